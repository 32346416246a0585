"""A chunk size set for all sequences (psv_set_attention_chunk): the matrix-core path's attention without the work list of the
step's lengths, which a step takes by itself only where the list does not fit or tuning has chosen so.  Against the CPU oracle
(tolerances of test_gpu_parity and test_gpu_int8; every byte of the cache outside the new rows untouched) for each cache, on both
sides of the rule that says which kernel appends the new rows (batch 16 and 17), and on the vector path (batch 2), with lengths that leave chunks empty and new
rows in a wave's first tile and beyond it.  A sequence's bits depend on the sequence alone then."""
import numpy as np
import pytest
import torch

import oracle
import test_gpu_int8 as q8
import test_gpu_parity as bf
from helpers import from_bits
from paper_2501_08192_amd import binding as psv
from paper_2501_08192_amd import synth
from paper_2501_08192_amd.harness import Session

pytestmark = pytest.mark.gpu

CACHES = {"head": ("bf16", "head"), "token": ("bf16", "token"), "int8": ("int8", "head")}
# block, tile and chunk edges, empty chunks behind the short ones; 641 and 897 are past a wave's first tile of a 640-token chunk
LENS = [900, 1, 16, 17, 128, 129, 255, 256, 257, 384, 640, 641, 897, 33, 513, 700, 5]


def workload(cache, batch):
    kv, layout = CACHES[cache]
    return synth.Workload("chunk", 1, 1024, 6, 2, 128, 256, batch, 900, batch % 2 == 1, (5.0, 5.0), kv_format=kv, kv_layout=layout)


def new_rows(w, lens, pt, shape):
    """Masks over the pools of a bf16 cache: the slots of the tokens being decoded, restated from the layouts."""
    k, v = np.zeros(shape[0], bool), np.zeros(shape[1], bool)
    for b in range(w.batch):
        t = int(lens[b]) - 1
        blk = int(pt[b, t // 16]) if pt is not None else b * w.blocks_per_seq + t // 16
        if w.kv_layout == "token":
            k[blk, t % 16] = v[blk, t % 16] = True
        else:
            k[blk, :, t % 16] = True
            v[blk, :, :, t % 16] = True
    return k, v


def check_against_oracle(s, lens):
    """One step of layer 0 against the oracle on the same inputs; returns the step's output."""
    w = s.w
    m = oracle.model(w.hidden, w.n_q_heads, w.n_kv_heads, w.head_dim, w.ffn, 16, w.rms_eps, w.rope_theta, kv_token_major=w.kv_layout == "token")
    s.seq_lens.copy_(torch.tensor(lens, dtype=torch.int32))
    pt = s.page_table_host.numpy() if w.paged else None
    before = s.host_pools(0)
    kr, vr = before[0].copy(), before[1].copy()
    x = oracle.decode_layer_x(m, s.host_layer(0), kr, vr, pt, w.blocks_per_seq, np.asarray(lens, np.int32), s.x_in.cpu().numpy().astype(np.float64))
    got = s.run().clone()
    bf.assert_close(got.cpu().numpy(), x, "chunk %d" % psv.psv_get_attention_chunk(s.ctx))
    kg, vg = s.host_pools(0)
    if w.kv_format == "int8":
        km, vm = q8.new_slot_mask_int8(kg.shape, w, lens, pt)
        for is_v, g, r in ((False, kg, kr), (True, vg, vr)):
            rows, scales = q8.appended_rows_int8(g, w, lens, pt, is_v)
            ref, ref_scales = q8.appended_rows_int8(r, w, lens, pt, is_v)
            np.testing.assert_allclose(scales, ref_scales, rtol=1e-3)
            assert (np.abs(rows - ref) <= 1.01 * ref_scales[..., None] + 1e-3 * np.abs(ref)).all()      # one code
    else:
        km, vm = new_rows(w, lens, pt, (kg.shape, vg.shape))
        for g, r, mask in ((kg, kr, km), (vg, vr, vm)):
            # one rounding to bf16 on either side of a boundary, and the fp32 sums (1e-4 absolute, as in test_gpu_parity)
            assert (np.abs(from_bits(g[mask]) - from_bits(r[mask])) <= 2.0 ** -7 * np.abs(from_bits(r[mask])) + 1e-4).all()
    assert np.array_equal(kg[~km], before[0][~km]) and np.array_equal(vg[~vm], before[1][~vm]), "cache touched outside the new rows"
    return got


@pytest.mark.parametrize("batch", [2, 3, 16, 17])
@pytest.mark.parametrize("cache", sorted(CACHES))
def test_uniform_chunks_match_oracle(cache, batch):
    w = workload(cache, batch)
    unit = 256 if cache == "int8" else 128
    with Session(w, seed=61) as s:
        own = check_against_oracle(s, LENS[:batch])
        for units in (1, 5 if unit == 128 else 3, -(-w.context // unit)):
            psv.psv_set_attention_chunk(s.ctx, units * unit)
            check_against_oracle(s, LENS[:batch])
        psv.psv_set_attention_chunk(s.ctx, 0)
        assert torch.equal(s.run(), own)                 # back to the library's own split


@pytest.mark.parametrize("cache", sorted(CACHES))
def test_with_uniform_chunks_a_sequence_does_not_see_its_neighbours(cache):
    w = workload(cache, 17)
    with Session(w, seed=62) as s:
        psv.psv_set_attention_chunk(s.ctx, 256)
        outs = []
        for others in (LENS[1:], [900] * 16, [1] * 16):
            s.seq_lens.copy_(torch.tensor([700] + others, dtype=torch.int32))
            outs.append(s.run()[0].clone())
        assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


def test_chunk_sizes_that_cannot_be_are_refused_and_change_nothing():
    w = synth.Workload("chunk", 1, 512, 4, 2, 128, 256, 3, 100, False, (0.0, 0.0))
    with Session(w, seed=63) as s:
        L = psv.lib()
        psv.psv_set_attention_chunk(s.ctx, 128)
        for bad in (1, 64, 127, 200, 256, 1 << 20, (1 << 32) - 128):
            assert L.psv_set_attention_chunk(s.ctx, bad) == psv.PSV_ERR_INVALID_ARG, bad
            assert psv.psv_get_attention_chunk(s.ctx) == 128
        assert L.psv_set_attention_chunk(None, 128) == psv.PSV_ERR_INVALID_ARG
        assert L.psv_get_attention_chunk(s.ctx, None) == psv.PSV_ERR_INVALID_ARG
    with Session(w.scaled(kv_format="int8"), seed=63) as s:
        assert psv.lib().psv_set_attention_chunk(s.ctx, 128) == psv.PSV_ERR_INVALID_ARG      # int8 tiles are twice as long
        psv.psv_set_attention_chunk(s.ctx, 256)
    with Session(w.scaled(context=256 * 128 + 16, batch=1), seed=63) as s:                     # more than 256 chunks of 128
        assert psv.lib().psv_set_attention_chunk(s.ctx, 128) == psv.PSV_ERR_INVALID_ARG
        psv.psv_set_attention_chunk(s.ctx, 256)


def test_tuning_keeps_the_split_by_length_where_it_is_the_faster_and_reports_its_chunk_size():
    """One long sequence among short ones, far from filling the chip: the library's own split takes the smallest chunks for the few
    tokens there are (measured 48 us a step), not those that divide the longest possible sequence (512 tokens, 53 us); the best
    uniform size (384) takes 51."""
    w = synth.Workload("tune", 1, 512, 4, 1, 128, 256, 24, 8192, False, (0.0, 0.0))
    with Session(w, seed=64) as s:
        s.seq_lens.copy_(torch.tensor([8192] + [64] * 23, dtype=torch.int32))
        own = s.run().clone()
        for rep in range(2):
            assert s.tune_attention() == 128 and psv.psv_get_attention_chunk(s.ctx) == 0
            assert torch.equal(s.run(), own)
        psv.psv_set_attention_chunk(s.ctx, 512)
        assert s.tune_attention() == 128 and psv.psv_get_attention_chunk(s.ctx) == 0       # whatever was set before
