"""Decode attention split by the lengths of the step, against the CPU oracle (tolerances and cache checks of test_gpu_parity and
test_gpu_int8): lengths at the edges of blocks, tiles and chunk units, one sequence far longer than the rest, more kv heads
times sequences than the chip has places for, contexts far below the longest possible one, and both sides of the rule that
says which kernel appends the new rows (batch 16 and 17)."""
import numpy as np
import pytest
import torch

import test_gpu_int8 as q8
import test_gpu_parity as bf
from paper_2501_08192_amd import binding as psv
from paper_2501_08192_amd import synth
from paper_2501_08192_amd.harness import Session

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257]


@pytest.mark.parametrize("batch,nkv,group,context,lens", [
    (17, 1, 4, 1500, EDGES[:-1] + [1500]),          # edges and one long sequence; the attention appends
    (16, 2, 3, 640, [640] + EDGES[1:-1]),           # the preparing kernel appends (bf16)
    (16, 2, 3, 640, [640] * 16),                    # all equal
    (24, 8, 1, 400, [400 - 16 * b for b in range(24)]),     # 56 places per kv head, 24 sequences
    (64, 8, 1, 300, [1] * 63 + [300]),              # fewer places than sequences: one chunk each
    (3, 1, 8, 3000, [7, 3000, 300]),                # most chunks of one sequence
    (5, 1, 2, 3000, [1, 2, 3, 4, 5]),               # nobody near the longest possible length
    (3, 1, 2, 20000, [20000, 5003, 1500]),          # merged by eight waves: 157 chunks, 40 and 12 (int8 79, 20 and 6)
    (4, 1, 2, 8100, [8100, 4100, 1030, 129]),       # merged by four: 64, 33, 9 and 2 (int8 32, 17, 5 and 1)
], ids=["edges", "b16", "b16_equal", "kv8", "one_chunk_each", "long", "short", "merge8", "merge4"])
@pytest.mark.parametrize("kv", ["bf16", "int8"])
@pytest.mark.parametrize("paged", [False, True], ids=["contiguous", "paged"])
def test_split_by_length(batch, nkv, group, context, lens, kv, paged):
    args = ("plan", 1, 1024, nkv * group, nkv, 256, batch, context)
    if kv == "int8":
        q8.check_step(q8.W(*args, ("bf16", "int8"), paged=paged), seed=91, seq_lens=lens, pool_slack=2 if paged else 0)
    else:
        bf.check_step(bf.W(*args, paged=paged), seed=91, seq_lens=lens, pool_slack=2 if paged else 0)


@pytest.mark.parametrize("fmt", [("bf16", "bf16", "head"), ("bf16", "bf16", "token"), ("int8", "int8", "head")], ids=["bf16", "token", "int8"])
@pytest.mark.parametrize("batch", [3, 17])
def test_empty_and_out_of_range_lengths_among_valid_ones(batch, fmt):
    """Lengths of zero, below it and beyond the descriptor's max_seq are empty sequences: nothing of theirs is appended, their
    attention is empty, and the other sequences' results are what they are with any other empty length in those places."""
    w = synth.Workload("gap", 1, 1024, 4, 2, 128, 256, batch, 600, False, (0.0, 0.0), weight_format=fmt[0], kv_format=fmt[1], kv_layout=fmt[2])
    with Session(w, seed=92, max_seq=400) as s:
        def run(empty):
            lens = [400 - 20 * b for b in range(batch)]
            for k, b in enumerate(range(1, batch, 2)):
                lens[b] = empty[k % len(empty)]
            s.seq_lens.copy_(torch.tensor(lens, dtype=torch.int32))
            out = s.run().clone()
            assert torch.isfinite(out).all()
            att = psv.psv_debug_read(s.ctx, psv.PSV_DBG_ATTN, np.zeros((batch, 4 * 128), np.float32))
            assert not att[1::2].any() and att[0::2].any(axis=1).all()
            return out

        first = run([0])
        k, v = s.k_pools[0].clone(), s.v_pools[0].clone()      # the valid sequences' rows are in; appending them again changes nothing
        assert torch.equal(run([500, -1, 401, 0, 2 ** 31 - 1, -2 ** 31]), first)
        assert torch.equal(s.k_pools[0], k) and torch.equal(s.v_pools[0], v)
        s.seq_lens.fill_(-5)                                    # nobody has anything
        assert torch.isfinite(s.run()).all()
        assert torch.equal(s.k_pools[0], k) and torch.equal(s.v_pools[0], v)
        assert torch.equal(run([0]), first)


@pytest.mark.parametrize("fmt", [("bf16", "bf16"), ("int8", "int8")], ids=["bf16", "int8"])
@pytest.mark.parametrize("batch", [3, 17])
def test_layer_ranges_chain_like_the_whole_step(batch, fmt):
    """A caller that runs its own collectives comes back between the layers: the list of the step's lengths is made in every call
    and is the same each time."""
    w = synth.Workload("range", 3, 1024, 4, 2, 128, 256, batch, 500, False, (0.0, 0.0), weight_format=fmt[0], kv_format=fmt[1])
    with Session(w, seed=93) as s:
        s.seq_lens.copy_(torch.tensor([max(1, 500 - 31 * b) for b in range(batch)], dtype=torch.int32))
        whole = s.run().clone()
        tmp = s.x_in.clone()
        for l in range(3):
            s.step(x_in=tmp, x_out=tmp, layer_begin=l, layer_end=l + 1)       # in place
        s.sync()
        assert torch.equal(tmp, whole)
        s.step(x_out=tmp, layer_begin=0, layer_end=2)
        s.step(x_in=tmp, x_out=tmp, layer_begin=2, layer_end=3)
        s.sync()
        assert torch.equal(tmp, whole)


def test_token_major_rows_beyond_a_waves_first_tile():
    """Seventeen sequences of up to 2300 tokens and two kv heads fill the chip, so chunks are longer than one tile of each wave and
    a new row lies in a wave's first tile, its later ones and the last partly filled one.  The same logical cache head-major gives
    the same bits, and that layout is held to the oracle above."""
    args = dict(name="tm", n_layers=1, hidden=1024, n_q_heads=4, n_kv_heads=2, head_dim=128, ffn=256, batch=17, context=2300,
                paged=True, window_us=(0.0, 0.0))
    lens = [2300 - 37 * b for b in range(17)]
    with Session(synth.Workload(**args, kv_layout="token"), seed=94) as a, Session(synth.Workload(**args), seed=94) as b:
        b.k_pools[0].copy_(a.k_pools[0].permute(0, 2, 1, 3))
        b.v_pools[0].copy_(a.v_pools[0].permute(0, 2, 3, 1))
        for s in (a, b):
            s.seq_lens.copy_(torch.tensor(lens, dtype=torch.int32))
        assert torch.equal(a.run(), b.run())
        assert torch.equal(a.k_pools[0].permute(0, 2, 1, 3), b.k_pools[0])
        assert torch.equal(a.v_pools[0].permute(0, 2, 3, 1), b.v_pools[0])
    bf.check_step(bf.W("hm", 1, 1024, 4, 2, 256, 17, 2300, paged=True), seed=94, seq_lens=lens)


@pytest.mark.parametrize("kv,unit", [("bf16", 128), ("int8", 256)])
@pytest.mark.parametrize("units", [4095, 4096])
def test_both_sides_of_the_longest_sequence_that_the_list_can_hold(units, kv, unit):
    """An entry of the list holds a chunk size of up to 4095 units; a context for longer sequences divides the longest possible one
    instead.  Same cache, same lengths as in a context for short ones: equal to rounding, and the same new rows.  Page-table
    entries past a sequence's blocks name block 0; what is read there is past every span."""
    max_seq = min(units * unit, 1 << 20)
    w = synth.Workload("far", 1, 512, 4, 1, 128, 256, 3, 700, True, (0.0, 0.0), kv_format=kv)
    with Session(w, seed=95) as s:
        s.seq_lens.copy_(torch.tensor([700, 1, 333], dtype=torch.int32))
        ref, k, v = s.run().clone(), s.k_pools[0].clone(), s.v_pools[0].clone()
        table = torch.zeros(3, max_seq // 16, dtype=torch.int32, device=s.device)
        table[:, :w.blocks_per_seq] = s.page_table
        ctx = psv.psv_create(psv.model_desc(1, 512, 4, 1, 256, 3, max_seq, kv_format=kv), s.main, s.side)
        try:
            psv.psv_set_layer_weights(ctx, 0, s.weights[0])
            psv.psv_set_kv(ctx, [s.k_pools[0]], [s.v_pools[0]], table, max_seq // 16, s.pool_blocks, s.seq_lens)
            out = torch.empty_like(ref)
            torch.cuda.synchronize()
            psv.psv_decode_step(ctx, s.x_in, out, 3, 0, 1)
            psv.psv_sync(ctx)
            assert torch.allclose(out, ref, rtol=1e-5, atol=1e-5)
            assert torch.equal(s.k_pools[0], k) and torch.equal(s.v_pools[0], v)
        finally:
            psv.psv_destroy(ctx)
