"""Attention over values of extreme sizes: what single precision holds is neither flushed to zero nor turned into a NaN."""
import numpy as np
import pytest
import torch

from paper_2501_08192_amd import binding as psv
from paper_2501_08192_amd import synth
from paper_2501_08192_amd.harness import Session

pytestmark = pytest.mark.gpu


def _attention(s, batch, nq):
    s.run()
    return torch.from_numpy(psv.psv_debug_read(s.ctx, psv.PSV_DBG_ATTN, np.zeros((batch, nq * 128), np.float32))).double()


@pytest.mark.parametrize("batch", [1, 3], ids=["vector", "matrix"])
@pytest.mark.parametrize("at", [0, 70, 299, 600], ids=["first", "second_tile", "fifth_tile", "late"])
def test_probabilities_below_the_normal_range_count_int8(batch, at):
    """One key 130 binary orders above the others, whose values are 1e43 times larger: the result is theirs.  2^-130 has 19 significant
    bits left in single precision; two digits of a query are 1.5e-5 of its largest element, 2e-6 of a score of 128 products, 2e-4 of
    2^score.  Held to 2e-3 (a flushed probability leaves an error of 1)."""
    T = 700
    w = synth.Workload("tiny", 1, 512, 1, 1, 128, 256, batch, T, False, (0.0, 0.0), rope_theta=0.0, kv_format="int8")
    with Session(w, seed=41, fused=0) as s:
        s.run()
        qkv = torch.from_numpy(psv.psv_debug_read(s.ctx, psv.PSV_DBG_QKV, np.zeros((batch, 3 * 128), np.float32))).double()
        k, v = s.k_pools[0].cpu(), s.v_pools[0].cpu()
        k_scale, v_scale = (p[:, 0, 2048:].contiguous().view(torch.float32).clone() for p in (k, v))
        k_code = k[:, 0, :2048].contiguous().view(torch.int8).view(-1, 16, 128).clone()
        k_code.zero_()
        v_scale.fill_(1e10)
        for b in range(batch):
            q = qkv[b, :128]
            blk, r = b * w.blocks_per_seq + at // 16, at % 16
            code = torch.round(q / q.abs().max() * 127)
            k_code[blk, r] = code.to(torch.int8)
            k_scale[blk, r] = 130.0 / (float(q @ code) * 0.08838834764831845 * 1.4426950408889634)
            v_scale[blk, r] = 1e-33
        k[:, 0, :2048] = k_code.view(-1, 2048).view(torch.uint8).view(k.dtype)
        k[:, 0, 2048:] = k_scale.view(torch.uint8).view(k.dtype)
        v[:, 0, 2048:] = v_scale.view(torch.uint8).view(v.dtype)
        s.k_pools[0].copy_(k)
        s.v_pools[0].copy_(v)
        got = _attention(s, batch, 1)
        k, v = s.k_pools[0].cpu(), s.v_pools[0].cpu()          # with the new rows
        rows = lambda p, channel_major: (p[:, 0, :2048].contiguous().view(torch.int8).double().view(-1, 128, 16).transpose(1, 2) if channel_major
                                         else p[:, 0, :2048].contiguous().view(torch.int8).double().view(-1, 16, 128)) \
            * p[:, 0, 2048:].contiguous().view(torch.float32).double()[..., None]
        kd, vd = rows(k, False).reshape(batch, -1, 128)[:, :T], rows(v, True).reshape(batch, -1, 128)[:, :T]
        for b in range(batch):
            ref = torch.softmax(kd[b] @ qkv[b, :128] * 128 ** -0.5, 0) @ vd[b]
            assert float((got[b] - ref).norm() / ref.norm()) < 2e-3, b


@pytest.mark.parametrize("kv", ["bf16", "int8"])
@pytest.mark.parametrize("batch,context", [(1, 6000), (1, 20000), (3, 6000), (3, 20000)])      # four and eight waves a merge, both forms
def test_an_overflowing_sum_stays_an_infinity(batch, context, kv):
    """Values of 3e38 whose sums leave the range, in more chunks than the merge requests at once: infinite, as each chunk's sum is."""
    w = synth.Workload("huge", 1, 512, 1, 1, 128, 256, batch, context, False, (0.0, 0.0), kv_format=kv)
    with Session(w, seed=43, fused=0) as s:
        s.k_pools[0].zero_()
        if kv == "bf16":
            s.v_pools[0].fill_(3e38)
        else:
            v = s.v_pools[0].cpu()
            v[..., :2048] = 127
            v[..., 2048:] = torch.full((16,), 2.4e36, dtype=torch.float32).view(torch.uint8).view(v.dtype)
            s.v_pools[0].copy_(v)
        got = _attention(s, batch, 1)
        assert bool((got == float("inf")).all()), got[:, :4]
