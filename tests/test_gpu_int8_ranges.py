"""int8 projections on the matrix cores at the edges of their tiling: K ranges of one block of 128 elements up to several rounds of
the four-block ring and remainders of every size, one to four batch tiles with full and nearly empty last tiles, both layouts.
Every stage against the product in 64 bits of the GPU's own input to it.  The bound is the operand's: two digits with a step of
max|block| / 32258 are 2.5e-5 of a Gaussian operand's rms and 5e-5 of a heavier-tailed one's; three times that.  A block left out
or taken twice is 1 / sqrt(blocks) > 0.1."""
import numpy as np
import pytest
import torch

from paper_2501_08192_amd import binding as psv
from paper_2501_08192_amd import synth
from paper_2501_08192_amd.harness import Session

pytestmark = pytest.mark.gpu

# H, nq, nkv, F, batch, layout: K of QKV and gate | up is H, of O nq * 128, of down F
CASES = [
    (512, 4, 1, 256, 3, "row"), (512, 1, 1, 1280, 16, "tiled"), (1536, 12, 4, 2304, 17, "row"), (2048, 16, 2, 2816, 33, "tiled"),
    (1024, 8, 8, 768, 64, "row"), (8192, 10, 2, 6400, 49, "tiled"), (16384, 2, 1, 3328, 5, "row"), (8192, 16, 2, 7168, 48, "row"),
    (4096, 14, 2, 9472, 16, "tiled"), (4096, 4, 1, 1792, 32, "row"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "H%d_F%d_b%d_%s" % (c[0], c[3], c[4], c[5]))
def test_every_stage_against_64_bits_from_its_own_input(case):
    H, nq, nkv, F, B, layout = case
    w = synth.Workload("i8", 1, H, nq, nkv, 128, F, B, 40, False, (0.0, 0.0), weight_format="int8", weight_layout=layout)
    with Session(w, seed=31) as s:
        out = s.run().double()
        rd = lambda which, cols: torch.from_numpy(psv.psv_debug_read(s.ctx, which, np.zeros((B, cols), np.float32))).to(s.device).double()
        qkv, att, y, m = rd(psv.PSV_DBG_QKV, w.qkv_rows), rd(psv.PSV_DBG_ATTN, nq * 128), rd(psv.PSV_DBG_Y, H), rd(psv.PSV_DBG_M, F)
        lw = synth.layer_weights(w, 0, 31, s.device)
        x = s.x_in.double()
        norm = lambda t, g: t / torch.sqrt((t * t).mean(-1, keepdim=True) + w.rms_eps) * lw[g].double()
        lin = lambda t, n: t @ (lw["w_" + n].double() * lw["s_" + n].double()[:, None]).T.contiguous()
        gate = lin(norm(y, "g_mlp"), "gate")
        for name, got, ref in (("qkv", qkv, lin(norm(x, "g_attn"), "qkv")), ("o", y - x, lin(att, "o")),
                               ("gate_up", m, gate * torch.sigmoid(gate) * lin(norm(y, "g_mlp"), "up")), ("down", out - y, lin(m, "down"))):
            e = float((got - ref).norm() / ref.norm())
            assert e < 1.5e-4, (name, e)
