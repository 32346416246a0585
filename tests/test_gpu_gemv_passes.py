"""Gate | up of the vector path: the weights of two passes in flight for two to many passes with full and ragged last ones, an even
and an odd number of them, groups of 128 to 512 threads a row, rows that end inside a group's reach, rows longer than 4096; one pass,
where a group has four rows at most (groups of 64 threads always do: the path ends at 8192 rows); both formats.  The stage against the product in
64 bits of the GPU's own input to it: fp32 sums of up to 8192 products leave about 1e-6, held to 1e-5 (a row of another pass, or
one that was not summed, is of the order of 1)."""
import numpy as np
import pytest
import torch

from paper_2501_08192_amd import binding as psv
from paper_2501_08192_amd import synth
from paper_2501_08192_amd.harness import Session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["bf16", "int8"])
@pytest.mark.parametrize("batch,H,F", [
    (1, 4096, 2304), (2, 4096, 2560), (2, 4096, 3584), (1, 4096, 8192),      # groups of a whole workgroup: 2, 2, 2 and 4 passes
    (1, 4096, 5120), (2, 4096, 4352),                                         # ... and 3
    (2, 1536, 7936), (1, 2048, 8192), (1, 1024, 4352), (2, 1024, 8192),      # groups of 256, 256, 128 and 128 threads: 2 passes
    (2, 512, 8192), (1, 1024, 2816),                                          # groups of 64 and 128 threads: one pass
    (1, 8192, 1280), (1, 8192, 2304), (1, 6144, 7168), (1, 8192, 8192),      # rows longer than 4096: 2, 3, 7 and 8 passes
])
def test_gate_up_of_every_number_of_passes(batch, H, F, fmt):
    w = synth.Workload("passes", 1, H, 2, 1, 128, F, batch, 20, False, (0.0, 0.0), weight_format=fmt)
    with Session(w, seed=23, fused=0) as s:
        s.run()
        assert psv.psv_get_stats(s.ctx)["kernels_per_layer"] == 5         # the vector path, a kernel per operator
        rd = lambda which, cols: torch.from_numpy(psv.psv_debug_read(s.ctx, which, np.zeros((batch, cols), np.float32))).to(s.device).double()
        y, m = rd(psv.PSV_DBG_Y, H), rd(psv.PSV_DBG_M, F)
        lw = synth.layer_weights(w, 0, 23, s.device)
        mat = lambda n: (lw["w_" + n].double() * (lw["s_" + n].double()[:, None] if fmt == "int8" else 1.0)).T.contiguous()
        h = y / torch.sqrt((y * y).mean(-1, keepdim=True) + w.rms_eps) * lw["g_mlp"].double()
        gate = h @ mat("gate")
        ref = gate * torch.sigmoid(gate) * (h @ mat("up"))
        assert float((m - ref).norm() / ref.norm()) < 1e-5
