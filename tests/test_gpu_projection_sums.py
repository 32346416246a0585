"""Distance of the matrix-core QKV sums from 64 bits.  The operand is exact here (a bf16 input times a bf16 gain has 16 significant
bits, which the two bf16 planes hold), so what is left is the rounding of fp32 sums: m roundings of a running sum that grows as a
random walk give a distance that grows as sqrt(m).  Measured with 44 roundings a K range 2.44e-7, with 32 2.18e-7, with 22 1.73e-7.
The bound is what 32 roundings give: neither a longer range nor a longer chain may cost precision."""
import numpy as np
import pytest
import torch

from paper_2501_08192_amd import binding as psv
from paper_2501_08192_amd import synth
from paper_2501_08192_amd.harness import Session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["row", "tiled"])
@pytest.mark.parametrize("batch", [3, 17, 33, 64])      # one to four batch tiles
def test_qkv_sums_are_no_further_from_64_bits_than_short_ranges_were(batch, layout):
    w = synth.Workload("sums", 1, 8192, 16, 2, 128, 256, batch, 32, False, (0.0, 0.0), weight_layout=layout)
    with Session(w, seed=7) as s:
        s.run()
        got = torch.from_numpy(psv.psv_debug_read(s.ctx, psv.PSV_DBG_QKV, np.zeros((batch, w.qkv_rows), np.float32))).cuda().double()
        lw = synth.layer_weights(w, 0, 7, s.device)
        x = s.x_in.double()
        x = x / torch.sqrt((x * x).mean(-1, keepdim=True) + w.rms_eps) * lw["g_attn"].double()
        ref = x @ lw["w_qkv"].double().T
        assert float((got - ref).norm() / ref.norm()) < 2.2e-7
