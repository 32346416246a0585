"""Gate | up projections whose ranges begin at multiples of 4 KiB are walked from another slab on in every row tile: every slab once (each
stage against the product in 64 bits of the GPU's own input to it; bound as in test_gpu_stage_errors, two bf16 planes), the same
bits in both layouts and launched into a communication window or not."""
import numpy as np
import pytest
import torch

from paper_2501_08192_amd import binding as psv
from paper_2501_08192_amd import synth
from paper_2501_08192_amd.harness import Session, default_policy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [16, 17, 33, 64])      # one to four batch tiles
def test_turned_ranges(batch):
    H, F = 8192, 7168          # four ranges of 32 slabs
    outs = []
    for layout in ("row", "tiled"):
        w = synth.Workload("turn", 2, H, 2, 1, 128, F, batch, 20, False, (15.0, 15.0), weight_layout=layout)
        with Session(w, seed=19) as s:
            outs.append(s.run().clone())
            rd = lambda which, cols: torch.from_numpy(psv.psv_debug_read(s.ctx, which, np.zeros((batch, cols), np.float32))).to(s.device).double()
            y, m = rd(psv.PSV_DBG_Y, H), rd(psv.PSV_DBG_M, F)
            lw = synth.layer_weights(w, 1, 19, s.device)
            h = y / torch.sqrt((y * y).mean(-1, keepdim=True) + w.rms_eps) * lw["g_mlp"].double()
            gate = h @ lw["w_gate"].double().T.contiguous()
            ref = gate * torch.sigmoid(gate) * (h @ lw["w_up"].double().T.contiguous())
            assert float((m - ref).norm() / ref.norm()) < 2e-5
            for policy in (default_policy(w), default_policy(w, prelaunch=0)):
                s.set_policy(policy)
                assert torch.equal(s.run(), outs[-1])
                if policy.prelaunch and s.overlap:
                    assert psv.psv_debug_last_step_prelaunches(s.ctx) == (2 if batch <= 16 else 0)
    assert torch.equal(outs[0], outs[1])
