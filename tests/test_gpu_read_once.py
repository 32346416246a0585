"""A model that exceeds the memory-side cache is read with other load instructions (non-temporal) than one that fits; nothing else differs.
The same layer as the only one of its model and as the first of eighty (the others are described but not materialised): the same
bits, on the vector path, with one to four batch tiles, for every layout, and launched into a window."""
import pytest
import torch

from paper_2501_08192_amd import binding as psv
from paper_2501_08192_amd import synth
from paper_2501_08192_amd.harness import Session, default_policy

pytestmark = pytest.mark.gpu


def _same_bits(layers, weights_once, kv_once, *shape, **formats):
    """Two numbers of layers, the rule's answers for the larger one (none for the smaller), and bits that agree."""
    outs = []
    for n_layers in layers:
        w = synth.Workload("once", n_layers, *shape, (8.0, 8.0), **formats)
        with Session(w, seed=29, layers=[0]) as s:
            s.seq_lens.copy_(torch.tensor([max(1, w.context - 11 * b) for b in range(w.batch)], dtype=torch.int32))
            out = [s.run().clone()]
            s.set_policy(default_policy(w, budget_bytes=1 << 40))
            out.append(s.run().clone())
            assert psv.psv_debug_last_step_read_once(s.ctx) == ((weights_once, kv_once) if n_layers == layers[1] else (False, False))
            outs.append(out + [s.k_pools[0].clone(), s.v_pools[0].clone()])
    assert torch.isfinite(outs[0][0]).all() and torch.equal(outs[0][0], outs[0][1])
    for a, b in zip(*outs):
        assert torch.equal(a.view(torch.int16) if a.dtype == torch.bfloat16 else a, b.view(torch.int16) if b.dtype == torch.bfloat16 else b)


@pytest.mark.parametrize("batch,weights,kv,layout,kv_layout,paged", [
    (1, "bf16", "bf16", "row", "head", True), (2, "bf16", "bf16", "row", "token", False), (1, "int8", "int8", "row", "head", True),
    (3, "bf16", "bf16", "tiled", "head", True), (17, "bf16", "bf16", "tiled", "token", True), (33, "bf16", "int8", "tiled", "head", False),
    (64, "bf16", "bf16", "tiled", "head", True), (16, "bf16", "bf16", "row", "head", False), (40, "int8", "int8", "tiled", "head", True),
    (3, "int8", "bf16", "tiled", "head", False), (17, "int8", "int8", "tiled", "head", True), (64, "int8", "bf16", "tiled", "head", True),
])
def test_same_bits_as_the_only_layer_and_as_the_first_of_many(batch, weights, kv, layout, kv_layout, paged):
    _same_bits((1, 80), True, True, 1024, 8, 2, 128, 1024, batch, 700, paged,        # 11.5 MB a layer in bf16, 5.8 MB in int8
               weight_format=weights, kv_format=kv, kv_layout=kv_layout, weight_layout=layout)


@pytest.mark.parametrize("batch,weights", [(1, "bf16"), (2, "bf16"), (1, "int8")])
def test_same_bits_with_two_passes_of_weights_in_flight(batch, weights):
    _same_bits((1, 8), True, True, 4096, 8, 2, 128, 3584, batch, 100, False, weight_format=weights)       # 109 MB a layer in bf16


@pytest.mark.parametrize("batch", [5, 17, 33, 64])
@pytest.mark.parametrize("weights", ["bf16", "int8"])
def test_same_bits_over_long_ranges(batch, weights):
    """Ranges of up to eleven int8 blocks or twenty-two slabs: several rounds of the rings of weights in flight, and their remainders."""
    _same_bits((1, 4), True, True, 4096, 2, 1, 128, 9472, batch, 90, False, weight_format=weights, kv_format="bf16", weight_layout="tiled")     # 240 MB a layer in bf16


def test_same_bits_where_only_the_cache_exceeds_it():
    _same_bits((1, 16), False, True, 1024, 8, 2, 128, 1024, 33, 700, True, weight_layout="tiled")         # 184 MB of weights


def test_the_cache_counts_as_far_as_it_is_read():
    """Weights fit the memory-side cache, the largest cache the context can hold does not: keys and values are read that way for a step
    whose planned context and batch exceed it, not for a short one of the same context, and the bits are the same."""
    w = synth.Workload("live", 4, 1024, 8, 8, 128, 1024, 16, 4096, False, (0.0, 0.0))      # 60 MB of weights, up to 1 GiB of cache
    with Session(w, seed=3) as s:
        outs = []
        for context, batch, want in ((4096, 16, True), (700, 16, False), (4096, 2, False), (16, 1, False), (900, 16, True)):
            psv.psv_set_policy(s.ctx, psv.prefetch_policy(mode=0), batch, context)
            s.seq_lens.fill_(16)
            psv.psv_decode_step(s.ctx, s.x_in, s.x_out, batch, 0, w.n_layers)
            s.sync()
            assert psv.psv_debug_last_step_read_once(s.ctx) == (False, want), (context, batch)
            if batch == 16:
                outs.append(s.x_out.clone())
        assert all(torch.equal(o, outs[0]) for o in outs)
