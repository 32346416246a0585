"""Decode attention split by the lengths of the step, against the CPU oracle (tolerances and cache checks of test_gpu_parity and
test_gpu_int8): lengths at the edges of blocks, tiles and chunk units, one sequence far longer than the rest, more kv heads
times sequences than the chip has places for, contexts far below the longest possible one, and both sides of the rule that
says which kernel appends the new rows (batch 16 and 17)."""
import pytest

import test_gpu_int8 as q8
import test_gpu_parity as bf

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
], ids=["edges", "b16", "b16_equal", "kv8", "one_chunk_each", "long", "short"])
@pytest.mark.parametrize("kv", ["bf16", "int8"])
@pytest.mark.parametrize("paged", [False, True], ids=["contiguous", "paged"])
def test_split_by_length(batch, nkv, group, context, lens, kv, paged):
    args = ("plan", 1, 1024, nkv * group, nkv, 256, batch, context)
    if kv == "int8":
        q8.check_step(q8.W(*args, ("bf16", "int8"), paged=paged), seed=91, seq_lens=lens, pool_slack=2 if paged else 0)
    else:
        bf.check_step(bf.W(*args, paged=paged), seed=91, seq_lens=lens, pool_slack=2 if paged else 0)
