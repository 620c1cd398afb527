"""Register tiles of the selection: the same lists whichever tile the bound on the blocks leads to, at the tiles' edges, against
the path that reads its keys from memory and against a sort of the scores on the host."""
import numpy as np
import pytest
import torch

from dsk_testutil import dev_i32
from test_gpu_select_short import _run, _tables

pytestmark = pytest.mark.gpu


def _sorted_slots(t, scores, seq, k):
    """Slots of sequence `seq` that a head with these block scores takes: best score first, then lowest index."""
    lo, hi = (int(x) for x in t.cu_blocks[seq: seq + 2].cpu())
    sb = t.slot_base[lo: hi + 1].cpu().numpy()
    slot_score = np.repeat(scores[lo:hi].cpu().numpy(), np.diff(sb))
    return sb[0] + np.sort(np.argsort(-slot_score, kind="stable")[:k])


@pytest.mark.parametrize("blocks", [[4093], [4094], [3, 6141], [6142, 1], [1, 8189], [8190], [2, 12285], [5, 12286], [3, 16381, 40],
                                    [16382], [20000]], ids=str)
@pytest.mark.parametrize("b", [1, 16])
def test_every_register_tile_selects_alike(blocks, b):
    rng = np.random.default_rng([b, max(blocks)])
    t = _tables(rng, blocks, 2, 1, b, room=30000)
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    q = torch.randn(t.B, 2, 128, generator=g, device="cuda").bfloat16()
    for budget in (b, 129 * b, 3000 * b):                                  # several rounds of the list of chosen blocks
        memory = _run(t, q, budget, max_blocks_per_seq=300)                # outgrown: read from memory
        # bounds that fit, and one that leaves the tile to the length of the sequence
        for kw in (dict(max_blocks_per_seq=max(blocks)), dict(max_blocks_per_seq=max(blocks) + 1), dict(max_blocks_per_seq=16381),
                   dict()):
            got = _run(t, q, budget, **kw)
            for name, x, y in zip(("slot", "start", "len", "count"), got, memory):
                assert torch.equal(x, y), (name, budget, kw)
        for s in range(t.B):
            for h in range(2):
                n = int(got[3][s, h])
                np.testing.assert_array_equal(got[0][s, h, :n].cpu().numpy(), _sorted_slots(t, got[4][h], s, budget // b))


def test_tiles_by_the_length_of_regions():
    """Tables with a region per sequence under a bound for the largest tile: the tile goes by the blocks in use, not by the region."""
    rng = np.random.default_rng(12)
    sizes, used = [9000, 13000, 17000, 4000], [8100, 12285, 16900, 0]
    t = _tables(rng, sizes, 2, 1, 8, room=100)
    ends = np.concatenate([[0], np.cumsum(sizes)])
    base = t.block_start.clone()
    for lo, hi in zip(ends, ends[1:]):                                     # inside a region positions and slots count from 0
        t.block_start[lo:hi] = base[lo:hi] - base[lo]
        t.slot_base[lo:hi] -= t.slot_base[lo].clone()
    t.blocks_used, t.seq_row0 = dev_i32(used), dev_i32([5, 0, 100000, 7])
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    q = torch.randn(4, 2, 128, generator=g, device="cuda").bfloat16()
    for budget in (8, 1500 * 8):
        memory = _run(t, q, budget, max_blocks_per_seq=300)
        for kw in (dict(max_blocks_per_seq=16381), dict()):
            for x, y in zip(_run(t, q, budget, **kw)[:4], memory):
                assert torch.equal(x, y), (budget, kw)
        assert memory[3].cpu().tolist() == [[min(budget // 8, 1500)] * 2] * 3 + [[0, 0]]
