"""The selection of short sequences scores its blocks in the same launch.  Compared bit by bit with the two launches that
longer sequences take (a bound on the blocks, or its absence, decides which runs), which the decode tests compare with the
oracle."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from dsk_testutil import dev_i32

pytestmark = pytest.mark.gpu


def _tables(rng, blocks, Hq, Hkv, b, room):
    """Tables and summaries of sequences with these numbers of blocks, without the pass that would make them."""
    lens = [rng.integers(1, 3 * b, size=n) for n in blocks]
    flat = np.concatenate(lens) if sum(blocks) else np.zeros(0, np.int64)
    cap = sum(blocks) + room
    bs = np.concatenate([[0], np.cumsum(flat), np.zeros(room + 4, np.int64)])
    sb = np.concatenate([[0], np.cumsum(-(-flat // b)), np.zeros(room + 4, np.int64)])
    ksum = torch.from_numpy(rng.standard_normal((Hkv, cap, 2, 128)).astype(np.float32)).cuda().bfloat16()
    ksum = torch.stack([ksum.amin(2), ksum.amax(2)], 2).contiguous()
    ksum[:, : sum(blocks): 7] = ksum[:, :1].clone()                        # ties
    t = SimpleNamespace()
    t.B, t.Hq, t.Hkv, t.b, t.max_blocks_total = len(blocks), Hq, Hkv, b, cap
    t.cu_blocks, t.block_start, t.slot_base = dev_i32(np.concatenate([[0], np.cumsum(blocks)])), dev_i32(bs), dev_i32(sb)
    t.ksum = ksum
    return t


def _run(t, q, budget, **kw):
    import paper_2602_03184_amd as dsk
    sel = dsk.make_select_args(t, q, budget, want_scores=True, **kw)
    for x in (sel.sel_slot, sel.sel_start, sel.sel_len, sel.sel_count):
        x.fill_(-7)
    sel.scores.fill_(0)
    dsk.dsk_select_topk(sel.args)
    torch.cuda.synchronize()
    return [x.clone() for x in (sel.sel_slot, sel.sel_start, sel.sel_len, sel.sel_count, sel.scores)]


GROUPS = [(1, 1), (8, 2), (6, 2), (16, 1), (28, 4), (32, 8), (10, 10)]
BLOCKS = [[1], [127], [128], [129], [255], [256], [200, 0, 1, 256, 0], [5] * 11, [0, 0, 40]]


@pytest.mark.parametrize("Hq,Hkv", GROUPS)
@pytest.mark.parametrize("blocks", BLOCKS, ids=str)
def test_one_launch_equals_two(blocks, Hq, Hkv):
    rng = np.random.default_rng([Hq, Hkv, len(blocks), max(blocks)])
    b = int(rng.choice([1, 8, 16]))
    t = _tables(rng, blocks, Hq, Hkv, b, room=2000)                        # 2000: no bound would let it run in one launch
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    q = torch.randn(t.B, Hq, 128, generator=g, device="cuda").bfloat16()
    budgets = dev_i32(rng.integers(0, 80 * b, size=t.B))
    n = sum(blocks)
    for budget in (b, 37 * b, 5000 * b):
        for kw in (dict(), dict(shared=True), dict(budget_per_seq=budgets)):
            two = _run(t, q, budget, **kw)
            one = _run(t, q, budget, max_blocks_per_seq=max(max(blocks), 1), **kw)
            short = _run(t, q, budget, max_blocks_per_seq=3, **kw)         # a bound that is too small
            for name, x, y, z in zip(("slot", "start", "len", "count"), one, two, short):
                assert torch.equal(x, y) and torch.equal(z, y), (name, budget, kw)
            assert torch.equal(one[4][:, :n], two[4][:, :n]) and torch.equal(short[4][:, :n], two[4][:, :n])


def test_beyond_the_tile_and_regions():
    """More blocks than any bound promises; tables with a region per sequence, of which one is empty and one full."""
    rng = np.random.default_rng(9)
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    t = _tables(rng, [3000, 20, 600], 8, 2, 16, room=100)
    q = torch.randn(3, 8, 128, generator=g, device="cuda").bfloat16()
    two, one = _run(t, q, 640), _run(t, q, 640, max_blocks_per_seq=200)
    assert all(torch.equal(x, y) for x, y in zip(one[:4], two[:4])) and torch.equal(one[4][:, :3620], two[4][:, :3620])

    t = _tables(rng, [200, 100, 256], 8, 2, 16, room=900)
    base = t.block_start.clone()
    for s, (lo, hi) in enumerate([(0, 200), (200, 300), (300, 556)]):     # inside a region positions and slots count from 0
        t.block_start[lo:hi] = base[lo:hi] - base[lo]
        t.slot_base[lo:hi] -= t.slot_base[lo].clone()
    t.blocks_used, t.seq_row0 = dev_i32([199, 0, 255]), dev_i32([1000, 50, 7])
    two, one = _run(t, q, 640), _run(t, q, 640, max_blocks_per_seq=255)
    assert all(torch.equal(x, y) for x, y in zip(one[:4], two[:4]))
    assert torch.equal(one[4][:, :556], two[4][:, :556])                   # what a region has in reserve is scored too


@pytest.mark.parametrize("blocks", [[257], [300, 20], [511, 512], [20, 513, 200]], ids=str)
@pytest.mark.parametrize("Hq,Hkv", [(8, 2), (6, 2)])
def test_sequences_that_outgrow_the_bounds(blocks, Hq, Hkv):
    """A sequence with a few more blocks than the caller's bounds say: up to 512 they are scored into the workgroup's own
    memory, beyond that through the workspace."""
    rng = np.random.default_rng([Hq, len(blocks), max(blocks)])
    t = _tables(rng, blocks, Hq, Hkv, 16, room=2000)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    q = torch.randn(t.B, Hq, 128, generator=g, device="cuda").bfloat16()
    n = sum(blocks)
    two = _run(t, q, 37 * 16)
    for kw in (dict(max_blocks_per_seq=250), dict(max_blocks_per_seq=100), dict(max_blocks_used=n - 7, max_blocks_per_seq=256),
               dict(max_blocks_used=19, max_blocks_per_seq=256)):
        one = _run(t, q, 37 * 16, **kw)
        for x, y in zip(one[:4], two[:4]):
            assert torch.equal(x, y), kw
        assert torch.equal(one[4][:, :n], two[4][:, :n]), kw
