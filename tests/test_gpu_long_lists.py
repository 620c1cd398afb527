"""The attention kernel for long lists: a workgroup per CU, each with many slots of one head.  Lists given directly (no
selection in front), against attention over the same rows in 64 bits."""
import math

import numpy as np
import pytest
import torch

from dsk_testutil import dev_i32, rel_err

pytestmark = pytest.mark.gpu


def _lists(rng, B, H, k, b, L, counts):
    start, length = np.zeros((B, H, k), np.int32), np.zeros((B, H, k), np.int32)
    for s in range(B):
        for h in range(H):
            n = int(counts[s, h])
            length[s, h, :n] = rng.integers(1, b + 1, size=n)
            start[s, h, :n] = np.sort(rng.integers(0, L - b, size=n))
            length[s, h, n:] = b                      # behind the count: not to be read
    return start, length


def _want(q, K, V, start, length, counts, div):
    B, Hq, _ = q.shape
    G = Hq // K.shape[0]
    out, lse = np.zeros((B, Hq, 128)), np.full((B, Hq), -np.inf)
    qd, Kd, Vd = q.double(), K.double(), V.double()
    for s in range(B):
        for h in range(Hq):
            n = int(counts[s, h // div])
            if n == 0:
                continue
            rows = np.concatenate([np.arange(a, a + l) for a, l in zip(start[s, h // div, :n], length[s, h // div, :n])])
            rows = torch.from_numpy(rows).cuda()
            z = Kd[h // G][rows] @ qd[s, h] / math.sqrt(128.0)
            lse[s, h] = float(torch.logsumexp(z, 0))
            out[s, h] = (torch.softmax(z, 0) @ Vd[h // G][rows]).cpu().numpy()
    return out, lse


# (B, Hq, Hkv, k, b, lists per head on the kernel for long lists, shared lists on the kernel of their own): one list a head
# with 32 slots, one more, a slot count beyond the 64 spans of a wavefront; several chunks; runs of chunks on XCDs of their
# own (4, 2, 1 and 3 groups); heads without groups; several rounds of workgroups and lists too long for them; every width and tile of the shared kernel,
# slots of one and two tiles of 16 rows, at the slot counts it starts with and well above them
SHAPES = [(8, 32, 8, 32, 16, True, False), (8, 32, 8, 33, 16, True, False), (8, 32, 8, 545, 8, True, True),
          (2, 32, 8, 163, 32, True, False), (1, 28, 4, 257, 16, True, False), (1, 16, 2, 515, 8, True, False),
          (1, 8, 1, 129, 16, False, False), (1, 40, 40, 245, 16, True, False), (3, 6, 1, 40, 16, False, False),
          (8, 40, 8, 121, 16, False, True), (3, 16, 2, 16, 32, False, False), (1, 28, 4, 40, 64, False, False),
          (4, 16, 8, 97, 32, False, True), (5, 24, 8, 83, 17, True, True), (4, 40, 8, 200, 32, False, True),
          (12, 56, 8, 33, 9, True, True), (6, 11, 1, 520, 16, False, True), (16, 8, 4, 49, 16, False, True),
          (8, 16, 8, 150, 32, True, True), (8, 24, 8, 139, 17, False, True), (12, 56, 8, 83, 9, True, True),
          (8, 11, 1, 810, 16, True, True), (16, 8, 4, 121, 16, True, True), (16, 32, 8, 64, 16, True, True), (16, 32, 8, 65, 16, True, True), (16, 32, 8, 100, 32, False, True)]


def _partials_left(att, lay):
    """Number of partials that a call wrote into a workspace that held NaN."""
    ml = att.keep[-1].view(torch.uint8).cpu().numpy()[lay.ml_offset: lay.acc_offset].view(np.float32).reshape(-1, 2)
    return int((~np.isnan(ml[:, 1])).sum())


@pytest.mark.parametrize("B,Hq,Hkv,k,b,is_long,on_shared_kernel", SHAPES)
@pytest.mark.parametrize("layout", ["hnd", "nhd"])
def test_long_lists(B, Hq, Hkv, k, b, is_long, on_shared_kernel, layout):
    import paper_2602_03184_amd as dsk
    rng = np.random.default_rng([B, Hq, Hkv, k, b])
    g = torch.Generator(device="cuda")
    g.manual_seed(k)
    L = 3001
    K, V = (torch.randn(Hkv, L, 128, generator=g, device="cuda").bfloat16() for _ in range(2))
    if layout == "nhd":
        K, V = (x.permute(1, 0, 2).contiguous().permute(1, 0, 2) for x in (K, V))
    q = torch.randn(B, Hq, 128, generator=g, device="cuda").bfloat16()
    for shared in (False, True):
        H = Hkv if shared else Hq
        if shared and Hq == Hkv:
            continue
        counts = np.minimum(k, rng.integers(0, 2 * k, size=(B, H)))
        counts.flat[-1], counts.flat[0] = 0, k
        start, length = _lists(rng, B, H, k, b, L, counts)
        flags = dsk.DSK_ATTN_SHARED_SELECTION if shared else 0
        att = dsk.make_attn_args(q, K, V, dev_i32(start), dev_i32(length), dev_i32(counts), b, flags=flags, want_bf16=True)
        lay = dsk.dsk_attn_partials_layout(att.args)
        assert lay.nchunks * lay.slots_per_chunk >= k
        if shared:                                        # the others cut lists that are to be left in parts into 8 or 16
            assert (lay.slots_per_chunk not in (8, 16)) == on_shared_kernel
        att.out.fill_(7.0)
        att.keep[-1].fill_(255)
        dsk.dsk_sparse_decode_attn(att.args)
        torch.cuda.synchronize()
        if not shared:
            used = -(-counts // lay.slots_per_chunk)      # of short chunks, as they are left in parts
            left, short = _partials_left(att, lay), int(used[used > 1].sum())
            assert left < short if is_long else left == short
        again = dsk.make_attn_args(q, K, V, dev_i32(start), dev_i32(length), dev_i32(counts), b, flags=flags)
        dsk.dsk_sparse_decode_attn(again.args)
        torch.cuda.synchronize()
        out, lse = _want(q, K, V, start, length, counts, Hq // H)
        # 32-bit sums of some thousand products and softmax terms: a few 1e-6 of the largest output
        assert rel_err(att.out.cpu().numpy(), out) <= 1e-5
        got = att.lse.cpu().numpy()
        np.testing.assert_allclose(got, lse, rtol=0, atol=1e-5)           # -inf where nothing is selected
        assert torch.equal(att.out.bfloat16(), att.out_bf16)
        assert torch.equal(att.out, again.out) and torch.equal(att.lse, again.lse)


def _spans_in_and_outside_the_cache(b, B, Hq, Hkv, k, shared, kernel):
    """kernel: the one that is to run, "8" and "16" the one for short chunks of so many slots."""
    import paper_2602_03184_amd as dsk
    rng = np.random.default_rng([b, B, Hq, k])
    g = torch.Generator(device="cuda")
    g.manual_seed(b)
    L, H = 1500, Hkv if shared else Hq
    K, V = (torch.randn(Hkv, L, 128, generator=g, device="cuda").bfloat16() for _ in range(2))
    q = torch.randn(B, Hq, 128, generator=g, device="cuda").bfloat16()
    counts = rng.integers(1, k + 1, size=(B, H))
    counts[0, 0], counts[0, -1] = k, 0
    start, length = _lists(rng, B, H, k, b, L, counts)
    edges = np.array([1, 2, 4, 5, 7, 8, 15, 16, 17, 31, 32, 33, 48, 49, 63, 64, b - 1, b])
    length[:, :, ::2] = rng.choice(edges[edges <= b], size=length[:, :, ::2].shape)
    start[:, :, 1::4] = L - length[:, :, 1::4]                             # ends with the cache
    bad = (start.copy(), length.copy())
    if k > 8:
        bad[0][:, :, 3], bad[0][:, :, 6] = L - length[:, :, 3] + 1, -1     # leave the cache: skipped
        bad[1][:, :, 7] = 0
        keep = np.array([j for j in range(k) if j not in (3, 6, 7)])
    else:
        keep = np.arange(k)
    n_kept = np.array([[int((keep < counts[s, h]).sum()) for h in range(H)] for s in range(B)])
    args = dsk.make_attn_args(q, K, V, dev_i32(bad[0]), dev_i32(bad[1]), dev_i32(counts), b,
                              flags=dsk.DSK_ATTN_SHARED_SELECTION if shared else 0)
    args.keep[-1].fill_(255)
    dsk.dsk_sparse_decode_attn(args.args)
    torch.cuda.synchronize()
    lay = dsk.dsk_attn_partials_layout(args.args)
    if kernel == "shared":
        assert lay.slots_per_chunk not in (8, 16)
    else:                                                                  # the long lists' kernel leaves fewer partials
        used = -(-counts // lay.slots_per_chunk) * (Hq // H)
        left, short = _partials_left(args, lay), int(used[used > Hq // H].sum())
        assert left < short if kernel == "long" else left == short
        assert kernel == "long" or lay.slots_per_chunk == int(kernel)
    want, want_lse = _want(q, K, V, start[:, :, keep], length[:, :, keep], n_kept, Hq // H)
    assert rel_err(args.out.cpu().numpy(), want) <= 1e-5                   # sums of 32 bits
    np.testing.assert_allclose(args.lse.cpu().numpy(), want_lse, rtol=0, atol=1e-5)   # -inf where nothing is selected


@pytest.mark.parametrize("b", [33, 48, 64, 65, 100, 127, 128])
@pytest.mark.parametrize("B,Hq,Hkv,k,shared,large", [(2, 6, 2, 21, False, False), (1, 28, 4, 8, False, False), (3, 8, 8, 9, False, False),
                                                     (2, 8, 2, 17, True, False), (16, 16, 4, 8, False, False), (16, 16, 4, 16, False, True),
                                                     (9, 19, 1, 21, False, True),
                                                     (12, 40, 8, 12, True, True), (33, 16, 16, 7, False, True)])
def test_slots_of_more_than_32_rows(b, B, Hq, Hkv, k, shared, large):
    """Slots around the 16 and 32 rows that are folded first, and of the rows behind them; launches of up to 256 workgroups of 8
    slots and of more, where slots of up to 127 rows, and of shared lists, go two to a wavefront."""
    assert (B * Hq * -(-k // 8) > 256) == large
    _spans_in_and_outside_the_cache(b, B, Hq, Hkv, k, shared, "8")


@pytest.mark.parametrize("b", [1, 5, 8])
@pytest.mark.parametrize("B,Hq,Hkv,k,shared,kernel", [(1, 4, 2, 21, False, "16"), (24, 32, 8, 31, False, "8"), (8, 32, 8, 67, False, "long"),
                                                      (4, 8, 8, 600, False, "long"), (8, 32, 8, 99, True, "shared"),
                                                      (8, 16, 2, 203, True, "shared"), (16, 4, 2, 131, True, "shared")])
def test_slots_of_up_to_8_rows(b, B, Hq, Hkv, k, shared, kernel):
    """Two slots in a wavefront's 16 rows: odd numbers of them, skipped ones in between; workgroups of 8 and 16 slots, the kernels
    for long and for shared lists with 2, 4 and 8 heads a tile."""
    _spans_in_and_outside_the_cache(b, B, Hq, Hkv, k, shared, kernel)


def test_long_lists_skip_spans_outside_the_cache():
    """Slots whose span leaves the cache, or is empty, add nothing; a caller that merges itself keeps its short chunks."""
    import paper_2602_03184_amd as dsk
    B, Hq, Hkv, k, b, L = 8, 32, 8, 64, 16, 1000
    rng = np.random.default_rng(5)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    K, V = (torch.randn(Hkv, L, 128, generator=g, device="cuda").bfloat16() for _ in range(2))
    q = torch.randn(B, Hq, 128, generator=g, device="cuda").bfloat16()
    counts = np.full((B, Hq), k)
    start, length = _lists(rng, B, Hq, k, b, L, counts)
    keep = rng.random((B, Hq, k)) < 0.7
    keep[0, 0] = False                                             # a head with nothing left
    bad_start = np.where(keep, start, rng.choice([-1, L - 1, L, 2 ** 30], size=start.shape)).astype(np.int32)
    bad_len = np.where(keep | (bad_start != L - 1), length, 2).astype(np.int32)
    att = dsk.make_attn_args(q, K, V, dev_i32(bad_start), dev_i32(bad_len), dev_i32(counts), b)
    att.keep[-1].fill_(255)
    dsk.dsk_sparse_decode_attn(att.args)
    torch.cuda.synchronize()
    cut = np.zeros((B, Hq), np.int64)
    s2, l2 = np.zeros_like(start), np.zeros_like(length)
    for s in range(B):
        for h in range(Hq):
            n = cut[s, h] = int(keep[s, h].sum())
            s2[s, h, :n], l2[s, h, :n] = start[s, h][keep[s, h]], length[s, h][keep[s, h]]
    out, lse = _want(q, K, V, s2, l2, cut, 1)
    assert rel_err(att.out.cpu().numpy(), out) <= 1e-5
    assert np.isinf(att.lse.cpu().numpy()[0, 0]) and float(att.out[0, 0].abs().max()) == 0.0
    assert _partials_left(att, dsk.dsk_attn_partials_layout(att.args)) == 0                          # one chunk a list
    part = dsk.make_attn_args(q, K, V, dev_i32(start), dev_i32(length), dev_i32(counts), b, flags=dsk.DSK_ATTN_PARTIALS_ONLY)
    assert dsk.dsk_attn_partials_layout(part.args).nchunks > 1
    assert part.args.workspace_bytes == att.args.workspace_bytes


@pytest.mark.parametrize("wide", ["K", "V", "KV"])
@pytest.mark.parametrize("b", [16, 32])
def test_token_strides_of_any_size(wide, b):
    """K and V whose rows lie 2^24 elements and more apart, or as far apart as each likes, per head and shared: the same rows
    as in a cache without gaps, the partials where the layout says whatever the strides."""
    import paper_2602_03184_amd as dsk
    B, Hq, Hkv, k, L = 8, 28, 4, 100, 48
    rng = np.random.default_rng(b)
    g = torch.Generator(device="cuda")
    g.manual_seed(b)
    K, V = (torch.randn(Hkv, L, 128, generator=g, device="cuda").bfloat16() for _ in range(2))
    q = torch.randn(B, Hq, 128, generator=g, device="cuda").bfloat16()

    def spread(x, stride):                                         # 1.6 GB for 2^24 + 8
        y = torch.empty((L - 1) * stride + Hkv * 128, dtype=x.dtype, device="cuda").as_strided((Hkv, L, 128), (128, stride, 1))
        y.copy_(x)
        return y
    Kw = spread(K, (1 << 24) + 8 if "K" in wide else 128 * Hkv + 8)
    Vw = spread(V, (1 << 24) + 8 if "V" in wide else 128 * Hkv + 64)
    for shared in (False, True):
        H = Hkv if shared else Hq
        counts = np.minimum(k, rng.integers(0, 2 * k, size=(B, H)))
        counts.flat[0] = k
        start, length = _lists(rng, B, H, k, b, L, counts)
        flags = dsk.DSK_ATTN_SHARED_SELECTION if shared else 0
        args = (dev_i32(start), dev_i32(length), dev_i32(counts), b)
        att = dsk.sparse_decode_attn(q, Kw, Vw, *args, flags=flags)
        near, far = (dsk.make_attn_args(q, x, y, *args, flags=flags | dsk.DSK_ATTN_PARTIALS_ONLY) for x, y in ((K, V), (Kw, Vw)))
        for p in (near, far):
            p.keep[-1].fill_(255)
            dsk.dsk_sparse_decode_attn(p.args)
        torch.cuda.synchronize()
        out, lse = _want(q, K, V, start, length, counts, Hq // H)
        assert rel_err(att.out.cpu().numpy(), out) <= 1e-5          # as in test_long_lists
        np.testing.assert_allclose(att.lse.cpu().numpy(), lse, rtol=0, atol=1e-5)
        assert torch.equal(near.keep[-1], far.keep[-1])             # same chunks, same sums


# (B, Hq, Hkv, k): chunks of the merged call (4), two where that call needs no merge, one slot more than the chunks divide
@pytest.mark.parametrize("B,Hq,Hkv,k", [(8, 32, 8, 128), (16, 64, 16, 64), (8, 28, 4, 129)])
def test_partials_of_shared_lists(B, Hq, Hkv, k):
    """Partials of a shared list, merged on the host by the documented formula, against the call that merges them."""
    import paper_2602_03184_amd as dsk
    rng = np.random.default_rng([B, Hq, k])
    g = torch.Generator(device="cuda")
    g.manual_seed(k)
    L, b = 2001, 16
    K, V = (torch.randn(Hkv, L, 128, generator=g, device="cuda").bfloat16() for _ in range(2))
    q = torch.randn(B, Hq, 128, generator=g, device="cuda").bfloat16()
    counts = np.full((B, Hkv), k)
    start, length = _lists(rng, B, Hkv, k, b, L, counts)
    full, part = (dsk.make_attn_args(q, K, V, dev_i32(start), dev_i32(length), dev_i32(counts), b,
                                     flags=dsk.DSK_ATTN_SHARED_SELECTION | f) for f in (0, dsk.DSK_ATTN_PARTIALS_ONLY))
    dsk.dsk_sparse_decode_attn(full.args)
    dsk.dsk_sparse_decode_attn(part.args)
    torch.cuda.synchronize()
    lay = dsk.dsk_attn_partials_layout(part.args)
    assert lay.nchunks == -(-k // lay.slots_per_chunk) and lay.nchunks >= 2
    assert part.args.workspace_bytes == full.args.workspace_bytes
    raw = part.keep[-1].view(torch.uint8).cpu().numpy()
    n = B * Hq * lay.nchunks
    ml = raw[lay.ml_offset: lay.ml_offset + n * 8].view(np.float32).reshape(B, Hq, lay.nchunks, 2).astype(np.float64)
    acc = raw[lay.acc_offset: lay.acc_offset + n * 512].view(np.float32).reshape(B, Hq, lay.nchunks, 128).astype(np.float64)
    w = np.exp2(ml[..., 0] - ml[..., 0].max(-1, keepdims=True))
    out = (acc * w[..., None]).sum(2) / (ml[..., 1] * w).sum(2)[..., None]
    assert rel_err(full.out.cpu().numpy(), out) <= 1e-5        # 32-bit sums in two orders, as in test_long_lists


# (B, Hq, Hkv, k, b, shared): chunks of 16, 8 and 8 slots a head; a list that a group shares in short chunks and, from 3072
# slots on, in two and in more chunks
SHORT_COUNTS = [(2, 8, 2, 50, 16, False), (8, 32, 8, 128, 16, False), (1, 8, 8, 20, 64, False), (2, 8, 2, 50, 32, True),
                (8, 32, 8, 128, 16, True), (16, 64, 16, 64, 16, True), (8, 28, 4, 129, 32, True)]


@pytest.mark.parametrize("B,Hq,Hkv,k,b,shared", SHORT_COUNTS)
def test_partials_of_lists_that_fit_one_chunk(B, Hq, Hkv, k, b, shared):
    """Every list with a slot leaves its partials where the layout says, also one that fits its first chunk: merged by the
    documented formula they are the merged call's result."""
    import paper_2602_03184_amd as dsk
    rng = np.random.default_rng([B, Hq, k, b])
    g = torch.Generator(device="cuda")
    g.manual_seed(k)
    L = 2001
    K, V = (torch.randn(Hkv, L, 128, generator=g, device="cuda").bfloat16() for _ in range(2))
    q = torch.randn(B, Hq, 128, generator=g, device="cuda").bfloat16()
    H = Hkv if shared else Hq
    flags = dsk.DSK_ATTN_SHARED_SELECTION if shared else 0
    counts = np.full((B, H), k)
    start, length = _lists(rng, B, H, k, b, L, counts)
    cnt = dev_i32(counts)
    full, part = (dsk.make_attn_args(q, K, V, dev_i32(start), dev_i32(length), cnt, b, flags=flags | f)
                  for f in (0, dsk.DSK_ATTN_PARTIALS_ONLY))
    lay = dsk.dsk_attn_partials_layout(part.args)
    per = lay.slots_per_chunk
    assert lay.nchunks > 1 and lay.nchunks * per >= k
    some = np.array([1, per, 0, per + 1, per - 1, k, 2, k + 3])
    counts = some[np.arange(B * H) % len(some)].reshape(B, H)
    cnt.copy_(dev_i32(counts))
    part.keep[-1].fill_(255)                                       # NaN wherever no partial is written
    dsk.dsk_sparse_decode_attn(full.args)
    dsk.dsk_sparse_decode_attn(part.args)
    torch.cuda.synchronize()
    raw = part.keep[-1].view(torch.uint8).cpu().numpy()
    n = B * Hq * lay.nchunks
    ml = raw[lay.ml_offset: lay.ml_offset + n * 8].view(np.float32).reshape(B, Hq, lay.nchunks, 2).astype(np.float64)
    acc = raw[lay.acc_offset: lay.acc_offset + n * 512].view(np.float32).reshape(B, Hq, lay.nchunks, 128).astype(np.float64)
    out, lse = full.out.cpu().numpy(), full.lse.cpu().numpy()
    for s in range(B):
        for h in range(Hq):
            c = min(int(counts[s, h // (Hq // H)]), k)
            used = -(-c // per)
            assert np.isnan(ml[s, h, used:]).all() and np.isnan(acc[s, h, used:]).all()
            if c == 0:
                assert float(part.out[s, h].abs().max()) == 0.0 and float(part.lse[s, h]) == -np.inf
                continue
            m, l = ml[s, h, :used].T
            w = np.exp2(m - m.max())
            # 32-bit sums in two orders, as in test_long_lists
            assert rel_err(out[s, h], (acc[s, h, :used] * w[:, None]).sum(0) / (l * w).sum()) <= 1e-5
            assert abs(lse[s, h] - math.log(2.0) * (m.max() + math.log2((l * w).sum()))) <= 1e-5
            if used == 1:
                assert rel_err(part.out[s, h].cpu().numpy(), out[s, h]) <= 1e-5
                assert abs(float(part.lse[s, h]) - lse[s, h]) <= 1e-5


# short chunks of one and of several, long lists whole and in chunks, slots of more than 32 rows in small and in large launches;
# shared lists in tiles of 2, 4 and 8 heads
LOGIT_LISTS = [(1, 4, 2, 7, 8, False), (2, 8, 2, 50, 16, False), (2, 8, 2, 50, 32, False), (8, 32, 8, 65, 8, False),
               (8, 32, 8, 33, 16, False), (2, 32, 8, 163, 32, False), (1, 40, 40, 245, 16, False), (2, 8, 2, 5, 64, False),
               (1, 28, 4, 40, 64, False), (3, 28, 4, 61, 40, False), (8, 32, 8, 33, 64, False), (8, 16, 8, 203, 8, True),
               (8, 32, 8, 128, 16, True), (8, 56, 8, 128, 32, True)]


@pytest.mark.parametrize("B,Hq,Hkv,k,b,shared", LOGIT_LISTS)
@pytest.mark.parametrize("scale,size", [(1e6, 1.0), (1e9, 1.0), (1e12, 1.0), (0.0, 2e5)])
def test_logits_of_any_size(B, Hq, Hkv, k, b, shared, scale, size):
    """Logits up to 1e14, far beyond where neighbours of 32 bits lie one apart: all the weight is on the best row of a list
    (rows that are well apart), on every kernel."""
    import paper_2602_03184_amd as dsk
    rng = np.random.default_rng([B, Hq, k, b])
    g = torch.Generator(device="cuda")
    g.manual_seed(k + b)
    L, H, G = 3001, Hkv if shared else Hq, Hq // Hkv
    K, V = (torch.randn(Hkv, L, 128, generator=g, device="cuda").bfloat16() for _ in range(2))
    K, q = (K.float() * size).bfloat16(), (torch.randn(B, Hq, 128, generator=g, device="cuda") * size).bfloat16()
    counts = np.full((B, H), k)
    start, length = _lists(rng, B, H, k, b, L, counts)
    att = dsk.make_attn_args(q, K, V, dev_i32(start), dev_i32(length), dev_i32(counts), b, scale=scale,
                             flags=dsk.DSK_ATTN_SHARED_SELECTION if shared else 0)
    dsk.dsk_sparse_decode_attn(att.args)
    torch.cuda.synchronize()
    out, lse = att.out.cpu().numpy(), att.lse.cpu().numpy()
    by = scale or 1.0 / math.sqrt(128.0)
    Kd, qd, checked = K.double(), q.double(), 0
    heads = rng.permutation(B * Hq)[:32]
    for s, h in zip(heads // Hq, heads % Hq):
        at = h // G if shared else h
        rows = np.unique(np.concatenate([np.arange(a, a + n) for a, n in zip(start[s, at], length[s, at])]))
        z = (Kd[h // G][torch.from_numpy(rows).cuda()] @ qd[s, h]).cpu().numpy()
        first, second = np.sort(z)[::-1][:2]
        # a dot is a sum of 128 products of some size^2 in 32 bits, wrong by some 1e-5 size^2 at most
        if (first - second) * by < 200.0 or first - second < 1e-2 * size * size:
            continue
        checked += 1
        times = sum(int(a <= rows[z.argmax()] < a + n) for a, n in zip(start[s, at], length[s, at]))
        want = V[h // G, int(rows[z.argmax()])].float().cpu().numpy()
        assert rel_err(out[s, h], want) <= 1e-6                    # weights of 1 and 0; the same row in several slots
        assert abs(lse[s, h] - (first * by + math.log(times))) <= 1e-5 * abs(first * by)
    assert checked >= len(heads) // 2


# chunks a list in several wavefronts: short chunks, long lists, shared lists in tiles of 4 and 8 heads, slots of two tiles; slots of
# which a wavefront takes two at a time (an odd number of them), or which lie in one or two to a wavefront beyond 32 rows
@pytest.mark.parametrize("B,Hq,Hkv,k,b,shared", [(2, 8, 2, 50, 16, False), (8, 32, 8, 128, 16, False), (8, 32, 8, 128, 32, False),
                                                 (8, 32, 8, 128, 16, True), (8, 56, 8, 128, 32, True), (2, 8, 2, 51, 8, False),
                                                 (12, 32, 8, 35, 8, False), (8, 32, 8, 121, 8, False), (8, 32, 8, 121, 8, True),
                                                 (2, 8, 2, 51, 64, False), (8, 32, 8, 121, 64, False)])
def test_values_that_are_not_finite_stay_where_they_are(B, Hq, Hkv, k, b, shared):
    """A NaN in a query, a row of K or a row of V, or an infinity in V, shows in the outputs that depend on it and in no other:
    not in the other heads of a group, whose logits share matrix products, nor in other lists or channels.  Where a logit is
    NaN no sum of weights is above zero and the result is that of an empty list, on every kernel."""
    import paper_2602_03184_amd as dsk
    rng = np.random.default_rng([B, Hq, k, b])
    g = torch.Generator(device="cuda")
    g.manual_seed(b)
    L = 4001
    K, V = (torch.randn(Hkv, L, 128, generator=g, device="cuda").bfloat16() for _ in range(2))
    q = torch.randn(B, Hq, 128, generator=g, device="cuda").bfloat16()
    H, G = (Hkv if shared else Hq), Hq // Hkv
    counts = np.full((B, H), k)
    start, length = _lists(rng, B, H, k, b, L - 200, counts)       # the last rows are in the lists below only
    # rows L-1, L-2, L-3 as the only row of a slot and L-10 inside one
    lists = {"K": (0, 0), "V": (0, 1), "inf": (1, 0), "inside": (1, 1)}
    for (s, h), row, n, at in zip(lists.values(), (L - 1, L - 2, L - 3, L - 12), (1, 1, 1, 5), (0, k - 1, 9, 30)):
        start[s, h, at], length[s, h, at] = row, n
    out0, lse0 = _want(q, K, V, start, length, counts, G if shared else 1)
    kv = lambda h: h if shared else h // G                          # KV head of a list
    K[kv(0), L - 1, 7] = float("nan")
    V[kv(1), L - 2, 5] = float("nan")
    V[kv(0), L - 3, 9] = float("inf")
    K[kv(1), L - 10, 100] = float("nan")
    q[0, Hq - 1, 3] = float("nan")
    att = dsk.make_attn_args(q, K, V, dev_i32(start), dev_i32(length), dev_i32(counts), b,
                             flags=dsk.DSK_ATTN_SHARED_SELECTION if shared else 0)
    dsk.dsk_sparse_decode_attn(att.args)
    torch.cuda.synchronize()
    out, lse = att.out.cpu().numpy(), att.lse.cpu().numpy()
    bad, bad_lse = np.zeros(out.shape, bool), np.zeros(lse.shape, bool)

    def heads(name):
        s, h = lists[name]
        return s, slice(h * G, (h + 1) * G) if shared else h
    for name in ("K", "inside"):
        bad[heads(name)], bad_lse[heads(name)] = True, True
    bad[heads("V") + (5,)] = True
    bad[heads("inf") + (9,)] = True
    bad[0, Hq - 1], bad_lse[0, Hq - 1] = True, True
    empty = np.broadcast_to(bad_lse[..., None], out.shape)
    np.testing.assert_array_equal(~np.isfinite(out), bad & ~empty)
    np.testing.assert_array_equal(lse == -np.inf, bad_lse)
    assert not out[empty].any()
    assert rel_err(out[~bad], out0[~bad]) <= 1e-5                  # as in test_long_lists
    np.testing.assert_allclose(lse[~bad_lse], lse0[~bad_lse], rtol=0, atol=1e-5)
