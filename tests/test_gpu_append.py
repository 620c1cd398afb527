"""GPU parity of dsk_append_tokens (Sec. 4.1, incremental update during decoding): after every
append the block table, the slot map and the summaries must equal, bit for bit, what the oracle
computes from scratch on the grown sequence, and the index of the first rewritten chunk must be
the oracle's."""
import numpy as np
import pytest
import torch

from oracle import dynsplit_oracle as O
from dsk_testutil import (assert_bf16_of, bf16_bits_of, canon_zero, dev_bf16, dev_i32, dev_u8, gpu_case, oracle_means_bf16,
                          oracle_summaries)

pytestmark = pytest.mark.gpu


def _dsk():
    import paper_2602_03184_amd as dsk
    return dsk


class _Seq:
    """One sequence on the device with room to grow, its oracle-side candidates, and a
    compression of its first L0 tokens."""

    def __init__(self, K_bits, V_bits, token_ids, delim_ids, wq, L0, C, delta, a_num, a_den, b, want_vsum=False,
                 max_blocks_total=None, Hq=None, summary_mode=0):
        dsk = _dsk()
        self.dsk = dsk
        self.K_bits, self.V_bits = K_bits, V_bits
        self.tok, self.delim, self.wq = np.asarray(token_ids), np.asarray(delim_ids), np.asarray(wq)
        self.C, self.delta, self.a_num, self.a_den, self.b = C, delta, a_num, a_den, b
        self.L_cap = K_bits.shape[1]
        self.K, self.V = dev_bf16(K_bits), dev_bf16(V_bits)
        self.d_tok, self.d_delim, self.d_wq = dev_i32(self.tok), dev_i32(self.delim), dev_u8(self.wq[None])
        self.pos, self.cls = O.extract_candidates(self.tok, self.delim)
        cap = dsk.dsk_block_capacity(self.L_cap, 1, C - delta) if max_blocks_total is None else max_blocks_total
        L_first = max(L0, 1)          # an empty start is made from a one-token table emptied below
        self.comp = dsk.compress(
            cu_seqlens=dev_i32([0, L_first]), max_seqlen=L_first, Hq=Hq or K_bits.shape[0], K=self.K, V=self.V,
            stages=dsk.DSK_STAGE_CANDIDATES | dsk.DSK_STAGE_SEGMENT | dsk.DSK_STAGE_SUMMARIES,
            token_ids=self.d_tok, delim_ids=self.d_delim, n_class=len(self.delim), class_weight_q=self.d_wq,
            C_=C, delta=delta, alpha_num=a_num, alpha_den=a_den, b=b, total_tokens=L_first,
            max_cand_total=self.L_cap, max_blocks_total=cap, want_vsum=want_vsum, summary_mode=summary_mode)
        if L0 == 0:
            torch.cuda.synchronize()
            self.comp.cu_blocks.zero_()
            self.comp.block_start[:4].zero_()
            self.comp.slot_base[:4].zero_()
        self.app = dsk.make_appender(self.comp, self.K, self.V, self.d_tok, self.d_delim, self.d_wq, C_=C,
                                     delta=delta, alpha_num=a_num, alpha_den=a_den, b=b)
        self.L = L0
        torch.cuda.synchronize()
        assert int(self.comp.dev_status.item()) == 0
        self.ora = self.oracle_table(L0) if L0 > 0 else np.zeros(1, dtype=np.int64)

    def oracle_table(self, n):
        m = self.pos < n
        return O.dd_select(n, self.pos[m], self.cls[m], self.wq, self.C, self.delta, self.a_num, self.a_den)

    def append(self, n_new, check_status=True):
        L_new = self.L + n_new
        m = self.pos < L_new
        want, i0 = O.dd_select_append(self.ora, L_new, self.pos[m], self.cls[m], self.wq, self.C, self.delta,
                                      self.a_num, self.a_den)
        self.app.step(self.L, L_new)
        torch.cuda.synchronize()
        if check_status:
            assert int(self.comp.dev_status.item()) == 0
        self.L, self.ora = L_new, want
        return want, i0

    def check_tables(self, want, i0):
        nblk = len(want) - 1
        assert int(self.comp.cu_blocks.cpu()[1]) == nblk
        np.testing.assert_array_equal(self.comp.block_start.cpu().numpy()[: nblk + 1], want)
        np.testing.assert_array_equal(self.comp.slot_base.cpu().numpy()[: nblk + 1], O.slot_map(want, self.b))
        assert int(self.app.first_recomputed.item()) == i0
        # chunks before i0 are untouched, so slot_base[i0] is the same in the old and the new table
        assert int(self.app.first_stale_slot.item()) == int(O.slot_map(want, self.b)[i0])

    def check_summaries(self, want, vsum=False):
        nblk = len(want) - 1
        got = bf16_bits_of(self.comp.vsum if vsum else self.comp.ksum)[:, :nblk]
        mn, mx = oracle_summaries((self.V_bits if vsum else self.K_bits)[:, : self.L], want)
        np.testing.assert_array_equal(canon_zero(got[:, :, 0]), canon_zero(mn))
        np.testing.assert_array_equal(canon_zero(got[:, :, 1]), canon_zero(mx))


def test_decode_loop_one_token_at_a_time_then_bursts():
    case = gpu_case(1)
    wl, cfg = case.wl, case.cfg
    seq = _Seq(wl.K, wl.V, wl.token_ids, wl.delim_ids, wl.class_weight_q[0], 1000, int(wl.C[0]), int(wl.delta[0]),
               cfg.a_num, cfg.a_den, cfg.b)
    for step in range(300):
        want, i0 = seq.append(1)
        seq.check_tables(want, i0)
        if step % 60 == 59:
            seq.check_summaries(want)
    for burst in (7, 64, 500, 0, 1):
        want, i0 = seq.append(burst)
        seq.check_tables(want, i0)
        seq.check_summaries(want)
    # the grown table is the table of a compression from scratch
    np.testing.assert_array_equal(want, seq.oracle_table(seq.L))


@pytest.mark.parametrize("Hkv", [1, 5])
def test_a_range_of_more_blocks_than_the_launch_has_workgroups(Hkv):
    """Thousands of rewritten blocks in one update: a workgroup of the summaries takes several of them."""
    rng = np.random.default_rng(Hkv)
    L, C, delta = 12000, 4, 2
    tok = np.where(rng.random(L) < 0.2, rng.integers(0, 3, L), 99)
    bits = [bf16_bits_of(torch.from_numpy(rng.standard_normal((Hkv, L, 128)).astype(np.float32)).bfloat16()) for _ in range(2)]
    seq = _Seq(bits[0], bits[1], tok, [0, 1, 2], [9, 5, 7], 50, C, delta, 5, 10, 4, want_vsum=True)
    want, i0 = seq.append(L - 50)
    assert len(want) - i0 > 2048
    seq.check_tables(want, i0)
    seq.check_summaries(want)
    seq.check_summaries(want, vsum=True)


def test_append_with_gqa_heads_and_v_summaries_then_decode():
    dsk = _dsk()
    case = gpu_case(2, seqlens=[6000])
    wl, cfg = case.wl, case.cfg
    seq = _Seq(wl.K, wl.V, wl.token_ids, wl.delim_ids, wl.class_weight_q[0], 3000, int(wl.C[0]), int(wl.delta[0]),
               cfg.a_num, cfg.a_den, cfg.b, want_vsum=True, Hq=cfg.Hq)
    r = np.random.default_rng(5)
    while seq.L < 5900:
        want, i0 = seq.append(int(r.integers(1, 90)))
        seq.check_tables(want, i0)
    seq.check_summaries(want)
    seq.check_summaries(want, vsum=True)
    # selection and attention on the grown cache = those on a cache compressed from scratch
    scratch = dsk.compress(
        cu_seqlens=dev_i32([0, seq.L]), max_seqlen=seq.L, Hq=cfg.Hq, K=seq.K, V=seq.V,
        stages=dsk.DSK_STAGE_CANDIDATES | dsk.DSK_STAGE_SEGMENT | dsk.DSK_STAGE_SUMMARIES,
        token_ids=seq.d_tok, delim_ids=seq.d_delim, n_class=cfg.n_class, class_weight_q=seq.d_wq,
        C_=seq.C, delta=seq.delta, alpha_num=cfg.a_num, alpha_den=cfg.a_den, b=cfg.b, total_tokens=seq.L)
    q = dev_bf16(wl.q[0])
    a = dsk.select_topk(seq.comp, q, cfg.T)
    b_ = dsk.select_topk(scratch, q, cfg.T)
    torch.cuda.synchronize()
    for name in ("sel_slot", "sel_start", "sel_len", "sel_count"):
        assert torch.equal(getattr(a, name), getattr(b_, name)), name
    oa = dsk.sparse_decode_attn(q, seq.K, seq.V, a.sel_start, a.sel_len, a.sel_count, cfg.b)
    ob = dsk.sparse_decode_attn(q, seq.K, seq.V, b_.sel_start, b_.sel_len, b_.sel_count, cfg.b)
    torch.cuda.synchronize()
    assert torch.equal(oa.out, ob.out)


@pytest.mark.parametrize("C,delta,a_num,everywhere", [(100, 99, 10, True), (8, 0, 5, False), (1, 0, 5, False),
                                                      (14, 7, 5, False), (40, 39, 0, True)])
def test_append_edge_parameters(C, delta, a_num, everywhere):
    """C - delta = 1 with delimiters everywhere and alpha = 1 gives one-token chunks, i.e. more
    open chunks than one wavefront counts at a time; delta = 0 and C = 1 have no search range;
    alpha = 0 ignores the weights."""
    case = gpu_case(1)
    wl, cfg = case.wl, case.cfg
    L_cap = 1500
    tok = wl.token_ids[:L_cap].copy()
    wq = wl.class_weight_q[0].copy()
    if everywhere:
        tok[:] = wl.delim_ids[3]
        wq[:] = 7
    seq = _Seq(wl.K[:, :L_cap], wl.V[:, :L_cap], tok, wl.delim_ids, wq, 400, C, delta, a_num, 10, 4)
    for n_new in (1, 1, 1, 2, 3, 1, 50, 1, 1, 300, 1, 199, 1):
        want, i0 = seq.append(n_new)
        seq.check_tables(want, i0)
    seq.check_summaries(want)
    if everywhere and delta == C - 1 and a_num == 10:
        assert len(want) - 1 == seq.L - C + 1             # one-token chunks, then the last chunk of C tokens


@pytest.mark.parametrize("C", [32, 33, 64, 65, 96, 97, 200])
@pytest.mark.parametrize("mean", [False, True])
def test_append_chunk_lengths_around_the_rows_in_flight(C, mean):
    """Whole chunks of C tokens (no delimiter, delta 0) and an open one that grows: up to 32 rows at a time, or up to 96 (C up to 64)."""
    rng = np.random.default_rng(C)
    L = 6 * C + 9
    K = (rng.standard_normal((3, L, 128)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    V = K[::-1].copy()
    seq = _Seq(K, V, np.full(L, 7), [1, 2], np.array([9, 5], np.uint8), 2 * C - 3, C, 0, 5, 10, 16, want_vsum=True,
               summary_mode=int(mean))
    for n in (1, 2, 1, 33, C - 1, 1, 2 * C + 5):
        want, i0 = seq.append(n)
        seq.check_tables(want, i0)
        if not mean:
            seq.check_summaries(want)
            seq.check_summaries(want, vsum=True)
            continue
        for bits, sums in ((K, seq.comp.ksum), (V, seq.comp.vsum)):
            got = bf16_bits_of(sums)[:, : len(want) - 1]
            np.testing.assert_array_equal(got[:, :, 0], got[:, :, 1])
            assert_bf16_of(got[:, :, 0], oracle_means_bf16(bits[:, : seq.L], want, range(3)))


@pytest.mark.parametrize("mean", [False, True])
def test_append_chunks_of_more_rows_than_are_in_flight(mean):
    """Chunks of 65 to 127 tokens around C = 64, each up to its delimiter: one or two rounds of up to 96 rows, of which 16 at a
    time are left out where a block has none."""
    rng = np.random.default_rng(7)
    lens = [97, 112, 113, 127, 96, 81, 80, 65, 128 - 1, 99, 111, 126]
    ends = np.cumsum(lens)
    L = int(ends[-1]) + 40
    K = (rng.standard_normal((3, L, 128)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    tok = np.full(L, 7)
    tok[ends - 1] = 1
    seq = _Seq(K, K, tok, [1, 2], np.array([9, 5], np.uint8), 5, 64, 63, 10, 10, 16, summary_mode=int(mean))
    for n in [1, 300, 1, 150, 250, 1, 1] + [L]:
        want, i0 = seq.append(min(n, L - seq.L))
        seq.check_tables(want, i0)
        if not mean:
            seq.check_summaries(want)
            continue
        got = bf16_bits_of(seq.comp.ksum)[:, : len(want) - 1]
        np.testing.assert_array_equal(got[:, :, 0], got[:, :, 1])
        assert_bf16_of(got[:, :, 0], oracle_means_bf16(K[:, : seq.L], want, range(3)))
    assert set(np.diff(want)) >= {97, 112, 113, 127}


def test_append_from_an_empty_sequence():
    case = gpu_case(1)
    wl, cfg = case.wl, case.cfg
    seq = _Seq(wl.K[:, :600], wl.V[:, :600], wl.token_ids[:600], wl.delim_ids, wl.class_weight_q[0], 0, 24, 12,
               5, 10, 16)
    for n_new in (1, 1, 10, 24, 100, 400):
        want, i0 = seq.append(n_new)
        seq.check_tables(want, i0)
    seq.check_summaries(want)


def test_append_reports_capacity_and_table_mismatch():
    dsk = _dsk()
    case = gpu_case(1)
    wl, cfg = case.wl, case.cfg
    seq = _Seq(wl.K[:, :2000], wl.V[:, :2000], wl.token_ids[:2000], wl.delim_ids, wl.class_weight_q[0], 500, 24,
               12, 5, 10, 16, max_blocks_total=30)
    seq.append(1500, check_status=False)                  # ~83 chunks do not fit 30
    assert int(seq.comp.dev_status.item()) == dsk.DSK_ERR_CAPACITY
    assert int(seq.comp.cu_blocks.cpu()[1]) == 30
    seq.comp.dev_status.zero_()
    seq.app.step(1234, 1300, check=True)                  # the table does not end at 1234
    torch.cuda.synchronize()
    assert int(seq.comp.dev_status.item()) == dsk.DSK_ERR_SHAPE
    # host-side validation
    seq.app.args.len_new = 10
    seq.app.args.len_old = 20
    assert dsk.dsk_append_tokens(seq.app.args, check=False) == dsk.DSK_ERR_SHAPE
    seq.app.args.len_old, seq.app.args.len_new = 0, 10
    seq.app.args.delta = seq.app.args.C
    assert dsk.dsk_append_tokens(seq.app.args, check=False) == dsk.DSK_ERR_PARAM


@pytest.mark.parametrize("C, delta, share, a_num, steps", [
    (40, 39, 1.0, 10, [1, 1, 3]),            # chunks of one token: more open chunks than one ballot covers
    (700, 600, 0.05, 5, [1, 2, 400]),        # more searched tokens than the window holds
    (24, 12, 0.04, 5, [1000, 1001, 1]),      # 2 * delta + new tokens: as many as the window holds, and one more
    (24, 12, 0.04, 5, [1, 255, 256, 257]),   # full and partial rounds of window loads
])
def test_append_token_window_edges(C, delta, share, a_num, steps):
    r = np.random.default_rng(C + delta)
    L0 = 2500
    total = L0 + sum(steps)
    K = r.integers(0x3F00, 0x4000, size=(1, total, 128)).astype(np.uint16)
    tok = np.where(r.random(total) < share, r.integers(0, 3, size=total), 9)
    q = _Seq(K, K, tok, [0, 1, 2], [10, 10, 7] if share < 1.0 else [10, 10, 10], L0, C, delta, a_num, 10, 16)
    for n in steps:
        q.check_tables(*q.append(n))


@pytest.mark.parametrize("n_class, delta", [(16, 2), (64, 0), (64, 4), (64, 31), (20, 9)])
def test_append_more_classes_than_searched_positions(n_class, delta):
    """More new tokens than the window holds, so that the search classifies them itself, with fewer positions in a
    search range than there are classes: the ids and weights of the lanes without a position count too."""
    r = np.random.default_rng(n_class + delta)
    L0, new = 700, 1500
    K = r.integers(0x3F00, 0x4000, size=(1, L0 + new, 128)).astype(np.uint16)
    tok = np.where(r.random(L0 + new) < 0.5, r.integers(0, n_class, size=L0 + new), 9999)
    q = _Seq(K, K, tok, np.arange(n_class), r.integers(0, 11, size=n_class).astype(np.uint8), L0, 32, delta, 7, 10, 16)
    q.check_tables(*q.append(new))
