"""GPU parity of the delimiter-importance stage of dsk_compress (Alg. 1 on one layer, sampled
candidates, class weights in tenths) against the fp64 oracle."""
import math

import numpy as np
import pytest
import torch

from oracle import dynsplit_oracle as O
from workloads import make_workload
from dsk_testutil import dev_bf16, dev_i32, dev_u8

pytestmark = pytest.mark.gpu

SCORE_TOL = 2e-5      # fp32 MFMA accumulation + fp32 softmax vs fp64
EDGE_TOL = 1e-3       # a weight may differ by one tenth only this close to a rounding edge


def _run(cfg_id, **ov):
    import paper_2602_03184_amd as dsk
    wl = make_workload(cfg_id, with_kv=True, with_qwin=True, **ov)
    cfg = wl.cfg
    K = dev_bf16(wl.K)
    prior = np.full((cfg.B, cfg.n_class), 3, np.uint8)
    comp = dsk.compress(
        cu_seqlens=dev_i32(wl.cu_seqlens), max_seqlen=int(wl.seqlens.max()), Hq=cfg.Hq, K=K, V=None,
        stages=dsk.DSK_STAGE_CANDIDATES | dsk.DSK_STAGE_IMPORTANCE,
        token_ids=dev_i32(wl.token_ids), delim_ids=dev_i32(wl.delim_ids), n_class=cfg.n_class,
        M=cfg.M, W=cfg.W, R=cfg.R, alpha_imp=cfg.alpha_imp, qwin=dev_bf16(wl.qwin), class_weight_q=dev_u8(prior))
    torch.cuda.synchronize()
    assert int(comp.dev_status.item()) == 0
    return wl, comp, prior


def _check(wl, comp, prior, seqs=None):
    cfg = wl.cfg
    samp = comp.samp_pos.cpu().numpy()
    score = comp.samp_score.cpu().numpy()
    mean = comp.class_mean.cpu().numpy()
    wq = comp.class_weight_q.cpu().numpy()
    scale = 1.0 / math.sqrt(128.0)
    worst = 0.0
    for s in (range(cfg.B) if seqs is None else seqs):
        lo, hi = int(wl.cu_seqlens[s]), int(wl.cu_seqlens[s + 1])
        Kf = O.widen_bf16(wl.K[:, lo:hi])
        pos, cls = O.extract_candidates(wl.token_ids[lo:hi], wl.delim_ids)
        want_samp = O.sample_candidates(pos, cls, cfg.n_class, cfg.M, cfg.R, cfg.W, hi - lo)
        np.testing.assert_array_equal(samp[s], np.where(want_samp >= 0, want_samp + lo, -1))
        s_or = np.zeros((cfg.n_class, cfg.M))
        for c in range(cfg.n_class):
            for m in range(cfg.M):
                t = int(want_samp[c, m])
                if t < 0:
                    assert math.isnan(score[s, c, m])
                    continue
                qw = O.widen_bf16(wl.qwin[s, c * cfg.M + m])          # [W, Hq, D]
                s_or[c, m] = O.delimiter_importance(qw, Kf, t, cfg.R, cfg.alpha_imp, scale)
                err = abs(float(score[s, c, m]) - s_or[c, m])
                worst = max(worst, err)
                assert err <= SCORE_TOL, (s, c, m, t, float(score[s, c, m]), s_or[c, m])
        wq_or, mean_or, edge = O.class_weights(s_or, want_samp, cfg.alpha_imp, prior[s])
        for c in range(cfg.n_class):
            if math.isnan(mean_or[c]):
                assert math.isnan(mean[s, c]) and wq[s, c] == prior[s, c]
                continue
            assert abs(float(mean[s, c]) - mean_or[c]) <= SCORE_TOL
            if edge[c] > EDGE_TOL:
                assert int(wq[s, c]) == int(wq_or[c]), (s, c, mean_or[c])
            else:
                assert abs(int(wq[s, c]) - int(wq_or[c])) <= 1
    return worst


def test_importance_single_head_small():
    wl, comp, prior = _run(1)
    print("cfg1 worst |s_gpu - s_oracle| = %.2e" % _check(wl, comp, prior))


def test_importance_gqa4_llama_shape():
    wl, comp, prior = _run(2, seqlens=[12288])
    print("cfg2 worst = %.2e" % _check(wl, comp, prior))


def test_importance_gqa8_two_row_tiles_and_odd_window():
    wl, comp, prior = _run(2, seqlens=[6000], Hkv=4, W=5, R=100, M=3, alpha_imp=0.5)
    print("G=8 worst = %.2e" % _check(wl, comp, prior))


def test_importance_mha_ragged_batch():
    wl, comp, prior = _run(5, B=3, seqlens=[3000, 150, 5000], Hq=6, Hkv=6, M=4)
    print("MHA ragged worst = %.2e" % _check(wl, comp, prior))


def test_importance_feeds_segmentation_in_one_call():
    """All four stages in one dsk_compress call: weights estimated on the GPU drive DD-Select."""
    import paper_2602_03184_amd as dsk
    wl = make_workload(2, with_kv=True, with_qwin=True, seqlens=[8192])
    cfg = wl.cfg
    prior = np.full((1, cfg.n_class), 3, np.uint8)
    comp = dsk.compress(
        cu_seqlens=dev_i32(wl.cu_seqlens), max_seqlen=8192, Hq=cfg.Hq, K=dev_bf16(wl.K), V=None,
        stages=dsk.DSK_STAGE_ALL, token_ids=dev_i32(wl.token_ids), delim_ids=dev_i32(wl.delim_ids),
        n_class=cfg.n_class, M=cfg.M, W=cfg.W, R=cfg.R, alpha_imp=cfg.alpha_imp, qwin=dev_bf16(wl.qwin),
        class_weight_q=dev_u8(prior), C_=30, delta=15, alpha_num=5, alpha_den=10, b=16)
    torch.cuda.synchronize()
    assert int(comp.dev_status.item()) == 0
    wq = comp.class_weight_q.cpu().numpy()[0]
    pos, cls = O.extract_candidates(wl.token_ids, wl.delim_ids)
    bs = O.dd_select(8192, pos, cls, wq, 30, 15, 5, 10)     # oracle segmentation with the GPU's weights
    nb = len(bs) - 1
    assert int(comp.cu_blocks.cpu()[1]) == nb
    np.testing.assert_array_equal(comp.block_start.cpu().numpy()[: nb + 1], bs)


def test_importance_mean_over_layers():
    """Three layers (their own keys and window queries) through stage IMPORTANCE with the running
    sum: after the last call the class means and weights are those of the oracle's expectation
    over (layer, head, query); the per-layer scores of each call are still reported."""
    import paper_2602_03184_amd as dsk
    layers = [make_workload(2, with_kv=True, with_qwin=True, seqlens=[7000], M=4) for _ in range(1)]
    wl = layers[0]
    cfg = wl.cfg
    # further layers: same tokens (the positions are a property of the text), other keys and queries
    r = np.random.default_rng(77)
    from workloads import f32_to_bf16_bits
    Ks = [wl.K, wl.V, f32_to_bf16_bits(r.standard_normal(wl.K.shape, dtype=np.float32))]
    qwins = [wl.qwin, f32_to_bf16_bits(r.standard_normal(wl.qwin.shape, dtype=np.float32)),
             f32_to_bf16_bits(r.standard_normal(wl.qwin.shape, dtype=np.float32))]
    prior = np.full((1, cfg.n_class), 3, np.uint8)
    wq_dev = dev_u8(prior)
    acc = torch.zeros(1, cfg.n_class, cfg.M, dtype=torch.float32, device="cuda")
    comp = None
    per_layer = []
    for l in range(3):
        comp = dsk.compress(
            cu_seqlens=dev_i32(wl.cu_seqlens), max_seqlen=7000, Hq=cfg.Hq, K=dev_bf16(Ks[l]), V=None,
            stages=dsk.DSK_STAGE_CANDIDATES | dsk.DSK_STAGE_IMPORTANCE,
            token_ids=dev_i32(wl.token_ids), delim_ids=dev_i32(wl.delim_ids), n_class=cfg.n_class,
            M=cfg.M, W=cfg.W, R=cfg.R, alpha_imp=cfg.alpha_imp, qwin=dev_bf16(qwins[l]), class_weight_q=wq_dev,
            samp_score_sum=acc, imp_layers=l + 1)
        torch.cuda.synchronize()
        per_layer.append(comp.samp_score.cpu().numpy()[0].copy())
    samp = comp.samp_pos.cpu().numpy()[0]
    scale = 1.0 / math.sqrt(128.0)
    Kf = [O.widen_bf16(k) for k in Ks]
    s_or = np.zeros((cfg.n_class, cfg.M))
    for c in range(cfg.n_class):
        for m in range(cfg.M):
            t = int(samp[c, m])
            if t < 0:
                continue
            qs = [O.widen_bf16(qw[0, c * cfg.M + m]) for qw in qwins]
            s_or[c, m] = O.delimiter_importance_layers(qs, Kf, t, cfg.R, cfg.alpha_imp, scale)
            for l in range(3):           # each call still reports its own layer
                one = O.delimiter_importance(qs[l], Kf[l], t, cfg.R, cfg.alpha_imp, scale)
                assert abs(float(per_layer[l][c, m]) - one) <= SCORE_TOL
            assert abs(float(acc[0, c, m]) / 3.0 - s_or[c, m]) <= SCORE_TOL
    wq_or, mean_or, edge = O.class_weights(s_or, samp, cfg.alpha_imp, prior[0])
    mean = comp.class_mean.cpu().numpy()[0]
    wq = wq_dev.cpu().numpy()[0]
    for c in range(cfg.n_class):
        if math.isnan(mean_or[c]):
            assert math.isnan(mean[c]) and wq[c] == prior[0, c]
            continue
        assert abs(float(mean[c]) - mean_or[c]) <= SCORE_TOL
        if edge[c] > EDGE_TOL:
            assert int(wq[c]) == int(wq_or[c])
        else:
            assert abs(int(wq[c]) - int(wq_or[c])) <= 1


# ---------------------------------------------------------------------------------------------
# the kernel that packs the query rows, with the samples ranked by a launch in front (several
# sequences, or more than 256 samples) and by itself, and Alg. 1 at the full 128K context
# ---------------------------------------------------------------------------------------------
def test_importance_many_workgroups_gqa_batch():
    """Llama-3-8B head shape, 4 sequences of 16 classes x 8 samples: ranked by the launch in front."""
    wl, comp, prior = _run(5, B=4, seqlens=[3300, 2100, 4000, 2600])
    cfg = wl.cfg
    assert not _on_the_few_rows_kernel(cfg.B, 4000, cfg.Hq, cfg.Hkv, cfg.n_class * cfg.M, cfg.W, cfg.R)
    print("many-workgroup GQA batch worst = %.2e" % _check(wl, comp, prior))


def test_importance_many_workgroups_mha():
    """Llama2-13B head shape (40 KV heads, no grouping), one sequence: ranked by the kernel itself, four samples
    in a row tile."""
    wl, comp, prior = _run(4, seqlens=[6000])
    cfg = wl.cfg
    assert cfg.n_class * cfg.M <= 256
    assert not _on_the_few_rows_kernel(1, 6000, cfg.Hq, cfg.Hkv, cfg.n_class * cfg.M, cfg.W, cfg.R)
    print("many-workgroup MHA worst = %.2e" % _check(wl, comp, prior))


def test_importance_at_full_128k_context_both_launch_shapes():
    """Stage IMPORTANCE alone at 131072 tokens with sample positions given by the caller, spread
    over the whole context (the first and the last admissible position, the middle, tile edges),
    so that the key loop runs thousands of tiles and nearly all of them lie in the discarded
    region.  512 samples run packed, ranked by the launch in front, a 6-sample call on the kernel for few
    rows, in key ranges; a handful of samples (all 32 heads, every window query) is compared with the oracle."""
    import paper_2602_03184_amd as dsk
    from workloads import f32_to_bf16_bits
    wl = make_workload(3, with_kv=True, with_qwin=False)
    cfg = wl.cfg
    L = wl.total_tokens
    assert L == 131072
    n_class, M = 16, 32
    n_samp = n_class * M
    assert n_samp > 256 and not _on_the_few_rows_kernel(1, L, cfg.Hq, cfg.Hkv, n_samp, cfg.W, cfg.R)
    assert _on_the_few_rows_kernel(1, L, cfg.Hq, cfg.Hkv, 6, cfg.W, cfg.R)
    r = np.random.default_rng(2024)
    t_all = r.integers(cfg.R, L - cfg.W, size=n_samp).astype(np.int64)
    t_all[0] = cfg.R                      # first admissible position
    t_all[1] = L - 1 - cfg.W              # last admissible position: the window ends at the last token
    t_all[2] = L // 2                     # middle
    t_all[3] = 32 * 1000 - 1              # last key of a 32-key tile
    t_all[4] = 4096 + cfg.R               # retained region starts on a tile edge
    t_all[n_samp - 1] = 97 * 1024 + 13
    checked = [0, 1, 2, 3, 4, n_samp - 1]
    qwin_bits = f32_to_bf16_bits(r.standard_normal((1, n_samp, cfg.W, cfg.Hq, 128), dtype=np.float32))
    K = dev_bf16(wl.K)
    scale = 1.0 / math.sqrt(128.0)
    Kf = O.widen_bf16(wl.K)
    want = {j: O.delimiter_importance(O.widen_bf16(qwin_bits[0, j]), Kf, int(t_all[j]), cfg.R, cfg.alpha_imp, scale)
            for j in checked}
    del Kf

    def run(samp_idx, n_class_, M_):
        samp = torch.from_numpy(t_all[samp_idx].astype(np.int32).reshape(1, n_class_, M_)).cuda()
        qw = dev_bf16(np.ascontiguousarray(qwin_bits[:, samp_idx]))
        comp = dsk.compress(
            cu_seqlens=dev_i32(wl.cu_seqlens), max_seqlen=L, Hq=cfg.Hq, K=K, V=None,
            stages=dsk.DSK_STAGE_IMPORTANCE, n_class=n_class_, M=M_, W=cfg.W, R=cfg.R, alpha_imp=cfg.alpha_imp,
            samp_pos=samp, qwin=qw, class_weight_q=dev_u8(np.full((1, n_class_), 3, np.uint8)))
        torch.cuda.synchronize()
        assert int(comp.dev_status.item()) == 0
        return comp.samp_score.cpu().numpy().reshape(-1)

    big = run(np.arange(n_samp), n_class, M)              # packed
    assert np.isfinite(big).all() and (big >= -cfg.alpha_imp - 1e-5).all() and (big <= 1.0 + 1e-5).all()
    small = run(np.asarray(checked), 2, 3)                # few rows: the checked samples alone
    worst = 0.0
    for i, j in enumerate(checked):
        for got in (float(big[j]), float(small[i])):
            worst = max(worst, abs(got - want[j]))
            assert abs(got - want[j]) <= SCORE_TOL, (j, int(t_all[j]), got, want[j])
    print("128K importance worst |s_gpu - s_oracle| = %.2e over %d samples" % (worst, len(checked)))


# ---------------------------------------------------------------------------------------------
# stage IMPORTANCE on positions given by the caller, odd shapes (all on the kernel for few rows but the one with
# 512 rows per sample; the packed kernel's edges are in test_importance_packed_rows)
# ---------------------------------------------------------------------------------------------
@pytest.mark.parametrize(
    "B, L, Hq, Hkv, n_class, M, W, R, spread, imp_scale",
    [
        (1, 700, 1, 1, 1, 1, 1, 1, 1.0, 0.0),            # one row; the regions meet at every position
        (1, 1500, 4, 4, 3, 7, 8, 20, 1.0, 0.0),          # 8 rows per sample, regions narrower than a tile
        (1, 2100, 6, 2, 5, 3, 5, 100, 1.0, 0.0),         # 15 rows per sample
        (1, 1300, 8, 1, 2, 2, 64, 128, 1.0, 0.0),        # 512 rows per sample: a sample fills two items
        (1, 900, 2, 2, 16, 16, 2, 64, 1.0, 0.0),         # 256 samples
        (1, 900, 2, 2, 16, 17, 2, 64, 1.0, 0.0),         # 272
        (3, 1100, 4, 1, 4, 3, 8, 128, 1.0, 0.0),         # several sequences
        (270, 90, 1, 1, 1, 2, 3, 16, 1.0, 0.0),          # many sequences
        (1, 3000, 4, 1, 4, 4, 8, 128, 40.0, 0.0),        # logits of hundreds: the maximum moves often
        (1, 1200, 4, 1, 4, 4, 8, 128, 1.0, 0.5),         # a caller's logit scale
    ])
def test_importance_given_positions(B, L, Hq, Hkv, n_class, M, W, R, spread, imp_scale):
    import paper_2602_03184_amd as dsk
    from workloads import f32_to_bf16_bits
    r = np.random.default_rng(B * L + Hq + M)
    n_samp = n_class * M
    lens = np.full(B, L)
    if B > 1:
        lens[1::2] = L // 2 + 7
    cu = np.concatenate([[0], np.cumsum(lens)])
    t = np.stack([r.integers(0, n, size=n_samp) for n in lens])       # also t < R and windows cut by the end
    t[:, 0] = lens - 1                                                # no key behind the sample but its own
    if n_samp > 3:
        t[:, 1] = 0
        t[:, 2] = t[:, 3]                                             # equal positions
    samp = t + cu[:-1, None]
    if n_samp > 4:
        samp[0, 4] = -1                                               # an absent sample
    if B > 1:
        samp[B - 1] = -1                                              # a sequence without samples
    K_bits = f32_to_bf16_bits(r.standard_normal((Hkv, int(cu[-1]), 128), dtype=np.float32) * np.float32(spread))
    q_bits = f32_to_bf16_bits(r.standard_normal((B, n_samp, W, Hq, 128), dtype=np.float32))
    wq = dev_u8(np.full((B, n_class), 3, np.uint8))
    kw = dict(cu_seqlens=dev_i32(cu), max_seqlen=int(lens.max()), Hq=Hq, K=dev_bf16(K_bits), V=None,
              stages=dsk.DSK_STAGE_IMPORTANCE, n_class=n_class, M=M, W=W, R=R, alpha_imp=1.0, imp_scale=imp_scale,
              samp_pos=dev_i32(samp.reshape(B, n_class, M)), qwin=dev_bf16(q_bits), class_weight_q=wq)
    got = dsk.compress(**kw).samp_score.cpu().numpy().reshape(B, n_samp)
    again = dsk.compress(**kw).samp_score.cpu().numpy().reshape(B, n_samp)
    np.testing.assert_array_equal(got, again)                         # fixed reduction orders
    Kf = O.widen_bf16(K_bits)
    scale = imp_scale if imp_scale != 0.0 else 1.0 / math.sqrt(128.0)
    # the logits' rounding (fp32, up to |z| units) is the error of the exponentials
    tol = SCORE_TOL * max(1.0, spread / 4)
    seqs = range(B) if B < 8 else (0, 1, 2, 255, 256, B - 2, B - 1)
    for s in seqs:
        for j in (range(n_samp) if n_samp < 30 else (0, 1, 2, 3, 4, n_samp // 2, n_samp - 1)):
            if samp[s, j] < 0:
                assert math.isnan(got[s, j])
                continue
            want = O.delimiter_importance(O.widen_bf16(q_bits[s, j]), Kf[:, cu[s]: cu[s + 1]], int(t[s, j]), R, 1.0, scale)
            assert abs(float(got[s, j]) - want) <= tol, (s, j, int(t[s, j]), float(got[s, j]), want)


# ---------------------------------------------------------------------------------------------
# both kernels of the stage at the sizes where they can go wrong, against plain torch in 64 bits
# ---------------------------------------------------------------------------------------------
def _on_the_few_rows_kernel(B, L, Hq, Hkv, n, W, R):
    """The launch rule, on the keys that a calibration's first occurrences reach: a bound on the work (row tiles of
    four samples times key tiles) and on the chain of a sample with several row tiles, or a handful of rows."""
    rows = W * (Hq // Hkv)
    row_tiles, keys = -(-rows // 32), min(L, R + W + 48 * n)
    limit = 16384 if B == 1 and n <= 256 else 26000 + 300 * B
    work = -(-n // 4) * Hkv * B * row_tiles * -(-keys // 32)
    return ((work <= limit and (row_tiles == 1 or row_tiles * keys <= 1024))
            or (row_tiles == 1 and n <= 8 and n * rows <= 64))


def _score64(q, K, t, R, alpha, scale):
    """s_t of one sample: q [W, Hq, D], K [Hkv, L, D]."""
    W_, Hq, D = q.shape
    Hkv, L, _ = K.shape
    n = min(t + W_, L - 1) + 1
    qg = q.double().view(W_, Hkv, Hq // Hkv, D).permute(1, 2, 0, 3).reshape(Hkv, -1, D)
    z = (qg @ K[:, :n].double().transpose(1, 2).contiguous() * scale).view(Hkv, Hq // Hkv, W_, n)
    pos = torch.arange(n, device=K.device)
    reach = pos[None] <= t + 1 + torch.arange(W_, device=K.device)[:, None]
    p = torch.softmax(z.masked_fill(~reach, float("-inf")), -1)
    kept = p[..., max(0, t - R + 1): t + 1].sum(-1)
    lost = p[..., : max(0, t - R) + 1].sum(-1)
    return float((kept - alpha * lost).mean())


def _compare_with_64_bits(B, L, Hq, Hkv, n_class, M, W, R, positions, few, spread=1.0, imp_scale=0.0, check=40, alpha=1.0):
    import paper_2602_03184_amd as dsk
    n = n_class * M
    assert _on_the_few_rows_kernel(B, L, Hq, Hkv, n, W, R) == few
    r = np.random.default_rng(L + Hq + n)
    g = torch.Generator(device="cuda")
    g.manual_seed(L + n)
    lens = np.full(B, L)
    lens[1::2] = max(1, L // 2)
    cu = np.concatenate([[0], np.cumsum(lens)])
    t = np.stack([r.integers(0, x, size=n) for x in lens])
    t[0, : len(positions)] = positions
    samp = t + cu[:-1, None]
    if n > 4:
        samp[0, n - 1] = -1                                           # an absent sample
    K = (torch.randn(Hkv, int(cu[-1]), 128, generator=g, device="cuda") * spread).bfloat16()
    q = torch.randn(B, n, W, Hq, 128, generator=g, device="cuda").bfloat16()
    wq = dev_u8(np.full((B, n_class), 3, np.uint8))
    kw = dict(cu_seqlens=dev_i32(cu), max_seqlen=L, Hq=Hq, K=K, V=None, stages=dsk.DSK_STAGE_IMPORTANCE,
              n_class=n_class, M=M, W=W, R=R, alpha_imp=alpha, imp_scale=imp_scale,
              samp_pos=dev_i32(samp.reshape(B, n_class, M)), qwin=q, class_weight_q=wq)
    comp = dsk.compress(**kw)
    got = comp.samp_score.cpu().numpy().reshape(B, n)
    np.testing.assert_array_equal(got, dsk.compress(**kw).samp_score.cpu().numpy().reshape(B, n))
    mean = comp.class_mean.cpu().numpy()
    scale = imp_scale if imp_scale != 0.0 else 1.0 / math.sqrt(128.0)
    tol = SCORE_TOL * max(1.0, spread / 4)                            # rounding of logits of that size, as above
    for s in (range(B) if B < 8 else (0, 1, B // 2, B - 1)):
        for j in (range(n) if n <= check else sorted(set(range(len(positions))) | {n // 2, n - 2, n - 1})):
            if samp[s, j] < 0:
                assert math.isnan(got[s, j])
                continue
            want = _score64(q[s, j], K[:, cu[s]: cu[s + 1]], int(t[s, j]), R, alpha, scale)
            assert abs(float(got[s, j]) - want) <= tol, (s, j, int(t[s, j]), float(got[s, j]), want)
        # the means add the scores in sample order, in 32 bits
        np.testing.assert_allclose(mean[s], np.nanmean(got[s].reshape(n_class, M).astype(np.float64), axis=1), atol=1e-6)


@pytest.mark.parametrize(
    "B, L, Hq, Hkv, n_class, M, W, R, positions",
    [
        (1, 700, 1, 1, 1, 3, 1, 1, [0, 699]),                             # one row a sample, a group that is not full
        (1, 900, 4, 2, 2, 3, 8, 128, [0, 31, 32, 899, 891]),              # second group of two samples, windows cut
        (1, 510, 8, 1, 2, 2, 8, 64, [0, 200, 509]),                       # two row tiles a sample
        (3, 300, 2, 2, 3, 4, 8, 300, [299, 0]),                           # ragged; nothing is discarded but key 0
        (32, 100, 32, 32, 1, 4, 8, 16, [99]),                             # 1024 groups: 3 samples and 4 wavefronts
        (1, 4096, 8, 2, 2, 2, 8, 128, [4095, 4087, 2000]),                # the longest in one range
        (1, 4097, 8, 2, 2, 2, 8, 128, [4096, 2079, 2080, 2071]),          # two ranges: 2080 keys, then the rest
        (1, 20000, 4, 4, 1, 5, 8, 5000, [19999, 3991, 3992, 3999, 4000]), # five ranges, retained over two
        (2, 20000, 8, 2, 2, 1, 4, 128, [7999, 12345]),                    # two sequences over ranges of 4000
        (1, 131072, 8, 8, 2, 2, 8, 128, [131071, 70000, 4095, 200]),      # 32 ranges
        (50000, 20, 1, 1, 1, 8, 2, 4, [19, 0]),                           # more sums than statistics of a packed launch
    ])
def test_importance_few_rows(B, L, Hq, Hkv, n_class, M, W, R, positions):
    """Calls on the kernel for few query rows, whole and in key ranges."""
    _compare_with_64_bits(B, L, Hq, Hkv, n_class, M, W, R, positions, few=True, alpha=0.75)


@pytest.mark.parametrize(
    "B, L, Hq, Hkv, n_class, M, W, R, spread, imp_scale",
    [
        (1, 8300, 1, 1, 16, 16, 1, 128, 1.0, 0.0),       # 256 samples of one row: the largest ranked inside the kernel
        (1, 14000, 2, 2, 16, 17, 2, 20, 1.0, 0.0),       # 272: ranked by the launch in front; narrow regions
        (1, 8300, 6, 2, 16, 12, 5, 100, 1.0, 0.0),       # 15 rows per sample: samples straddle row tiles
        (3, 3000, 8, 8, 16, 4, 8, 128, 1.0, 0.0),        # several sequences
        (270, 180, 4, 1, 1, 2, 64, 16, 1.0, 0.0),        # more sequences than one launch plans
        (1, 3000, 4, 1, 4, 4, 16, 128, 40.0, 0.0),       # logits of hundreds: the reference moves often
        (1, 3000, 4, 1, 4, 4, 16, 128, 1.0, 0.5),        # a caller's logit scale
        (1, 500, 8, 1, 16, 40, 64, 128, 1.0, 0.0),       # 1280 items: several per thread of the plan, past the table's LDS
        (1, 3000, 1, 1, 64, 64, 1, 64, 1.0, 0.0),        # the most samples of a sequence
    ])
def test_importance_packed_rows(B, L, Hq, Hkv, n_class, M, W, R, spread, imp_scale):
    """Calls on the kernel that packs the rows, where its packing, ranking and plan have their edges."""
    n = n_class * M
    positions = [L - 1, 0, L // 3, L // 3][: min(n, 4)]
    _compare_with_64_bits(B, L, Hq, Hkv, n_class, M, W, R, positions, few=False, spread=spread, imp_scale=imp_scale)


@pytest.mark.parametrize("L", [300, 600, 1000, 1400, 1900, 2300, 4000, 9000])
def test_importance_rows_of_many_pieces(L):
    """Two groups of query rows, cut into pieces of four stages: 2 to 37 pieces a row for the finishing kernel."""
    _compare_with_64_bits(1, L, 8, 1, 2, 2, 16, 64, [L - 17, L - 18, L - 40], few=False)


def test_importance_ranks_positions_beyond_19_bits():
    """A sequence of more than 2^19 tokens: the sort keys leave out the lowest bit of a position, so neighbours
    tie and an item's length counts from the later one."""
    L = 600001
    positions = [L - 1, L - 2, L - 10, 524288, 524289, 524287, 300, 64 * 9000 + 55]
    _compare_with_64_bits(1, L, 1, 1, 1, 8, 64, 128, positions, few=False)


@pytest.mark.parametrize("B, L, Hkv, n_class, M, few", [(2, 400, 2, 4, 2, True), (1, 30000, 2, 4, 2, True),
                                                        (1, 9000, 2, 16, 12, False), (3, 3000, 8, 16, 4, False)])
def test_importance_in_a_graph(B, L, Hkv, n_class, M, few):
    """The stage recorded once and replayed on other queries, with eager calls on the same workspace in between."""
    import paper_2602_03184_amd as dsk
    n, W, R = n_class * M, 8, 128
    assert _on_the_few_rows_kernel(B, L, Hkv, Hkv, n, W, R) == few
    g = torch.Generator(device="cuda")
    g.manual_seed(L)
    K = torch.randn(Hkv, B * L, 128, generator=g, device="cuda").bfloat16()
    qs = [torch.randn(B, n, W, Hkv, 128, generator=g, device="cuda").bfloat16() for _ in range(3)]
    t = torch.randint(R, L - W, (B, n), generator=g, device="cuda", dtype=torch.int32)
    samp = (t + torch.arange(0, B * L, L, device="cuda", dtype=torch.int32)[:, None]).view(B, n_class, M).contiguous()
    q = qs[0].clone()
    comp = dsk.compress(cu_seqlens=dev_i32(np.arange(B + 1) * L), max_seqlen=L, Hq=Hkv, K=K, V=None,
                        stages=dsk.DSK_STAGE_IMPORTANCE, n_class=n_class, M=M, W=W, R=R, alpha_imp=1.0, samp_pos=samp,
                        qwin=q, class_weight_q=dev_u8(np.full((B, n_class), 3, np.uint8)))
    want = []
    for x in qs:
        q.copy_(x)
        dsk.dsk_compress(comp.args)
        want.append((comp.samp_score.clone(), comp.class_mean.clone(), comp.class_weight_q.clone()))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        dsk.dsk_compress(comp.args)
    for x, (score, mean, weight) in [(qs[i], want[i]) for i in (0, 1, 2, 0)]:
        q.copy_(x)
        comp.samp_score.fill_(7.0)
        comp.class_mean.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(comp.samp_score, score) and torch.equal(comp.class_mean, mean)
        assert torch.equal(comp.class_weight_q, weight)
        dsk.dsk_compress(comp.args)
