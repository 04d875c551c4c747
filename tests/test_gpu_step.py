"""GPU parity of xc_step against the oracle: loss, dZ, touched ids, updated rows."""
import numpy as np
import pytest
import torch

from oracle import astra_oracle as orc
from paper_2409_20156_amd import synth
from tests.parity import TOL, check_bf16_rows, check_rows_close, dtype_name, f64

pytestmark = pytest.mark.gpu


def _inputs(seed, B, L, d, dtype, k_p, k_h, k_r, zipf=1.0, law="uniform:1:3"):
    dev = "cuda:0"
    W = synth.make_matrix(seed, synth.TAG_W, L, d, dtype, dev)
    Z = synth.make_matrix(seed, synth.TAG_Z, B, d, dtype, dev)
    pos = synth.zipf_positives(seed, B, L, zipf, law if k_p > 1 else "one", k_p)
    Z = synth.add_positive_signal(Z, W, pos)
    Z64, W64 = f64(Z), f64(W)
    sl, _ = orc.mine_negatives(Z64, W64, k_h) if k_h else (np.zeros((B, 0), np.int32), None)
    neg, logq = orc.sample_negatives(sl, B, k_h, k_r, L, seed=seed + 17)
    return Z, W, pos, neg, logq, Z64, W64


def _run_and_check(Z, W, pos, neg, logq, Z64, W64, lr, kind):
    import paper_2409_20156_amd as xc
    name = dtype_name(Z)
    tol = TOL[name]
    dev = Z.device
    Wg = W.clone()
    out = xc.xc_step(Z, Wg, torch.tensor(pos, device=dev), torch.tensor(neg, device=dev),
                     torch.tensor(logq, device=dev), lr, kind=kind, want_rows=True)
    torch.cuda.synchronize()
    ref = orc.xc_step(Z64, W64, pos, neg, logq, lr, kind=kind, storage=name)
    loss = float(out["loss"].item())
    assert abs(loss - ref["loss"]) <= tol * abs(ref["loss"]), (loss, ref["loss"])
    floor = None
    if kind == orc.LOSS_SOFTMAX:
        # dZ_i = (sum_j p_j w_j - mean of the positives' rows) / B: two sums of size max|w_j| each, which
        # cancel when the candidates are few and the positives among them many
        floor = np.array([2.0 / Z64.shape[0] * (np.abs(W64[[l for l, _ in c]]).max() if c else 0.0)
                          for c in ref["coef"]])
    check_rows_close(out["dZ"].cpu().numpy(), ref["dZ"], tol, "dZ", floor=floor)
    nt = int(out["n_touched"].item())
    touched = out["touched"][:nt].cpu().numpy()
    assert nt == len(ref["touched"]) and (touched == ref["touched"]).all()
    rows = f64(out["W_rows"][:nt])
    new = f64(Wg)
    assert (new[touched] == rows).all()                          # W_rows_out is a copy of the stored rows
    if name == "f32":
        # the update itself must match to the float tolerance
        # ... up to the float32 rounding of the stored row itself (one ulp of w per side)
        dg, dw = rows - W64[touched], ref["W_rows"] - W64[touched]
        slack = 2.0 ** -23 * np.abs(W64[touched]).max(axis=1, keepdims=True)
        scale = np.abs(dw).max(axis=1, keepdims=True)
        assert (np.abs(dg - dw) <= 5 * tol * scale + slack).all(), "delta W"
        check_rows_close(rows, ref["W_rows"], tol, "W rows")
    else:
        check_bf16_rows(rows, ref["W_rows"], W64[touched], "W rows")
    mask = np.ones(W64.shape[0], bool)
    mask[touched] = False
    assert (new[mask] == W64[mask]).all()                        # untouched rows are bit-identical
    return out, ref


@pytest.mark.parametrize("kind", [orc.LOSS_BCE, orc.LOSS_SOFTMAX])
@pytest.mark.parametrize("B,L,d,dtype,k_p,k_h,k_r", [
    (32, 4096, 64, torch.float32, 1, 8, 16),          # Tiny
    (37, 500, 72, torch.bfloat16, 3, 5, 40),          # heavy duplicates, ragged everything
    (20, 3000, 20, torch.float32, 2, 4, 30),          # 80-byte fp32 rows
    (48, 20000, 768, torch.bfloat16, 4, 64, 256),     # config-2 row shape
    (16, 9000, 256, torch.bfloat16, 3, 50, 300),      # config-5 row shape
    (9, 2000, 2048, torch.bfloat16, 2, 8, 24),        # longest supported row
    # few pairs for the number of labels (2 P <= L): most labels have one pair and get their row updated inside
    # the gather (BCE), the others are listed for the row update kernel
    (64, 200000, 256, torch.bfloat16, 3, 50, 300),    # config-5 row shape
    (40, 150000, 768, torch.bfloat16, 4, 64, 256),
    (33, 90000, 72, torch.bfloat16, 3, 5, 40),        # ragged rows
])
def test_step_matches_oracle(B, L, d, dtype, k_p, k_h, k_r, kind):
    print("case", B, L, d, dtype, k_p, k_h, k_r, kind, flush=True)
    Z, W, pos, neg, logq, Z64, W64 = _inputs(3, B, L, d, dtype, k_p, k_h, k_r)
    lr = 0.05 if dtype == torch.bfloat16 else 0.3
    _run_and_check(Z, W, pos, neg, logq, Z64, W64, lr, kind)


def test_step_masks_positives_and_padding_and_out_of_range_ids():
    B, L, d = 4, 300, 64
    Z, W, pos, neg, logq, Z64, W64 = _inputs(5, B, L, d, torch.float32, 3, 4, 12)
    neg[0, 2] = pos[0, 0]           # a positive among the hard negatives
    neg[1, 7] = pos[1, 0]           # ... and among the random ones
    neg[2, 3] = -1
    neg[3, 5] = L + 5               # out of range: ignored, not dereferenced
    pos[3, 2] = L
    for kind in (orc.LOSS_BCE, orc.LOSS_SOFTMAX):
        _run_and_check(Z, W, pos, neg, logq, Z64, W64, 0.2, kind)


def test_step_softmax_with_two_labels_that_are_both_positive():
    # every negative is masked (it is one of the two positives): dZ_i = (p_0 - 1/2)(w_0 - w_1)/B, a difference
    # of two sums that nearly cancel, so the error is measured against the size of those sums
    B, L, d, n_neg = 177, 2, 128, 60
    W = synth.make_matrix(12, synth.TAG_W, L, d, torch.float32, "cuda:0")
    Z = synth.make_matrix(12, synth.TAG_Z, B, d, torch.float32, "cuda:0")
    Z64, W64 = f64(Z), f64(W)
    rng = np.random.default_rng(12)
    pos = np.tile(np.array([[0, 1]], dtype=np.int32), (B, 1))
    neg = rng.integers(0, L, size=(B, n_neg)).astype(np.int32)
    logq = np.log(rng.uniform(0.05, 1.0, size=(B, n_neg))).astype(np.float32)
    for kind in (orc.LOSS_SOFTMAX, orc.LOSS_BCE):
        _run_and_check(Z, W, pos, neg, logq, Z64, W64, 0.2, kind)


def test_step_shared_positive_is_summed_once_per_pair():
    B, L, d = 64, 100, 64
    Z, W, pos, neg, logq, Z64, W64 = _inputs(6, B, L, d, torch.float32, 1, 2, 6)
    pos[:, 0] = 42
    out, ref = _run_and_check(Z, W, pos, neg, logq, Z64, W64, 0.1, orc.LOSS_BCE)
    assert 42 in ref["touched"]


def test_step_without_negatives_or_without_positives():
    B, L, d = 8, 200, 64
    Z, W, pos, neg, logq, Z64, W64 = _inputs(7, B, L, d, torch.float32, 2, 3, 9)
    empty_i = np.zeros((B, 0), np.int32)
    empty_f = np.zeros((B, 0), np.float32)
    _run_and_check(Z, W, pos, empty_i, empty_f, Z64, W64, 0.1, orc.LOSS_BCE)
    _run_and_check(Z, W, empty_i, neg, logq, Z64, W64, 0.1, orc.LOSS_BCE)
    _run_and_check(Z, W, np.full((B, 2), -1, np.int32), neg, logq, Z64, W64, 0.1, orc.LOSS_SOFTMAX)


@pytest.mark.parametrize("L", [1000, 60000])              # row updates by the update kernel alone / mostly inside the gather
def test_step_is_bitwise_reproducible(L):
    import paper_2409_20156_amd as xc
    Z, W, pos, neg, logq, _, _ = _inputs(8, 40, L, 768, torch.bfloat16, 4, 16, 100)
    dev = Z.device
    res = []
    for _ in range(2):
        Wg = W.clone()
        out = xc.xc_step(Z, Wg, torch.tensor(pos, device=dev), torch.tensor(neg, device=dev),
                         torch.tensor(logq, device=dev), 0.05)
        torch.cuda.synchronize()
        res.append((out["loss"].cpu(), out["dZ"].cpu(), Wg.cpu()))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
    assert torch.equal(res[0][2].view(torch.int16), res[1][2].view(torch.int16))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_step_many_long_segments(dtype):
    """Every label is shared by 17 pairs (more than a lane group takes alone) and there are enough
    such labels that lane groups exceed their queue of shared segments: both the cooperative
    path and the in-place path of the row update are exercised, and the result is reproducible."""
    B, L, d, k_p, n = 1088, 90000, 64, 1, 1280            # 64 blocks of 17 queries with the same negatives
    Z = synth.make_matrix(8, synth.TAG_Z, B, d, dtype, "cuda:0")
    W = synth.make_matrix(8, synth.TAG_W, L, d, dtype, "cuda:0")
    blk = np.arange(B) // 17
    neg = (blk[:, None] * n + np.arange(n)[None, :]).astype(np.int32)          # < 64 * 1280 = 81920
    pos = (81920 + np.arange(B) % 5000).astype(np.int32).reshape(B, 1)         # positives elsewhere
    logq = np.full((B, n), np.log(0.5), dtype=np.float32)
    lr = 0.05 if dtype == torch.bfloat16 else 0.3
    out, ref = _run_and_check(Z, W, pos, neg, logq, f64(Z), f64(W), lr, orc.LOSS_BCE)
    assert len(ref["touched"]) == 64 * n + B
    # which long segments a workgroup shares and which a lane group sums alone is a function of the
    # data, not of timing: three runs give the same bits
    import paper_2409_20156_amd as xc
    res = []
    for _ in range(3):
        Wg = W.clone()
        xc.xc_step(Z, Wg, torch.tensor(pos, device="cuda:0"), torch.tensor(neg, device="cuda:0"),
                   torch.tensor(logq, device="cuda:0"), lr)
        torch.cuda.synchronize()
        res.append(Wg.view(torch.int16 if dtype == torch.bfloat16 else torch.int32).cpu())
    assert torch.equal(res[0], res[1]) and torch.equal(res[0], res[2])


def test_step_long_segments_beyond_the_queue_are_reproducible_and_exact():
    """307 200 labels of 17 pairs each: every lane group of the row update meets more long segments than
    it may queue for the whole workgroup, so the later ones are summed by the group alone.  Which path a
    segment takes is a function of its position only; three runs give the same bits, and sampled rows
    of both kinds match the oracle on the sub-problem of the label's 17 queries."""
    import paper_2409_20156_amd as xc
    B, L, d, n, lr = 2176, 320000, 64, 2400, 0.05             # 128 blocks of 17 queries with the same negatives
    dev = "cuda:0"
    Z = synth.make_matrix(9, synth.TAG_Z, B, d, torch.bfloat16, dev)
    W = synth.make_matrix(9, synth.TAG_W, L, d, torch.bfloat16, dev)
    blk = np.arange(B) // 17
    neg = (blk[:, None] * n + np.arange(n)[None, :]).astype(np.int32)          # < 128 * 2400 = 307200
    pos = (310000 + np.arange(B) % 5000).astype(np.int32).reshape(B, 1)
    logq = np.full((B, n), np.log(0.5), dtype=np.float32)
    tp, tn, tl = (torch.tensor(a, device=dev) for a in (pos, neg, logq))
    res = []
    for _ in range(3):
        Wg = W.clone()
        out = xc.xc_step(Z, Wg, tp, tn, tl, lr)
        torch.cuda.synchronize()
        res.append(Wg)
    assert int(out["n_touched"].item()) == 128 * n + B
    assert torch.equal(res[0].view(torch.int16), res[1].view(torch.int16))
    assert torch.equal(res[0].view(torch.int16), res[2].view(torch.int16))
    rng = np.random.default_rng(9)
    labels = np.concatenate([rng.integers(0, 200000, size=12), rng.integers(270000, 307200, size=12)])
    Z64 = f64(Z)
    for l in labels:
        qsel = np.where(blk == l // n)[0]
        rows = f64(W[int(l):int(l) + 1])
        ref = orc.xc_step(Z64[qsel], rows, np.full((len(qsel), 1), -1, np.int32),
                          np.zeros((len(qsel), 1), np.int32), logq[qsel, :1], lr * len(qsel) / B, storage="bf16")
        gsum = sum(abs(g) for c in ref["coef"] for _, g in c)
        slack = 2e-6 * lr * len(qsel) / B * gsum * np.abs(Z64[qsel]).max()
        check_bf16_rows(f64(res[0][int(l):int(l) + 1]), ref["W_rows"], rows, "row %d" % l,
                        max_mismatch_frac=3.0 / d, slack=[slack])   # one row of 64 elements: at most three one ulp off


@pytest.mark.parametrize("B,L,d,k_p,n_neg,masked", [
    (96, 8, 64, 2, 640, 0.0),         # 4 label buckets of ~15 000 pairs each: buckets streamed, not held in registers
    (96, 700, 64, 4, 300, 0.6),       # most pairs masked (-1 / out of range): they bypass the buckets
    (33, 2, 64, 1, 50, 0.0),          # the smallest label set that takes the bucket path
    (40, 4_300_000, 64, 3, 200, 0.2),  # more labels than 2047 buckets of 2048: digit-by-digit rounds
    (64, 4_194_303, 16, 2, 300, 0.1),  # 22-bit keys that just miss the split into buckets
    (50, 30_000_000, 8, 3, 500, 0.3),  # 25-bit keys: three rounds
    (20, 1, 64, 1, 30, 0.5),           # a single label
])
def test_step_sort_paths(B, L, d, k_p, n_neg, masked):
    """The pair sort behind the row update: bucket sizes far above and below a workgroup's tile,
    masked pairs, and the wide-key path, all against the oracle (touched ids exact)."""
    rng = np.random.default_rng(L + B)
    dtype = torch.float32
    Z = synth.make_matrix(21, synth.TAG_Z, B, d, dtype, "cuda:0")
    W = synth.make_matrix(21, synth.TAG_W, L, d, dtype, "cuda:0")
    pos = rng.integers(0, L, size=(B, k_p)).astype(np.int32)
    for i in range(B):                                        # distinct positives per query, -1 padded
        _, first = np.unique(pos[i], return_index=True)
        dup = np.ones(k_p, bool)
        dup[first] = False
        pos[i, dup] = -1
    neg = rng.integers(0, L, size=(B, n_neg)).astype(np.int32)
    if masked > 0:
        m = rng.random((B, n_neg)) < masked
        neg[m] = np.where(rng.random(int(m.sum())) < 0.5, -1, L + 5).astype(np.int32)
    logq = np.log(rng.uniform(0.05, 1.0, size=(B, n_neg))).astype(np.float32)
    _run_and_check(Z, W, pos, neg, logq, f64(Z), f64(W), 0.2, orc.LOSS_BCE)


@pytest.mark.parametrize("dtype,L,d", [
    (torch.float32, 3_400_000, 128),       # 1.7 GB: the gather and the update both stream the rows
    (torch.float32, 700_000, 128),         # 0.36 GB: only the update does
    (torch.bfloat16, 1_500_000, 128),      # 0.38 GB, bf16
])
def test_step_on_a_matrix_larger_than_the_last_level_cache(dtype, L, d):
    """Above 256 MB (update) and 1.5 GB (gather) the rows of W are loaded and stored with the non-temporal
    hint, in kernel instances of their own: same results."""
    B, k_p, n_neg = 48, 3, 300
    rng = np.random.default_rng(L)
    Z = synth.make_matrix(31, synth.TAG_Z, B, d, dtype, "cuda:0")
    W = synth.make_matrix(31, synth.TAG_W, L, d, dtype, "cuda:0")
    pos = np.stack([rng.choice(L, size=k_p, replace=False) for _ in range(B)]).astype(np.int32)
    neg = rng.integers(0, L, size=(B, n_neg)).astype(np.int32)
    neg[:, :40] = neg[0, :40]                                # labels shared by every query: long segments
    neg[rng.random((B, n_neg)) < 0.05] = -1
    logq = np.log(rng.uniform(0.05, 1.0, size=(B, n_neg))).astype(np.float32)
    for kind in (orc.LOSS_BCE, orc.LOSS_SOFTMAX):
        _run_and_check(Z, W, pos, neg, logq, f64(Z), f64(W), 0.2, kind)


def test_step_wide_keys_in_a_narrow_label_range():
    """25-bit keys whose labels all fall into a narrow range (and a few at the far end): most digit values of the
    upper rounds are empty and a few hold everything."""
    B, L, d, k_p, n_neg = 600, 30_000_000, 8, 2, 700
    rng = np.random.default_rng(77)
    Z = synth.make_matrix(23, synth.TAG_Z, B, d, torch.float32, "cuda:0")
    W = synth.make_matrix(23, synth.TAG_W, L, d, torch.float32, "cuda:0")
    pos = np.stack([rng.choice(100_000, size=k_p, replace=False) for _ in range(B)]).astype(np.int32) + 7_000_000
    neg = (rng.integers(0, 100_000, size=(B, n_neg)) + 7_000_000).astype(np.int32)
    neg[:, -5:] = L - 1 - np.arange(5)                       # and a few at the far end of the label range
    logq = np.log(rng.uniform(0.05, 1.0, size=(B, n_neg))).astype(np.float32)
    _run_and_check(Z, W, pos, neg, logq, f64(Z), f64(W), 0.2, orc.LOSS_BCE)


@pytest.mark.parametrize("B,n_neg,L", [
    (1, 1, 300), (31, 32, 50), (32, 31, 4096), (41, 24, 4096),                  # 2, 1023, 1024, 1025 pairs
    (32, 63, 4096), (683, 2, 4096), (64, 63, 700), (64, 63, 3000000),           # 2048, 2049, 4096 pairs; 64-bit elements
    (241, 16, 3000000), (30, 30, 3000000), (1, 4095, 40),                       # 4097 pairs; few labels
    (683, 2, 4200000), (64, 63, 4200000), (241, 16, 4200000),                   # 2049, 4096, 4097 pairs with wide keys
])
def test_step_small_pair_sort(B, n_neg, L):
    """Steps of up to 4096 pairs sort them in one workgroup: both element widths, one to four elements per thread, a last
    one partly filled, masked pairs among them; labels with one and with many pairs; and the sizes just behind that line."""
    print("case", B, n_neg, L, flush=True)
    Z, W, pos, neg, logq, Z64, W64 = _inputs(31, B, L, 8, torch.float32, 1, 0, n_neg)
    neg[0, n_neg // 2] = -1
    neg[B // 2, 0] = pos[B // 2, 0]
    for kind in (orc.LOSS_BCE, orc.LOSS_SOFTMAX):
        _run_and_check(Z, W, pos, neg, logq, Z64, W64, 0.2, kind)
