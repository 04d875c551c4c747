"""Searches of up to 2048 fp32 queries find the groups that can hold an answer with 16-bit products; what they return is the fp32
search's, bit for bit (the general kernel's, forced), whatever the rows are: also where the 16-bit maxima do not settle a query
and the fp32 kernels take it."""
import pytest
import torch

from paper_2409_20156_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(monkeypatch, Z, W, k):
    """A search from scratch, bit for bit the fp32 kernels'.  Returns what its workspace says of the route, (many, few): 1 if the fp32 kernels
    had to take some query tile of a sweep on fp16 copies, or some query of 16-bit maxima; 0 if none; -1 if there was no such search."""
    import paper_2409_20156_amd as xc
    ws = torch.empty(xc.mine_workspace(Z.shape[0], W.shape[0], Z.shape[1], k, xc.XC_F32), dtype=torch.uint8, device=DEV)
    ws[:256].fill_(0xff)
    ids, sc = (t.clone() for t in xc.mine_negatives(Z, W, k, want_scores=True, workspace=ws))
    words = ws[:256].view(torch.int32).tolist()
    monkeypatch.setenv("XC_MINE_GENERAL", "1")
    want, want_sc = xc.mine_negatives(Z, W, k, want_scores=True)
    monkeypatch.delenv("XC_MINE_GENERAL")
    assert torch.equal(ids, want)
    assert torch.equal(sc.view(torch.int32), want_sc.view(torch.int32))
    return words[0], words[32] if Z.shape[0] <= 2048 else -1          # (of more queries the word is a tile's)


def _inputs(Zq, L, d):
    return (synth.make_matrix(81, synth.TAG_Z, Zq, d, torch.float32, DEV), synth.make_matrix(81, synth.TAG_W, L, d, torch.float32, DEV))


@pytest.mark.parametrize("Zq,L,d,k", [
    (17, 10000003, 4, 5), (32, 1400001, 28, 100),   # one block of 32 queries; a step of seven chunks, of one
    (33, 700003, 32, 128), (64, 600001, 36, 7),     # four blocks of 16
    (65, 50021, 300, 32), (128, 15021, 768, 20),    # eight; a query block that fits LDS with four
    (17, 4096, 4, 5), (100, 20000, 256, 20),        # too few products: the fp32 kernels
    (129, 2100001, 8, 100),                         # groups of 32 labels
    (200, 130, 64, 128),                            # fewer groups than k
    (513, 30011, 100, 50), (1025, 20001, 300, 32),  # 256 threads per query at the end
])
def test_sizes(monkeypatch, Zq, L, d, k):
    many, few = _check(monkeypatch, *_inputs(Zq, L, d), k)
    fp32 = (Zq, L) in ((17, 4096), (100, 20000), (200, 130))
    assert (many, few) == (-1, -1 if fp32 else 0)


@pytest.mark.parametrize("Zq,L,d,k", [(64, 50021, 768, 5), (1000, 50021, 300, 32), (2560, 40011, 128, 32), (2560, 40011, 320, 32)])
@pytest.mark.parametrize("scale", [1e-12, 1e-6, 1e-3, 37.0, 3e4, 1e8, 1e14])
def test_scale_of_the_rows_does_not_matter(monkeypatch, Zq, L, d, k, scale):
    """fp16's range is brought to W's, whatever that is: no query is left to the fp32 kernels.  Most of the sixteen rows that tell it are
    ordinary ones here, the others zero, far longer or no numbers."""
    import paper_2409_20156_amd as xc
    Z, W = _inputs(Zq, L, d)
    W *= scale
    sample = [(2 * i + 1) * L // 32 for i in range(16)]
    W[sample[0]] = 0.0
    W[sample[3], 1] = float("nan")
    W[sample[7]] *= 1000.0
    ws = torch.empty(xc.mine_workspace(Zq, L, d, k, xc.XC_F32), dtype=torch.uint8, device=DEV)
    ws[:256].fill_(0xff)
    xc.mine_negatives(Z, W, k, workspace=ws)
    words = ws[:256].view(torch.int32).tolist()
    assert (words[0], words[32]) == ((-1, 0) if Zq <= 1000 else (0, -1))
    assert _check(monkeypatch, Z, W, k) == (words[0], words[32])


@pytest.mark.parametrize("Zq", [40, 600])
@pytest.mark.parametrize("rows", ["zero", "mostly zero", "equal", "pairs", "large", "tiny", "wide", "inf", "nan", "far", "common", "queries"])
def test_odd_rows(monkeypatch, Zq, rows):
    L, d, k = 20011 if Zq > 100 else 200011, 100, 32
    Z, W = _inputs(Zq, L, d)
    if rows == "zero":
        W.zero_()
    elif rows == "mostly zero":                      # all other scores negative: the answer is zero rows, the first ones
        Z.abs_()
        W.abs_().neg_()
        W[torch.arange(L, device=DEV) % 10 != 3] = 0.0
    elif rows == "equal":
        W[:] = W[5].clone()
    elif rows == "pairs":                            # rows an ulp apart, far too close for 16 bits to tell
        W[1::2] = W[0:L - 1:2]
        W[1::2, 7] = torch.nextafter(W[1::2, 7], W[1::2, 7] + 1)
    elif rows == "large":
        W[::50] *= 1e5                               # beyond fp16
    elif rows == "tiny":
        W *= 1e-9
    elif rows == "wide":
        W *= torch.logspace(-20, 10, L, device=DEV)[:, None]
    elif rows == "inf":
        W[77, 3] = float("inf")
        W[9000, 50] = -float("inf")
    elif rows == "nan":
        W[123] = float("nan")
        W[20000, 99] = float("nan")
    elif rows == "far":                              # as many large maxima side by side as there are threads
        W[:3000] *= 4.0
    elif rows == "common":                           # a part of all rows that is three times the rest
        W += 3.0 * d ** -0.5
        Z += 3.0 * d ** -0.5
    else:
        Z[0] = 0.0
        Z[1] *= 1e20
        Z[2] *= 1e-20
        Z[3, 5] = float("inf")
        Z[4, 6] = float("nan")
        Z[5] *= -1e30
        Z[6, 1:] = 0.0
    # some query is left to the fp32 kernels: ties by the thousand, rows of all sizes, a group in six beyond fp16, queries out of its range
    left = rows in ("mostly zero", "equal", "large", "wide", "queries")
    assert _check(monkeypatch, Z, W, k) == (-1, 1 if left else 0)


# ---- many queries: the sweep runs on fp16 copies, what it leaves is scored in fp32
def _thresholds(monkeypatch, Z, W, k, margin):
    """A search from scratch, then from its thresholds on the same rows; the ids and scores of the second are those of the fp32 kernels."""
    import paper_2409_20156_amd as xc
    ws = torch.empty(xc.mine_workspace(Z.shape[0], W.shape[0], Z.shape[1], k, xc.XC_F32), dtype=torch.uint8, device=DEV)
    xc.mine_negatives(Z, W, k, workspace=ws)
    W[::3] *= 0.9                                    # fewer labels than k reach some of the thresholds
    ids, sc = xc.mine_negatives(Z, W, k, want_scores=True, workspace=ws, warm_margin=margin)
    repeats = int(ws[:4].view(torch.int32).item())
    monkeypatch.setenv("XC_MINE_GENERAL", "1")
    want, want_sc = xc.mine_negatives(Z, W, k, want_scores=True)
    monkeypatch.delenv("XC_MINE_GENERAL")
    assert torch.equal(ids, want)
    assert torch.equal(sc.view(torch.int32), want_sc.view(torch.int32))
    return repeats


@pytest.mark.parametrize("Zq,L,d,k", [
    (2049, 60001, 100, 50),                         # 256-byte copies: the row kernel, items of 256 queries
    (8300, 40010, 128, 10), (4100, 30010, 252, 128),  # items of 512; 512-byte copies
    (4097, 20010, 260, 100), (3000, 20003, 772, 64),   # the general kernel; a stage that is mostly padding
    (2100, 9000, 2048, 20),                         # the longest rows
    (300, 1300000, 512, 30),                        # fewer queries: a workgroup each at the end
    (2300, 4300000, 60, 16),                        # copies of more than one chunk
    (16500, 8192, 512, 5),                          # few labels
])
def test_many_queries(monkeypatch, Zq, L, d, k):
    Z, W = _inputs(Zq, L, d)
    assert _check(monkeypatch, Z, W, k) == (0, -1)
    _thresholds(monkeypatch, Z, W, k, 0.1)


@pytest.mark.parametrize("Zq,L,d,k", [
    (2560, 40011, 128, 32), (8300, 40010, 128, 16), (4100, 30010, 252, 100),       # the row kernel, items of 256 and 512 queries
    (2560, 40011, 320, 32), (4097, 20010, 260, 100), (2300, 4300000, 60, 16),       # the general kernel; copies of more than one chunk
])
@pytest.mark.parametrize("rows", ["element", "far element", "row", "rows", "norms", "inf", "nan", "zero rows"])
def test_rows_that_stand_out_cost_their_own_tile(monkeypatch, Zq, L, d, k, rows):
    """A few rows far longer than the others, beyond fp16 or no numbers: no query tile is left to the fp32 kernels for them."""
    Z, W = _inputs(Zq, L, d)
    if rows == "element":
        W[L // 3, 5] = 2000.0
    elif rows == "far element":
        W[77, 5] = -3e9
    elif rows == "row":
        W[L // 3] *= 100.0
    elif rows == "rows":
        W[100:110] *= 30.0
        W[L - 1] *= 1000.0
    elif rows == "norms":
        W *= torch.exp(0.7 * torch.randn((L, 1), device=DEV, generator=torch.Generator(device=DEV).manual_seed(1)))
    elif rows == "inf":
        W[L // 2, 3] = float("inf")
    elif rows == "nan":
        W[L - 3] = float("nan")
    else:
        W[torch.arange(L, device=DEV) // 300 % 4 == 1] = 0.0         # whole tiles among them
    assert _check(monkeypatch, Z, W, k) == (0, -1)


@pytest.mark.parametrize("rows", ["zero", "mostly zero", "equal", "pairs", "large", "tiny", "wide", "inf", "nan", "rising", "queries"])
@pytest.mark.parametrize("Zq,L,d,k", [
    (2560, 40011, 320, 32),                         # the general kernel
    (2560, 40011, 128, 32), (8300, 40011, 252, 32),   # the row kernel, items of 256 and 512 queries
])
def test_many_queries_odd_rows(monkeypatch, Zq, L, d, k, rows):
    Z, W = _inputs(Zq, L, d)
    if rows == "zero":
        W.zero_()
    elif rows == "mostly zero":
        Z.abs_()
        W.abs_().neg_()
        W[torch.arange(L, device=DEV) % 10 != 3] = 0.0
    elif rows == "equal":
        W[:] = W[5].clone()
    elif rows == "pairs":
        W[1::2] = W[0:L - 1:2]
        W[1::2, 7] = torch.nextafter(W[1::2, 7], W[1::2, 7] + 1)
    elif rows == "large":
        W[::50] *= 1e5
    elif rows == "tiny":
        W *= 1e-9
    elif rows == "wide":
        W *= torch.logspace(-20, 2, L, device=DEV)[:, None]
    elif rows == "inf":
        W[77, 3] = float("inf")
        W[9000, 50] = -float("inf")
    elif rows == "nan":
        W[123] = float("nan")
        W[40010, 99] = float("nan")
    elif rows == "rising":                           # the scores of two query tiles rise along the label range: lists run over
        W[:, 0] = torch.linspace(0, 20, L, device=DEV)
        Z[256:512, 0] = 3.0
        Z[1000, 0] = 3.0
    else:
        Z[0] = 0.0
        Z[1] *= 1e20
        Z[300] *= 1e-20
        Z[800, 5] = float("inf")
        Z[1400, 6] = float("nan")
        Z[2500, 1:] = 0.0
    # some query tile is left to the fp32 kernels: more labels than a list holds pass, or a query is out of fp16's range
    left = rows in ("zero", "mostly zero", "equal", "large", "wide", "rising", "queries")
    assert _check(monkeypatch, Z, W, k) == (1 if left else 0, -1)


def test_thresholds_too_high_are_repeated(monkeypatch):
    Z, W = _inputs(3000, 30000, 320)
    assert _thresholds(monkeypatch, Z, W, 50, 0.0) == 1


@pytest.mark.parametrize("Zq", [300, 700, 2000])
def test_unsettled_queries_beside_settled_ones(monkeypatch, Zq):
    """Fewer than 2048 queries: the four waves of a query agree on whether its tile is given up, whatever the other queries of the tile
    find out meanwhile.  From thresholds that are too high for some queries of every tile, with a query that is no number and one
    out of fp16's range."""
    import paper_2409_20156_amd as xc
    L, d, k = 60001, 320, 32
    Z, W = _inputs(Zq, L, d)
    ws = torch.empty(xc.mine_workspace(Zq, L, d, k, xc.XC_F32), dtype=torch.uint8, device=DEV)
    for margin in (0.0, 0.02, 0.1):
        xc.mine_negatives(Z, W, k, workspace=ws)                # (the thresholds; from scratch these may come from another kernel)
        Y = Z.clone()
        Y[::37] *= 0.9                                          # these queries' scores sink below their thresholds
        Y[11, 5] = float("nan")
        Y[Zq - 5] *= 1e25
        ids, sc = (t.clone() for t in xc.mine_negatives(Y, W, k, want_scores=True, workspace=ws, warm_margin=margin))
        assert int(ws[:4].view(torch.int32).item()) == 1
        monkeypatch.setenv("XC_MINE_GENERAL", "1")
        want, want_sc = xc.mine_negatives(Y, W, k, want_scores=True)
        monkeypatch.delenv("XC_MINE_GENERAL")
        assert torch.equal(ids, want)
        assert torch.equal(sc.view(torch.int32), want_sc.view(torch.int32))


@pytest.mark.parametrize("Zq,L,d,k", [(2560, 40011, 320, 32), (4100, 30010, 128, 100)])
def test_workspace_without_room_for_copies(monkeypatch, Zq, L, d, k):
    """A byte less than the copies need: the fp32 kernels search, with the same answer, from scratch and from thresholds."""
    import paper_2409_20156_amd as xc
    Z, W = _inputs(Zq, L, d)
    need = xc.mine_workspace(Zq, L, d, k, xc.XC_F32)
    full, less = (torch.empty(n, dtype=torch.uint8, device=DEV) for n in (need, need - 1))
    for margin in (None, 0.05):
        full[:4].fill_(0xff)
        less[:4].fill_(0xff)
        ids, sc = (t.clone() for t in xc.mine_negatives(Z, W, k, want_scores=True, workspace=full, warm_margin=margin))
        l_ids, l_sc = xc.mine_negatives(Z, W, k, want_scores=True, workspace=less, warm_margin=margin)
        assert torch.equal(ids, l_ids) and torch.equal(sc.view(torch.int32), l_sc.view(torch.int32))
        assert int(full[:4].view(torch.int32).item()) == 0                              # on copies
        assert int(less[:4].view(torch.int32).item()) == (-1 if margin is None else 0)   # a search from scratch in fp32 leaves the word alone
