"""A label's score has the same bits in every search kernel: whichever route a call takes - from scratch, from thresholds,
through the 8-bit filter, the row kernel in either width or the general kernel - ids and scores are equal bit for bit, and
identical rows of W, which tie, come in the order of their ids wherever they were scored."""
import pytest
import torch

from paper_2409_20156_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _inputs(seed, Zq, L, d, dtype):
    return (synth.make_matrix(seed, synth.TAG_Z, Zq, d, dtype, DEV), synth.make_matrix(seed, synth.TAG_W, L, d, dtype, DEV))


def _cold(Z, W, k, ws=None):
    import paper_2409_20156_amd as xc
    return xc.mine_negatives(Z, W, k, want_scores=True, workspace=ws)


def _all_routes(monkeypatch, Z, W, k, forced, margins=(0.0, 0.1)):
    """The result of the default route, after comparing every other one with it."""
    import paper_2409_20156_amd as xc
    code = xc.XC_BF16 if Z.dtype == torch.bfloat16 else xc.XC_F32
    ws = torch.empty(xc.mine_workspace(Z.shape[0], W.shape[0], Z.shape[1], k, code), dtype=torch.uint8, device=DEV)
    ids, sc = (t.clone() for t in _cold(Z, W, k, ws))
    for margin in margins:                                          # from the thresholds of a search of any route
        w_ids, w_sc = xc.mine_negatives(Z, W, k, want_scores=True, workspace=ws, warm_margin=margin)
        assert torch.equal(ids, w_ids) and torch.equal(sc, w_sc), margin
        assert int(ws[:4].view(torch.int32).item()) == 0, margin    # the k-th score reaches itself: no repeat, also without a margin
        _cold(Z, W, k, ws)
    for name, value in forced:
        monkeypatch.setenv(name, value)
        f_ids, f_sc = _cold(Z, W, k)
        monkeypatch.delenv(name)
        assert torch.equal(ids, f_ids) and torch.equal(sc, f_sc), (name, value)
    return ids, sc


def _takes_few(Z, W, k, **kw):
    """Whether a call takes the search of few queries: two launches, whatever the size."""
    from paper_2409_20156_amd import binding
    binding.mine_negatives(Z, W, k, **kw)
    binding.profile_reset()
    binding.profile_enable(True)
    binding.mine_negatives(Z, W, k, **kw)
    binding.profile_enable(False)
    n = binding.profile_collect()
    binding.profile_reset()
    return n["mine_tile"][1] == 1 and n["mine_select"][1] == 1


GENERAL, NARROW, WIDE = ("XC_MINE_GENERAL", "1"), ("XC_MINE_ROWS", "narrow"), ("XC_MINE_ROWS", "wide")


@pytest.mark.parametrize("Zq,L,d,k", [(4100, 1050001, 128, 100), (4300, 1100000, 256, 50)])
def test_filter_scores_as_the_other_kernels_do(monkeypatch, Zq, L, d, k):
    """Rows before label 2^17 are scored by the row kernel, rows behind it after the filter."""
    Z, W = _inputs(71, Zq, L, d, torch.bfloat16)
    early = torch.arange(1000, device=DEV) * 131
    late = L - 1 - 701 * torch.arange(1000, device=DEV)
    W[late] = W[early]
    q = torch.arange(1000, device=DEV) * 4
    Z[q] += W[early]                                                # a query beside each pair of equal rows
    ids, sc = _all_routes(monkeypatch, Z, W, k, [NARROW, WIDE, GENERAL])
    at = ids[q].eq(early[:, None].to(torch.int32)).int().argmax(dim=1)
    assert bool((ids[q, at] == early).all())
    later = ids[q].eq(late[:, None].to(torch.int32)).int().argmax(dim=1)
    assert bool((ids[q, later] == late).all()) and bool((later == at + 1).all())
    assert torch.equal(sc[q, at], sc[q, later])


@pytest.mark.parametrize("Zq,L,d,k", [
    (1000, 50021, 300, 32),                # rows of 1200 bytes: a step of three chunks at the end
    (300, 20000, 68, 64),                  # 272 bytes: a step of one chunk
    (520, 9000, 76, 128),                  # 304 bytes: three chunks; one workgroup of 256 threads per query at the end
    (64, 30000, 768, 50),                  # two blocks of queries fit LDS
    (16, 5000, 300, 40), (17, 5001, 300, 40), (33, 5017, 256, 40),     # one, two and four blocks of 16 queries; ragged labels
    (9, 3000, 1216, 20),                   # the longest rows of which two blocks of queries fit LDS, and longer ones
    (40, 3001, 1220, 20),
    (3, 2100000, 8, 100), (20, 2100016, 8, 100),                       # groups of 32 labels
])
def test_few_queries_score_as_the_general_kernel_does_fp32(monkeypatch, Zq, L, d, k):
    Z, W = _inputs(72, Zq, L, d, torch.float32)
    n = min(Zq, 200)
    late = L - 1 - 7 * torch.arange(n, device=DEV)
    W[:n] *= 3.0                            # (the longest rows: among the best of their own query)
    W[late] = W[:n].clone()
    Z[:n] += W[:n]
    assert _takes_few(Z, W, k)
    ids, sc = _all_routes(monkeypatch, Z, W, k, [GENERAL])
    at = ids[:n].eq(torch.arange(n, device=DEV, dtype=torch.int32)[:, None]).int().argmax(dim=1)
    q = torch.arange(n, device=DEV)
    assert bool((ids[q, at + 1] == late).all()) and torch.equal(sc[q, at], sc[q, at + 1])


@pytest.mark.parametrize("Zq,L,d,k", [
    (512, 60000, 768, 5),                  # rows that the general kernel takes
    (1000, 50000, 256, 50),                # ... that the row kernel takes
    (300, 20000, 40, 64),                  # 80 bytes: a step of one chunk at the end
    (20, 3000, 1152, 20),
    (5, 2100000, 64, 100),                 # groups of 32 labels
])
def test_few_queries_score_as_the_other_kernels_do_bf16(monkeypatch, Zq, L, d, k):
    Z, W = _inputs(73, Zq, L, d, torch.bfloat16)
    forced = [GENERAL, NARROW, WIDE] if d * 2 % 128 == 0 and d * 2 <= 512 else [GENERAL]
    assert _takes_few(Z, W, k)
    _all_routes(monkeypatch, Z, W, k, forced)


@pytest.mark.parametrize("Zq,L,d,dtype,k,warm,few", [
    (96, 40000, 2304, torch.bfloat16, 100, False, True),          # up to 96 queries always
    (256, 200000, 256, torch.bfloat16, 100, False, True),         # from scratch against the row kernel
    (1000, 50000, 256, torch.bfloat16, 50, False, True),
    (256, 400000, 64, torch.bfloat16, 5, True, True),             # from thresholds: by the estimates
    (256, 4000000, 64, torch.bfloat16, 5, True, False),
    (256, 5000, 2304, torch.bfloat16, 100, False, False),         # long lists of long rows read again
    (256, 50000, 768, torch.bfloat16, 5, True, True),
    (512, 60000, 768, torch.bfloat16, 5, False, True),
    (1024, 98301, 768, torch.bfloat16, 50, False, False),         # enough tiles for the general kernel
    (2048, 24573, 2304, torch.bfloat16, 5, False, False),         # two blocks of queries in LDS only
    (1257, 118938, 256, torch.bfloat16, 100, False, True),        # more tiles than six per compute unit: by the estimates all the same
    (276, 652935, 1024, torch.bfloat16, 20, False, True),
    (643, 361318, 128, torch.bfloat16, 20, False, True),
    (690, 793300, 1024, torch.bfloat16, 20, False, False),
    (235, 1200071, 96, torch.bfloat16, 50, False, True),          # up to 256 queries from scratch
    (256, 10000000, 128, torch.bfloat16, 50, True, True),         # from thresholds, long label ranges
    (256, 100000, 768, torch.float32, 50, True, True),            # fp32 up to 256 queries
    (1024, 60000, 300, torch.float32, 32, False, True),
    (1024, 70000, 2304, torch.float32, 5, False, False),
    (264, 10771, 256, torch.float32, 20, False, True),            # too few products for 16-bit maxima, against copies
    (560, 8264, 256, torch.float32, 5, False, True),
    (910, 6435, 200, torch.float32, 20, False, True),
    (293, 4253, 768, torch.float32, 100, False, False),
])
def test_searches_take_the_faster_route(monkeypatch, Zq, L, d, dtype, k, warm, few):
    """Either side of the lines between the search of few queries and the others; the result is the same."""
    import paper_2409_20156_amd as xc
    Z, W = _inputs(74, Zq, L, d, dtype)
    code = xc.XC_BF16 if dtype == torch.bfloat16 else xc.XC_F32
    ws = torch.empty(xc.mine_workspace(Zq, L, d, k, code), dtype=torch.uint8, device=DEV)
    ids, sc = (t.clone() for t in _cold(Z, W, k, ws))
    assert _takes_few(Z, W, k, workspace=ws, warm_margin=0.1 if warm else None) == few
    monkeypatch.setenv("XC_MINE_ROWS", "narrow")                  # the other side of the line
    ids_o, sc_o = _cold(Z, W, k)
    monkeypatch.delenv("XC_MINE_ROWS")
    assert torch.equal(ids, ids_o) and torch.equal(sc, sc_o)
