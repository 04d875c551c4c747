"""The 8-bit filter in front of the search of large pools over long ranges of short bf16 rows: the result has to be that
of the bf16 kernels (forced through XC_MINE_ROWS) on everything the filter can meet - rows that 8 bits describe well and
badly, rows that are no numbers, scores that rise along the label range so that its lists run over - and, on sampled
queries, that of 64-bit scores."""
import numpy as np
import pytest
import torch

from paper_2409_20156_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _search(Z, W, k, ws=None):
    import paper_2409_20156_amd as xc
    ids, sc = xc.mine_negatives(Z, W, k, want_scores=True, workspace=ws)
    torch.cuda.synchronize()
    return ids, sc


def _room(Zq, L, d, k):
    """A workspace, and the filter's state in it after a search: [tiles of 256 queries given up, 1 if switched off]."""
    import paper_2409_20156_amd as xc
    need = xc.mine_workspace(Zq, L, d, k, xc.XC_BF16)
    ws = torch.zeros(need, dtype=torch.uint8, device=DEV)
    words = 4 * ((Zq + 255) // 256 + 3)                             # the last part of the workspace
    return ws, ws[need - (words + 255) // 256 * 256:][:8].view(torch.int32)


def _same_as_bf16(monkeypatch, Z, W, k, ws=None):
    """Bit for bit: what passes the filter is scored in the bf16 kernels' order of sums."""
    ids, sc = _search(Z, W, k, ws)
    monkeypatch.setenv("XC_MINE_ROWS", "narrow")
    ids_b, sc_b = _search(Z, W, k)
    monkeypatch.delenv("XC_MINE_ROWS")
    assert torch.equal(ids, ids_b) and torch.equal(sc, sc_b)
    return ids, sc


def _check_exact(Z, W, ids, sc, k, n=24):
    """Sampled queries against 64-bit scores over all labels."""
    q = torch.linspace(0, Z.shape[0] - 1, n, device=DEV).long()
    best = None
    for r in range(0, W.shape[0], 1 << 20):
        s = Z[q].double() @ W[r:r + (1 << 20)].double().T
        v = torch.topk(s, min(k, s.shape[1]), dim=1)[0]
        best = v if best is None else torch.topk(torch.cat([best, v], 1), k, dim=1)[0]
    assert float(((sc[q].double() - best).abs() / best.abs().clamp(min=1e-3)).max()) <= 1e-5
    own = (Z[q].double()[:, None, :] * W[ids[q].long()].double()).sum(-1)
    assert float(((own - best).abs() / best.abs().clamp(min=1e-3)).max()) <= 1e-5


@pytest.mark.parametrize("Zq,L,d,k", [
    (4096, 1 << 20, 256, 50),              # the smallest it takes; whole tiles
    (4100, 1050001, 128, 100),             # ragged queries and labels
    (5000, 2300007, 256, 64),              # two chunks and a remainder
    (9001, 1100000, 128, 1),
    (4097, 1048577, 256, 128),             # one label beyond a whole tile, maximum k
])
def test_q8_matches_bf16_search(monkeypatch, Zq, L, d, k):
    print("case", Zq, L, d, k, flush=True)
    W = synth.make_matrix(41, synth.TAG_W, L, d, torch.bfloat16, DEV)
    Z = synth.make_matrix(41, synth.TAG_Z, Zq, d, torch.bfloat16, DEV)
    ids, sc = _same_as_bf16(monkeypatch, Z, W, k)
    _check_exact(Z, W, ids, sc, k)


def _base(seed=43, Zq=4300, L=1100000, d=256):
    return (synth.make_matrix(seed, synth.TAG_Z, Zq, d, torch.bfloat16, DEV),
            synth.make_matrix(seed, synth.TAG_W, L, d, torch.bfloat16, DEV))


def test_q8_uneven_rows(monkeypatch):
    """Outliers that cost their tile its resolution, rows of very different lengths, zero rows and tiles, elements near
    the ends of the range, and queries of the same kinds."""
    Z, W = _base()
    L = W.shape[0]
    W[::1000, 7] = 3.0                                              # a spike in every 16th tile
    W[200000:300000] *= torch.logspace(-3, 1.5, 100000, device=DEV)[:, None].to(torch.bfloat16)
    W[400000:420000] = 0.0
    W[500000:500064] = 1e-20
    W[600000] = 1e18
    W[L - 1] = W[5] * 4
    Z[3, 0] = 9.0
    Z[17] *= 1e-3
    Z[18] = 0.0
    Z[19] = 1e-20
    Z[20] = 1e16
    ids, sc = _same_as_bf16(monkeypatch, Z, W, 50)
    ok = torch.ones(Z.shape[0], dtype=torch.bool, device=DEV)
    ok[[18, 19, 20]] = False
    _check_exact(Z[ok], W, ids[ok], sc[ok], 50)


def test_q8_rows_that_are_no_numbers(monkeypatch):
    Z, W = _base(44)
    W[300000:300100] = float("nan")
    W[700001, 3] = float("inf")
    W[800002, 4] = -float("inf")
    Z[9, 1] = float("nan")
    Z[4200, 0] = float("inf")
    ids, _ = _same_as_bf16(monkeypatch, Z, W, 50)
    assert bool((ids[9] == -1).all())
    good = torch.arange(Z.shape[0], device=DEV) != 9
    assert not bool(((ids[good] >= 300000) & (ids[good] < 300100)).any())


def test_q8_queries_that_cannot_gain_do_not_cost_their_tile_the_filter(monkeypatch):
    """A zero query (a padded pool), one with a NaN and one with an infinity in every tile of 256 queries: once k labels are
    held, no later one can enter, so nothing passes for them and no list runs over."""
    Z, W = _base(46)
    Z[5::256] = 0.0
    Z[9::256, 1] = float("nan")
    Z[77::256, 0] = float("inf")
    W[700001, 3] = float("inf")                                     # (0 * inf is no number; the tile of 64 rows passes whole)
    W[800000, 0] = 0.0
    ws, state = _room(Z.shape[0], W.shape[0], 256, 50)
    ids, _ = _same_as_bf16(monkeypatch, Z, W, 50, ws)
    assert state.cpu().tolist() == [0, 0]
    assert bool((ids[5::256] == torch.arange(50, device=DEV, dtype=torch.int32)).all())
    assert bool((ids[9::256] == -1).all())


def test_q8_scores_that_rise_along_the_labels(monkeypatch):
    """Every label beats the threshold of those before it: the lists run over, the query tiles are given up and searched in
    bf16.  First for all queries but 2000..2999, which prefer small ids (exact products; rows are equal in long runs, so ties
    everywhere), then for one tile of queries among random ones."""
    L, d, Zq, k = 1100000, 128, 4200, 60
    W = (torch.arange(L, dtype=torch.float32, device=DEV)[:, None] / 65536.0 * torch.ones(d, device=DEV)[None, :]).to(torch.bfloat16)
    Z = torch.ones((Zq, d), dtype=torch.bfloat16, device=DEV)
    Z[2000:3000] *= -1.0
    ws, state = _room(Zq, L, d, k)
    ids, sc = _same_as_bf16(monkeypatch, Z, W, k, ws)
    assert state[0].item() > 0
    rows = ids[:, :-1].long(), ids[:, 1:].long()                    # equal rows come in the order of their ids
    assert bool((rows[0] < rows[1])[sc[:, :-1] == sc[:, 1:]].all())
    Z[:] = synth.make_matrix(5, synth.TAG_Z, Zq, d, torch.bfloat16, DEV)
    W = synth.make_matrix(5, synth.TAG_W, L, d, torch.bfloat16, DEV)
    W[:, 0] = (0.3 * torch.arange(L, device=DEV) / L).to(torch.bfloat16)
    Z[:, 0] = 0.0
    Z[256:300] = 0.0
    Z[256:300, 0] = 1.0
    ids, sc = _same_as_bf16(monkeypatch, Z, W, k, ws)
    assert state[0].item() > 0 and state[1].item() == 0             # some tiles, and the filter goes on for the others
    _check_exact(Z, W, ids, sc, k)


@pytest.mark.parametrize("Zq,given_up", [
    (4300, [0]),                           # work items of one tile of 256 queries; the first
    (4300, [16]),                          # the last, ragged one
    (4300, [1, 4, 5, 11]),
    (16200, [62]),                         # work items of two tiles
    (16200, [0, 1, 7, 30, 63]),
])
def test_q8_few_tiles_given_up(monkeypatch, Zq, given_up):
    """A query out of the filter's range makes its tile of 256 queries run over: those tiles alone are searched in bf16, in more
    slices of the labels than a search of the whole pool has."""
    L, d, k = 1100000, 128, 60
    W = synth.make_matrix(47, synth.TAG_W, L, d, torch.bfloat16, DEV)
    Z = synth.make_matrix(47, synth.TAG_Z, Zq, d, torch.bfloat16, DEV)
    q = torch.tensor([256 * t + 3 for t in given_up], device=DEV)
    Z[q] *= 2.0 ** 60
    ws, state = _room(Zq, L, d, k)
    ids, sc = _same_as_bf16(monkeypatch, Z, W, k, ws)
    assert state[0].item() >= len(given_up) and state[1].item() == 0
    Z[q] *= 2.0 ** -60
    ids2, sc2 = _search(Z, W, k, ws)
    assert torch.equal(ids, ids2) and torch.equal(sc[q], sc2[q] * 2.0 ** 60)


@pytest.mark.parametrize("n_tiles,off", [(8, 0), (17, 1)])
def test_q8_is_switched_off_by_what_one_chunk_gives_up(monkeypatch, n_tiles, off):
    """Four chunks of labels.  Eight tiles of seventeen given up in each are worth it (they do not add up from chunk to chunk),
    all of them are not."""
    Zq, L, d, k = 4300, 4500000, 256, 50
    W = synth.make_matrix(48, synth.TAG_W, L, d, torch.bfloat16, DEV)
    Z = synth.make_matrix(48, synth.TAG_Z, Zq, d, torch.bfloat16, DEV)
    Z[3:256 * n_tiles:256] *= 2.0 ** 60
    ws, state = _room(Zq, L, d, k)
    _same_as_bf16(monkeypatch, Z, W, k, ws)
    assert state.cpu().tolist() == [17 if off else 4 * n_tiles, off]


def test_q8_needs_its_room_and_is_reproducible(monkeypatch):
    import paper_2409_20156_amd as xc
    Z, W = _base(45)
    need = xc.mine_workspace(Z.shape[0], W.shape[0], 256, 50, xc.XC_BF16)
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    ws.random_(0, 255)
    a = _search(Z, W, 50, ws)
    ws.random_(0, 255)
    b = _search(Z, W, 50, ws)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    c = _search(Z, W, 50, ws[:need - 256])                          # without the filter's room: the bf16 search
    assert torch.equal(a[0], c[0]) and torch.equal(a[1], c[1])
    # a warm search after it starts from its thresholds
    ids, sc = xc.mine_negatives(Z, W, 50, want_scores=True, workspace=ws, warm_margin=0.05)
    xc.mine_negatives(Z, W, 50, workspace=ws)
    ids, sc = xc.mine_negatives(Z, W, 50, want_scores=True, workspace=ws, warm_margin=0.05)
    torch.cuda.synchronize()
    assert int(ws[:4].view(torch.int32).item()) == 0
    assert torch.equal(a[0], ids) and torch.equal(a[1], sc)
