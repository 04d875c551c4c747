"""The general search kernel's dense first phase (all scores of its tiles written, the best k taken by one wave per query)
against the oracle, forced through XC_MINE_GENERAL: the three widths of the selection (4, 8 and 16 tiles), row lengths with and without a tail, equal
scores (more pass the bound than the list holds), scores that are no numbers, fewer scores than k."""
import numpy as np
import pytest
import torch

from oracle import astra_oracle as orc
from paper_2409_20156_amd import synth
from tests.parity import check_topk, f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(autouse=True)
def _general(monkeypatch):
    monkeypatch.setenv("XC_MINE_GENERAL", "1")


def _run(Z, W, k):
    import paper_2409_20156_amd as xc
    ids, sc = xc.mine_negatives(Z, W, k, want_scores=True)
    torch.cuda.synchronize()
    return ids.cpu().numpy(), sc.cpu().numpy()


@pytest.mark.parametrize("Zq,L,d,dtype,k", [
    (300, 16 * 256, 64, torch.bfloat16, 5),       # 16 tiles: four of them dense
    (300, 13 * 256 + 9, 64, torch.bfloat16, 100), # 13 tiles: six of them dense, what half of the range allows
    (520, 9000, 128, torch.bfloat16, 40),         # eight dense tiles
    (257, 9000, 768, torch.bfloat16, 128),        # maximum k: every half of a lane's scores has its maximum taken
    (700, 12001, 100, torch.float32, 100),        # fp32 with a tail, ragged last tile
    (40, 20000, 40, torch.bfloat16, 1),           # 80-byte rows, mostly empty query tile
    (2600, 8300, 64, torch.bfloat16, 64),         # eleven query tiles
])
def test_dense_phase_matches_oracle(Zq, L, d, dtype, k):
    print("case", Zq, L, d, dtype, k, flush=True)
    W = synth.make_matrix(51, synth.TAG_W, L, d, dtype, DEV)
    Z = synth.make_matrix(51, synth.TAG_Z, Zq, d, dtype, DEV)
    ids, sc = _run(Z, W, k)
    ids_o, sc_o = orc.mine_negatives(f64(Z), f64(W), k)
    check_topk(ids, sc, ids_o, sc_o, f64(Z), f64(W))


# labels, k, dense tiles
_WIDTHS = [(9000, 100, 16), (9000, 40, 8), (3337, 100, 6), (4096, 5, 4)]


@pytest.mark.parametrize("L,k,tiles", _WIDTHS)
def test_dense_phase_equal_scores_order_by_id(L, k, tiles):
    W = torch.zeros((L, 64), dtype=torch.bfloat16, device=DEV)
    Z = synth.make_matrix(1, synth.TAG_Z, 300, 64, torch.bfloat16, DEV)
    ids, _ = _run(Z, W, k)
    assert (ids == np.arange(k)[None, :]).all()
    W = torch.ones((L, 64), dtype=torch.bfloat16, device=DEV)      # some above the ties, on either side of the dense tiles
    Z = torch.ones((300, 64), dtype=torch.bfloat16, device=DEV)
    better = np.concatenate([np.arange(70, 1500, 100), np.arange(L - 5, L)])
    W[torch.as_tensor(better, device=DEV)] = 2.0
    ids, _ = _run(Z, W, k)
    rest = np.setdiff1d(np.arange(L), better)
    assert (ids == np.concatenate([better, rest])[None, :k]).all()


@pytest.mark.parametrize("L,k,tiles", _WIDTHS)
def test_dense_phase_scores_that_are_no_numbers(L, k, tiles):
    d = 64
    W = synth.make_matrix(3, synth.TAG_W, L, d, torch.bfloat16, DEV)
    Z = synth.make_matrix(3, synth.TAG_Z, 300, d, torch.bfloat16, DEV)
    W[:256 * tiles + 10] = float("nan")                            # all of the dense tiles, but for
    few = k // 2
    W[10:10 + few] = synth.make_matrix(4, synth.TAG_W, few, d, torch.bfloat16, DEV)        # fewer numbers there than k
    Z[7] = float("nan")
    ids, sc = _run(Z, W, k)
    assert (ids[7] == -1).all() and np.isneginf(sc[7]).all()
    W64 = f64(W)
    good = np.flatnonzero(~np.isnan(W64).any(axis=1))
    q = np.setdiff1d(np.arange(300), [7])
    ids_o, sc_o = orc.mine_negatives(f64(Z)[q], W64[good], k)
    remap = np.full(L, -1)
    remap[good] = np.arange(len(good))
    check_topk(remap[ids[q]], sc[q], ids_o, sc_o, f64(Z)[q], W64[good])
