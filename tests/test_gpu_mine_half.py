"""Searches of up to 2048 fp32 queries find the groups that can hold an answer with 16-bit products; what they return is the fp32
search's, bit for bit (the general kernel's, forced), whatever the rows are: also where the 16-bit maxima do not settle a query
and the fp32 kernels take it."""
import pytest
import torch

from paper_2409_20156_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(monkeypatch, Z, W, k):
    import paper_2409_20156_amd as xc
    ids, sc = (t.clone() for t in xc.mine_negatives(Z, W, k, want_scores=True))
    monkeypatch.setenv("XC_MINE_GENERAL", "1")
    want, want_sc = xc.mine_negatives(Z, W, k, want_scores=True)
    monkeypatch.delenv("XC_MINE_GENERAL")
    assert torch.equal(ids, want)
    assert torch.equal(sc.view(torch.int32), want_sc.view(torch.int32))


def _inputs(Zq, L, d):
    return (synth.make_matrix(81, synth.TAG_Z, Zq, d, torch.float32, DEV), synth.make_matrix(81, synth.TAG_W, L, d, torch.float32, DEV))


@pytest.mark.parametrize("Zq,L,d,k", [
    (17, 4096, 4, 1), (32, 5001, 28, 100),          # one block of 32 queries; a step of seven chunks, of one
    (33, 5003, 32, 128), (64, 9001, 36, 7),         # four blocks of 16
    (65, 8191, 300, 32), (128, 5021, 768, 20),      # eight; a query block that fits LDS with four
    (129, 2100001, 8, 100),                         # groups of 32 labels
    (200, 130, 64, 128),                            # fewer groups than k
    (513, 30011, 100, 50), (1025, 20001, 300, 32),  # 256 threads per query at the end
])
def test_sizes(monkeypatch, Zq, L, d, k):
    _check(monkeypatch, *_inputs(Zq, L, d), k)


@pytest.mark.parametrize("Zq", [40, 600])
@pytest.mark.parametrize("rows", ["zero", "mostly zero", "equal", "pairs", "large", "tiny", "wide", "inf", "nan", "far", "queries"])
def test_odd_rows(monkeypatch, Zq, rows):
    L, d, k = 20011, 100, 32
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
    else:
        Z[0] = 0.0
        Z[1] *= 1e20
        Z[2] *= 1e-20
        Z[3, 5] = float("inf")
        Z[4, 6] = float("nan")
        Z[5] *= -1e30
        Z[6, 1:] = 0.0
    _check(monkeypatch, Z, W, k)
