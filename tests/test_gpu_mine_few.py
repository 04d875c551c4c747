"""The search of few queries (group maxima, then the k best groups again) against the oracle and against the general
kernel, at the sizes where it can go wrong: query blocks of 16 and their remainders, rows that are no multiple of the
64-byte step, fewer groups than k, groups of more than 16 labels, ties across groups, scores that are no numbers."""
import numpy as np
import pytest
import torch

from oracle import astra_oracle as orc
from paper_2409_20156_amd import synth
from tests.parity import check_topk, f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _run(Z, W, k, **kw):
    import paper_2409_20156_amd as xc
    ids, sc = xc.mine_negatives(Z, W, k, want_scores=True, **kw)
    torch.cuda.synchronize()
    return ids.cpu().numpy(), sc.cpu().numpy()


@pytest.mark.parametrize("Zq,L,d,dtype,k", [
    (1, 16, 8, torch.bfloat16, 16),             # one group, one chunk, k = L
    (15, 33, 32, torch.bfloat16, 5),            # 33 labels: a tile of one label
    (16, 5000, 40, torch.bfloat16, 128),        # 80-byte rows: a step of one chunk at the end
    (17, 5001, 768, torch.bfloat16, 100),       # two query blocks
    (33, 70000, 104, torch.bfloat16, 64),       # four query blocks, three in use
    (64, 16 * 1024, 256, torch.bfloat16, 1),
    (65, 4100, 768, torch.bfloat16, 20),        # a second group of query blocks
    (256, 9000, 768, torch.bfloat16, 20),
    (256, 9000, 256, torch.bfloat16, 128),
    (5, 3000, 2048, torch.bfloat16, 9),         # 4096-byte rows: fewer query blocks fit LDS
    (40, 3000, 1152, torch.bfloat16, 9),        # 2304-byte rows: two query blocks, two groups of them
    (1, 1000, 4608, torch.bfloat16, 3),         # the longest row it takes (9216 bytes)
    (7, 2500, 4, torch.float32, 31),
    (100, 20000, 68, torch.float32, 64),
    (31, 2100000, 8, torch.bfloat16, 100),      # groups of 32 labels
    (3, 4300001, 8, torch.bfloat16, 128),       # groups of 64 labels
])
def test_few_queries_match_oracle(Zq, L, d, dtype, k):
    print("case", Zq, L, d, dtype, k, flush=True)
    W = synth.make_matrix(21, synth.TAG_W, L, d, dtype, DEV)
    Z = synth.make_matrix(21, synth.TAG_Z, Zq, d, dtype, DEV)
    ids, sc = _run(Z, W, k)
    Z64, W64 = f64(Z), f64(W)
    ids_o, sc_o = orc.mine_negatives(Z64, W64, k)
    check_topk(ids, sc, ids_o, sc_o, Z64, W64)
    assert all(len(set(row)) == k for row in ids.tolist()) and (np.diff(sc, axis=1) <= 0).all()


# 4300001: more tied candidates than the key list holds; from 512 queries on a query has 256 threads and a list of 1024 keys,
# which 128 groups of 16 tied labels overflow, from more than 512 groups with the same maximum
@pytest.mark.parametrize("Zq,L,d", [(3, 1000, 8), (3, 2200000, 8), (3, 4300001, 8), (512, 1900, 64), (700, 40000, 64)])
def test_few_queries_equal_scores_order_by_id(Zq, L, d):
    W = torch.ones((L, d), dtype=torch.bfloat16, device=DEV)
    Z = torch.ones((Zq, d), dtype=torch.bfloat16, device=DEV)
    ids, sc = _run(Z, W, 128)
    assert (ids == np.arange(128)[None, :]).all() and (sc == d).all()
    W[L // 2:L // 2 + 40] = 2.0                                   # some better, the rest still tied
    ids, sc = _run(Z, W, 128)
    want = np.concatenate([np.arange(L // 2, L // 2 + 40), np.arange(88)])
    assert (ids == want[None, :]).all()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_few_queries_scores_that_are_no_numbers(monkeypatch, dtype):
    """NaN is never taken, infinities order as numbers, slots without a score get -1: as the general kernel does."""
    L, d, k = 3000, 64, 100
    W = synth.make_matrix(3, synth.TAG_W, L, d, dtype, DEV)
    Z = synth.make_matrix(3, synth.TAG_Z, 20, d, dtype, DEV)
    W[::7] = float("nan")
    W[5, 0] = float("inf")
    W[33, 3] = -float("inf")
    W[70:400] = float("nan")                                      # whole groups without a score
    Wn = torch.full_like(W, float("nan"))
    Wn[100:150] = W[501:551]                                      # fewer scores than k
    Z[4] = 0.0                                                    # 0 * inf
    Z[5] = float("nan")
    for M in (W, Wn):
        ids, sc = _run(Z, M, k)
        monkeypatch.setenv("XC_MINE_GENERAL", "1")
        ids_g, sc_g = _run(Z, M, k)
        monkeypatch.delenv("XC_MINE_GENERAL")
        assert (ids == ids_g).all() and (sc == sc_g).all()        # bit for bit
        assert (ids[5] == -1).all()


def test_few_queries_warm_call_needs_no_repeat():
    import paper_2409_20156_amd as xc
    Zq, L, d, k = 40, 9000, 128, 50
    W = synth.make_matrix(8, synth.TAG_W, L, d, torch.bfloat16, DEV)
    Z = synth.make_matrix(8, synth.TAG_Z, Zq, d, torch.bfloat16, DEV)
    ws = torch.empty(xc.mine_workspace(Zq, L, d, k, xc.XC_BF16), dtype=torch.uint8, device=DEV)
    ws.random_(0, 255)
    a = _run(Z, W, k, workspace=ws, warm_margin=0.1)
    assert ws[:8].view(torch.int32).cpu().tolist() == [0, 0]
    b = _run(Z, W, k)
    assert (a[0] == b[0]).all() and (a[1] == b[1]).all()


@pytest.mark.parametrize("Zq,L,d,k,dtype", [
    (1, 4097, 64, 5, torch.bfloat16), (16, 5001, 72, 30, torch.bfloat16), (17, 5021, 120, 30, torch.bfloat16),     # one stage; two, of which the
    (33, 5033, 136, 30, torch.bfloat16), (65, 33, 1032, 30, torch.bfloat16),                       # second has one chunk, ...; fewer tiles than waves
    (64, 30011, 768, 20, torch.bfloat16), (8, 5003, 2304, 20, torch.bfloat16),                     # no room for the stages; one block of queries
    (20, 2200003, 64, 100, torch.bfloat16), (3, 400011, 384, 9, torch.bfloat16),                   # read past the caches, groups of 32 labels
    (1, 4099, 32, 5, torch.float32), (16, 5003, 100, 60, torch.float32), (9, 150001, 512, 20, torch.float32),
    (100, 1048577, 96, 20, torch.bfloat16), (100, 1048575, 96, 20, torch.bfloat16),                # either side of the line to half lines
    (257, 503317, 200, 20, torch.bfloat16), (1100, 20011, 504, 9, torch.bfloat16),                 # ... of five blocks; of LDS that leaves slots idle
])
@pytest.mark.parametrize("shift", [0, 8])
def test_rows_read_by_lines(monkeypatch, Zq, L, d, k, dtype, shift):
    """The ids and scores of the general kernel, also where the rows of W begin within a line (W 16 or 32 bytes off)."""
    import paper_2409_20156_amd as xc
    Z = synth.make_matrix(91, synth.TAG_Z, Zq, d, dtype, DEV)
    W = torch.empty(L * d + shift, dtype=dtype, device=DEV)[shift:].view(L, d)
    W.copy_(synth.make_matrix(91, synth.TAG_W, L, d, dtype, DEV))
    ids, sc = (t.clone() for t in xc.mine_negatives(Z, W, k, want_scores=True))
    monkeypatch.setenv("XC_MINE_GENERAL", "1")
    want, want_sc = xc.mine_negatives(Z, W, k, want_scores=True)
    monkeypatch.delenv("XC_MINE_GENERAL")
    assert torch.equal(ids, want)
    assert torch.equal(sc, want_sc)


def test_few_queries_up_to_the_scratch_limit():
    """The group maxima fill the lists' 512 MiB but for 3 MB: what 16-bit maxima of fp32 rows need beside them does not
    count for bf16 rows (one launch that reads W, not phases)."""
    import paper_2409_20156_amd as xc
    from paper_2409_20156_amd import binding
    Zq, L, d, k = 96, 1390000 * 256, 8, 5
    W = torch.empty((L, d), dtype=torch.bfloat16, device=DEV).normal_(0.0, d ** -0.5)
    Z = synth.make_matrix(7, synth.TAG_Z, Zq, d, torch.bfloat16, DEV)
    W[-7:] = 4.0 * W[-7:]
    binding.profile_reset()
    binding.profile_enable(True)
    ids, sc = xc.mine_negatives(Z, W, k, want_scores=True)
    binding.profile_enable(False)
    torch.cuda.synchronize()
    prof = binding.profile_collect()
    assert prof["mine_tile"][1] == 1 and prof["mine_select"][1] == 1
    best = torch.zeros((Zq, 0), device=DEV)
    for r in range(0, L, 1 << 22):
        best = torch.cat([best, torch.topk(Z.float() @ W[r:r + (1 << 22)].float().T, k, dim=1)[0]], dim=1).topk(k, dim=1)[0]
    assert torch.allclose(sc, best, rtol=1e-5, atol=1e-6)
