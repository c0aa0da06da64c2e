"""The selection's kernels at the edges of their lists and tiles, against the
oracle: key places counted by several workgroups, the ordered fold of listed
rows over several tiles of trees, outputs that share memory with the list, and
the merge of the streamed explorer's sorted lists."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2411_10764_amd import ml2  # noqa: E402

DEV = "cuda:0"


def _topk(score, valid, k):
    n = score.shape[0]
    s, v = torch.from_numpy(score).to(DEV), torch.from_numpy(valid).to(DEV)
    idx = torch.full((k,), -7, dtype=torch.int32, device=DEV)
    top = torch.empty(k, device=DEV)
    num = torch.empty(1, dtype=torch.int32, device=DEV)
    ws = torch.empty(ml2.ml2_topk_workspace_bytes(n, k), dtype=torch.uint8, device=DEV)
    ml2.ml2_filter_topk(v, s, k, idx, top, num, ws)
    torch.cuda.synchronize()
    return idx.cpu().numpy(), top.cpu().numpy(), int(num.item())


# pools above the one-workgroup limit (8,192): ties that fill the threshold
# bin, all distinct, few included, none included; k around 64 keys and 1,024
@pytest.mark.parametrize("n", [8193, 20000, 300001])
@pytest.mark.parametrize("k", [1, 63, 64, 65, 1023, 1025, 16384])
def test_topk_places(n, k):
    rng = np.random.default_rng(n + k)
    for kind in range(4):
        score = rng.standard_normal(n).astype(np.float32)
        if kind == 0:
            score = np.round(score * 4) / 4  # many ties
        valid = (rng.random(n) < (0.6, 0.6, 0.003, 0.0)[kind]).astype(np.uint8)
        score[rng.random(n) < 0.01] = rng.choice(
            np.array([np.nan, np.inf, -np.inf, 0.0, -0.0], np.float32))
        score = np.ascontiguousarray(score, np.float32)
        got, want = _topk(score, valid, k), oracle.topk(valid, score, k)
        assert got[2] == want[2]
        assert np.array_equal(got[0], want[0])
        assert np.array_equal(got[1].view(np.uint32), want[1].view(np.uint32))


# trees around the fold's tiles of 128, list lengths around 64 entries and the
# 1,024 keys of a tile; repeated and out-of-range rows
@pytest.mark.parametrize("trees,depth", [(1, 4), (127, 5), (129, 6), (300, 3)])
@pytest.mark.parametrize("m", [1, 64, 65, 1025, 2100])
@pytest.mark.parametrize("shared", [False, True])
def test_rerank_places(trees, depth, m, shared):
    n, F, keep = 5000, 20, max(1, m // 2)
    A = gen.perfect_ensemble(31, 3, trees, depth, F, 10, 0.1)
    X = gen.features(31, n, F, 10)
    rng = np.random.default_rng(m + trees)
    rows = rng.integers(-3, n + 3, m).astype(np.int32)
    rows[m // 2:] = rows[:m - m // 2]
    want = oracle.rerank(A, X, rows, keep)
    a = ml2.ml2_load_ensemble(A)
    Xd, rd = torch.from_numpy(X).to(DEV), torch.from_numpy(rows).to(DEV)
    rs = torch.empty(m, device=DEV)
    idx = rd if shared else torch.empty(keep, dtype=torch.int32, device=DEV)
    top = torch.empty(keep, device=DEV)
    num = torch.empty(1, dtype=torch.int32, device=DEV)
    ws = torch.empty(ml2.ml2_rerank_workspace_bytes(a, m), dtype=torch.uint8, device=DEV)
    ml2.ml2_rerank(a, Xd, rd, keep, rs, idx, top, num, ws, m=m)
    torch.cuda.synchronize()
    assert np.array_equal(rs.cpu().numpy().view(np.uint32), want[0].view(np.uint32))
    assert np.array_equal(idx.cpu().numpy()[:keep], want[1])
    assert np.array_equal(top.cpu().numpy().view(np.uint32), want[2].view(np.uint32))
    assert int(num.item()) == want[3]
    a.free()


# deep trees: lists up to 256 entries and wide rows gather their features,
# longer lists of narrow rows walk in tiles
@pytest.mark.parametrize("trees,depth", [(9, 10), (5, 11), (3, 12)])
@pytest.mark.parametrize("F", [20, 64, 130])
@pytest.mark.parametrize("m", [1, 65, 256, 257, 1025])
def test_rerank_deep(trees, depth, F, m):
    n, keep = 3000, max(1, m // 2)
    A = gen.perfect_ensemble(32, 3, trees, depth, F, F // 2, 0.1)
    X = gen.features(32, n, F, F // 2)
    rows = np.random.default_rng(m + F).integers(-3, n + 3, m).astype(np.int32)
    want = oracle.rerank(A, X, rows, keep)
    a = ml2.ml2_load_ensemble(A)
    Xd, rd = torch.from_numpy(X).to(DEV), torch.from_numpy(rows).to(DEV)
    rs, top = torch.empty(m, device=DEV), torch.empty(keep, device=DEV)
    idx = torch.empty(keep, dtype=torch.int32, device=DEV)
    num = torch.empty(1, dtype=torch.int32, device=DEV)
    ws = torch.empty(ml2.ml2_rerank_workspace_bytes(a, m), dtype=torch.uint8, device=DEV)
    ml2.ml2_rerank(a, Xd, rd, keep, rs, idx, top, num, ws)
    torch.cuda.synchronize()
    assert np.array_equal(rs.cpu().numpy().view(np.uint32), want[0].view(np.uint32))
    assert np.array_equal(idx.cpu().numpy(), want[1])
    assert np.array_equal(top.cpu().numpy().view(np.uint32), want[2].view(np.uint32))
    assert int(num.item()) == want[3]
    a.free()


# held and chunk lists of every fill, chunks that overlap in part and wholly
@pytest.mark.parametrize("k", [1, 5, 64, 1000, 4096])
def test_stream_merge(k):
    n, F = 9000, 12
    V = gen.perfect_ensemble(33, 1, 8, 4, F, F, 0.5)
    P = gen.perfect_ensemble(33, 2, 6, 4, F, F, 0.1)  # few distinct scores: ties
    X = gen.features(33, n, F, F)
    keep = max(1, k // 2)
    spans = [(0, 3000), (2000, 3000), (2000, 3000), (8990, 10), (5000, 3500), (0, 9000)]
    v, p = ml2.ml2_load_ensemble(V), ml2.ml2_load_ensemble(P)
    ex = ml2.StreamExplorer(v, p, None, 9000, k, keep, 3)
    Xd = torch.from_numpy(X).to(DEV)
    idx = torch.empty(keep, dtype=torch.int32, device=DEV)
    top = torch.empty(keep, device=DEV)
    num = torch.empty(1, dtype=torch.int32, device=DEV)
    chunks = [(r, X[r:r + c]) for r, c in spans]
    want = oracle.explore_stream(V, P, None, chunks, k, keep, 3)
    for w in want:
        ex.begin()
        for r, c in spans:
            ex.chunk(Xd[r:r + c], r)
        ex.end(idx, top, num)
        torch.cuda.synchronize()
        assert int(num.item()) == w[2]
        assert np.array_equal(idx.cpu().numpy(), w[0])
        assert np.array_equal(top.cpu().numpy().view(np.uint32), w[1].view(np.uint32))
