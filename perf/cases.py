"""The scoring work that an explorer program has this library do, as cases to time.

A case holds sizes only.  `prepare` builds what such a program has in hand (a
pool of candidates on the device, loaded ensembles, output buffers), `run`
makes one pass through the public calls of paper_2411_10764_amd.ml2.

Pools: knob columns are integers 0..8 and hidden columns lognormal(0, 1), a
share of them missing (NaN) where the models take missing values.  Models:
perfect trees, or ragged ones with default directions, whose split features
are uniform over the model's columns and whose thresholds come from the
column's own distribution; validity leaves are N(0, 0.5) with the margin bias
set so that a stated share of the pool is rejected, performance leaves
N(0, 0.1).

Margins and scores are float32 left folds in tree order, so every output is
determined bit for bit and the tolerance is "exact".
"""
import math
import types

import numpy as np
import torch

from paper_2411_10764_amd import ml2

KNOBS = 9          # knob values 0 .. 8
RAGGED_PATH = 5.0  # mean splits per walk of the ragged trees grown here
GROWN_NODES = 255  # largest ragged tree


def _case(name, call, n, F, K, v, p, k, invalid, *, a=(0, 0), keep=0, pad=0, visible=False,
          ragged=False, missing=0.0, chunk=0):
    return {"name": name, "call": call, "n": n, "F": F, "K": K, "pad": pad,
            "v_trees": v[0], "v_depth": v[1], "p_trees": p[0], "p_depth": p[1],
            "a_trees": a[0], "a_depth": a[1], "k": k, "keep": keep, "invalid": invalid,
            "visible": visible, "ragged": ragged, "missing": missing, "chunk": chunk}


def listed():
    return [
        # A small proposal batch scored in an interactive tuning loop: launches
        # and latency count.
        _case("score_4k_f32", "score", 4096, 32, 16, (50, 5), (50, 5), 32, 0.65),
        # One layer's search space, scored and cut to its best.
        _case("step_262k_f64", "step", 262144, 64, 32, (200, 6), (200, 6), 128, 0.40),
        # An odd pool: rows that are neither aligned nor a multiple of four wide.
        _case("step_1m_f37_odd", "step", 1000003, 37, 18, (150, 5), (300, 7), 100, 0.50, pad=4),
        # A merged space of several layers.
        _case("step_4m_f96", "step", 4194304, 96, 48, (500, 8), (500, 8), 512, 0.50),
        # The largest pool: the benchmark's 16M x 128 scoring step.
        _case("step_16m_f128", "step", 16777216, 128, 64, (300, 6), (1000, 8), 1024, 0.52),
        # A space that is mostly invalid, with deep performance trees.
        _case("step_8m_f64_d10", "step", 8388608, 64, 32, (200, 6), (800, 10), 256, 0.90),
        # Small models over the largest pool: reading the pool bounds it.
        _case("score_16m_f128_small", "score", 16777216, 128, 64, (40, 5), (40, 5), 1024, 0.49),
        # An explorer round after retraining: V and P on the visible columns,
        # model A on all of them.
        _case("round_16m_visible", "round", 16777216, 128, 64, (300, 6), (1000, 8), 1024, 0.50,
              a=(300, 12), keep=512, visible=True),
        # The same with models of the paper's sizes: P and A ragged, depth 14,
        # missing hidden values.
        _case("round_16m_ragged", "round", 16777216, 128, 64, (300, 5), (300, 14), 20, 0.50,
              a=(300, 14), keep=10, visible=True, ragged=True, missing=0.05),
        # A round over a pool that arrives in uneven chunks.
        _case("stream_3m_ragged", "stream", 3000017, 96, 40, (200, 5), (300, 14), 64, 0.60,
              a=(200, 14), keep=32, ragged=True, missing=0.05, chunk=700001),
        # The selection alone over stored scores: top-k, then model A.
        _case("select_16m", "select", 16777216, 128, 64, (0, 0), (0, 0), 1024, 0.50,
              a=(300, 12), keep=512),
        # Performance alone over a whole pool of the widest rows, deepest
        # perfect trees.
        _case("perf_500k_f256_d12", "perf", 500000, 256, 128, (0, 0), (100, 12), 0, 0.0),
    ]


def _visits(c):
    n = c["n"]
    ragged = c["ragged"]
    p_path = RAGGED_PATH if ragged else c["p_depth"]
    a_path = RAGGED_PATH if ragged else c["a_depth"]
    kept = n * (1.0 - c["invalid"])
    chunks = -(-n // c["chunk"]) if c["chunk"] else 1
    return (n * c["v_trees"] * c["v_depth"] + kept * c["p_trees"] * p_path
            + chunks * c["k"] * c["a_trees"] * a_path)


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    most = max(_visits(c) for c in listed())
    while True:
        call = rng.choice(["score", "step", "step", "step", "round", "stream", "select", "perf"])
        n = log_int(2000, 16777216)
        F = log_int(16, 160)
        if rng.random() < 0.5:
            F = -(-F // 4) * 4
        K = max(4, F // 2)
        pad = 0 if rng.random() < 0.6 else rng.randint(1, 7)
        ragged = call in ("step", "round", "stream") and rng.random() < 0.4
        vd = rng.randint(4, 6)
        v = (log_int(40, 300), vd)
        p = (log_int(40, 300), 14) if ragged else (log_int(40, 1000), rng.randint(5, 10))
        if call == "score":  # models small enough for one pass
            p = (log_int(20, 60), vd)
            v = (log_int(20, 60), vd)
        a, keep = (0, 0), 0
        k = log_int(8, min(2048, max(9, n // 4)))
        if call in ("round", "stream", "select"):
            a = (log_int(40, 300), 14 if ragged else rng.randint(8, 12))
            keep = max(1, k // 2)
        if call in ("perf", "select"):
            v = (0, 0)
        if call == "select":
            p = (0, 0)
        invalid = 0.0 if call == "perf" else round(rng.uniform(0.3, 0.9), 2)
        c = _case("", call, n, F, K, v, p, 0 if call == "perf" else k, invalid, a=a, keep=keep,
                  pad=pad, visible=call == "round" and rng.random() < 0.5, ragged=ragged,
                  missing=0.05 if ragged else 0.0,
                  chunk=max(1, n // rng.randint(2, 5)) if call == "stream" else 0)
        del c["name"]
        if _visits(c) <= most and n * (F + pad) <= 16777216 * 128:
            return c


# ---- inputs -------------------------------------------------------------------

def _thresholds(rng, feat, K):
    knob = rng.integers(0, KNOBS, feat.shape).astype(np.float32)
    hidden = np.exp(rng.standard_normal(feat.shape)).astype(np.float32)
    return np.where(feat < K, knob, hidden).astype(np.float32)


def _perfect(rng, trees, depth, F, K, sigma):
    internal, nodes = (1 << depth) - 1, (2 << depth) - 1
    left = np.full((trees, nodes), -1, np.int32)
    right = np.full((trees, nodes), -1, np.int32)
    feat = np.full((trees, nodes), -1, np.int32)
    thr = np.zeros((trees, nodes), np.float32)
    val = np.zeros((trees, nodes), np.float32)
    i = np.arange(internal, dtype=np.int32)
    left[:, :internal] = 2 * i + 1
    right[:, :internal] = 2 * i + 2
    feat[:, :internal] = rng.integers(0, F, (trees, internal))
    thr[:, :internal] = _thresholds(rng, feat[:, :internal], K)
    val[:, internal:] = sigma * rng.standard_normal((trees, nodes - internal))
    return types.SimpleNamespace(
        num_features=F, base_score=0.0, default_left=None, depth=depth,
        offsets=np.arange(trees + 1, dtype=np.int64) * nodes, left=left.ravel(),
        right=right.ravel(), feature=feat.ravel(), threshold=thr.ravel(), value=val.ravel())


def _grown(rng, trees, depth, F, K, sigma):
    """Ragged trees of at most `depth` levels, grown breadth-first: a node at
    depth d splits with probability 0.9 * 0.9^(d-1), the root always."""
    off, left, right = [0], [], []
    for _ in range(trees):
        u = rng.random(GROWN_NODES)
        lv, lf, rt = [0], [], []
        i = 0
        while i < len(lv):
            d = lv[i]
            if len(lv) + 2 <= GROWN_NODES and d < depth and (
                    d == 0 or u[i] < 0.9 * 0.9 ** (d - 1)):
                lf.append(len(lv))
                rt.append(len(lv) + 1)
                lv += [d + 1, d + 1]
            else:
                lf.append(-1)
                rt.append(-1)
            i += 1
        left += lf
        right += rt
        off.append(len(left))
    left, right = np.array(left, np.int32), np.array(right, np.int32)
    split = left >= 0
    feat = np.where(split, rng.integers(0, F, left.shape), -1).astype(np.int32)
    return types.SimpleNamespace(
        num_features=F, base_score=0.0, depth=depth, offsets=np.array(off, np.int64), left=left,
        right=right, feature=feat,
        threshold=np.where(split, _thresholds(rng, feat, K), 0).astype(np.float32),
        value=np.where(split, 0, sigma * rng.standard_normal(left.shape)).astype(np.float32),
        default_left=(split & (rng.random(left.shape) < 0.5)).astype(np.uint8))


def _pool(case, seed):
    n, F, K = case["n"], case["F"], case["K"]
    g = torch.Generator(device="cuda").manual_seed(seed * 7919 + 1)
    X = torch.zeros(n, F + case["pad"], device="cuda")
    step = 1 << 20
    for r in range(0, n, step):
        m = min(step, n - r)
        X[r:r + m, :K] = torch.randint(0, KNOBS, (m, K), generator=g, device="cuda").float()
        h = torch.randn(m, F - K, generator=g, device="cuda").exp_()
        if case["missing"]:
            gone = torch.rand(m, F - K, generator=g, device="cuda") < case["missing"]
            h = h.masked_fill_(gone, math.nan)
        X[r:r + m, K:F] = h
    return X[:, :F]


def _leaves(ens, X):
    """Leaf value of every tree for every row of X: [rows, trees], float32."""
    dev = X.device
    left, right = (torch.from_numpy(a.astype(np.int64)).to(dev) for a in (ens.left, ens.right))
    feat = torch.from_numpy(ens.feature.astype(np.int64)).to(dev).clamp_(min=0)
    thr, val = (torch.from_numpy(a).to(dev) for a in (ens.threshold, ens.value))
    off = torch.from_numpy(ens.offsets[:-1]).to(dev)
    dl = None if ens.default_left is None else torch.from_numpy(ens.default_left).to(dev).bool()
    u = off.expand(X.shape[0], -1).contiguous()
    for _ in range(ens.depth):
        x = X.gather(1, feat[u])
        go_left = x < thr[u]
        if dl is not None:
            go_left |= x.isnan() & dl[u]
        child = torch.where(go_left, left[u], right[u])
        u = torch.where(child < 0, u, off + child)
    return val[u]


def _models(case, seed, X):
    rng = np.random.default_rng(seed * 104729 + 17)
    F, K = case["F"], case["K"]
    seen = K if case["visible"] else F
    grow = _grown if case["ragged"] else _perfect
    v = p = a = None
    if case["v_trees"]:
        v = _perfect(rng, case["v_trees"], case["v_depth"], seen, K, 0.5)
        sample = _leaves(v, X[:8192]).double().sum(1)
        v.base_score = float(np.float32(-torch.quantile(sample, case["invalid"]).item()))
    if case["p_trees"]:
        p = grow(rng, case["p_trees"], case["p_depth"], seen, K, 0.1)
    if case["a_trees"]:
        a = grow(rng, case["a_trees"], case["a_depth"], F, K, 0.1)
    return v, p, a


def _stored_scores(case, seed):
    """A scored pool: the mask, and scores as a performance model gives them."""
    g = torch.Generator(device="cuda").manual_seed(seed * 6007 + 3)
    n = case["n"]
    valid = (torch.rand(n, generator=g, device="cuda") >= case["invalid"]).to(torch.uint8)
    score = torch.randn(n, generator=g, device="cuda") * 1.5
    return valid, score.masked_fill_(valid == 0, -math.inf)


def prepare(case, seed):
    X = _pool(case, seed)
    v, p, a = (None if m is None else ml2.ml2_load_ensemble(m) for m in _models(case, seed, X))
    n, k, keep = case["n"], case["k"], case["keep"]
    s = types.SimpleNamespace(call=case["call"], X=X, v=v, p=p, a=a, k=k, keep=keep)

    def out(m, dtype):
        return torch.empty(max(m, 1), dtype=dtype, device="cuda")

    if s.call in ("score", "step"):
        s.pipe = ml2.Pipeline(v, p, n, k, with_margin=True)
    elif s.call == "perf":
        s.score = out(n, torch.float32)
    else:
        s.idx, s.top, s.num = out(keep, torch.int32), out(keep, torch.float32), out(1, torch.int32)
    if s.call == "round":
        s.explorer = ml2.Explorer(v, p, a, n, k, keep, 4)
    if s.call == "stream":
        s.explorer = ml2.StreamExplorer(v, p, a, case["chunk"], k, keep, 4)
        s.chunks = [(X[r:r + case["chunk"]], r) for r in range(0, n, case["chunk"])]
    if s.call == "select":
        s.valid, s.score = _stored_scores(case, seed)
        s.rows, s.held, s.found = out(k, torch.int32), out(k, torch.float32), out(1, torch.int32)
        s.ws = out(ml2.ml2_topk_workspace_bytes(n, k), torch.uint8)
        s.row_scores = out(k, torch.float32)
        s.a_ws = out(ml2.ml2_rerank_workspace_bytes(a, k), torch.uint8)
    return s


def run(s):
    if s.call == "step":
        q = s.pipe
        q.run(s.X)
        return {"valid": q.valid, "margin": q.margin, "score": q.score, "idx": q.idx,
                "top": q.top, "num": q.num}
    if s.call == "score":
        q = s.pipe
        ml2.ml2_score(s.v, s.p, s.X, q.valid, q.margin, q.score)
        ml2.ml2_filter_topk(q.valid, q.score, q.k, q.idx, q.top, q.num, q.ws, q.ws_bytes, q.n)
        return {"valid": q.valid, "margin": q.margin, "score": q.score, "idx": q.idx,
                "top": q.top, "num": q.num}
    if s.call == "perf":
        ml2.ml2_score_perf(s.p, s.X, None, s.score)
        return {"score": s.score}
    if s.call == "round":  # the first round after the models changed
        s.explorer.reset()
        s.explorer.round(s.X, s.idx, s.top, s.num)
        return {"idx": s.idx, "top": s.top, "num": s.num}
    if s.call == "stream":
        s.explorer.reset()
        s.explorer.begin()
        for X, r in s.chunks:
            s.explorer.chunk(X, r)
        s.explorer.end(s.idx, s.top, s.num)
        return {"idx": s.idx, "top": s.top, "num": s.num}
    ml2.ml2_filter_topk(s.valid, s.score, s.k, s.rows, s.held, s.found, s.ws)
    ml2.ml2_rerank(s.a, s.X, s.rows, s.keep, s.row_scores, s.idx, s.top, s.num, s.a_ws)
    return {"rows": s.rows, "held": s.held, "row_scores": s.row_scores, "idx": s.idx,
            "top": s.top, "num": s.num}


def work(case):
    n, F, kept = case["n"], case["F"], case["n"] * (1.0 - case["invalid"])
    seen = case["K"] if case["visible"] else F
    call, k = case["call"], case["k"]
    if call == "select":
        nbytes = 5 * n + 4 * k * F
    elif call == "perf":
        nbytes = 4 * n * F + 4 * n
    elif call in ("score", "step"):
        nbytes = 4 * n * F + 9 * n
    else:  # mask and scores stay with the explorer
        nbytes = 4 * n * seen
    # one comparison for each node on a walk, one addition for each leaf
    leaves = n * case["v_trees"] + kept * case["p_trees"] + k * case["a_trees"]
    return {"bytes": int(nbytes), "flops": int(_visits(case) + leaves)}


def tolerance(case):
    return "exact"


def _folds(ens, X, rows=None):
    """The margins of X's rows (or of the listed ones): the float32 left fold
    that defines the result, and the sum of the same leaves in 64 bits."""
    n = X.shape[0] if rows is None else rows.shape[0]
    step = max(1, (1 << 26) // (len(ens.offsets) - 1))
    f32, f64 = [], []
    for r in range(0, n, step):
        x = X[r:r + step] if rows is None else X[rows[r:r + step]]
        leaf = _leaves(ens, x[:, :ens.num_features])
        m = torch.full((x.shape[0],), ens.base_score, dtype=torch.float32, device=X.device)
        for t in range(leaf.shape[1]):
            m = m + leaf[:, t]
        f32.append(m)
        f64.append(leaf.double().sum(1) + ens.base_score)
    return torch.cat(f32), torch.cat(f64)


def _best(score, ok, k):
    """The k best included rows by (score desc, row asc)."""
    row = torch.nonzero(ok).flatten()
    return row[torch.sort(score[row], descending=True, stable=True).indices[:k]]


def exact(case, seed):
    call, k, keep = case["call"], case["k"], case["keep"]
    if _visits(case) > 1e10:
        return None
    X = _pool(case, seed)
    v, p, a = _models(case, seed, X)

    def padded(x, m):
        return torch.cat([x, x.new_full((max(m, 1) - x.shape[0],), -math.inf)])

    if call == "perf":
        return {"score": _folds(p, X)[1]}
    if call == "select":
        valid, score = _stored_scores(case, seed)
        rows = _best(score, valid != 0, k)
        s32, s64 = _folds(a, X, rows)
        order = torch.sort(s32, descending=True, stable=True).indices[:keep]
        return {"rows": None, "held": padded(score[rows].double(), k),
                "row_scores": padded(s64, k), "idx": None, "top": padded(s64[order], keep),
                "num": None}
    m32, m64 = _folds(v, X)
    ok = m32 > 0
    s32, s64 = _folds(p, X)
    rows = _best(s32, ok, k)
    if call in ("score", "step"):
        return {"valid": None, "margin": m64, "score": s64.masked_fill(~ok, -math.inf),
                "idx": None, "top": padded(s64[rows], k), "num": None}
    a32, a64 = _folds(a, X, rows)
    order = torch.sort(a32, descending=True, stable=True).indices[:keep]
    return {"idx": None, "top": padded(a64[order], keep), "num": None}
