"""Performance cases of the GED-Walk library: what a user has it compute.

A case names a graph family with its sizes, a call (one group's score, a batch
of scores, a greedy maximisation) and the call's sizes.  ``prepare`` builds the
graph from the seed and hands it to the library, as a program does once;
``run`` is one call on the resident graph.  The sizes are those of
``bench.py``'s workloads and of the serving mix (``serve.SERVE_GRAPHS``).
"""
import math

import numpy as np
import torch

from paper_1910_13874_amd import ged, inputs

EPS = 1e-4
RMAT = (0.57, 0.19, 0.19)


def listed():
    return [
        # The smallest call: one group of a thousand-vertex network, the
        # latency an interactive tool sees (28 walk lengths, launch-bound).
        dict(name="score_er1k", kind="score", graph="er", n=1000, deg=10, size=5),
        # An ordinary single query: a power-law network of a million vertices.
        dict(name="score_ba1m", kind="score", graph="ba", n=1000000, m=5, size=5),
        # The largest single query: R-MAT scale 22, 128 M arcs.
        dict(name="score_rmat22", kind="score", graph="rmat", scale=22, ef=16, size=5),
        # A directed network (web links, citations): the level-by-level chain.
        dict(name="score_directed_rmat17", kind="score", graph="rmat", scale=17, ef=8,
             directed=True, size=37),
        # Many candidate groups of a small uniform network (a serving lane).
        dict(name="batch_er10k", kind="batch", graph="er", n=10000, deg=8, groups=256, smax=100),
        # The batched workload's graph, with a ragged last tile.
        dict(name="batch_ba2m", kind="batch", graph="ba", n=2000000, m=8, groups=1000, smax=200),
        # A serving lane on a skewed graph whose deeper counts exceed 32 bits.
        dict(name="batch_rmat20", kind="batch", graph="rmat", scale=20, ef=16, groups=250,
             smax=100),
        # Choosing a group: the small call, ...
        dict(name="greedy_er1k", kind="greedy", graph="er", n=1000, deg=10, k=5),
        # ... an ordinary one, ...
        dict(name="greedy_ba1m", kind="greedy", graph="ba", n=1000000, m=5, k=10),
        # ... and the headline configuration.
        dict(name="greedy_rmat22", kind="greedy", graph="rmat", scale=22, ef=16, k=100),
        # The directed and the weighted variant of the maximisation.
        dict(name="greedy_directed_rmat17", kind="greedy", graph="rmat", scale=17, ef=8,
             directed=True, k=10),
        dict(name="greedy_weighted_ba100k", kind="greedy", graph="ba", n=100000, m=5,
             weighted=True, k=10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: a call and a graph family at random, sizes spread over
    the logarithm of the range the listed cases span."""
    c = {"kind": rng.choice(["score", "batch", "greedy", "greedy", "score"])}
    fam = rng.choice(["er", "ba", "rmat", "directed", "weighted"])
    big = c["kind"] == "score"
    if fam == "er":
        c.update(graph="er", n=_log_int(rng, 700, 150000), deg=rng.choice([6, 8, 10, 16]))
    elif fam == "ba":
        c.update(graph="ba", n=_log_int(rng, 2000, 2000000 if big else 1000000),
                 m=rng.choice([4, 5, 8]))
    elif fam == "weighted":
        c.update(graph="ba", n=_log_int(rng, 2000, 150000), m=rng.choice([3, 5]), weighted=True)
    elif fam == "directed":
        c.update(graph="rmat", scale=rng.randint(11, 18), ef=rng.choice([4, 8]), directed=True)
    else:
        c.update(graph="rmat", scale=rng.randint(12, 21 if big else 20), ef=rng.choice([8, 16]))
    if c["kind"] == "score":
        c["size"] = min(_log_int(rng, 1, 300), _vertices(c) // 4)
    elif c["kind"] == "batch":
        # no more arc-columns than the listed batches traverse
        most = min(1200, max(8, int(7e9 / _arcs(c))))
        c["groups"] = _log_int(rng, 3, most)
        c["smax"] = rng.choice([10, 100, 200])
    else:
        c["k"] = _log_int(rng, 1, 25)
        if fam in ("er", "ba") and rng.random() < 0.3:
            c["eta"] = 0.1  # the stochastic variant
    return c


# ----------------------------------------------------------------- inputs --

def _vertices(c):
    return c["n"] if "n" in c else 1 << c["scale"]


def _arcs(c):
    """Stored arcs of the case's graph (R-MAT: before duplicates are merged)."""
    if c["graph"] == "er":
        return c["n"] * c["deg"]
    if c["graph"] == "ba":
        return 2 * c["n"] * c["m"]
    return (1 if c.get("directed") else 2) * (c["ef"] << c["scale"])


def _rmat(scale, ef, directed, seed):
    """R-MAT edges without loops or duplicates as CSR of in-neighbours, both
    arcs of each edge or (directed) one of them, built on the GPU."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    gen = torch.Generator(device=dev).manual_seed(seed)
    n, m = 1 << scale, ef << scale
    a, b, c = RMAT
    src = torch.zeros(m, dtype=torch.int64, device=dev)
    dst = torch.zeros_like(src)
    for _ in range(scale):
        r = torch.rand(m, generator=gen, device=dev)
        low = r >= a + b  # lower half of the quadrant matrix
        src.mul_(2).add_(low)
        dst.mul_(2).add_((r >= a + b + c) | ((r >= a) & ~low))
    lo, hi = torch.minimum(src, dst), torch.maximum(src, dst)
    key = torch.unique((lo * n + hi)[lo != hi])
    del src, dst, lo, hi, r, low
    lo, hi = key // n, key % n
    if directed:
        flip = torch.rand(key.numel(), generator=gen, device=dev) < 0.5
        arcs = torch.where(flip, hi * n + lo, key)
    else:
        arcs = torch.cat([key, hi * n + lo])
    arcs = torch.sort(arcs).values
    row_ptr = torch.searchsorted(arcs, torch.arange(n + 1, device=dev) * n)
    col = (arcs % n).to(torch.int32)
    return inputs.Graph(n=n, row_ptr=row_ptr.cpu().numpy(), col_idx=col.cpu().numpy(),
                        name="rmat", directed=directed)


def _graph(c, seed):
    """The case's graph and, for weighted cases, its arc weights
    (D^-1/2 A D^-1/2)."""
    if c["graph"] == "er":
        return inputs.erdos_renyi(c["n"], c["n"] * c["deg"] // 2, seed), None
    if c["graph"] == "rmat":
        return _rmat(c["scale"], c["ef"], bool(c.get("directed")), seed), None
    g = inputs.barabasi_albert(c["n"], c["m"], seed)
    if not c.get("weighted"):
        return g, None
    deg = np.diff(g.row_ptr).astype(np.float64)
    rows = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    return g, 1.0 / np.sqrt(deg[rows] * deg[g.col_idx])


def _alpha(g, w):
    """1 / (maximum out-degree + 1); weighted graphs: half the inverse of the
    largest weighted out-degree."""
    if w is not None:
        return 0.5 / float(np.bincount(g.col_idx, weights=w, minlength=g.n).max())
    return 1.0 / (int(np.bincount(g.col_idx, minlength=g.n).max()) + 1.0)


def _groups(c, n, seed):
    if c["kind"] == "score":
        return np.array([0, c["size"]], dtype=np.int64), inputs.group(n, c["size"], seed + 7)
    return inputs.groups(n, c["groups"], 1, min(c["smax"], n), seed + 7)


def prepare(case, seed):
    g, w = _graph(case, seed + 1)
    gg = ged.GedGraph.from_graph(g, weights=w)
    alpha = _alpha(g, w)
    gg.prepare(alpha, EPS)
    st = {"case": case, "gg": gg, "alpha": alpha, "seed": seed}
    if case["kind"] in ("score", "batch"):
        st["offsets"], st["members"] = _groups(case, g.n, seed)
    return st


def run(state):
    c, gg, alpha = state["case"], state["gg"], state["alpha"]
    if c["kind"] == "score":
        s, ell, bound = gg.score(state["members"], alpha, EPS, with_info=True)
        return {"score": np.array([s]), "ell": np.array([ell]), "bound": np.array([bound])}
    if c["kind"] == "batch":
        return {"scores": gg.score_batch(state["offsets"], state["members"], alpha, EPS)}
    if "eta" in c:
        r = gg.greedy_stochastic(c["k"], alpha, EPS, eta=c["eta"], seed=state["seed"] + 3)
    else:
        r = gg.greedy(c["k"], alpha, EPS)
    return {"group": r["group"], "ell": r["ell"], "L1": r["L1"], "U2": r["U2"], "L2": r["L2"],
            "B": r["B"], "score": np.array([r["score"]])}


def work(case):
    """The graph once (row pointers, sources, weights), the groups and the
    results; one multiply-add per arc for each group scored or vertex chosen."""
    n, arcs = _vertices(case), _arcs(case)
    cols = {"score": 1, "batch": case.get("groups", 1), "greedy": case.get("k", 1)}[case["kind"]]
    members = {"score": case.get("size", 0), "batch": cols * case.get("smax", 0) // 2,
               "greedy": cols}[case["kind"]]
    per_arc = 12 if case.get("weighted") else 4
    return {"bytes": 4.0 * (n + 1) + per_arc * arcs + 4.0 * members + 8.0 * cols,
            "flops": 2.0 * arcs * cols}


# ------------------------------------------------------------------ exact --

def _levels(A, deg, alpha, n):
    """Total walk levels t_0 .. t_ell* and the tail bound (Eq. comb-bound)."""
    t = [torch.ones(n, dtype=torch.float64, device=A.device)]
    while True:
        t.append(alpha * (A @ t[-1]))
        bound = alpha * (deg / (1.0 - alpha * deg)) * float(t[-1].sum())
        if bound < EPS:
            return t, bound


def _matrix(g, w, dev):
    vals = np.ones(g.nnz) if w is None else w
    return torch.sparse_csr_tensor(torch.from_numpy(g.row_ptr), torch.from_numpy(g.col_idx).long(),
                                   torch.from_numpy(vals), size=(g.n, g.n)).to(dev)


def _exact_scores(A, t, alpha, offsets, members):
    """Level-by-level hit chains (Section 3.1.1) of all groups, 64 at a time."""
    G, n = len(offsets) - 1, A.shape[0]
    out = []
    for g0 in range(0, G, 64):
        cols = min(64, G - g0)
        mask = torch.zeros(n, cols, dtype=torch.bool, device=A.device)
        for j in range(cols):
            mem = members[offsets[g0 + j]:offsets[g0 + j + 1]]
            mask[torch.from_numpy(mem).long().to(A.device), j] = True
        h = mask.to(torch.float64)
        tot = torch.zeros(cols, dtype=torch.float64, device=A.device)
        for ti in t[1:]:
            h = alpha * (A @ h)
            h = torch.where(mask, ti[:, None], h)
            tot += h.sum(0)
        out.append(tot.cpu().numpy())
    return np.concatenate(out)


def _exact_greedy(A, g, alpha, deg, k):
    """Greedy on a small graph from the dense matrix: the exact gains of every
    vertex at every step (Section 3.2.2), ties to the smaller id."""
    n = g.n
    A = A.to_dense()
    t0 = torch.ones(n, dtype=torch.float64, device=A.device)
    out = {"group": [], "ell": [], "L1": [], "U2": [], "L2": [], "B": []}
    inS = torch.zeros(n, dtype=torch.bool, device=A.device)
    eye = torch.eye(n, dtype=torch.float64, device=A.device)
    ell = 1
    while len(out["group"]) < k:
        t = t0
        for _ in range(ell):
            t = alpha * (A @ t)
        B = alpha * (deg / (1.0 - alpha * deg)) * float(t.sum())
        free = (~inS).to(torch.float64)
        m, D, L = free.clone(), eye * free[:, None], torch.zeros(n, dtype=torch.float64,
                                                                 device=A.device)
        for _ in range(ell):
            m = free * (alpha * (A @ m))
            D = free[:, None] * (alpha * (A @ D))
            D[torch.arange(n), torch.arange(n)] = m
            L += D.sum(0)
        gains = L.cpu().numpy()
        gains[inS.cpu().numpy()] = -1.0
        order = np.lexsort((np.arange(n), -gains))
        u, v = int(order[0]), int(order[1])
        if gains[u] <= gains[v] + B - EPS / k:
            ell *= 2
            continue
        for key, x in zip(out, (u, ell, gains[u], gains[v] + B, gains[v], B)):
            out[key].append(x)
        inS[u] = True
    return {key: np.array(x) for key, x in out.items()}


def exact(case, seed):
    if case["kind"] == "greedy" and ("eta" in case or case.get("directed") or
                                     case.get("weighted") or _vertices(case) > 1500):
        return None
    if case["kind"] == "batch" and float(_arcs(case)) * case["groups"] > 4e10:
        return None
    g, w = _graph(case, seed + 1)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    A = _matrix(g, w, dev)
    alpha = _alpha(g, w)
    deg = float(np.bincount(g.col_idx, weights=w, minlength=g.n).max())
    t, bound = _levels(A, deg, alpha, g.n)
    if case["kind"] == "greedy":
        r = _exact_greedy(A, g, alpha, deg, case["k"])
        members = r["group"].astype(np.int32)
        r["score"] = _exact_scores(A, t, alpha, [0, len(members)], members)
        return r
    offsets, members = _groups(case, g.n, seed)
    s = _exact_scores(A, t, alpha, offsets, members)
    if case["kind"] == "batch":
        return {"scores": s}
    return {"score": s, "ell": np.array([len(t) - 1]), "bound": np.array([bound])}
