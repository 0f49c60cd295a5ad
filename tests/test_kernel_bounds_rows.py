"""Index arithmetic of the row sums over 16-bit counts, the lower arcs, the
segments that finish long rows and the slices of small graphs, emulated on the
CPU (no GPU), on the graphs and with the partition of test_kernel_bounds."""
import numpy as np
import pytest

from paper_1910_13874_amd import inputs
from test_kernel_bounds import (K_BLOCK, K_LDS, check_plan_matches_emulation, check_quads,
                                check_step, graphs, internal_csr, partition)

INLINE_FIX_SEGS = 2048


def check_quad_rows(rp, ci, n, C, NC, cut_div, rng):
    """Phase 2 of a 16-bit row block with NC columns per lane: lane t takes
    columns NC*k .. of row slot t/(LA*tpr), striding the row's arcs by tpr, and
    the tpr lanes of a row lie in one wavefront; every row and column is summed
    once, from staged slots only, and stored inside its level."""
    GU, LA = C // 4, C // NC
    blocks, _, _ = partition(rp, C, GU, cut_div)
    x = rng.integers(0, 65535, (n, C)).astype(np.int64)
    picked = sorted(set([0, len(blocks) - 1] + rng.integers(0, max(1, len(blocks)), 6).tolist()))
    for b in picked if blocks else []:
        r0, r1, p0, p1 = blocks[b]
        nrows, arcs = r1 - r0, p1 - p0
        vals = x[ci[p0:p1]]                      # [arcs][C] staged halves
        assert 2 * vals.size <= 8 * K_LDS        # LDS bytes
        assert arcs <= K_LDS                     # 32-bit sums of 16-bit values
        tpr = min(64 // LA, 64)
        while tpr > 1 and nrows * LA * tpr > K_BLOCK:
            tpr >>= 1
        assert LA * tpr <= 64
        rstep = K_BLOCK // LA // tpr
        t = np.arange(K_BLOCK)
        k, s, slot = t & (LA - 1), (t // LA) & (tpr - 1), t // LA // tpr
        assert (t // 64 == (slot * LA * tpr) // 64).all()  # a row's lanes: one wavefront
        # early loads of the combining step
        assert (r0 + np.minimum(slot, nrows - 1)).max() < n
        seen = np.zeros((nrows, LA), int)
        for rl0 in range(0, nrows, rstep):
            rl = rl0 + slot
            for lane in np.flatnonzero((rl < nrows) & (s == 0)):
                row = rl[lane]
                j0, j1 = rp[r0 + row] - p0, rp[r0 + row + 1] - p0
                idx = np.concatenate([np.arange(j0 + q, j1, tpr) for q in range(tpr)])
                assert idx.size == j1 - j0 and (idx.size == 0 or idx.max() * LA + k[lane] < arcs * LA)
                cols = slice(NC * k[lane], NC * k[lane] + NC)
                want = x[ci[rp[r0 + row]:rp[r0 + row + 1]], cols].sum(axis=0)
                assert (vals[idx, cols].sum(axis=0) == want).all()
                assert (r0 + row) * C + NC * k[lane] + NC <= n * C
                seen[row, k[lane]] += 1
        assert (seen == 1).all()


def lower_csr(rp, ci):
    """Of each row the sources before it: a prefix of the row."""
    rows = np.repeat(np.arange(len(rp) - 1), np.diff(rp))
    low = ci < rows
    rl = np.concatenate([[0], np.cumsum(np.bincount(rows[low], minlength=len(rp) - 1))])
    for v in range(0, len(rp) - 1, max(1, len(rp) // 50)):
        m = rl[v + 1] - rl[v]
        assert low[rp[v]:rp[v] + m].all() and not low[rp[v] + m:rp[v + 1]].any()
    return rl.astype(np.int64), ci[low]


@pytest.mark.parametrize("g", graphs(), ids=lambda g: g.name or str(g.n))
def test_quad_rows_and_lower_arcs(g):
    from paper_1910_13874_amd import ged
    rng = np.random.default_rng(3)
    rp, ci = internal_csr(g)
    sides = [(rp, ci)]
    if not g.directed:
        rl, cl = lower_csr(rp, ci)
        assert 2 * rl[-1] == rp[-1]
        sides.append((rl, cl))
        for C in (1, 2, 8, 64):
            check_step(rl, cl, g.n, C)
            if C >= 2:
                check_step(rl, cl, g.n, C, pairs=True, cut_div=2)
        for C in (4, 64):
            check_quads(rl, cl, g.n, C, 1, g.n // 8)
        for U, cut_div in ((1, 1), (4, 2), (16, 1)):
            check_plan_matches_emulation(ged, rl, cl, g.n, U, cut_div)
    for r, c in sides:
        for C in (4, 8, 16, 32, 64):
            for NC in (2, 4):
                check_quad_rows(r, c, g.n, C, NC, 1, rng)
        check_quad_rows(r, c, g.n, 16, 4, 4, rng)


@pytest.mark.parametrize("g", graphs(), ids=lambda g: g.name or str(g.n))
def test_segments_finish_rows(g):
    """The last of a long row's segments adds them: 64 lanes, S = 64/C per
    column in strides of 4 S and S, take every segment of the row once; the
    counters' buffer covers every partition that counts."""
    rp, ci = internal_csr(g)
    for C, U in [(c, c) for c in (1, 2, 4, 8, 16, 32, 64)] + [(8, 2), (64, 16), (64, 32)]:
        for cut_div in (1, 4):
            _, segs, lrows = partition(rp, C, U, cut_div)
            first = {}
            for q, (r, _, _) in enumerate(segs):
                first.setdefault(r, []).append(q)
            if len(segs) <= INLINE_FIX_SEGS:
                assert len(lrows) <= INLINE_FIX_SEGS
            S = 64 // C
            t = np.arange(64)
            for r in lrows:
                q0, q1 = first[r][0], first[r][-1] + 1
                assert first[r] == list(range(q0, q1))
                for c in {0, C - 1}:
                    took = []
                    for lane in t[(t & (C - 1)) == c]:
                        q = q0 + lane // C
                        while q + 3 * S < q1:
                            took += [q + k * S for k in range(4)]
                            q += 4 * S
                        took += list(range(q, q1, S))
                    assert sorted(took) == list(range(q0, q1))


def slices(rp, ci, n, L):
    """The slices of one direction: (chunks sorted by length, off, col, rows of
    several chunks with their first slots)."""
    ch, multi, first, slots = [], [], [], 0
    for v in range(n):
        d = int(rp[v + 1] - rp[v])
        if d <= L:
            ch.append((v, int(rp[v]), d, -1))
            continue
        multi.append(v)
        first.append(slots)
        for j in range(int(rp[v]), int(rp[v + 1]), L):
            ch.append((v, j, min(L, int(rp[v + 1]) - j), slots))
            slots += 1
    first.append(slots)
    ch.sort(key=lambda c: -c[2])
    ns = (len(ch) + 63) // 64
    off = np.concatenate([[0], np.cumsum([(ch[64 * s][2] + 3) // 4 for s in range(ns)])])
    col = np.full(int(off[-1]) * 256, n, np.int64)
    for c, (v, j0, d, _) in enumerate(ch):
        s, lane = c // 64, c % 64
        for j in range(d):
            col[((off[s] + j // 4) * 64 + lane) * 4 + j % 4] = ci[j0 + j]
    return ch, off, col, multi, first, slots


@pytest.mark.parametrize("name", ["er", "star", "dir", "edgeless", "ba"])
def test_small_graph_slices(name):
    """A level over the slices is the product with the CSR: every arc once,
    padding reads the zero behind the vector, chunks of a row meet in their
    slots, and the vector, slots and bits fit the workgroup's LDS."""
    if name == "star":
        leaf = np.arange(1, 5000, dtype=np.int32)
        g = inputs.from_edges(5000, np.zeros(4999, np.int32), leaf)
    elif name == "dir":
        r = inputs.uniform_ints(2 * 9000, 2000, 61)
        g = inputs.from_edges(2000, r[0::2], r[1::2], symmetrize=False)
    else:
        g = {"er": lambda: inputs.erdos_renyi(1500, 9000, 7),
             "ba": lambda: inputs.barabasi_albert(3000, 9, 2),
             "edgeless": lambda: inputs.from_edges(70, [], [])}[name]()
    rp, ci = internal_csr(g)
    n = g.n
    L = 16 if rp[-1] <= 32 << 10 else 32
    ch, off, col, multi, first, slots = slices(rp, ci, n, L)
    assert 8 * (n + 1 + slots + len(multi) + 16) + 4 * ((n + 31) // 32) <= 160 * 1024 - 1024
    assert n < 1 << 16 and -(-len(off[1:]) // 16) <= 18
    x = np.append(np.random.default_rng(1).integers(0, 1000, n), 0).astype(np.int64)
    y, part = np.zeros(n, np.int64), np.zeros(max(slots, 1), np.int64)
    for c, (v, _, _, slot) in enumerate(ch):
        s, lane = c // 64, c % 64
        at = ((np.arange(off[s], off[s + 1])[:, None] * 64 + lane) * 4 + np.arange(4)).ravel()
        assert at.size <= 4 * (L // 4) and (at.size == 0 or at.max() < col.size)
        total = x[col[at]].sum()
        if slot < 0:
            y[v] = total
        else:
            part[slot] = total
    for m, v in enumerate(multi):  # eight lanes stride the row's slots
        y[v] = sum(part[first[m] + k:first[m + 1]:8].sum() for k in range(8))
    rows = np.repeat(np.arange(n), np.diff(rp))
    assert (y == np.bincount(rows, weights=x[ci], minlength=n).astype(np.int64)).all()


def test_unchecked_tile_pushes():
    """Tile pushes add to member rows below the hubs' test without asking: every
    sum stays within omega_2 (so a 16-bit half of at most 2^16 - 2 never
    carries), and rows outside the group hold the counts of the checked push.
    Groups around hubs, their neighbours and each other."""
    g = inputs.barabasi_albert(3000, 6, 8)
    rp, ci = internal_csr(g)
    n = g.n
    deg = np.diff(rp)
    hubs = int((deg > 128).sum())
    assert 0 < hubs < n and (deg[:hubs] > 128).all()
    rows = np.repeat(np.arange(n), deg)
    omega2 = np.bincount(rows, weights=deg[ci], minlength=n).astype(np.int64)
    rng = np.random.default_rng(2)
    near = ci[rp[hubs]:rp[hubs + 1]]
    for S in (np.array([0]), np.unique(near), np.unique(rng.integers(0, n, 400)),
              np.arange(hubs + 40), np.arange(n)):
        member = np.zeros(n, bool)
        member[S] = True
        cnt1 = np.bincount(ci[member[rows]], minlength=n)          # one per arc s -> y
        cnt2 = np.bincount(ci[member[rows]], weights=deg[rows[member[rows]]], minlength=n)
        src = ~member[rows] & (cnt1[rows] > 0)                      # arcs y -> x of the worklist
        add = src & ~((ci < hubs) & member[ci])
        cnt2 = (cnt2 + np.bincount(ci[add], weights=cnt1[rows[add]], minlength=n)).astype(np.int64)
        assert (cnt2 <= omega2).all()
        checked = src & ~member[ci]
        want = np.bincount(ci[member[rows]], weights=deg[rows[member[rows]]], minlength=n) + \
            np.bincount(ci[checked], weights=cnt1[rows[checked]], minlength=n)
        assert (cnt2[~member] == want[~member]).all()
