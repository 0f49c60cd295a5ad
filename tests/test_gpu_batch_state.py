"""What a batch leaves in the handle's workspace for the next one: sequences of
batches, settings and profiled calls whose later results would show counts or
buffers kept from an earlier one (GPU, against the CPU oracle)."""
import numpy as np
import pytest

import oracle
from paper_1910_13874_amd import inputs

pytestmark = pytest.mark.gpu

REL = 1e-9


@pytest.fixture(scope="module")
def ged():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_1910_13874_amd import ged
    return ged


def rel(a, b):
    return abs(a - b) / max(abs(b), 1e-300)


def flat(groups):
    off = np.concatenate([[0], np.cumsum([len(S) for S in groups])]).astype(np.int64)
    return off, np.concatenate(groups).astype(np.int32)


class Pair:
    """A heavy batch (level 2 gathered, 16-bit copies) and a light one (level 2
    pushed) on a skewed graph, with the oracle's scores."""

    def __init__(self, ged, tile):
        g = inputs.rmat(14, 16, seed=43)
        self.gg = ged.GedGraph.from_graph(g)
        self.alpha, self.eps = g.default_alpha(), 1e-4  # FP64 stored levels
        if tile:
            self.gg.set_batch_tile(tile)
            self.gg.set_batch_row_cut(1)
        by_deg = np.argsort(-g.degrees, kind="stable").astype(np.int32)
        heavy = [by_deg[:1], np.sort(by_deg[:40])] + [inputs.group(g.n, 300, 10 + j)
                                                      for j in range(70)]
        low = by_deg[g.degrees[by_deg] > 0][-3:]
        light = [low[j:j + 1] for j in range(3)] * 24  # as many tiles
        self.heavy, self.light = flat(heavy), flat(light)
        self.want_heavy = [oracle.score(g, S, self.alpha, self.eps)[0] for S in heavy[:4]]
        self.want_light = [oracle.score(g, S, self.alpha, self.eps)[0] for S in light[:3]]

    def steps(self, batch):
        """Step launches of a batch of 72 groups (profiled, so eager)."""
        self.gg.profile_enable(True)
        self.gg.score_batch(*batch, self.alpha, self.eps)
        n = self.gg.profile_read()["launches"]
        self.gg.profile_enable(False)
        return n

    def run_heavy(self):
        s = self.gg.score_batch(*self.heavy, self.alpha, self.eps)
        assert max(rel(x, c) for x, c in zip(s, self.want_heavy)) <= REL
        return s

    def run_light(self):
        s = self.gg.score_batch(*self.light, self.alpha, self.eps)
        assert max(rel(x, self.want_light[j % 3]) for j, x in enumerate(s)) <= REL


@pytest.mark.parametrize("tile", [0, 16, 64])
def test_pushed_batch_after_replayed_gathered_batch(ged, tile):
    """A replay of the captured heavy batch leaves level 2 as the capture did:
    the pushed batch after it starts from zero counts, also where a call in
    between cleared them (a profiled batch, which runs eagerly and keeps the
    captured graph; a new width race)."""
    p = Pair(ged, tile)
    first = p.run_heavy()
    if tile:  # one more step per tile where level 2 is gathered
        assert p.steps(p.heavy) == p.steps(p.light) + -(-72 // tile)
    p.run_light()
    p.run_heavy()                  # captured
    p.gg.profile_enable(True)
    p.run_light()                  # eager: level 2 cleared, the capture kept
    p.gg.profile_enable(False)
    assert np.array_equal(p.run_heavy(), first)  # replayed
    p.run_light()
    if tile == 0:
        p.run_heavy()
        p.gg.set_batch_tile(0)     # the race's narrow tiles clear level 2
        p.run_heavy()
        p.run_light()
    p.gg.close()


@pytest.mark.parametrize("kind", ["directed", "undirected"])
def test_captured_batch_after_wider_long_rows(ged, kind):
    """A captured batch is replayed after profiled (eager) batches at narrower
    tiles and lower row-split thresholds, whose partitions have more long rows:
    the long rows' counters are those it was captured with."""
    n = 60_000
    hubs = [(h, 140 + 90 * h) for h in range(60)] + [(60, 9000), (61, 50_000)]
    r = inputs.uniform_ints(2 * 40_000, n, 5).astype(np.int32)
    src = np.concatenate([r[0::2]] + [np.arange(100, 100 + d, dtype=np.int32) for _, d in hubs])
    dst = np.concatenate([r[1::2]] + [np.full(d, h, np.int32) for h, d in hubs])
    g = inputs.from_edges(n, src, dst, symmetrize=kind != "directed")
    gg = ged.GedGraph.from_graph(g)
    alpha, eps = 0.5 * oracle.default_alpha(g, None), 1e-3
    groups = [inputs.group(n, 5, 1), np.array([60], np.int32), np.array([0, 30, 61], np.int32),
              inputs.group(n, 300, 2)] * 17
    off, mem = flat(groups)
    want = [oracle.score(g, S, alpha, eps)[0] for S in groups[:4]]

    def batch(tile, cut, profiled=False):
        gg.set_batch_tile(tile)
        gg.set_batch_row_cut(cut)
        gg.profile_enable(profiled)
        s = gg.score_batch(off, mem, alpha, eps)
        gg.profile_enable(False)
        assert max(rel(x, want[j % 4]) for j, x in enumerate(s)) <= REL, (tile, cut)
        return s

    first = batch(64, 1)
    for tile, cut in ((32, 4), (16, 4), (8, 1)):
        batch(tile, cut, True)
        assert np.array_equal(batch(64, 1), first)
    s = gg.score(groups[3], alpha, eps)
    assert rel(s, want[3]) <= REL and gg.score(groups[3], alpha, eps) == s
    gg.close()


def test_captured_16bit_batch_after_wider_copy(ged):
    """A batch in the 16-bit layout with two stored levels is replayed after a
    profiled batch at twice the width with one stored level: the same bytes of
    stored levels, but a larger 16-bit copy, which the capture has to follow."""
    g = inputs.erdos_renyi(30_000, 120_000, 11)
    gg = ged.GedGraph.from_graph(g)
    gg.set_count16(0)
    alpha = 0.4 / g.max_degree
    eps_of = {}
    for e in range(80):
        eps = 10.0 ** (4 - 0.25 * e)
        eps_of.setdefault(gg.prepare(alpha, eps)[0], eps)
    groups = [inputs.group(g.n, 3 + 5 * j, j) for j in range(20)]
    off, mem = flat(groups)

    def batch(tile, ell, profiled=False):
        gg.set_batch_tile(tile)
        gg.set_batch_row_cut(1)
        gg.profile_enable(profiled)
        s = gg.score_batch(off, mem, alpha, eps_of[ell])
        gg.profile_enable(False)
        assert gg.count16_hub() == 0
        for j in (0, 7, 19):
            assert rel(s[j], oracle.score(g, groups[j], alpha, eps_of[ell])[0]) <= REL
        return s

    first = batch(8, 10)
    batch(16, 8, True)
    assert np.array_equal(batch(8, 10), first)
    gg.close()


def test_more_groups_than_one_launch(ged):
    """A batch on a small graph with more groups than one launch of a workgroup
    each takes (2^22 groups are 2^32 threads): every score is that of its
    group, whichever launch it fell into."""
    g = inputs.erdos_renyi(40, 90, 3)
    gg = ged.GedGraph.from_graph(g)
    alpha, eps = g.default_alpha(), 1e-2
    G = (1 << 22) + 1000
    mem = (np.arange(G, dtype=np.int64) * 7 % g.n).astype(np.int32)
    s = gg.score_batch(np.arange(G + 1, dtype=np.int64), mem, alpha, eps)
    one = np.array([oracle.score(g, np.array([v], np.int32), alpha, eps)[0] for v in range(g.n)])
    assert (np.abs(s - one[mem]) <= REL * one[mem]).all()  # isolated vertices score 0
    gg.close()


@pytest.mark.parametrize("keep_order", [False, True])
@pytest.mark.parametrize("tile,count16", [(2, -1), (8, 0), (64, -1), (64, 0)])
def test_pushed_tiles_with_member_hubs(ged, keep_order, tile, count16):
    """Pushed tiles whose groups hold hubs (tested as members by the push),
    their neighbours and vertices around the test's degree line (128), in the
    32-bit and the 16-bit layout and with the caller's vertex order."""
    g = inputs.barabasi_albert(40_000, 3, 12)
    gg = ged.GedGraph.from_graph(g, keep_order=keep_order)
    gg.set_batch_tile(tile)
    gg.set_batch_row_cut(1)
    if count16 < 0:
        gg.set_count16(-1)
    by_deg = np.argsort(-g.degrees, kind="stable").astype(np.int32)
    line = int((g.degrees > 128).sum())
    assert 8 < line < 2000
    hub = by_deg[0]
    groups = [by_deg[:1], by_deg[:20], by_deg[line - 2:line + 2], by_deg[line:line + 1],
              np.concatenate([[hub], g.col_idx[g.row_ptr[hub]:g.row_ptr[hub + 1]][:50]]),
              inputs.group(g.n, 30, 4)] + [np.concatenate([by_deg[j:j + 1], inputs.group(g.n, 20, j)])
                                           for j in range(2, 70)]
    groups = [np.unique(S).astype(np.int32) for S in groups]
    alpha, eps = g.default_alpha(), 1e-4
    s = gg.score_batch(*flat(groups), alpha, eps)
    for j in list(range(8)) + [40, 73]:
        assert rel(s[j], oracle.score(g, groups[j], alpha, eps)[0]) <= REL, (tile, j)
    gg.close()
