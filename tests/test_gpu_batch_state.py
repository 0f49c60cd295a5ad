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
