"""The step kernels on graphs that scores, batches and greedy runs otherwise
take through one workgroup (ged_small.hip): the oracle comparisons of
test_gpu_parity with profiling left on, which keeps every call on the steps,
and the sizes at which the choice changes."""
import numpy as np
import pytest

import oracle
import test_gpu_parity as parity
from paper_1910_13874_amd import inputs

pytestmark = pytest.mark.gpu

REL = 1e-9


@pytest.fixture(scope="module")
def ged():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_1910_13874_amd import ged
    return ged


class Stepped:
    """The module with graph handles that stay profiled."""

    def __init__(self, ged):
        self._ged = ged
        self.handles = []
        outer = self

        class GedGraph(ged.GedGraph):
            def __init__(self, *a, **k):
                super().__init__(*a, **k)
                self.steps = 0
                outer.handles.append(self)
                super().profile_enable(True)

            def profile_enable(self, on=True):  # restarts the record, never ends it
                self.steps += self.profile_read()["launches"]
                super().profile_enable(True)

            def close(self):
                if getattr(self, "_h", None) is not None:
                    self.steps += self.profile_read()["launches"]
                super().close()

        self.GedGraph = GedGraph

    def __getattr__(self, name):
        return getattr(self._ged, name)


@pytest.mark.parametrize("test,args", [
    ("test_score_parity", ("er1k",)), ("test_greedy_parity", ("er1k", 5)),
    ("test_split_ell_sweep", ("er",)), ("test_split_ell_sweep", ("ba",)),
    ("test_split_ell_sweep", ("weighted",)), ("test_directed_score_and_greedy", ()),
    ("test_greedy_width_parity", (0,)), ("test_greedy_width_parity", (2,)),
    ("test_greedy_width_parity", (16,)), ("test_greedy_multigraph", ()),
    ("test_greedy_gain_layout", ()), ("test_greedy_ties_smallest_id", ()),
    ("test_weighted_parity", ()), ("test_stochastic_greedy_parity", ()),
    ("test_score_pushed_level3", ("sparse_er",)), ("test_score_pushed_level3", ("multigraph",)),
    ("test_split_count_layout", ("sparse_er",)), ("test_greedy_selection_ties", (1025,)),
    ("test_batch_matches_solo_and_oracle", ())],
    ids=lambda x: x if isinstance(x, str) else "-".join(map(str, x)))
def test_by_steps(ged, test, args):
    m = Stepped(ged)
    getattr(parity, test)(m, *args)
    assert m.handles and all(h.steps > 0 for h in m.handles)


@pytest.mark.parametrize("n,m,kind", [(6144, 16_000, "weighted"), (6145, 16_000, "weighted"),
                                      (8192, 16_000, "plain"), (8193, 16_000, "plain"),
                                      (10_240, 30_000, "directed"), (10_241, 30_000, "directed"),
                                      (14_337, 55_000, "weighted"), (16_385, 30_000, "directed")])
def test_around_the_choice(ged, n, m, kind):
    """Scores, a greedy run and batches of 64 and 65 groups on both sides of
    the sizes up to which one workgroup runs a single chain, and up to the
    largest whose batches do."""
    g = parity._random_graph(n, m, 5 + n, kind == "directed")
    w = None
    if kind == "weighted":
        deg = g.degrees.astype(np.float64)
        rows = np.repeat(np.arange(g.n), g.degrees)
        w = 1.0 / np.sqrt(deg[rows] * deg[g.col_idx])
    gg = ged.GedGraph.from_graph(g, weights=w)
    alpha, eps = 0.5 * oracle.default_alpha(g, w), 1e-3
    groups = [inputs.group(n, 1 + j, 3 + j) for j in range(65)]
    off = np.concatenate([[0], np.cumsum([len(S) for S in groups])]).astype(np.int64)
    mem = np.concatenate(groups).astype(np.int32)
    s64 = gg.score_batch(off[:65], mem[:off[64]], alpha, eps)
    s65 = gg.score_batch(off, mem, alpha, eps)
    assert np.array_equal(s64, s65[:64])  # a group's bits do not depend on the batch
    for j in (0, 30, 64):
        want = oracle.score(g, groups[j], alpha, eps, w=w)[0]
        assert parity.rel(gg.score(groups[j], alpha, eps), want) <= REL
        assert parity.rel(s65[j], want) <= REL, j
    rev = inputs.reverse(g) if kind == "directed" else None
    parity.compare_greedy(gg.greedy(2, alpha, eps),
                          oracle.greedy(g, 2, alpha, eps, w=w, **({"rev": rev} if rev else {})),
                          (kind, n))
    gg.close()
