"""Plans with aggregations in chunks of high colours, beside their plain use:
which of the other aggregations take their sorted entries, last passes of
fewer colourings, fixed areas and batches, neighbour ranges with weights."""
import numpy as np
import pytest

import graphgen as gg
import oracle as O
import paper_2009_11665_amd as sg

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32s": 1e-5}  # bounds of the modes
CAT12 = [-1, 0, 1, 2, 3, 4, 5, 1, 2, 3, 4, 5]


def random_graph(n, deg, seed, weighted=False):
    rng = np.random.default_rng(seed)
    e = np.sort(rng.integers(0, n, (int(n * deg), 2)), axis=1)
    e = np.unique(e[e[:, 0] != e[:, 1]], axis=0)
    e = e[rng.permutation(len(e))[:int(n * deg / 2)]]
    w = rng.uniform(0.5, 1.5, len(e)) if weighted else None
    return gg.from_edge_list(n, [(int(a), int(b)) for a, b in e], w)


@pytest.mark.parametrize("par,k", [(gg.PATH8, 12), (CAT12, 13), (gg.BINTREE15, 15)])
@pytest.mark.parametrize("side", [-1, 1])
def test_sorted_entries_by_mean_degree(par, k, side):
    """Mean degrees on both sides of 8 k: staged rows and sorted entries of the
    aggregations of 220 to 495 sets; 66 and 78 sets are LDS sums on both."""
    n = 400
    G = random_graph(n, 8 * k + 4 * side, 3 * k + side)
    assert (G.nnz >= 8 * k * n) == (side > 0)
    g = sg.Graph.from_csr(G)
    plan = sg.Plan(par, k)
    c = sg.Colorings(g, k, 2, 2)
    for mode in ("fp32s", "fp64"):
        print("sorted entries", par, k, side, mode, flush=True)
        got = sg.count(plan, g, c, mode)["colorful"]
        with sg.tuned(flags=sg.TUNE_NO_COLOR_SKIP):
            full = sg.count(plan, g, c, "fp64")["colorful"]
        for j in range(2):
            f = O.count(G, par, k, O.colors(n, k, 2, j))[0]
            assert f > 0
            assert got[j] == pytest.approx(f, rel=TOL[mode])
            assert full[j] == pytest.approx(f, rel=TOL["fp64"])
