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


def ring(n, deg, weighted):
    """Every vertex and its deg nearest on a ring; weights of 0.5 to 1.5."""
    d = np.arange(1, deg // 2 + 1)
    ci = (np.arange(n)[:, None] + np.concatenate([-d, d])) % n
    w = 0.5 + (ci * np.arange(n)[:, None] % 97) / 96.0 if weighted else None
    order = np.argsort(ci, axis=1)
    ci = np.take_along_axis(ci, order, axis=1).astype(np.int32).reshape(-1)
    if weighted:
        w = np.take_along_axis(w, order, axis=1).astype(np.float32).reshape(-1)
    return sg.Graph(n, np.arange(n + 1, dtype=np.int64) * deg, ci, w)


def test_budget_counts_the_sorted_entries():
    """A budget that holds the tables but not the 24 MB of sorted entries beside them:
    the count runs in absolute tables (whose one-vertex multiply-adds the relative
    ones do not have), with the same results."""
    n, deg = 3000, 1000
    g = ring(n, deg, True)
    plan = sg.Plan(gg.PATH8, 12)
    tables = plan.info().bytes_per_vertex_fp32 * n
    assert tables < 8 * deg * n
    c = sg.Colorings(g, 12, 4, 3)
    ref = sg.count(plan, g, c, "fp64")["colorful"]
    for budget, absolute in ((tables + (2 << 20), True), (0, False)):
        print("budget", budget, flush=True)
        with sg.tuned(budget_bytes=budget):
            sg.profile_start()
            got = sg.count(plan, g, c, "fp32s")["colorful"]
            prof = sg.profile_stop()
        assert (prof["ema_single"]["launches"] > 0) == absolute
        np.testing.assert_allclose(got, ref, rtol=TOL["fp32s"])


@pytest.mark.parametrize("n,deg", [(3700, 8), (7000, 1000)])
def test_chunks_inside_the_fixed_area(n, deg):
    """sg2v_count_noalloc: sorted entries beside the tables in the area, and a graph
    whose 56 MB of sorted entries do not fit there with them (absolute tables)."""
    g = ring(n, deg, True)
    plan = sg.Plan(gg.PATH8, 12)
    c = sg.Colorings(g, 12, 4, 2)
    print("noalloc, chunks", n, deg, flush=True)
    ref = sg.count(plan, g, c, "fp64")["colorful"]
    got = sg.count_noalloc(plan, g, c, "fp32s")["colorful"]
    assert (np.asarray(ref) > 0).all()
    np.testing.assert_allclose(got, ref, rtol=TOL["fp32s"])
