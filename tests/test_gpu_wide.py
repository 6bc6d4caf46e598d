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


@pytest.mark.parametrize("weighted", [False, True])
def test_last_pass_of_fewer_colourings_sorts_again(weighted):
    n = 900
    G = random_graph(n, 12, 4, weighted)
    g = sg.Graph.from_csr(G)
    plan = sg.Plan(gg.PATH8, 12)
    c = sg.Colorings(g, 12, 6, 6)
    with sg.tuned(batch=4):
        for mode in ("fp64", "fp32s") + (() if weighted else ("u64",)):
            print("partial pass, chunks", weighted, mode, flush=True)
            r = sg.count(plan, g, c, mode)
            for j in range(6):
                f, u, _ = O.count(G, gg.PATH8, 12, O.colors(n, 12, 6, j), mode=O.U64 if mode == "u64" else O.FP64)
                if mode == "u64":
                    assert int(r["colorful_u64"][j]) == u
                else:
                    assert r["colorful"][j] == pytest.approx(f, rel=TOL[mode])


@pytest.mark.parametrize("flags", [0, 512])
def test_chunks_recorded_in_a_batch(flags):
    """Sorting and chunked aggregations inside the recorded graph, templates as parallel
    branches and one after another, replayed with eager work in between."""
    G = random_graph(2000, 10, 8)
    g = sg.Graph.from_csr(G)
    plans = [sg.Plan(gg.PATH8, 12), sg.Plan(gg.BINTREE7, 7), sg.Plan(CAT12, 13)]
    with sg.tuned(flags=flags):
        for mode in ("u64", "fp32s"):
            first = None
            for rep in range(3):
                print("batch, chunks", flags, mode, rep, flush=True)
                cf, _ = sg.count_batch(plans, g, 5, 3, mode)
                first = cf if first is None else first
                np.testing.assert_array_equal(cf, first)
                sg.count(plans[2], g, sg.Colorings(g, 13, 40 + rep, 2), mode)
            for p, plan in enumerate(plans):
                ref = sg.count(plan, g, sg.Colorings(g, plan.k, 5, 3), "fp64")["colorful"]
                np.testing.assert_allclose(first[p], ref, rtol=TOL["fp32s"])


def test_neighbour_ranges_with_weights():
    """Long tasks taken once per neighbour range, their weights with them."""
    G = gg.rmat(18, 25_000_000, seed=5)
    rows = np.repeat(np.arange(G.n, dtype=np.int64), np.diff(G.row_ptr))
    G.w = (0.5 + ((rows + G.col_idx) * 2654435761 % 997) / 996.0).astype(np.float32)
    plan = sg.Plan(gg.PATH8, 12)
    for relabel in (False, True):
        g = sg.Graph.from_csr(G, relabel=relabel)
        c = sg.Colorings(g, 12, 2, 1)
        print("ranges with weights", relabel, flush=True)
        f64 = sg.count(plan, g, c, "fp64")["colorful"][0]
        f32 = sg.count(plan, g, c, "fp32s")["colorful"][0]
        with sg.tuned(flags=sg.TUNE_NO_COLOR_SKIP):
            ref = sg.count(plan, g, c, "fp64")["colorful"][0]
        assert ref > 0
        assert f64 == pytest.approx(ref, rel=2 * TOL["fp64"])
        assert f32 == pytest.approx(ref, rel=TOL["fp32s"])


def core(size, n):
    """A complete graph of `size` vertices among n."""
    ci = np.broadcast_to(np.arange(size, dtype=np.int32), (size, size))[~np.eye(size, dtype=bool)]
    rp = np.minimum(np.arange(n + 1, dtype=np.int64), size) * (size - 1)
    return gg.Graph(n, rp, np.ascontiguousarray(ci), None)


@pytest.mark.parametrize("par,k,large,small,n", [
    ([-1] + [0] * 7, 8, 3000, 300, 200_000),           # the root's products
    ([-1] + [0] * 8, 9, 3000, 200, 200_000),           # a multiply-add before it
    (gg.PATH8, 8, 3000, 300, 250_000),                 # LDS sums of 8 sets
    ([-1] + list(range(9)), 10, 1750, 150, 150_000),   # staged rows of 120 sets
    ([-1] + list(range(11)), 12, 1000, 80, 1000),      # chunks
])
def test_sums_past_2_to_64_are_flagged(par, k, large, small, n):
    """Counts of a complete graph's vertices whose tables pass 2^64, and of a smaller
    one's whose do not; the isolated others make relative tables the faster ones."""
    plan = sg.Plan(par, k)
    for size in (large, small):
        G = core(size, n)
        g = sg.Graph.from_csr(G)
        c = sg.Colorings(g, k, 1, 1)
        _, u, over = O.count(G, par, k, O.colors(n, k, 1, 0), mode=O.U64)
        assert over == (size == large)
        print("overflow", par, k, size, flush=True)
        sg.profile_start()
        r = sg.count(plan, g, c, "u64")
        assert sg.profile_stop()["ema_single"]["launches"] == 0
        assert int(r["colorful_u64"][0]) == u
        assert r["overflow"] == over
