"""Counts in vertex-relative tables (the default) against the oracle and
against the absolute tables, at the sizes where their kernels change: one to
three output columns per lane, sums in LDS or staged rows, colour sets of one
to nearly all colours, rows of no entries, of several segments and in between,
vertex numbers around the rows of a wave, one and several colourings."""
import sys

import numpy as np
import pytest

import graphgen as gg
import oracle as O
import paper_2009_11665_amd as sg

pytestmark = pytest.mark.gpu

# bounds of the library's modes: FP64 rounding over the sums of a count, FP32
# with power-of-two frames
TOL = {"fp64": 1e-12, "fp32s": 1e-5}

TEMPLATES = [
    ([-1, 0], 2), ([-1, 0], 20),                       # histogram and root only
    ([-1, 0, 1], 3), ([-1, 0, 1], 20),                 # one aggregation; 190 sets
    ([-1, 0, 1, 2], 4), ([-1, 0, 1, 2], 12),           # widths 1..3; 220 sets
    ([-1, 0, 0, 0, 0], 6), (gg.PATH5, 9), (gg.BINTREE7, 7), (gg.BINTREE7, 9),
    (gg.PATH8, 8), (gg.CATERPILLAR10, 10),
    ([-1, 0, 1, 2, 3, 4, 5], 11), (gg.PATH8, 12),      # chunks by high colours
    (gg.BINTREE15, 15),                                # 6435 sets
    ([-1, 0, 1, 2, 3], 16),                            # 560 sets: absolute tables
]


def hubs(n, seed, weighted):
    """Hubs of n - 1, 300 and 255 neighbours, a ring, and isolated vertices at
    the end when there is room."""
    edges = set()
    last = n - max(0, min(7, n - 8))
    for v in range(1, last):
        edges.add((0, v))
        edges.add((min(v, (v % (last - 1)) + 1), max(v, (v % (last - 1)) + 1)))
    for hub, d in ((1, 300), (2, 255)):
        for v in range(last):
            if v > hub and v < hub + d:
                edges.add((hub, v))
    e = np.array([x for x in sorted(edges) if x[0] != x[1]])
    rng = np.random.default_rng(seed)
    perm = rng.permutation(n)
    w = rng.uniform(0.5, 1.5, len(e)) if weighted else None
    return gg.from_edge_list(n, [(int(perm[a]), int(perm[b])) for a, b in e], w)


@pytest.mark.parametrize("n", [5, 33, 1500])
@pytest.mark.parametrize("par,k", TEMPLATES)
def test_relative_tables_against_oracle_and_absolute(par, k, n):
    for weighted in (False, True):
        G = hubs(n, 11 * n + k, weighted)
        g = sg.Graph.from_csr(G)
        plan = sg.Plan(par, k)
        for ncol in (1, 6):
            c = sg.Colorings(g, k, 5, ncol, first=3)
            for mode in ("fp64", "fp32s") + (() if weighted else ("u64",)):
                print("relative", n, par, k, weighted, ncol, mode, flush=True)
                sys.stdout.flush()
                r = sg.count(plan, g, c, mode)
                with sg.tuned(flags=sg.TUNE_NO_COLOR_SKIP):
                    full = sg.count(plan, g, c, mode)
                for j in range(ncol):
                    col = O.colors(n, k, 5, 3 + j)
                    f, u, _ = O.count(G, par, k, col, mode=O.U64 if mode == "u64" else O.FP64)
                    if mode == "u64":
                        assert int(r["colorful_u64"][j]) == u == int(full["colorful_u64"][j])
                    else:
                        assert r["colorful"][j] == pytest.approx(f, rel=TOL[mode])
                        assert r["colorful"][j] == pytest.approx(full["colorful"][j], rel=2 * TOL[mode])


def test_relative_chunks_with_neighbour_ranges():
    """RMAT scale 18 (50M entries): long tasks are taken once per neighbour range;
    exact counts equal those in absolute tables, with and without renumbering."""
    G = gg.rmat(18, 25_000_000, seed=5)
    plan = sg.Plan(gg.BINTREE15, 15)
    got = []
    for relabel in (False, True):
        g = sg.Graph.from_csr(G, relabel=relabel)
        c = sg.Colorings(g, 15, 2, 1)
        print("ranges: relative", relabel, flush=True)
        got.append(int(sg.count(plan, g, c, "u64")["colorful_u64"][0]))
        f64 = sg.count(plan, g, c, "fp64")["colorful"][0]
        f32 = sg.count(plan, g, c, "fp32s")["colorful"][0]
        assert abs(f32 - f64) <= TOL["fp32s"] * f64
    with sg.tuned(flags=sg.TUNE_NO_COLOR_SKIP):
        print("ranges: absolute", flush=True)
        got.append(int(sg.count(plan, g, c, "u64")["colorful_u64"][0]))
    assert got[0] == got[1] == got[2] and got[0] % 128 == 0


def test_relative_tables_partial_pass_and_several_templates():
    """A last pass of fewer colourings, and templates that share tables."""
    G = hubs(700, 3, False)
    g = sg.Graph.from_csr(G, relabel=True)
    ts = sg.trees(6)
    plan = sg.Plan.multi(ts, 7)
    c = sg.Colorings(g, 7, 9, 5)
    with sg.tuned(batch=2):
        r = sg.count_multi(plan, g, c, "u64")
    for t, par in enumerate(ts):
        for j in range(5):
            assert int(r["colorful_u64"][t][j]) == O.count(G, par, 7, O.colors(700, 7, 9, j), mode=O.U64)[1]


def test_relative_overflow_flag():
    """Sums past 2^64 are flagged, and only those."""
    n = 1400
    G = hubs(n, 4, False)
    g = sg.Graph.from_csr(G)
    for par, k in (([-1, 0, 0, 0, 0, 0, 0], 7), (gg.PATH5, 5)):
        r = sg.count(sg.Plan(par, k), g, sg.Colorings(g, k, 1, 2), "u64")
        ref = [O.count(G, par, k, O.colors(n, k, 1, j), mode=O.U64) for j in range(2)]
        assert [int(x) for x in r["colorful_u64"]] == [x[1] for x in ref]
        assert r["overflow"] == any(x[2] for x in ref)


@pytest.mark.parametrize("n", [5, 33, 1500])
@pytest.mark.parametrize("par,k", [([-1, 0], 3), ([-1, 0, 1], 3), ([-1, 0, 0, 0], 5), (gg.PATH5, 7),
                                   (gg.BINTREE7, 7), (gg.CATERPILLAR10, 10), (gg.PATH8, 9)])
def test_relative_adjoint_against_oracle_and_absolute(par, k, n):
    """Per-entry derivatives: rows of no entries, long and segmented rows, one and
    two columns per lane, several colourings of either sign and of weight zero."""
    G = hubs(n, 7 * n + k, True)
    g = sg.Graph.from_csr(G)
    plan = sg.Plan(par, k)
    gcol = [1.0, 0.0, -0.75]
    c = sg.Colorings(g, k, 4, 3)
    ref = np.zeros(G.nnz)
    for j, a in enumerate(gcol):
        if a:
            ref += a * O.grad(G, par, k, O.colors(n, k, 4, j))[1]
    top = np.abs(ref).max()
    for mode, tol in (("fp64", 1e-10), ("fp32s", 2e-5)):
        print("adjoint", n, par, k, mode, flush=True)
        got = sg.count_grad(plan, g, c, gcol, mode).cpu().numpy()
        with sg.tuned(flags=sg.TUNE_NO_COLOR_SKIP):
            full = sg.count_grad(plan, g, c, gcol, mode).cpu().numpy()
        np.testing.assert_allclose(got, ref, rtol=tol, atol=tol * top)
        np.testing.assert_allclose(got, full, rtol=2 * tol, atol=2 * tol * top)


def test_adjoint_of_entries_without_reverse():
    """A row that repeats or lacks a reverse entry has the absolute adjoint: the
    derivative by every entry as it stands."""
    G = gg.from_edge_list(6, [(0, 1), (1, 2), (2, 3), (3, 4), (4, 5), (0, 5)], np.linspace(0.5, 1.5, 6))
    drop = int(G.row_ptr[3])  # first entry of vertex 3
    rp = G.row_ptr.copy()
    rp[4:] -= 1
    g = sg.Graph(6, rp, np.delete(G.col_idx, drop), np.delete(G.w, drop))
    plan = sg.Plan(gg.PATH5, 5)
    c = sg.Colorings(g, 5, 3, 2)
    a = sg.count_grad(plan, g, c, [1.0, 1.0], "fp64").cpu().numpy()
    with sg.tuned(flags=sg.TUNE_NO_COLOR_SKIP):
        b = sg.count_grad(plan, g, c, [1.0, 1.0], "fp64").cpu().numpy()
    np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("par,k", [(gg.BINTREE7, 7), (gg.BINTREE7, 8), ([-1, 0, 0, 1, 1], 5), ([-1, 0, 1, 0, 3], 6)])
@pytest.mark.parametrize("n", [20011, 24576])
def test_relative_multiply_add_in_row_groups(par, k, n):
    """Enough rows that threads of narrow outputs (6 to 35 columns) take several
    groups of rows each; a last tile of 11, 43, ... rows and whole tiles."""
    g = sg.Graph.from_csr(hubs(n, k, False))
    plan = sg.Plan(par, k)
    c = sg.Colorings(g, k, 5, 7)
    print("row groups", n, par, k, flush=True)
    got = {m: sg.count(plan, g, c, m) for m in ("u64", "fp64", "fp32s")}
    with sg.tuned(flags=sg.TUNE_NO_COLOR_SKIP):
        full = sg.count(plan, g, c, "u64")["colorful_u64"]
    for j in range(7):
        u = int(got["u64"]["colorful_u64"][j])
        assert u == int(full[j])
        for m in ("fp64", "fp32s"):
            assert got[m]["colorful"][j] == pytest.approx(float(u), rel=TOL[m])


@pytest.mark.parametrize("n,ncol", [(1000, 270), (120011, 20)])
def test_relative_passes_by_rows(n, ncol):
    """Colourings of a pass by its rows: more than the columns of the absolute
    tables would give (262 of path5 on 1000 vertices), fewer on a large graph (13
    of 120,011); a last pass of the rest.  Exact counts do not depend on it."""
    edges = [(v, (v * 7 + 3) % n) for v in range(n)] + [(v, (v + 1) % n) for v in range(n - 1)]
    g = sg.Graph.from_csr(gg.from_edge_list(n, sorted({(min(e), max(e)) for e in edges if e[0] != e[1]}), None))
    plan = sg.Plan(gg.PATH5, 5)
    c = sg.Colorings(g, 5, 8, ncol)
    print("passes", n, ncol, flush=True)
    r = sg.count(plan, g, c, "u64")["colorful_u64"]
    f = sg.count(plan, g, c, "fp32s")["colorful"]
    with sg.tuned(batch=7):
        s = sg.count(plan, g, c, "u64")["colorful_u64"]
    assert [int(x) for x in r] == [int(x) for x in s] and all(int(x) > 0 for x in r)
    for x, y in zip(r, f):
        assert y == pytest.approx(float(x), rel=TOL["fp32s"])
