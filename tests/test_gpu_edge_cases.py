"""Edge cases of the multi-template count, the renumbered graph and the
no-allocation count: every tree of 1 to 6 vertices counted per size in one
plan (one-vertex and one-edge templates included), k above t; renumbered
graphs registered from device tensors; sg2v_count_noalloc on a renumbered
graph."""
import sys

import numpy as np
import pytest

import graphgen as gg
import oracle as O
import paper_2009_11665_amd as sg

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("t", [1, 2, 3, 4, 5, 6])
def test_all_trees_of_a_size(t):
    G = gg.rmat(9, 2000, seed=3)
    k, seed, ncol = t + 1, 9, 2
    trees = sg.trees(t)
    g = sg.Graph.from_csr(G)
    c = sg.Colorings(g, k, seed, ncol)
    say("all trees of", t, "vertices:", len(trees))
    r = sg.count_multi(sg.Plan.multi(trees, k), g, c, "u64")
    f = sg.count_multi(sg.Plan.multi(trees, k), g, c, "fp64")
    for j in range(ncol):
        col = O.colors(G.n, k, seed, j)
        for q, par in enumerate(trees):
            _, u, _ = O.count(G, par, k, col, mode=O.U64)
            assert int(r["colorful_u64"][q, j]) == u, (q, j)
            assert f["colorful"][q, j] == pytest.approx(float(u), rel=1e-12, abs=1e-300)
    assert f["frequency"].sum() == pytest.approx(1.0, rel=1e-12)


def test_relabel_from_device_tensors():
    import torch
    G = gg.rmat(11, 12_000, seed=21)
    par, k, seed = gg.BINTREE7, 7, 5
    rp = torch.from_numpy(G.row_ptr.astype(np.int64)).cuda()
    ci = torch.from_numpy(G.col_idx.astype(np.int32)).cuda()
    g1 = sg.Graph(G.n, rp, ci, relabel=True)
    g0 = sg.Graph.from_csr(G)
    p = sg.Plan(par, k)
    a = sg.count(p, g1, sg.Colorings(g1, k, seed, 2), "u64")["colorful_u64"]
    b = sg.count(p, g0, sg.Colorings(g0, k, seed, 2), "u64")["colorful_u64"]
    np.testing.assert_array_equal(a, b)


def test_noalloc_on_renumbered_graph():
    G = gg.rmat(11, 12_000, seed=21)
    par, k, seed = gg.BINTREE7, 7, 8
    g = sg.Graph.from_csr(G, relabel=True)
    c = sg.Colorings(g, k, seed, 3)
    p = sg.Plan(par, k)
    ref = sg.count(p, g, c, "u64")
    na = sg.count_noalloc(p, g, c, "u64")
    np.testing.assert_array_equal(na["colorful_u64"], ref["colorful_u64"])
    _, u, _ = O.count(G, par, k, O.colors(G.n, k, seed, 2), mode=O.U64)
    assert int(na["colorful_u64"][2]) == u


@pytest.mark.parametrize("tuned", [{}, {"batch": 30000}])
def test_many_colourings_of_a_chunked_aggregation(tuned):
    """Chunks times colourings past the 65,535 blocks that a grid dimension holds
    (path of 8 with 12 colours: 4 chunks, 30,000 colourings of 8 vertices a pass)."""
    n, ncol = 8, 30000
    e = [(i, j) for i in range(n) for j in range(i + 1, n) if (i, j) != (2, 5)]
    g = sg.Graph.from_csr(gg.from_edge_list(n, e, None))
    plan = sg.Plan(gg.PATH8, 12)
    c = sg.Colorings(g, 12, 3, ncol)
    print("chunks x colourings", tuned, flush=True)
    got = {}
    with sg.tuned(**tuned):
        for m in ("u64", "fp64", "fp32s"):
            got[m] = sg.count(plan, g, c, m)
    with sg.tuned(batch=1000):
        ref = sg.count(plan, g, c, "u64")["colorful_u64"]
    assert [int(x) for x in got["u64"]["colorful_u64"]] == [int(x) for x in ref]
    assert sum(int(x) > 0 for x in ref[16384:]) > 100
    f = [float(x) for x in ref]
    np.testing.assert_allclose(got["fp64"]["colorful"], f, rtol=1e-12)
    np.testing.assert_allclose(got["fp32s"]["colorful"], f, rtol=1e-5)


@pytest.mark.parametrize("deg", [254, 256, 1030])
def test_rows_long_like_the_others_and_longer(deg):
    """Graphs whose rows all have about as many entries as a long row (one wave each),
    with a hub of twice their mean and more (whole blocks, two segments at 1030)."""
    n = 2 * deg + 100
    d = np.arange(1, deg // 2 + 1)
    e = {(i, int(j)) for i in range(n) for j in (i + d) % n}
    e |= {(0, j) for j in range(1, n)}
    G = gg.from_edge_list(n, sorted({(min(x), max(x)) for x in e}), None)
    g = sg.Graph.from_csr(G)
    Gw = gg.Graph(n, G.row_ptr, G.col_idx, (1.0 + (G.col_idx + np.repeat(np.arange(n), np.diff(G.row_ptr))) % 7).astype(np.float32))
    gw = sg.Graph.from_csr(Gw)
    for par, k in (([-1, 0, 1], 3), (gg.PATH5, 5), (gg.PATH8, 9)):
        plan = sg.Plan(par, k)
        c = sg.Colorings(g, k, 2, 2)
        say("rows of", deg, par, k)
        u = sg.count(plan, g, c, "u64")["colorful_u64"]
        f = sg.count(plan, gw, sg.Colorings(gw, k, 2, 2), "fp32s")["colorful"]
        h = sg.count_grad(plan, gw, sg.Colorings(gw, k, 2, 1), [1.0], "fp64").cpu().numpy()
        for j in range(2):
            col = O.colors(n, k, 2, j)
            assert int(u[j]) == O.count(G, par, k, col, mode=O.U64)[1] > 0
            assert f[j] == pytest.approx(O.count(Gw, par, k, col)[0], rel=1e-5)
        ref = O.grad(Gw, par, k, O.colors(n, k, 2, 0))[1]
        np.testing.assert_allclose(h, ref, rtol=1e-10, atol=1e-10 * np.abs(ref).max())


@pytest.mark.parametrize("deg,ncol,absolute", [(4, 24, False), (256, 24, True), (256, 1, False)])
@pytest.mark.parametrize("mode", ["u64", "fp64", "fp32s"])
def test_tables_by_estimated_time(deg, ncol, absolute, mode):
    """Path of 5 on a uniform graph of 6000 vertices: few columns, many colourings and
    a high degree run in absolute tables (which have one-vertex multiply-adds), the
    others in relative ones; counts do not depend on it."""
    n = 6000
    G = gg.csr(n, *gg.er_edges(n, n * deg // 2, 5))
    g = sg.Graph.from_csr(G)
    plan = sg.Plan(gg.PATH5, 5)
    c = sg.Colorings(g, 5, 2, ncol)
    say("tables by time", deg, ncol, mode)
    sg.profile_start()
    r = sg.count(plan, g, c, mode)
    prof = sg.profile_stop()
    assert (prof["ema_single"]["launches"] > 0) == absolute
    for j in (0, ncol - 1):
        f, u, _ = O.count(G, gg.PATH5, 5, O.colors(n, 5, 2, j), mode=O.U64 if mode == "u64" else O.FP64)
        if mode == "u64":
            assert int(r["colorful_u64"][j]) == u
        else:
            assert r["colorful"][j] == pytest.approx(f, rel={"fp64": 1e-12, "fp32s": 1e-5}[mode])


@pytest.mark.parametrize("mode", ["u64", "fp64", "fp32s"])
def test_tables_by_estimated_time_of_the_root(mode):
    """Binary tree of 7 with 14 colours: 34,320 products a vertex at the root, which the
    absolute tables' root takes faster; with 9 colours (560) relative ones are."""
    n = 3000
    G = gg.csr(n, *gg.er_edges(n, 3 * n, 5))
    g = sg.Graph.from_csr(G)
    for k, absolute in ((14, True), (9, False)):
        plan = sg.Plan(gg.BINTREE7, k)
        c = sg.Colorings(g, k, 2, 6)
        say("root's pairs", k, mode)
        sg.profile_start()
        r = sg.count(plan, g, c, mode)
        prof = sg.profile_stop()
        if mode != "fp32s":
            assert (prof["ema_single"]["launches"] > 0) == absolute
        f, u, _ = O.count(G, gg.BINTREE7, k, O.colors(n, k, 2, 5), mode=O.U64 if mode == "u64" else O.FP64)
        if mode == "u64":
            assert int(r["colorful_u64"][5]) == u
        else:
            assert r["colorful"][5] == pytest.approx(f, rel={"fp64": 1e-12, "fp32s": 1e-5}[mode])
