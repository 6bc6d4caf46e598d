"""FP32S over the range of the weights: counts and derivatives on a graph whose
weights all carry one power of two against FP64, whose exponents hold it."""
import numpy as np
import pytest

import graphgen as gg
import paper_2009_11665_amd as sg

pytestmark = pytest.mark.gpu

N = 1500


def graph(scale):
    """Hubs of 1499 and 300 neighbours (rows of two segments and of one), a path
    and random edges, weights of one to two times 2^scale."""
    rng = np.random.default_rng(5)
    edges = {(0, v) for v in range(1, N)} | {(1, v) for v in range(2, 302)} | {(v - 1, v) for v in range(1, N)}
    edges |= {(int(min(e)), int(max(e))) for e in rng.integers(0, N, (4000, 2)) if e[0] != e[1]}
    w = rng.uniform(1.0, 2.0, len(edges)) * 2.0 ** scale
    return gg.from_edge_list(N, sorted(edges), w)


# rooted at an end: every aggregation follows the one before it directly
PATHS = [([-1, 0], 3), ([-1, 0, 1], 3), ([-1, 0, 1, 2], 4), (gg.PATH5, 5),  # sums in LDS
         (gg.PATH5, 9), (gg.PATH8, 9),                                      # staged rows
         (gg.PATH8, 12)]                                                    # chunks by high colours
OTHERS = [(gg.BINTREE7, 7), (gg.CATERPILLAR10, 10)]


@pytest.mark.parametrize("scale", [-60, -35, 0, 35, 70])
@pytest.mark.parametrize("par,k", PATHS + OTHERS)
def test_fp32s_counts_at_any_scale_of_the_weights(par, k, scale):
    g = sg.Graph.from_csr(graph(scale))
    plan = sg.Plan(par, k)
    c = sg.Colorings(g, k, 7, 3)
    print("range", par, k, scale, flush=True)
    ref = np.asarray(sg.count(plan, g, c, "fp64")["colorful"])
    got = np.asarray(sg.count(plan, g, c, "fp32s")["colorful"])
    assert (ref > 0).all() and np.isfinite(ref).all()
    np.testing.assert_allclose(got, ref, rtol=1e-5)  # bound of the mode


@pytest.mark.parametrize("scale", [-60, 0, 70])
@pytest.mark.parametrize("par,k", PATHS[:-1] + OTHERS)  # no chunks in the adjoint
def test_fp32s_derivatives_at_any_scale_of_the_weights(par, k, scale):
    g = sg.Graph.from_csr(graph(scale))
    plan = sg.Plan(par, k)
    c = sg.Colorings(g, k, 7, 2)
    print("range, derivative", par, k, scale, flush=True)
    ref = sg.count_grad(plan, g, c, [1.0, -0.5], "fp64").cpu().numpy()
    got = sg.count_grad(plan, g, c, [1.0, -0.5], "fp32s").cpu().numpy()
    top = np.abs(ref).max()
    assert top > 0 and np.isfinite(top)
    np.testing.assert_allclose(got, ref, rtol=2e-5, atol=2e-5 * top)  # bound of the mode
