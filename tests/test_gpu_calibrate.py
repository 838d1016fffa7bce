"""Calibration at the edges of its groups of lanes: rows of 1 to 257 entries
around 16 and 64 lanes, perplexities just below a row's length, distances that
are near, nearly tied, tied and spread over many orders of magnitude."""
import numpy as np
import pytest

import oracle
from bars import P_TOL, rel_l2
from paper_2310_11186_amd import tsgne

pytestmark = pytest.mark.gpu

DEGREES = (1, 2, 3, 4, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 127, 128, 129, 257)


def star_graph(kind, seed):
    """One hub per degree of DEGREES with leaves of its own, and the hubs in a ring."""
    edges, n = [], len(DEGREES)
    for h, deg in enumerate(DEGREES):
        edges.append((h, (h + 1) % len(DEGREES)))
        own = range(n, n + max(0, deg - 2))
        edges += [(h, v) for v in own]
        n += len(own)
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, 3))
    if kind == "near":
        X = 100 + 1e-3 * X
    elif kind == "wide":
        X *= 10.0 ** rng.uniform(-6, 3, (n, 1))
    elif kind == "tied":
        X = np.round(X)
    return n, np.array(edges, np.int32), X.astype(np.float32)


@pytest.mark.parametrize("kind", ["spread", "near", "wide", "tied"])
@pytest.mark.parametrize("perp", [1.5, 2.9, 15.9, 30.0, 62.9, 100.0])
def test_calibration_at_group_edges(gpu, kind, perp):
    import torch
    n, edges, X = star_graph(kind, 7)
    rp, col = tsgne.tsgne_csr_from_edges(n, edges)
    g = tsgne.tsgne_build_P(*(torch.from_numpy(a).to(gpu) for a in (rp, col, X)), perp)
    ex = g.export()
    P, beta = oracle.build_P(*oracle.csr_from_edges(n, edges), X, perp)
    assert rel_l2(ex["P"], P) <= P_TOL
    assert np.array_equal(np.isinf(ex["beta"]), np.isinf(beta)) and np.array_equal(ex["beta"] == 0, beta == 0)
    fine = np.isfinite(beta) & (beta > 0)
    # both searches end at the rounding of the entropy (a few 1e-16 of log(perp) and of beta * distance),
    # which beta follows by 1 / (beta^2 Var): the oracle's own entropy is what both are held to
    for i in np.flatnonzero(fine):
        D = oracle.edge_sqdist(rp, col, X)[rp[i]:rp[i + 1]]
        d = D - D.min()
        e = np.exp(-ex["beta"][i] * d)
        H = np.log(e.sum()) + ex["beta"][i] * (d * e).sum() / e.sum()
        assert abs(H - np.log(np.float32(perp).astype(np.float64))) <= 1e-11, (i, DEGREES[i])
    g.close()


@pytest.mark.parametrize("d", [1, 15, 16, 17, 48, 63, 64, 65, 80, 127, 129])
@pytest.mark.parametrize("cut", [0, 1])                  # an even and an odd number of edges
def test_distances_at_group_edges(gpu, d, cut):
    """Coordinates around the sixteen lanes of an entry and the four loads of a lane."""
    import torch
    n, edges, _ = star_graph("spread", 7)
    edges = edges[:len(edges) - cut]
    X = np.random.default_rng(d).standard_normal((n, d)).astype(np.float32)
    rp, col = tsgne.tsgne_csr_from_edges(n, edges)
    g = tsgne.tsgne_build_P(*(torch.from_numpy(a).to(gpu) for a in (rp, col, X)), 15.0)
    P, _ = oracle.build_P(*oracle.csr_from_edges(n, edges), X, 15.0)
    assert rel_l2(g.export()["P"], P) <= P_TOL
    g.close()


@pytest.mark.parametrize("perp", [1.5, 3.0, 5.0, 9.0])
@pytest.mark.parametrize("near,far", [(1e-10, 1e10), (1e-30, 1e38), (2e-38, 1e38)])
def test_calibration_over_the_range_of_fp32(gpu, near, far, perp):
    """A hub with eight near and eight far leaves whose beta lies far from 1 / mean."""
    import torch
    n = 17
    edges = np.stack([np.zeros(16, np.int32), np.arange(1, 17, dtype=np.int32)], 1)
    X = np.concatenate([[0.0], near * np.linspace(1, 2, 8), far * np.linspace(1, 2, 8)]).astype(np.float32)[:, None]
    rp, col = tsgne.tsgne_csr_from_edges(n, edges)
    g = tsgne.tsgne_build_P(*(torch.from_numpy(a).to(gpu) for a in (rp, col, X)), perp)
    ex = g.export()
    P, beta = oracle.build_P(*oracle.csr_from_edges(n, edges), X, perp)
    assert rel_l2(ex["P"], P) <= P_TOL
    assert abs(ex["beta"][0] / beta[0] - 1.0) <= 1e-11
    g.close()
