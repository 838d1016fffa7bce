"""Launches at sizes where a launch dimension's 2^32 work-items are the limit:
a tile list of more than 2^24 tiles, whose last rows and normaliser have to be
there like the first ones'."""
import numpy as np
import pytest

from bars import Z_TOL, sample_rows
from paper_2310_11186_amd import tsgne

pytestmark = pytest.mark.gpu


@pytest.fixture()
def path_layout(gpu):
    """make(n): a path graph, a layout of it on the device and the same on the host."""
    import torch
    made = []

    def make(n):
        rp = np.zeros(n + 1, np.int32)
        rp[1:] = 2 * np.arange(1, n + 1) - 1
        rp[n] -= 1
        col = np.empty(2 * n - 2, np.int32)
        col[0::2] = np.arange(1, n)
        col[1::2] = np.arange(n - 1)
        g = tsgne.tsgne_graph_from_host_P(rp, col, np.full(2 * n - 2, 1.0 / (2 * n - 2), np.float32))
        made.append(g)
        Y = (30.0 * np.random.default_rng(n).standard_normal((n, 2))).astype(np.float32)
        return g, torch.from_numpy(Y).to(gpu), Y

    yield make
    for g in made:
        g.close()
    torch.cuda.empty_cache()


def check_repulsion(force_z, Z, Z16, Y, rows):
    """force_z: Z times the repulsive part of the sampled rows' gradients, 4 R_i.
    A term w^2 d of R_i carries at most 12 roundings of 2^-24 (d, two FMAs, a
    reciprocal within 1 ulp, its square and the product), and a sum in FP32 at
    most 64 more, so R_i is within 80 * 2^-24 of its terms' sizes added up."""
    Y = Y.astype(np.float64)
    for row, f in zip(rows, force_z):
        d = Y[row] - Y
        w2 = 1.0 / (1.0 + (d * d).sum(1)) ** 2
        exact, size = 4.0 * (w2[:, None] * d).sum(0), 4.0 * (w2 * np.hypot(d[:, 0], d[:, 1])).sum()
        assert np.hypot(*(f - exact)) <= 80 * 2.0 ** -24 * size, row
    assert abs(Z / Z16 - 1.0) <= 2 * Z_TOL     # both within Z_TOL of the exact one


def gradient(g, dY, rows, **kw):
    p = tsgne.tsgne_params_default(**kw)
    grad, Z = tsgne.tsgne_gradient(g, dY, 0.0, p)   # alpha = 0: the repulsion alone
    return -Z.item() * grad.cpu().numpy()[rows].astype(np.float64), Z.item()


def test_direct_tiles_of_four_rows(path_layout):
    # 4,141^2 tiles of 256 rows
    n = 1_060_000
    g, dY, Y = path_layout(n)
    rows = sample_rows(n, 200, 1)
    _, Z16 = gradient(g, dY, rows, tile_rows=16)
    fz, Z = gradient(g, dY, rows, tile_rows=4, repulsion=tsgne.TSGNE_REPULSION_DIRECT)
    check_repulsion(fz, Z, Z16, Y, rows)
