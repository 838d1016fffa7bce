"""Launches at sizes where a launch dimension's 2^32 work-items are the limit:
tile lists of more than 2^24 tiles and arrays of 2^28 and more nodes, whose last
rows have to be there like the first ones'."""
import numpy as np
import pytest

import oracle
from bars import P_TOL, Z_TOL, rel_l2, sample_rows
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


@pytest.mark.parametrize("rows_per_lane,n", [(2, 1_060_000), (4, 1_500_000)])
def test_symmetric_tiles_shared_by_waves(path_layout, gpu, rows_per_lane, n):
    # more than 2^24 workgroups of two tiles of 128 rows, of one of 256
    import torch
    g, dY, Y = path_layout(n)
    rows = sample_rows(n, 200, 2)
    _, Z16 = gradient(g, dY, rows, tile_rows=16)
    kl16 = tsgne.tsgne_kl(g, dY)
    fz, Z = gradient(g, dY, rows, tile_rows=rows_per_lane)                 # tiles and attraction together
    check_repulsion(fz, Z, Z16, Y, rows)
    g.set_timing(True)
    grad2, Z2 = tsgne.tsgne_gradient(g, dY, 0.0, tsgne.tsgne_params_default(tile_rows=rows_per_lane))
    g.set_timing(False)                                                    # a launch per phase
    assert Z2.item() == Z and np.array_equal(-Z * grad2.cpu().numpy()[rows].astype(np.float64), fz)
    assert abs(tsgne.tsgne_kl(g, dY) - kl16) <= 2 * Z_TOL                  # Z alone
    if rows_per_lane == 2:                                                 # the batch's launch, against a run's
        p = tsgne.tsgne_params_default(tile_rows=2, learning_rate=1.0)
        a, b = dY.clone(), dY.clone()
        tsgne.tsgne_run(g, a, 1, p)
        tsgne.tsgne_batch_run([g], [b], [1], p)
        assert not torch.equal(a, dY) and torch.equal(a, b)


def late_graph(n, edges, gpu):
    """CSR on the device of n nodes, of which the last 64 have the edges (numbered from the first of them)."""
    import torch
    rp, col = tsgne.tsgne_csr_from_edges(64, np.asarray(edges, np.int32))
    row_ptr = torch.zeros(n + 1, dtype=torch.int32, device=gpu)
    row_ptr[n - 64:] = torch.from_numpy(rp).to(gpu)
    return row_ptr, torch.from_numpy(col + (n - 64)).to(gpu), rp, col


def test_calibration_of_2_28_nodes(gpu):
    import torch
    n = 2 ** 28 + 100                                       # sixteen lanes each
    row_ptr, dcol, rp, col = late_graph(n, [(i, j) for i in range(0, 60, 2) for j in range(i + 1, 64, 3)], gpu)
    X = torch.zeros((n, 1), dtype=torch.float32, device=gpu)
    x = np.random.default_rng(28).standard_normal((64, 1)).astype(np.float32)
    X[n - 64:] = torch.from_numpy(x).to(gpu)
    g = tsgne.tsgne_build_P(row_ptr, dcol, X, 5.0)
    P = np.zeros(col.shape[0], np.float32)
    assert tsgne.lib().tsgne_graph_export(g.handle, None, None, None, P.ctypes.data, None) == tsgne.TSGNE_OK
    g.close()
    assert rel_l2(P, oracle.build_P(rp, col, x, 5.0)[0]) <= P_TOL


def test_kmeans_of_2_30_points(gpu):
    import torch
    n = 2 ** 30 + 300                                       # four lanes each
    h = n // 2
    Y = torch.zeros((n, 2), dtype=torch.float32, device=gpu)
    Y[h:] = 1.0
    labels, passes = tsgne.tsgne_kmeans(Y, torch.tensor([0, n - 1], dtype=torch.int32, device=gpu), 5)
    assert passes == 2 and not labels[:h].any() and bool((labels[h:] == 1).all())
    del Y, labels
    torch.cuda.empty_cache()


def test_hop_distances_of_2_30_nodes(gpu):
    import torch
    n = 2 ** 30 + 70                                        # decoded by four work-items each
    row_ptr, col, _, _ = late_graph(n, [(i, i + 1) for i in range(60, 63)], gpu)
    X, _ = tsgne.tsgne_shortest_path_embedding(row_ptr, col, torch.tensor([n - 1], dtype=torch.int32, device=gpu), 2.0)
    assert X[n - 4:, 0].tolist() == [3.0, 2.0, 1.0, 0.0] and bool((X[:n - 4] == 3.0).all())
    del X, row_ptr
    torch.cuda.empty_cache()


def test_permuted_rows_of_2_32_words(gpu):
    import torch
    n, words = 2 ** 20, 4100
    src = torch.arange(n, dtype=torch.int32, device=gpu)[:, None] + torch.arange(words, dtype=torch.int32, device=gpu)
    perm = torch.arange(n - 1, -1, -1, dtype=torch.int32, device=gpu)
    dst = tsgne.tsgne_permute_rows(src, perm)
    for rows in torch.arange(n, device=gpu).split(2 ** 17):
        assert torch.equal(dst[rows], src[n - 1 - rows])
    del src, dst, rows
    torch.cuda.empty_cache()


def test_neighbourhood_graph_of_2_26_nodes(gpu):
    n = 2 ** 26 + 100                                       # a wave each
    row_ptr, dcol, rp, col = late_graph(n, [(i, j) for i in range(0, 60, 2) for j in range(i + 1, 64, 3)], gpu)
    krp, kcol = tsgne.tsgne_knn_graph(row_ptr, dcol, 3)
    orp, ocol = oracle.knn_graph(rp, col, 3)
    assert not krp[:n - 64].any()
    assert np.array_equal(krp[n - 64:].cpu().numpy(), orp) and np.array_equal(kcol.cpu().numpy() - (n - 64), ocol)


def test_walks_of_2_26_nodes(gpu):
    import torch
    n = 2 ** 26 + 100                                       # a wave each
    row_ptr, dcol, _, _ = late_graph(n, [(0, i) for i in range(1, 64)], gpu)
    g = tsgne.tsgne_build_P_walks(row_ptr, dcol, torch.zeros((n, 1), dtype=torch.float32, device=gpu), 8, 2, 5)
    # a leaf's 8 walks go through the hub to any of the 63 leaves alike, so 504 of them have at most
    # 63 * 62 / 2 distinct ends and hardly fewer than 400; always to the same leaf they have 62
    nnz = g.info()[1]
    g.close()
    torch.cuda.empty_cache()
    assert 2 * 300 < nnz <= 63 * 62


def lattice(n, reach, gpu):
    """CSR on the device of a ring of n nodes, each joined to the `reach` before and after it."""
    import torch
    off = torch.cat([torch.arange(-reach, 0, device=gpu), torch.arange(1, reach + 1, device=gpu)])
    col = torch.remainder(torch.arange(n, device=gpu)[:, None] + off, n).to(torch.int32)
    for rows in (slice(0, reach), slice(n - reach, n)):
        col[rows] = col[rows].sort(1).values
    return (2 * reach * torch.arange(n + 1, device=gpu)).to(torch.int32), col.flatten()


def test_distances_of_2_29_entries(gpu):
    import torch
    n, reach = 2 ** 24, 17                                  # eight lanes an entry
    X = (torch.arange(n, device=gpu) % 2).to(torch.float32)[:, None].contiguous()
    row_ptr, col = lattice(n, reach, gpu)
    g = tsgne.tsgne_build_P(row_ptr, col, X, 20.0)
    P = np.zeros(col.numel(), np.float32)
    assert tsgne.lib().tsgne_graph_export(g.handle, None, None, None, P.ctypes.data, None) == tsgne.TSGNE_OK
    g.close()
    del row_ptr, col
    torch.cuda.empty_cache()
    small = [t.cpu().numpy() for t in lattice(64, reach, gpu)]
    oP = oracle.build_P(small[0], small[1], X[:64].cpu().numpy(), 20.0)[0].reshape(64, 2 * reach)[reach] * 64 / n
    assert np.abs(P.reshape(n, 2 * reach)[reach:n - reach] / oP.astype(np.float32) - 1).max() <= P_TOL


def test_attraction_of_2_29_nodes(gpu):
    import torch
    n = 2 ** 29 + 100                                       # eight lanes each
    rp, col = tsgne.tsgne_csr_from_edges(64, [(i, j) for i in range(0, 60, 2) for j in range(i + 1, 64, 3)])
    row_ptr = np.zeros(n + 1, np.int32)
    row_ptr[n - 64:] = rp
    P = np.full(col.shape[0], 1.0 / col.shape[0], np.float32)
    g = tsgne.tsgne_graph_from_host_P(row_ptr, col + np.int32(n - 64), P)
    Y = torch.zeros((n, 2), dtype=torch.float32, device=gpu)
    y = np.random.default_rng(29).standard_normal((64, 2)).astype(np.float32)
    Y[n - 64:] = torch.from_numpy(y).to(gpu)
    A = torch.full((n, 2), -1.0, dtype=torch.float64, device=gpu)
    tsgne.tsgne_attraction(g, Y, tsgne.TSGNE_PREC_SPLIT, A)
    assert not A[:n - 64].any()
    row, y64 = np.repeat(np.arange(64), np.diff(rp)), y.astype(np.float64)
    d = y64[row] - y64[col]
    pw = P / (1.0 + (d * d).sum(1))
    exact, size = np.zeros((64, 2)), np.zeros((64, 2))
    np.add.at(exact, row, pw[:, None] * d)
    np.add.at(size, row, np.abs(pw[:, None] * d))
    # FP32 terms of at most 8 roundings, FP64 sums
    assert (np.abs(A[n - 64:].cpu().numpy() - exact) <= 8 * 2.0 ** -24 * np.maximum(size, np.abs(pw).max())).all()
    g.close()
    del Y, A
    torch.cuda.empty_cache()
