"""ShortestPath embedding (section 2.3, eq. (8)) on the GPU: bit-exact against
the oracle's one-BFS-per-target definition."""
import numpy as np
import pytest

import oracle
from paper_2310_11186_amd import synth, tsgne

pytestmark = pytest.mark.gpu


def path_edges(n):
    return np.stack([np.arange(n - 1), np.arange(1, n)], 1).astype(np.int32)


def star_edges(n):
    return np.stack([np.zeros(n - 1, np.int32), np.arange(1, n, dtype=np.int32)], 1)


def run_both(gpu, n, edges, targets, l0):
    import torch
    rp, col = tsgne.tsgne_csr_from_edges(n, edges)
    X, levels = tsgne.tsgne_shortest_path_embedding(torch.from_numpy(rp).to(gpu), torch.from_numpy(col).to(gpu),
                                                    torch.from_numpy(np.asarray(targets, np.int32)).to(gpu), l0)
    l0_used = np.sqrt(col.shape[0] // 2) if l0 < 0 else l0
    return X.cpu().numpy(), oracle.shortest_path_embedding(rp, col, targets, l0_used), levels


CASES = [
    # (name, graph, d, l0)
    ("sbm_sparse", lambda: synth.small_sbm(500, 4, 2.2, 4, 3), 1, -1.0),
    ("sbm_sparse", lambda: synth.small_sbm(500, 4, 2.2, 4, 3), 33, 0.0),
    ("sbm_sparse", lambda: synth.small_sbm(500, 4, 2.2, 4, 3), 64, 2.5),
    ("sbm", lambda: synth.small_sbm(1500, 6, 5.0, 8, 4), 100, -1.0),
    ("sbm", lambda: synth.small_sbm(1500, 6, 5.0, 8, 4), 128, 3.0),
    ("dcsbm_hubs", lambda: synth.small_dcsbm(4000, 12000, 2.2, 10, 4, 5), 128, -1.0),
    ("dcsbm_hubs", lambda: synth.small_dcsbm(4000, 12000, 2.2, 10, 4, 5), 200, 1e9),
    ("dcsbm_hubs", lambda: synth.small_dcsbm(4000, 12000, 2.2, 10, 4, 5), 256, 4.0),
]


@pytest.mark.parametrize("name,make,d,l0", CASES, ids=["%s-d%d-l0%g" % (c[0], c[2], c[3]) for c in CASES])
def test_sp_bit_exact(gpu, name, make, d, l0):
    gi = make()
    targets = np.random.default_rng(d).choice(gi.n, d, replace=d > gi.n).astype(np.int32)
    X, oX, _ = run_both(gpu, gi.n, gi.edges, targets, l0)
    assert X.dtype == np.float32 and X.shape == (gi.n, d)
    assert np.array_equal(X, oX)


@pytest.mark.parametrize("n,l0", [(300, 1e6), (300, 37.5), (700, -1.0), (2, 0.5)])
def test_sp_path_graph_many_levels(gpu, n, l0):
    # distances up to n - 1: many level chunks and distance planes
    targets = np.array([0, n - 1, n // 2, n // 3, 0], np.int32)        # includes a repeat
    X, oX, levels = run_both(gpu, n, path_edges(n), targets, l0)
    assert np.array_equal(X, oX)
    used = np.sqrt(n - 1) if l0 < 0 else l0
    assert levels <= min(np.floor(used), n - 1)
    if l0 >= n:
        assert X[n - 1, 0] == n - 1


def test_sp_star_and_isolated(gpu):
    # one node of degree 999 (the wave-per-node path) and 50 isolated nodes
    n = 1050
    X, oX, _ = run_both(gpu, n, star_edges(1000), np.array([0, 5, 1020, 999], np.int32), 10.0)
    assert np.array_equal(X, oX)
    assert np.all(X[1000:, 0] == 11.0) and X[1020, 2] == 0.0


@pytest.mark.parametrize("n", [63, 64, 129, 7001])       # rows of a decoding block, one past two, hubs of 2 and 4 chunks
@pytest.mark.parametrize("d", [1, 2, 3, 4, 31, 32, 127, 255, 256])
def test_sp_hubs_and_target_counts(gpu, n, d):
    # two hubs, of all nodes and of every second one, whose levels alternate with a path of 14 off the last leaf
    far = np.arange(2, n, 2)
    edges = np.concatenate([star_edges(n), np.stack([np.ones_like(far), far], 1),
                            n - 1 + path_edges(15)]).astype(np.int32)
    targets = np.random.default_rng(n + d).choice(n + 14, d).astype(np.int32)
    targets[-1] = n + 13                                                # 15 levels from the hub: past the first 12
    X, oX, _ = run_both(gpu, n + 14, edges, targets, 1e6)
    assert np.array_equal(X, oX)


def test_sp_no_edges(gpu):
    import torch
    n = 40
    rp = torch.zeros(n + 1, dtype=torch.int32, device=gpu)
    col = torch.zeros(0, dtype=torch.int32, device=gpu)
    X, levels = tsgne.tsgne_shortest_path_embedding(rp, col, torch.tensor([3, 7], dtype=torch.int32, device=gpu))
    expect = np.ones((n, 2), np.float32)                                # default l0 = sqrt(0) = 0
    expect[3, 0] = expect[7, 1] = 0
    assert np.array_equal(X.cpu().numpy(), expect) and levels == 0


def test_sp_full_size(gpu):
    """The 300,000-node, 1,000,000-edge graph with 128 targets: every element."""
    import torch
    gi = synth.make("dcsbm300k")
    rp, col = tsgne.tsgne_csr_from_edges(gi.n, gi.edges)
    targets = np.random.default_rng(2310).choice(gi.n, 128, replace=False).astype(np.int32)
    X, levels = tsgne.tsgne_shortest_path_embedding(torch.from_numpy(rp).to(gpu), torch.from_numpy(col).to(gpu),
                                                    torch.from_numpy(targets).to(gpu))
    oX = oracle.shortest_path_embedding(rp, col, targets, np.sqrt(col.shape[0] // 2))
    assert np.array_equal(X.cpu().numpy(), oX)
    print("levels launched", levels, "max finite distance", oX[oX < np.sqrt(col.shape[0] // 2) + 1].max())


def test_sp_then_affinities(gpu):
    """GD = DR o GE (section 2, eq. (1)): the embedding feeds build_P unchanged."""
    import torch
    gi = synth.small_dcsbm(3000, 9000, 2.4, 12, 4, 9)
    rp, col = tsgne.tsgne_csr_from_edges(gi.n, gi.edges)
    d_rp, d_col = torch.from_numpy(rp).to(gpu), torch.from_numpy(col).to(gpu)
    targets = np.random.default_rng(5).choice(gi.n, 64, replace=False).astype(np.int32)
    X, _ = tsgne.tsgne_shortest_path_embedding(d_rp, d_col, torch.from_numpy(targets).to(gpu))
    g = tsgne.tsgne_build_P(d_rp, d_col, X, 30.0)
    oX = oracle.shortest_path_embedding(rp, col, targets, np.sqrt(col.shape[0] // 2))
    oP, _ = oracle.build_P(rp, col, oX, 30.0)
    P = g.export()["P"]
    assert np.linalg.norm(P - oP) <= 1e-6 * np.linalg.norm(oP)
    g.close()


def test_sp_rejects(gpu):
    import torch
    gi = synth.small_sbm(100, 2, 3.0, 4, 1)
    rp, col = tsgne.tsgne_csr_from_edges(gi.n, gi.edges)
    d_rp, d_col = torch.from_numpy(rp).to(gpu), torch.from_numpy(col).to(gpu)
    with pytest.raises(tsgne.TsgneError) as e:
        tsgne.tsgne_shortest_path_embedding(d_rp, d_col, torch.tensor([0, 100], dtype=torch.int32, device=gpu))
    assert e.value.status == tsgne.TSGNE_E_INVAL
    with pytest.raises(tsgne.TsgneError) as e:
        tsgne.tsgne_shortest_path_embedding(d_rp, d_col, torch.tensor([-1], dtype=torch.int32, device=gpu))
    assert e.value.status == tsgne.TSGNE_E_INVAL
    bad = col.copy()
    bad[0], bad[1] = bad[1], bad[0]
    with pytest.raises(tsgne.TsgneError) as e:
        tsgne.tsgne_shortest_path_embedding(d_rp, torch.from_numpy(bad).to(gpu),
                                            torch.tensor([0], dtype=torch.int32, device=gpu))
    assert e.value.status == tsgne.TSGNE_E_GRAPH


@pytest.mark.parametrize("far", [11, 12, 13, 23, 24, 25])     # the last level with a new node, around chunks of 12
@pytest.mark.parametrize("over", [-1.0, 0.0, 0.5, 1e6])       # the threshold, less that level
def test_sp_searches_that_end_around_a_chunk(gpu, far, over):
    n = far + 1
    targets = np.full(9, 0, np.int32)
    targets[::2] = n - 1
    X, oX, levels = run_both(gpu, n, path_edges(n), targets, far + over)
    assert np.array_equal(X, oX)
    assert levels <= min(np.floor(far + over), n - 1)
