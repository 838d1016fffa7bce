"""The step's launches: tiles and attraction together, and Z summed by the
update, give bit for bit what a launch per phase gives (phase timing takes
those), at sizes on both sides of a tile, of a round of the attraction's
workgroups over the XCDs and of the 8,192 tiles up to which Z has no launch of
its own."""
import numpy as np
import pytest

from paper_2310_11186_amd import synth, tsgne

pytestmark = pytest.mark.gpu

# 64-row tiles: 127 blocks are 8,128 tiles, 128 blocks 8,256
CASES = [(1, 1), (63, 1), (64, 1), (65, 2), (129, 1), (255, 4), (256, 4), (257, 4), (2049, 8), (8128, 1), (8129, 1),
         (8192, 1), (16257, 2), (3001, 16), (5000, 0), (20011, 0)]


@pytest.mark.parametrize("n,rows", CASES)
@pytest.mark.parametrize("precision", [tsgne.TSGNE_PREC_SPLIT, tsgne.TSGNE_PREC_FP32])
def test_fused_step_equals_its_phases(gpu, n, rows, precision):
    import torch
    rng = np.random.default_rng(n)
    if n >= 255:
        gi = synth.small_dcsbm(n, 4 * n, 2.3, 4, 4, n)   # hubs: rows of one lane group and of a wave
        rp, col = tsgne.tsgne_csr_from_edges(n, gi.edges)
    else:
        rp, col = tsgne.tsgne_csr_from_edges(n, [(i, i + 1) for i in range(n - 1)])
    deg = np.diff(rp)
    row = np.repeat(np.arange(n), deg)
    P = (1.0 / deg[row] + 1.0 / deg[col]).astype(np.float32)
    g = tsgne.tsgne_graph_from_host_P(rp, col, P / max(P.sum(), 1))
    p = tsgne.tsgne_params_default(tile_rows=rows, precision=precision, exaggeration_iters=2)
    start = [torch.from_numpy(a.astype(np.float32)).to(gpu) for a in
             (3.0 * rng.standard_normal((n, 2)), 0.1 * rng.standard_normal((n, 2)), rng.uniform(0.5, 1.5, (n, 2)))]
    out = []
    for timing in (False, True):
        g.set_timing(timing)
        Y, U, G = (t.clone() for t in start)
        grad, Z = torch.empty_like(Y), torch.empty(1, dtype=torch.float64, device=gpu)
        for t in range(3):
            tsgne.tsgne_step(g, Y, U, G, t, p, grad, Z)
        run = start[0].clone()
        tsgne.tsgne_run(g, run, 3, p)
        out.append([t.cpu().numpy() for t in (Y, U, G, grad, Z, run)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    g.close()
