"""Runs whose sampled steps take a launch per phase and whose others take the
fused one: the same layouts as unsampled runs and single steps, and the trace's
values those of tsgne_kl, on both sides of the 8,192 tiles up to which the update
sums Z, with the exaggeration's end beside a sampled step and apart from one."""
import numpy as np
import pytest

from paper_2310_11186_amd import synth, tsgne

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rows", [(8128, 1), (8129, 1), (500, 2), (500, 4), (3001, 0)])   # 8,128 and 8,256 tiles of 64
@pytest.mark.parametrize("variant", [tsgne.TSGNE_REPULSION_SYMMETRIC, tsgne.TSGNE_REPULSION_DIRECT])
@pytest.mark.parametrize("precision", [tsgne.TSGNE_PREC_SPLIT, tsgne.TSGNE_PREC_FP32])
@pytest.mark.parametrize("every,switch", [(1, 3), (3, 3), (3, 4), (5, 2)])
def test_sampled_and_fused_steps(gpu, n, rows, variant, precision, every, switch):
    import torch
    gi = synth.small_dcsbm(n, 4 * n, 2.3, 4, 4, n)
    rp, col = tsgne.tsgne_csr_from_edges(n, gi.edges)
    P = np.full(col.shape[0], 1.0 / col.shape[0], np.float32)
    g = tsgne.tsgne_graph_from_host_P(rp, col, P)
    kw = dict(tile_rows=rows, repulsion=variant, precision=precision, exaggeration_iters=switch, learning_rate=20.0)
    Y0 = torch.from_numpy(np.random.default_rng(n).standard_normal((n, 2)).astype(np.float32)).to(gpu)
    steps = 7
    plain, traced, single = Y0.clone(), Y0.clone(), Y0.clone()
    p = tsgne.tsgne_params_default(**kw)
    tsgne.tsgne_run(g, plain, steps, p)
    trace = tsgne.tsgne_run(g, traced, steps, tsgne.tsgne_params_default(kl_every=every, **kw))
    U, G = torch.zeros_like(Y0), torch.ones_like(Y0)
    kls = []
    for t in range(steps):
        tsgne.tsgne_step(g, single, U, G, t, p)
        if (t + 1) % every == 0:
            kls.append(tsgne.tsgne_kl(g, single))
    assert torch.equal(plain, traced) and torch.equal(plain, single)
    # in the split mode the sampled step's Z is bitwise the KL's own; in FP32 it is summed in FP32
    assert len(trace) == len(kls) == steps // every
    if precision == tsgne.TSGNE_PREC_SPLIT:
        assert np.array_equal(np.asarray(trace), np.asarray(kls))
    g.close()
