"""The CSR check's symmetry test: of an edge's two entries only the one whose far
row is the shorter searches it, so a missing entry shows either as a search
that finds nothing or as an entry that nothing found."""
import numpy as np
import pytest

import oracle
from paper_2310_11186_amd import tsgne

pytestmark = pytest.mark.gpu


def drop(rp, col, i, j):
    e = rp[i] + int(np.flatnonzero(col[rp[i]:rp[i + 1]] == j)[0])
    rp = rp.copy()
    rp[i + 1:] -= 1
    return rp, np.delete(col, e)


def star(leaves):        # a hub, its leaves, and a path among the first of them: long, short and equal rows
    hub = [(0, v) for v in range(1, leaves + 1)]
    path = [(v, v + 1) for v in range(1, leaves // 2)]
    return tsgne.tsgne_csr_from_edges(leaves + 1, np.array(hub + path, np.int32))


@pytest.mark.parametrize("leaves", [4, 255, 1500])       # one to several workgroups of 1,024 entries
@pytest.mark.parametrize("which", ["hub_to_leaf", "leaf_to_hub", "up", "down", "two_that_cancel"])
def test_one_sided_entries_are_refused(gpu, leaves, which):
    import torch
    rp, col = star(leaves)
    if which == "hub_to_leaf":
        rp, col = drop(rp, col, 0, leaves)
    elif which == "leaf_to_hub":
        rp, col = drop(rp, col, leaves, 0)
    elif which == "up":
        rp, col = drop(rp, col, 1, 2) if leaves > 4 else drop(rp, col, 0, 1)
    elif which == "down":
        rp, col = drop(rp, col, 2, 1) if leaves > 4 else drop(rp, col, 1, 0)
    else:                # as many searched as not, one of them found nothing
        rp, col = drop(rp, col, 0, leaves)
        rp, col = drop(rp, col, leaves - 1, 0)
    rp_d, col_d = torch.from_numpy(rp).to(gpu), torch.from_numpy(col).to(gpu)
    X = torch.zeros((leaves + 1, 2), dtype=torch.float32, device=gpu)
    for call in (lambda: tsgne.tsgne_build_P(rp_d, col_d, X, 2.0),
                 lambda: tsgne.tsgne_shortest_path_embedding(rp_d, col_d, torch.zeros(1, dtype=torch.int32, device=gpu))):
        with pytest.raises(tsgne.TsgneError) as e:
            call()
        assert e.value.status == tsgne.TSGNE_E_GRAPH


@pytest.mark.parametrize("leaves", [4, 255, 1500])
def test_mirror_of_hubs(gpu, leaves):
    import torch
    rp, col = star(leaves)
    X = torch.from_numpy(np.random.default_rng(1).standard_normal((leaves + 1, 2)).astype(np.float32)).to(gpu)
    ex = tsgne.tsgne_build_P(torch.from_numpy(rp).to(gpu), torch.from_numpy(col).to(gpu), X, 2.0).export()
    assert np.array_equal(ex["mirror"], oracle.mirror(rp, col))
