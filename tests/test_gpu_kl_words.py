"""KL's read-back: a pinned word per workspace while there are any (512), pageable
memory past them, and the words of freed graphs again."""
import threading

import numpy as np
import pytest

import oracle
from bars import kl_close
from paper_2310_11186_amd import tsgne

pytestmark = pytest.mark.gpu


def test_kl_with_more_graphs_than_pinned_words(gpu):
    import torch
    n = 40
    rp, col = tsgne.tsgne_csr_from_edges(n, [(i, (i + 1) % n) for i in range(n)])
    P = np.full(col.shape[0], 1.0 / col.shape[0], np.float32)
    Ys = [np.random.default_rng(k).standard_normal((n, 2)).astype(np.float32) for k in range(4)]
    exact = [oracle.kl(rp, col, P, Y.astype(np.float64)) for Y in Ys]
    dY = [torch.from_numpy(Y).to(gpu) for Y in Ys]
    graphs = [tsgne.tsgne_graph_from_host_P(rp, col, P) for _ in range(520)]
    for _ in range(2):
        for k, g in enumerate(graphs):
            assert kl_close(tsgne.tsgne_kl(g, dY[k % 4]), exact[k % 4]), k
        for g in graphs[::2]:
            g.close()
        graphs[::2] = [tsgne.tsgne_graph_from_host_P(rp, col, P) for _ in graphs[::2]]
    wrong = []

    def many(w):
        s = torch.cuda.Stream()
        for k in range(w, 520, 4):
            if not kl_close(tsgne.tsgne_kl(graphs[k], dY[w], s), exact[w]):
                wrong.append(k)
            graphs[k].close()

    threads = [threading.Thread(target=many, args=(w,)) for w in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
