"""Sparse products with rows of very different widths: a grid with a node
connected to thousands of others, whose Galerkin rows hold up to all coarse
columns.  Every route (a thread, a wavefront's table of each size, a
workgroup's table up to nearly full, global memory) must give the same
operators bit for bit."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _hub_laplacian(m, fan, seed):
    """Graph Laplacian plus identity of an m x m grid, its node 0 also tied weakly to `fan` others."""
    import scipy.sparse as sp

    rng = np.random.default_rng(seed)
    n = m * m
    i = np.arange(n).reshape(m, m)
    a = np.concatenate([i[:, :-1].ravel(), i[:-1].ravel(), np.zeros(fan, int)])
    b = np.concatenate([i[:, 1:].ravel(), i[1:].ravel(), 2 + rng.choice(n - 2, fan, replace=False)])
    w = np.concatenate([rng.uniform(0.5, 1.0, 2 * m * (m - 1)), np.full(fan, 1e-3)])
    g = sp.coo_matrix((np.concatenate([w, w]), (np.concatenate([a, b]), np.concatenate([b, a]))), shape=(n, n)).tocsr()
    g.sum_duplicates()
    s = (sp.diags(1.0 + np.asarray(g.sum(1)).ravel()) - g).tocsr()
    s.sort_indices()
    return s, np.stack([np.repeat(np.arange(m), m), np.tile(np.arange(m), m)], 1).astype(float)


def _levels(s, xy, route, monkeypatch):
    import paper_2602_05686_amd as amg

    if route:
        monkeypatch.setenv("MATAMG_SPGEMM_ROUTE", route)
    else:
        monkeypatch.delenv("MATAMG_SPGEMM_ROUTE", raising=False)
    h = amg.Hierarchy(s.indptr.astype(np.int32), s.indices.astype(np.int32), s.data, np.zeros((0, 4), np.int32),
                      np.zeros((0, 2, 2)), xy, amg.options(dim=2, soc="sa", max_coarse=12000, theta=0.02))
    st = h.stats()
    out = [h.level_csr(l, w) for l in range(st["levels"] - 1) for w in "PR"] + \
          [h.level_csr(l, "A") for l in range(1, st["levels"])]
    h.close()
    return out


# widest rows: a wavefront's middle and largest tables, the workgroup's table half and nearly full
@pytest.mark.parametrize("m,fan,widest", [(130, 100, 60), (130, 400, 200), (130, 900, 400), (230, 7000, 3500),
                                          (300, 9000, 5500)])
def test_every_route_gives_the_same_products(m, fan, widest, monkeypatch):
    s, xy = _hub_laplacian(m, fan, m)
    ref = _levels(s, xy, None, monkeypatch)
    assert max(int(np.diff(rp).max()) for rp, _, _ in ref) > widest
    # every row in global memory beyond 512 columns; all rows by wavefronts;
    # all by the workgroup's table beyond 16 columns; all by threads where they fit
    for route in ("64,512,0", "0,512,8192", "0,16,8192", "64,16,0"):
        got = _levels(s, xy, route, monkeypatch)
        assert len(got) == len(ref)
        for (rp0, c0, v0), (rp1, c1, v1) in zip(ref, got):
            assert np.array_equal(rp0, rp1) and np.array_equal(c0, c1) and np.array_equal(v0, v1)
