"""The device's row-block partition against the host walk (the setup compares
them itself under MATAMG_CHECK_PARTITION=1): one chunk of rows and several, their
edges, long rows at them, eight threads a row, chunks of several tiles."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

_TILE = 16384
_CHUNKS = 512


def _band(n, half, hubs, rng):
    """Entries (i, j) with |i - j| <= min(half_i, half_j), and each hub with its next 400 rows."""
    import scipy.sparse as sp

    i, j = [], []
    for d in range(1, int(half.max()) + 1):
        r = np.arange(n - d)
        r = r[np.minimum(half[:-d], half[d:]) >= d]
        i.append(r)
        j.append(r + d)
    for h in hubs:
        r = np.arange(h + 1, min(n, h + 401))
        i.append(np.full(r.size, h))
        j.append(r)
    i = np.concatenate(i) if i else np.zeros(0, np.int64)
    j = np.concatenate(j) if j else np.zeros(0, np.int64)
    b = sp.coo_matrix((np.ones(i.size), (i, j)), shape=(n, n)).tocsr()
    b.data[:] = -1.0
    a = (b + b.T).tocsr()
    a = (a + sp.diags(np.asarray(abs(a).sum(axis=1)).ravel() + 0.5)).tocsr()
    a.sort_indices()
    return a


@pytest.mark.parametrize("kind", ["three", "mixed", "long", "eight"])
@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, _TILE - 1, _TILE, _TILE + 1, 3 * _TILE + 77, 65536, 65537])
def test_partition(n, kind, monkeypatch):
    import paper_2602_05686_amd as amg

    rng = np.random.default_rng(n)
    half = {"three": np.ones(n, int), "mixed": rng.integers(1, 16, n), "long": rng.integers(1, 4, n),
            "eight": np.where(np.arange(n) % 1000 < 600, 60, 2)}[kind]
    half = np.minimum(half, max(n - 1, 1))
    hubs = [] if kind != "long" else [h for h in (0, 1, _TILE - 2, _TILE - 1, _TILE, 2 * _TILE, n - 402, n - 2) if 0 <= h < n - 1]
    a = _band(n, half, sorted(set(hubs)), rng)
    monkeypatch.setenv("MATAMG_CHECK_PARTITION", "1")
    h = amg.Hierarchy(a.indptr.astype(np.int32), a.indices.astype(np.int32), a.data, np.zeros((0, 2), np.int32),
                      np.zeros((0, 1, 1)), np.arange(n, dtype=np.float64)[:, None],
                      amg.options(dim=1, soc="sa", theta=0.0, max_coarse=500, max_levels=16))
    h.close()


def test_partition_of_many_tiles(monkeypatch):
    import paper_2602_05686_amd as amg

    n = _CHUNKS * _TILE + 3
    rp = np.concatenate([[0, 2], 2 + 3 * np.arange(1, n - 1), [3 * n - 2]]).astype(np.int32)
    col = (np.arange(n)[:, None] + np.array([-1, 0, 1])).ravel()[1:-1].astype(np.int32)
    val = np.tile([-1.0, 2.5, -1.0], n)[1:-1]
    monkeypatch.setenv("MATAMG_CHECK_PARTITION", "1")
    h = amg.Hierarchy(rp, col, val, np.zeros((0, 2), np.int32), np.zeros((0, 1, 1)),
                      np.arange(n, dtype=np.float64)[:, None], amg.options(dim=1, soc="sa", theta=0.0, max_levels=16))
    h.close()
