"""Operators some of whose row blocks reach 2^16 columns or further: blocks with
one to four windows of columns, with more (plain columns), with few repeated
columns and with one long row, alone and in one matrix."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _matrix(n, parts, hubs, rng):
    """Symmetric, diagonally dominant; rows lo..hi of parts couple to the given offsets (mod n)."""
    import scipy.sparse as sp

    i, j = [], []
    for lo, hi, offs in parts:
        r = np.arange(lo, hi)
        for d in offs:
            i.append(r)
            j.append((r + d) % n)
    for h, m in hubs:
        i.append(np.full(m, h))
        j.append((h + 1 + 7 * np.arange(m)) % n)
    i, j = np.concatenate(i), np.concatenate(j)
    keep = i != j
    i, j = i[keep], j[keep]
    b = sp.coo_matrix((-rng.uniform(0.5, 1.0, i.size), (i, j)), shape=(n, n)).tocsr()
    a = (b + b.T).tocsr()
    a = (a + sp.diags(np.asarray(abs(a).sum(axis=1)).ravel() + 1.0)).tocsr()
    a.sort_indices()
    return a


_NEAR = [1, 2, 3, 4, 5]
_CASES = {
    # (n, parts, hubs): narrow blocks but for those at the two ends
    "ring": (70000, [(0, 70000, _NEAR + [300, 301])], []),
    # the last column of a window, and the first beyond it
    "edge": (140000, [(0, 140000, [1, 2, 65535, 65536])], []),
    # three windows everywhere, four where they wrap
    "planes": (250000, [(0, 250000, [1, 2, 70000, 70001, 70002])], []),
    # more windows than are kept: plain columns in half of the blocks, in all
    "half": (400000, [(0, 150000, _NEAR + [6, 7, 8, 9]), (150000, 250000, [1, 66000, 132000])], []),
    "many": (400000, [(0, 400000, [1, 66000, 132000])], []),
    # one long row among narrow ones, and eight threads a row
    "long": (90000, [(0, 90000, _NEAR)], [(45000, 9000)]),
    "wide": (90000, [(0, 90000, list(range(1, 26)))], [(45000, 300)]),
}


@pytest.mark.parametrize("name", sorted(_CASES))
def test_product_over_windows(name):
    import torch

    import paper_2602_05686_amd as amg

    n, parts, hubs = _CASES[name]
    rng = np.random.default_rng(11)
    a = _matrix(n, parts, hubs, rng)
    rp, col, val = a.indptr.astype(np.int32), a.indices.astype(np.int32), a.data
    h = amg.Hierarchy(rp, col, val, np.zeros((0, 2), np.int32), np.zeros((0, 1, 1)),
                      np.arange(n, dtype=np.float64)[:, None], amg.options(dim=1, soc="sa", theta=0.0, max_coarse=16000))
    x = rng.standard_normal(n)
    xd = torch.as_tensor(x).cuda()
    y = torch.empty_like(xd)
    h.level_spmv(0, xd, y)
    got = y.cpu().numpy()
    # any order of a row's additions: each sum within (entries) eps of the sum of magnitudes
    ref = a @ x
    mag = abs(a) @ abs(x)
    length = np.diff(rp)
    assert np.all(np.abs(got - ref) <= 2.0 * length * 2.0**-53 * mag)
    h.close()
