"""Row dictionaries (operators whose rows repeat): the finest level's streaming
product must be the serial row sums bit for bit, whether its rows repeat
everywhere, in part or nowhere, and after an update that ends the repetition."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _serial(rp, col, val, x):
    """Row sums in stored order, one rounded product and one rounded addition at a time."""
    s = np.zeros(rp.shape[0] - 1)
    length = np.diff(rp)
    for k in range(int(length.max())):
        r = np.nonzero(length > k)[0]
        e = rp[r] + k
        s[r] = s[r] + val[e] * x[col[e]]
    return s


def _spmv(h, x):
    import torch

    xd = torch.as_tensor(x).cuda()
    y = torch.empty_like(xd)
    h.level_spmv(0, xd, y)
    return y.cpu().numpy()


# two and three directions; one workgroup, a few, groups of several row blocks
@pytest.mark.parametrize("shape", [(2, 2), (40, 3), (63, 65), (300, 211), (4, 4, 4), (9, 31, 5), (63, 61, 17), (97, 81, 33),
                                   (160, 131, 57)])
@pytest.mark.parametrize("kind", ["constant", "pieces", "one", "every"])
def test_finest_product_is_the_serial_sum(shape, kind):
    import paper_2602_05686_amd as amg
    from workloads import q1

    rng = np.random.default_rng(5)
    ne = int(np.prod(shape))
    k = np.ones(ne)
    if kind == "pieces":
        k = np.where(np.arange(ne) % (7 * shape[0]) < 3 * shape[0], 1.0, 1e4)
    elif kind == "one":
        k[ne // 2] = 3.0
    elif kind == "every":
        k = rng.uniform(0.5, 2.0, ne)
    dim = len(shape)

    def left(x):
        return np.isclose(x[:, 0], 0.0), np.zeros(x.shape[0])

    p = q1.assemble_q1("t", shape, (1.0,) * dim, q1._iso(k, dim), np.ones(ne), left)
    h = amg.Hierarchy.from_problem(p, max_levels=16)
    x = rng.standard_normal(p.n)
    assert np.array_equal(_spmv(h, x), _serial(p.rowptr, p.col, p.val, x))
    # values that repeat nowhere, then the first ones again
    scale = rng.uniform(1.0, 2.0, p.val.shape[0])
    rows = np.repeat(np.arange(p.n), np.diff(p.rowptr))
    diag = rows == p.col
    v2 = np.where(diag, p.val * scale, p.val)
    h.update_values(v2)
    assert np.array_equal(_spmv(h, x), _serial(p.rowptr, p.col, v2, x))
    h.update_values(p.val)
    assert np.array_equal(_spmv(h, x), _serial(p.rowptr, p.col, p.val, x))
    h.close()


# offsets in more windows than are staged, rows as wide as one thread sums,
# and one wider (no dictionary: eight lanes sum such a row, in their own order)
@pytest.mark.parametrize("width", [12, 32, 33])
def test_scattered_offsets(width):
    import paper_2602_05686_amd as amg

    n = 4000
    offs = np.unique(np.concatenate([[0], 97 * np.arange(1, width // 2 + 1), -97 * np.arange(1, width // 2 + 1)]))
    c = (np.arange(n)[:, None] + offs[None, :])
    ok = (c >= 0) & (c < n)
    v = np.broadcast_to(np.where(offs == 0, 2.0 * width, -1.0 / (1 + np.abs(offs))), c.shape)
    if width == 32:  # the outer two offsets in different rows: at most 32 entries a row
        ok &= (offs[None, :] != offs[-1]) | (np.arange(n)[:, None] < n // 2)
        ok &= (offs[None, :] != offs[0]) | (np.arange(n)[:, None] > n // 2)
    rp = np.concatenate([[0], np.cumsum(ok.sum(1))]).astype(np.int32)
    h = amg.Hierarchy(rp, c[ok].astype(np.int32), v[ok], np.zeros((0, 2), np.int32), np.zeros((0, 1, 1)),
                      np.arange(n, dtype=np.float64)[:, None], amg.options(dim=1))
    x = np.random.default_rng(3).standard_normal(n)
    y, ref = _spmv(h, x), _serial(rp, c[ok], v[ok], x)
    if width <= 32:
        assert np.diff(rp).max() == (13 if width == 12 else 32)
        assert np.array_equal(y, ref)
    else:
        # two orders of at most 33 terms
        assert np.all(np.abs(y - ref) <= 2 * 33 * 2.0 ** -53 * _serial(rp, c[ok], np.abs(v[ok]), np.abs(x)))
    h.close()
