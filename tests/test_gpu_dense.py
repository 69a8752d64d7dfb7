"""The coarsest level's dense inverse (64 x 64 tiles, 16-column panels,
matrix-core products) against numpy, on one-level hierarchies of full SPD
matrices at the edges of its tiles."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

COND = 1e3


def _spd(n, seed):
    rng = np.random.default_rng(seed)
    q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    a = (q * np.geomspace(1.0, COND, n)) @ q.T
    return 0.5 * (a + a.T)


def _hierarchy(a):
    import paper_2602_05686_amd as amg

    n = a.shape[0]
    rp = np.arange(0, n * n + 1, n, dtype=np.int32)
    col = np.tile(np.arange(n, dtype=np.int32), n)
    return amg.Hierarchy(rp, col, a.reshape(-1), np.zeros((0, 2), np.int32), np.zeros((0, 1, 1)),
                         np.arange(n, dtype=np.float64)[:, None], amg.options(dim=1))


def _inverse_times(a, r):
    import torch

    h = _hierarchy(a)
    assert h.stats()["levels"] == 1
    rd = torch.as_tensor(r).cuda()
    z = torch.empty_like(rd)
    h.vcycle(rd, z)
    out = z.cpu().numpy()
    h.close()
    return out


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 63, 64, 65, 127, 128, 129, 200, 321, 700])
def test_dense_inverse_matches_numpy(n):
    a = _spd(n, n)
    r = np.random.default_rng(1).standard_normal(n)
    z = _inverse_times(a, r)
    ref = np.linalg.solve(a, r)
    # Cholesky, inverse of the factor and its product: O(n eps cond) each
    assert np.linalg.norm(z - ref) <= 10 * n * 2.0 ** -53 * COND * np.linalg.norm(ref)


def test_far_exponents_take_the_plain_divisions():
    # a scale of 2^140 puts the factor's diagonal beyond the range of the
    # refined quotients; every rounding scales with it, so the two routes must
    # agree bit for bit
    n = 150
    a = _spd(n, 7)
    r = np.random.default_rng(2).standard_normal(n)
    assert np.array_equal(_inverse_times(a, r), _inverse_times(a * 2.0 ** 140, r) * 2.0 ** 140)


@pytest.mark.parametrize("bad", [0, 40, 64, 129])
def test_indefinite_matrix_is_refused(bad):
    import paper_2602_05686_amd as amg

    a = _spd(130, 3)
    a[bad, bad] = -1.0
    with pytest.raises(amg.AmgError) as e:
        _hierarchy(a)
    assert e.value.status == "NOT_SPD"
