"""The V-cycle's last levels in one workgroup: a solve is the server's, which
launches level by level, bit for bit, with one to several levels in the
workgroup and with none, in both precisions, and after updates."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _problem(shape, contrast):
    from workloads import q1

    rng = np.random.default_rng(int(np.prod(shape)))
    dim, ne = len(shape), int(np.prod(shape))
    k = 10.0 ** (contrast * rng.random(ne))

    def left(x):
        return np.isclose(x[:, 0], 0.0), np.zeros(x.shape[0])

    return q1.assemble_q1("t", shape, (1.0,) * dim, q1._iso(k, dim), np.ones(ne), left)


# coarsest sizes on both sides of the dense limit; a level that fits and one
# that does not; rows wider than one thread sums in sequence
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("smoother", [dict(), dict(cheb_degree=1), dict(cheb_degree=4), dict(cheb_degree=5), dict(smoother="jacobi")])
@pytest.mark.parametrize("shape,contrast,max_coarse", [((24, 20), 0.0, 60), ((64, 64), 6.0, 100), ((130, 121), 3.0, 50),
                                                       ((90, 100), 1.0, 300), ((16, 14, 12), 2.0, 40)])
def test_solve_is_the_servers(shape, contrast, max_coarse, smoother, precision):
    import paper_2602_05686_amd as amg

    p = _problem(shape, contrast)
    kw = dict(max_coarse=max_coarse, max_levels=16, precision=precision, **smoother)
    with amg.Server(budget_bytes=2 << 30, dim=p.dim, **kw) as srv:
        ref = srv.result(_done(srv, srv.submit(p, tol=1e-8, max_iter=60)))[0]
    h = amg.Hierarchy.from_problem(p, **kw)
    x, _ = h.solve(p.b, tol=1e-8, max_iter=60, raise_on_error=False)
    assert np.array_equal(x, ref)
    # other values, then the first ones again (four times: exact under the
    # square roots of the dense factor too)
    h.update_values(4.0 * p.val)
    h.update_values(p.val)
    x, _ = h.solve(p.b, tol=1e-8, max_iter=60, raise_on_error=False)
    assert np.array_equal(x, ref)
    h.update_values(4.0 * p.val)
    x2, _ = h.solve(4.0 * p.b, tol=1e-8, max_iter=60, raise_on_error=False)
    assert np.array_equal(x2, ref)
    h.close()


def _done(srv, rid):
    left = {rid}
    while left:
        left.difference_update(srv.poll(timeout_s=1.0))
    return rid
