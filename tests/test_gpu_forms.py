"""Which form the streaming kernels take each operator in (row dictionaries,
column windows, the last levels in one workgroup), at the sizes at which
test_gpu_rows, test_gpu_windows and test_gpu_tail compare results, and FP32
products in those forms against the same operations in 64 bits."""

import numpy as np
import pytest

import test_gpu_tail as tail
import test_gpu_windows as windows

pytestmark = pytest.mark.gpu


def _box(shape, kind):
    from workloads import q1

    dim, ne = len(shape), int(np.prod(shape))
    k = np.ones(ne)
    if kind == "pieces":
        k = np.where(np.arange(ne) % (7 * shape[0]) < 3 * shape[0], 1.0, 1e4)
    elif kind == "every":
        k = np.random.default_rng(5).uniform(0.5, 2.0, ne)

    def left(x):
        return np.isclose(x[:, 0], 0.0), np.zeros(x.shape[0])

    return q1.assemble_q1("t", shape, (1.0,) * dim, q1._iso(k, dim), np.ones(ne), left)


def _windows(name, **kw):
    import paper_2602_05686_amd as amg

    n, parts, hubs = windows._CASES[name]
    a = windows._matrix(n, parts, hubs, np.random.default_rng(11))
    return amg.Hierarchy(a.indptr.astype(np.int32), a.indices.astype(np.int32), a.data, np.zeros((0, 2), np.int32),
                         np.zeros((0, 1, 1)), np.arange(n, dtype=np.float64)[:, None],
                         amg.options(dim=1, soc="sa", theta=0.0, max_coarse=16000, **kw))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(40, 3), (63, 65), (300, 211), (9, 31, 5), (63, 61, 17), (97, 81, 33)])
def test_repeating_rows_have_dictionaries(shape, precision):
    import paper_2602_05686_amd as amg

    for kind in ("constant", "pieces", "every"):
        p = _box(shape, kind)
        h = amg.Hierarchy.from_problem(p, max_levels=16, precision=precision)
        repeats = kind != "every"
        assert (h.level_form(0)["dictionaries"] > 0) == repeats
        # an update that ends the repetition, and one that brings it back
        rows = np.repeat(np.arange(p.n), np.diff(p.rowptr))
        scale = np.random.default_rng(6).uniform(1.0, 2.0, p.val.shape[0])
        h.update_values(np.where(rows == p.col, p.val * scale, p.val))
        assert h.level_form(0)["dictionaries"] == 0
        h.update_values(p.val)
        assert (h.level_form(0)["dictionaries"] > 0) == repeats
        h.close()


# 9 entries a row at any size, 27 of them in few rows and in many
@pytest.mark.parametrize("shape,staged", [((520, 510), False), ((720, 700), False), ((40, 40, 40), False), ((97, 81, 33), True)])
def test_windows_are_staged_for_many_long_rows(shape, staged):
    import paper_2602_05686_amd as amg

    h = amg.Hierarchy.from_problem(_box(shape, "constant"), max_levels=16)
    f = h.level_form(0)
    assert f["dictionaries"] > 0 and bool(f["staged"]) == staged
    h.close()


@pytest.mark.parametrize("width,taken", [(12, True), (32, True), (33, False)])
def test_dictionary_rows_are_those_one_thread_sums(width, taken):
    import paper_2602_05686_amd as amg

    n = 4000
    offs = np.arange(-(width // 2), width // 2 + 1) if width % 2 else np.delete(np.arange(-(width // 2), width // 2 + 1), 0)
    c = np.arange(n)[:, None] + 97 * offs[None, :]
    ok = (c >= 0) & (c < n)
    # (symmetric but for the one offset that an even width lacks, which is zero)
    v = np.broadcast_to(np.where(offs == 0, 2.0 * width, -1.0 / (1 + np.abs(offs))), c.shape)
    v = np.where((width % 2 == 0) & (offs == width // 2), 0.0, v)
    rp = np.concatenate([[0], np.cumsum(ok.sum(1))]).astype(np.int32)
    assert np.diff(rp).max() == width
    h = amg.Hierarchy(rp, c[ok].astype(np.int32), v[ok], np.zeros((0, 2), np.int32), np.zeros((0, 1, 1)),
                      np.arange(n, dtype=np.float64)[:, None], amg.options(dim=1))
    assert (h.level_form(0)["dictionaries"] > 0) == taken
    h.close()


@pytest.mark.parametrize("name,columns,threads", [("ring", "windows", 1), ("edge", "windows", 1), ("planes", "windows", 1),
                                                  ("half", "windows", 1), ("many", "32-bit", 1), ("long", "windows", 1),
                                                  ("wide", "windows", 8)])
def test_wide_blocks_have_windows(name, columns, threads):
    h = _windows(name)
    f, nnz = h.level_form(0), h.stats()["nnz"][0]
    assert f["columns"] == columns and f["threads_per_row"] == threads and f["dictionaries"] == 0
    if name in ("ring", "edge", "planes"):
        assert f["windowed_entries"] == nnz
    elif columns == "windows":
        assert nnz // 2 <= f["windowed_entries"] < nnz  # some blocks have none
    h.close()


# (the first three as in test_gpu_tail; a coarsest level beyond the dense limit)
@pytest.mark.parametrize("shape,contrast,max_coarse,first", [((64, 64), 6.0, 100, {"fp64": 2, "fp32": 1}),
                                                             ((130, 121), 3.0, 50, {"fp64": 2, "fp32": 2}),
                                                             ((16, 14, 12), 2.0, 40, {"fp64": 2, "fp32": 2}),
                                                             ((130, 121), 3.0, 350, None)])
@pytest.mark.parametrize("smoother", [dict(), dict(cheb_degree=1), dict(cheb_degree=4), dict(cheb_degree=5), dict(smoother="jacobi")])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_last_levels_in_one_workgroup(shape, contrast, max_coarse, first, smoother, precision):
    import paper_2602_05686_amd as amg

    p = tail._problem(shape, contrast)
    h = amg.Hierarchy.from_problem(p, max_coarse=max_coarse, max_levels=16, precision=precision, **smoother)
    levels = h.stats()["levels"]
    taken = [bool(h.level_form(l)["one_workgroup"]) for l in range(levels)]
    start = levels if first is None or smoother.get("cheb_degree") == 5 else first[precision]
    assert taken == [l >= start for l in range(levels)]
    h.close()


# layered stacks: levels with rows of 110 to 170 entries among narrower ones
@pytest.mark.parametrize("n,max_coarse", [(16, 20), (24, 10), (24, 60), (30, 20)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_levels_with_long_rows_keep_their_launches(n, max_coarse, precision):
    import paper_2602_05686_amd as amg
    from workloads import layered_stack_3d

    p = layered_stack_3d(n=n, repeats=4)
    kw = dict(max_coarse=max_coarse, max_levels=16, precision=precision)
    h = amg.Hierarchy.from_problem(p, **kw)
    levels = h.stats()["levels"]
    longest = [max(int(np.diff(h.level_csr(l, w)[0]).max()) for w in "APR") for l in range(levels - 1)]
    taken = [bool(h.level_form(l)["one_workgroup"]) for l in range(levels)]
    start = levels - 1
    while longest[start - 1] <= 96:
        start -= 1
    # (the narrow levels below the first long row are few and small enough)
    assert any(100 < m <= 256 for m in longest[1:])
    assert taken == [l >= start and start < levels - 1 for l in range(levels)]
    with amg.Server(budget_bytes=2 << 30, dim=p.dim, **kw) as srv:
        ref = srv.result(tail._done(srv, srv.submit(p, tol=1e-8, max_iter=60)))[0]
    x, _ = h.solve(p.b, tol=1e-8, max_iter=60, raise_on_error=False)
    assert np.array_equal(x, ref)
    h.close()


# a request whose finest rows have dictionaries, and two with windows
@pytest.mark.parametrize("name", ["stack", "ring", "wide"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_admission_estimate_covers_the_forms(name, precision):
    import types

    import paper_2602_05686_amd as amg
    from workloads import layered_stack_3d

    kw = dict(precision=precision, max_levels=16)
    if name == "stack":
        p = layered_stack_3d(n=48, repeats=16)
    else:
        n, parts, hubs = windows._CASES[name]
        a = windows._matrix(n, parts, hubs, np.random.default_rng(11))
        p = types.SimpleNamespace(n=n, dim=1, rowptr=a.indptr.astype(np.int32), col=a.indices.astype(np.int32), val=a.data,
                                  elem_nodes=np.zeros((0, 2), np.int32), elem_sigma=np.zeros((0, 1, 1)),
                                  coords=np.arange(n, dtype=np.float64)[:, None], b=np.ones(n))
        kw.update(soc="sa", theta=0.0)
    with amg.Server(budget_bytes=8 << 30, dim=p.dim, **kw) as srv:
        _, _, timeline = srv.result(tail._done(srv, srv.submit(p, max_iter=3)))
        assert 0 < timeline["resident_bytes"] <= timeline["setup_peak_bytes"] <= timeline["est_bytes"]
        assert srv.stats()["estimate_exceeded"] == 0


def _csr(rcv, shape):
    import scipy.sparse as sp

    return sp.csr_matrix((rcv[2], rcv[1], rcv[0]), shape=shape)


def _integers(case):
    """A diagonally dominant matrix of integers, its diagonal powers of two: off-diagonals -1, or (`every`) -1 to -3
    at random; `pieces`: twice the diagonal in every other run of rows."""
    import scipy.sparse as sp

    if isinstance(case, str):
        n, parts, hubs = windows._CASES[case]
        off, kind = windows._matrix(n, parts, hubs, np.random.default_rng(11)), "every"
    else:
        shape, kind = case
        off = sp.identity(1)
        for m in shape[::-1]:
            off = sp.kron(off, sp.diags([np.ones(m - 1), np.ones(m), np.ones(m - 1)], [-1, 0, 1]))
    off = (off - sp.diags(off.diagonal())).tocsr()
    off.eliminate_zeros()
    off.data[:] = 1.0
    if kind == "every":
        up = sp.triu(off, format="csr")
        up.data[:] = np.random.default_rng(8).integers(1, 4, up.nnz)
        off = up + up.T
    diag = 2.0 ** np.ceil(np.log2(2.0 * np.ravel(off.sum(1))))
    if kind == "pieces":
        diag *= 1.0 + np.arange(diag.size) // (3 * shape[0]) % 2
    a = (sp.diags(diag) - off).tocsr()
    a.sort_indices()
    return a


# Dictionaries of 9- and 27-entry rows, of one and of several row blocks a group;
# no dictionaries; windows at one and at eight threads a row.  Integers, powers of
# two and an unsmoothed prolongator make everything up to the coarse right-hand
# side exact in FP32, the first product with A included.
@pytest.mark.parametrize("case,columns,dictionaries", [(((150, 130), "constant"), "16-bit", True),
                                                       (((63, 65), "pieces"), "16-bit", True),
                                                       (((33, 29, 21), "pieces"), "16-bit", True),
                                                       (((33, 29, 21), "every"), "16-bit", False),
                                                       (((58, 56, 51), "constant"), "16-bit", True),
                                                       ("ring", "windows", False), ("wide", "windows", False)])
def test_fp32_products_of_every_form(case, columns, dictionaries):
    import scipy.sparse as sp
    import scipy.sparse.linalg as spl
    import torch

    import paper_2602_05686_amd as amg

    u = 2.0 ** -24
    a = _integers(case)
    n = a.shape[0]
    h = amg.Hierarchy(a.indptr.astype(np.int32), a.indices.astype(np.int32), a.data, np.zeros((0, 2), np.int32),
                      np.zeros((0, 1, 1)), np.arange(n, dtype=np.float64)[:, None],
                      amg.options(dim=1, soc="sa", theta=0.0, max_coarse=min(16000, n // 2), precision="fp32", smoother="jacobi",
                                  jacobi_omega=0.5, jacobi_sweeps=1, omega_sym=0.0))
    f, st = h.level_form(0), h.stats()
    assert f["columns"] == columns and (f["dictionaries"] > 0) == dictionaries and st["levels"] == 2
    if dictionaries and n > 150000:
        assert f["dictionaries"] < f["blocks"]
    nc = st["n"][1]
    p = _csr(h.level_csr(0, "P"), shape=(n, nc))
    ac = sp.csc_matrix(_csr(h.level_csr(1, "A"), shape=(nc, nc)))
    b = np.random.default_rng(4).integers(-8, 9, n).astype(np.float64)
    rb = torch.as_tensor(b).cuda()
    z = torch.empty_like(rb)
    h.vcycle(rb, z)
    h.close()

    d = 0.5 / a.diagonal()
    x = d * b
    r = b - a @ x
    coarse = p.T @ r
    for exact in (x, r, coarse):
        assert np.array_equal(exact, exact.astype(np.float32))
    # the coarse solve is in 64 bits, rounded once (2 u: and a last bit of the inverse)
    e = spl.spsolve(ac, coarse)
    x = x + p @ e
    err = 2 * u * (abs(p) @ np.abs(e)) + u * np.abs(x)
    s = a @ x
    length = np.diff(a.indptr)
    res = b - s
    err_res = abs(a) @ err + (length + 1) * u * (abs(a) @ np.abs(x)) + u * np.abs(res)
    ref = x + d * res
    bound = 1.01 * (err + d * err_res + u * np.abs(ref))
    assert np.linalg.norm(bound) <= 1e-4 * np.linalg.norm(ref)
    off = np.abs(z.cpu().numpy() - ref)
    assert np.all(off <= bound), float(np.max(off / bound))
