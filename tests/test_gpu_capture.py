"""V-cycles and finest products recorded in a graph by the caller, replayed after
amg_update_values: the replay reads the hierarchy as it is, whether the finest
rows repeated when it was recorded, repeat now, or repeat in other numbers.
Every replay must equal the direct call bit for bit (Jacobi: its weight is part of
the launches, and the values do not change it)."""

import numpy as np
import pytest

from test_gpu_forms import _box

pytestmark = pytest.mark.gpu


def _record(h, r, z, y):
    import torch

    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        s = torch.cuda.current_stream()
        h.vcycle(r, z, stream=s)
        h.level_spmv(0, r, y, stream=s)
    return g


# gathering and staged groups (the last two, in FP64), of 9 and 27 entries a row;
# one row block a group and several
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(40, 3), (300, 211), (63, 61, 17), (65, 63, 33), (97, 81, 33)])
def test_replay_after_update(shape, precision):
    import torch

    import paper_2602_05686_amd as amg

    vals = {kind: _box(shape, kind) for kind in ("constant", "pieces", "every")}
    p = vals["constant"]
    rows = np.repeat(np.arange(p.n), np.diff(p.rowptr))
    # the diagonal in several sizes, so that each group has more different rows
    step = np.where(rows == p.col, 1.0 + 0.25 * (rows // (5 * shape[0]) % 3), 1.0)
    states = {"constant": p.val, "steps": p.val * step, "pieces": vals["pieces"].val, "every": vals["every"].val}
    h = amg.Hierarchy.from_problem(p, max_levels=16, max_coarse=100, precision=precision, smoother="jacobi")
    rng = np.random.default_rng(3)
    r = torch.from_numpy(rng.standard_normal(p.n)).cuda()
    z, y, z0, y0 = (torch.empty_like(r) for _ in range(4))
    graphs = {}
    forms = []
    for at, state in enumerate(["constant", "every", "steps", "constant", "pieces", "every", "pieces", "constant"]):
        print(f"[gpu-case] capture {shape} {precision}: {at} {state}", flush=True)
        if at:
            h.update_values(states[state])
        forms.append(h.level_form(0)["dictionaries"])
        h.vcycle(r, z0)
        h.level_spmv(0, r, y0)
        torch.cuda.synchronize()
        if at < 5:
            graphs[at] = _record(h, r, z, y)
        for rep in range(3):
            for k, g in graphs.items():
                z.fill_(7.0)
                y.fill_(7.0)
                torch.cuda.synchronize()
                g.replay()
                torch.cuda.synchronize()
                assert torch.equal(z, z0) and torch.equal(y, y0), (at, state, k, rep)
            r.mul_(-1.0)  # (eager work between: the next replays are of other input)
            h.vcycle(r, z0)
            h.level_spmv(0, r, y0)
            torch.cuda.synchronize()
    assert forms[0] > 0 and forms[1] == 0 and forms[4] > 0 and forms[-1] > 0
    h.close()
