"""bench.py's line on stdout: the contract's fields in full and the main figures
of the other parts, short enough for logs that keep the last few kilobytes."""

import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

CONTRACT = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
            "vs_baseline", "dtype", "data", "config")
_X = 1234567.123456789


def _stats():
    return dict(mean=_X, std=_X, median=_X, min=_X, max=_X)


def _vcycle():
    return dict(ms=_X, alg_bytes=_X, alg_GBps=_X, frac_of_peak=_X, fine_smoother_us=_X, fine_smoother_GBps=_X)


def _form():
    return dict(status="OK", iterations=2576, rel_res=_X, levels=[7189057] * 11, op_complexity=_X,
                t_setup_ms_stats=_stats(), t_solve_ms_stats=_stats(), step_ms_stats=_stats(), dof_per_s=_X,
                solve_only_dof_per_s=_X, vcycle=_vcycle(), rel_err_vs_closed_form=_X)


def _record():
    row = dict(refine=4, h="h/16", dof=13096800, nnz=337005600, kappa=_X, theta=_X, status="OK", levels=6,
               op_complexity=_X, iterations=51, cost=_X, t_setup_ms=_X, t_solve_ms=_X)
    return dict(
        metric="DOF/s to rel-res 1e-8 (setup + AMG-PCG solve)", value=_X, unit="DOF/s", n_gpus=1, steps=20, warmup=5,
        ms_per_step=_X, higher_is_better=True, scaling="weak", vs_baseline=None, dtype="f64", data="synthetic",
        config=dict(workload="layered stack " * 8, dof=2146689, nnz=56210557, theta=0.08, tol=1e-8),
        solve_only_dof_per_s=_X, t_setup_ms=_X, t_solve_ms=_X, step_ms_stats=_stats(), t_setup_ms_stats=_stats(),
        t_solve_ms_stats=_stats(), iterations_per_step=[108], iterations=108, rel_res_true=_X,
        rel_err_vs_closed_form=_X, levels=[2146689] * 8, op_complexity=_X, vcycle=_vcycle(),
        seeded_x0=dict(seeds=5, iterations=[105] * 5, t_solve_ms_median=_X, solve_only_dof_per_s_median=_X),
        roofline=dict(bound="hbm", kernel="k" * 100, achieved=_X, peak=_X, unit="GB/s", frac=_X, traffic=_X,
                      avg_launch_us=_X, launches=100, alg_bytes_per_launch=_X,
                      achievable=dict(read_GBps=_X, copy_GBps=_X, fill_GBps=_X), frac_of_achievable_read=_X),
        fp32_form=dict(_form(), t_solve_s=_X, speedup_vs_fp64_solve=_X, speedup_per_iteration=_X,
                       speedup_vs_fp64_vcycle=_X, rel_err_vs_fp64_form=_X, x0_seeds=dict(v=[_X] * 20),
                       aniso=dict(workload="w" * 80, n=912673, nnz=22720485, fp64=_form(), fp32=_form(), speedup=_X)),
        layered192=dict(workload="w" * 100, n=7189057, nnz=1, fp64=_form(), fp32=_form(), speedup=_X),
        serving=dict(requests=256, p50_latency_s=_X, p99_latency_s=_X, solves_per_s=_X,
                     status_counts=dict(OK=201, NOT_CONVERGED=55), not_converged_requests=list(range(55)),
                     converged_only=dict(requests=201, solves_per_s=_X), alone_vs_mix=[dict(request=1)] * 2),
        studies=dict(compare=dict(rows=[row] * 36), sweep=dict(rows=[row] * 400), annulus=dict(rows=[row] * 50)),
        cpu_baseline=dict(value=_X, unit="DOF/s", cores=1, kind="oracle", sample="s" * 150, t_setup_s=_X, t_solve_s=_X,
                          iterations=103, status=0, rel_res=_X, host_cpu="AMD EPYC", host_threads=16))


def test_line_is_short_and_complete():
    import bench

    rec = _record()
    assert len(json.dumps(rec)) > 100000
    line = json.dumps(bench.headline(rec))
    assert len(line) < 7000
    got = json.loads(line)
    for k in CONTRACT:
        assert got[k] == rec[k]
    assert got["roofline"]["traffic"] and got["fp32_form"]["vcycle"]["ms"] and got["layered192"]["fp32"]["iterations"] == 2576
    assert got["serving"]["converged_only"]["requests"] == 201 and got["studies"]["sweep"] == "400 rows"


def test_line_of_a_partial_run():
    import bench

    rec = dict(_record(), fp32_form=None, layered192=None, serving=None, studies=None, cpu_baseline=None, seeded_x0=None)
    got = json.loads(json.dumps(bench.headline(rec)))
    assert all(got[k] == rec[k] for k in CONTRACT) and got["serving"] is None


def test_roofline_names_the_kernel_that_ran():
    import bench

    form = dict(threads_per_row=1, block_entries=4096, blocks=1, columns="16-bit", windowed_entries=0, dictionaries=7,
                staged=1, one_workgroup=0)
    assert "k_rows" in bench.smoother_kernel(form)
    assert "k_stream" in bench.smoother_kernel(dict(form, dictionaries=0))
