"""Host-only parts of the CG loop (paper_2602_05686_amd/csrc/cg_host.h),
driven by a small g++ program."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_05686_amd", "csrc")


def _run(tmp_path, body, *flags):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include <cstdio>\n#include "cg_host.h"\nusing namespace matamg;\n' + body)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", *flags, "-I", CSRC, str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout + res.stderr
    return res.stdout


def test_a_v_cycle_goes_ahead_only_where_the_next_step_needs_it(tmp_path):
    _run(tmp_path, r"""
#define CHECK(c) do { if (!(c)) { std::printf("FAIL line %d: %s\n", __LINE__, #c); return 1; } } while (0)
int main() {
    CHECK(!look_ahead(1, 1, 100, 1.0, 0.1, 1e-8));   // one level: the first step as a rule ends the solve
    CHECK(look_ahead(2, 1, 100, 1.0, 0.1, 1e-8));
    CHECK(!look_ahead(2, 100, 100, 1.0, 0.1, 1e-8)); // the last step allowed
    CHECK(!look_ahead(2, 5, 100, 1e-7, 0.1, 1e-8));  // foreseen at the tolerance
    CHECK(look_ahead(2, 5, 100, 1e-6, 0.1, 1e-8));
    return 0;
}
""")
