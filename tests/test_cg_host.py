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


_WAIT = r"""
#include <atomic>
#include <chrono>
#include <ctime>
#include <sched.h>
#include <thread>
using us = std::chrono::microseconds;
static double seconds(clockid_t c) { timespec t; clock_gettime(c, &t); return t.tv_sec + 1e-9 * t.tv_nsec; }
static bool never() { return false; }
"""


def test_waiting_threads_share_a_core(tmp_path):
    # two threads on one core hand a number to and fro: a waiter that kept the
    # core until the scheduler took it would hold each of the 400 turns up for a
    # time slice of some milliseconds
    out = _run(tmp_path, _WAIT + r"""
int main() {
    cpu_set_t all, one;
    sched_getaffinity(0, sizeof all, &all);
    int cpu = 0;
    while (!CPU_ISSET(cpu, &all)) ++cpu;
    CPU_ZERO(&one);
    CPU_SET(cpu, &one);
    sched_setaffinity(0, sizeof one, &one);
    std::atomic<int> turn{0};
    auto play = [&](int me) {
        for (int k = me; k < 400; k += 2) {
            if (!wait_until(false, [&] { return turn.load() == k; }, never)) return;
            turn.store(k + 1);
        }
    };
    const double t = seconds(CLOCK_MONOTONIC);
    std::thread other(play, 1);
    play(0);
    other.join();
    std::printf("%f", seconds(CLOCK_MONOTONIC) - t);
    return turn.load() == 400 ? 0 : 1;
}
""", "-pthread")
    assert float(out) < 0.4, f"{float(out) / 400 * 1e3:.2f} ms a turn"


def test_a_long_wait_gives_its_core_back(tmp_path):
    out = _run(tmp_path, _WAIT + r"""
int main() {
    std::atomic<bool> done{false};
    std::thread setter([&] { std::this_thread::sleep_for(us(400000)); done = true; });
    const double c = seconds(CLOCK_THREAD_CPUTIME_ID);
    const bool ok = wait_until(true, [&] { return done.load(); }, never);
    std::printf("%f", seconds(CLOCK_THREAD_CPUTIME_ID) - c);
    setter.join();
    return ok ? 0 : 1;
}
""", "-pthread")
    assert float(out) < 0.2  # of 0.4 s


def test_a_wait_for_nothing_ends(tmp_path):
    _run(tmp_path, _WAIT + r"""
int main() {
    if (wait_until(true, never, [] { return true; })) return 1;
    if (wait_until(false, never, [] { return true; })) return 2;
    // what arrived just before the stream went idle still counts
    bool there = false;
    return wait_until(true, [&] { return there; }, [&] { there = true; return true; }) ? 0 : 3;
}
""", "-pthread")
