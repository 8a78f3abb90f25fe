"""Arithmetic of the waits in a cluster of workgroups (wd_spin.h), on the host."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "wd_spin.h"
extern "C" int arrived(unsigned now, unsigned target) { return wd::arrived(now, target); }
// ticks that looks `step` apart take until the wait is beyond its limit; one of them comes `pause` late
extern "C" unsigned long long limit(unsigned long long step, unsigned long long pause) {
  unsigned long long now = 1ull << 40;
  wd::SpinClock c(now);
  for (unsigned long long i = 0, run = 0;; ++i) {
    now += step + (i == 1 ? pause : 0);
    run += step;
    if (c.beyond(now)) return run;
  }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("spin")
    (d / "spin.cpp").write_text(SRC)
    out = str(d / "libspin.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_1804_03243_amd", "csrc"),
                    "-o", out, str(d / "spin.cpp")], check=True)
    so = ctypes.CDLL(out)
    so.limit.restype = ctypes.c_uint64
    so.limit.argtypes = [ctypes.c_uint64] * 2
    return so


@pytest.mark.parametrize("base", [0, 1 << 20, (1 << 31) - 40, (1 << 32) - 40])
def test_barrier_count_runs_over(lib, base):
    """Barriers of 32 workgroups across 2^31 and 2^32: nobody passes before the
    last arrival, everybody passes after it, up to a whole barrier later."""
    gen = base
    for _ in range(4):
        target = gen + 32
        for k in range(32):
            assert not lib.arrived((gen + k) % 2 ** 32, target % 2 ** 32), (gen, k)
        for k in range(32):
            assert lib.arrived((target + k) % 2 ** 32, target % 2 ** 32), (gen, k)
        gen = target


@pytest.mark.parametrize("step", [40, 100, 900])
def test_limit_counts_running_time(lib, step):
    """Two seconds of looks at the clock, however long the queue was off the
    device between two of them."""
    two, ten_us = 200_000_000, 1000
    assert two <= lib.limit(step, 0) <= two + step
    assert two - ten_us <= lib.limit(step, 0) - step <= two
    for pause in (10 ** 6, 10 * two, 10 ** 12):
        assert two - ten_us <= lib.limit(step, pause) <= two + step
