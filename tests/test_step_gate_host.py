"""Whether a step runs, and how a failing step is reported, past 2^31 steps (csrc/mx_internal.hpp: the
code of the first stage's gate, on the host).  Small tubes take that many steps in hours; a
gate of 32 bits would stop such a run without a report.  Host-only build: no GPU needed."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r'''
#include <cstdio>
#include "mx_internal.hpp"
int main() {
  static_assert(sizeof(mx::DevCtrl::fail_step) == sizeof(mx::DevCtrl::step[0]), "as wide as the count");
  const long long steps[] = {0, 1, 2147483646LL, 2147483647LL, 2147483648LL, 1LL << 40};
  for (long long n : steps) {
    // no failure; the next step failing (its own later workgroups still run it); the last one failed
    std::printf("%lld %d %d %d %d\n", n, mx::step_runs(mx::NO_FAILURE, n), mx::step_runs(n + 1, n),
                mx::step_runs(n, n), mx::reported_fail_step(n));
  }
  std::printf("none %d %d\n", mx::reported_fail_step(mx::NO_FAILURE), mx::step_runs(0, 0));
}
'''


def test_steps_past_32_bits_run(tmp_path):
    hipcc = shutil.which('hipcc') or '/opt/rocm/bin/hipcc'
    if not os.path.exists(hipcc):
        pytest.skip('hipcc not available')
    src, exe = tmp_path / 'gate.cpp', str(tmp_path / 'gate')
    src.write_text(SRC)
    subprocess.run([hipcc, '-x', 'hip', '--offload-arch=gfx950', '-O1', '-std=c++17',
                    '-I' + os.path.join(ROOT, 'paper_2401_15233_amd', 'csrc'), str(src), '-o', exe], check=True,
                   stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    lines = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split('\n')
    for line in lines[:6]:
        n, free, running, failed, reported = (int(x) for x in line.split())
        assert (free, running, failed) == (1, 1, 0), line
        assert reported == min(n, 2 ** 31 - 1), line
    assert lines[6] == 'none 0 0'       # a loaded state that failed its check runs no step
