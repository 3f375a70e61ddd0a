"""The reversed replay of an iteration that the adjoint differentiates through
(csrc/replay.hpp): every iterate once, last to first, also where a segment is
longer than what is kept of it.  The header is compiled for the host."""
import os
import subprocess

import pytest

from paper_2511_17701_amd import build

PROGRAM = r"""
#include <cstdio>
#include "replay.hpp"
int main() {
  for (int n = 1; n <= 1200; ++n) {
    int want = n - 1, steps = 0;
    bool ok = true;
    grpic::reverse_iterates<16>(
        n, 0.0, 0.5, [&](double& a, double& b) { a += 1.0; b += 1.0; ++steps; },
        [&](double a, double b) { ok = ok && a == want && b == want + 0.5; --want; });
    if (!ok || want != -1) { printf("n %d\n", n); return 1; }
    if (n <= 256 && steps > 2 * n) { printf("n %d: %d steps\n", n, steps); return 1; }
  }
  return 0;
}
"""


def test_reverse_iterates(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "replay.cpp", tmp_path / "replay"
    src.write_text(PROGRAM)
    csrc = os.path.join(build.HERE, "csrc")
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-I", csrc, str(src), "-o", str(exe)],
                   check=True, timeout=300)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout
