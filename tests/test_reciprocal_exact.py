"""The two quotients that the kernels take from a product with a reciprocal and one residual step, q0 = a * inv,
q = fma(fma(-d, q0, a), inv, q0), against the correctly rounded a / d: a grid corner's fraction, for every
remainder of every denominator 2 * blocks up to 2^18 (corner_rcp), and c / 255 for every byte (unit8).  A C
program with the CPU's fused multiply-add, which rounds as the GPU's."""
import os
import shutil
import subprocess

import pytest

SOURCE = r"""
#include <math.h>
#include <stdio.h>
static float residual(float a, float d, float inv) {
  const float q0 = a * inv;
  return fmaf(fmaf(-d, q0, a), inv, q0);
}
int main(void) {
  long bad = 0, checked = 0;
#pragma omp parallel for schedule(dynamic, 256) reduction(+ : bad, checked)
  for (int den = 2; den <= 1 << 18; den += 2) {
    const float d = (float)den, inv = 1.0f / d;
    int wrong = 0;
    for (int r = 0; r < den; ++r) wrong += residual((float)r, d, inv) != (float)r / d;
    bad += wrong;
    checked += den;
  }
  for (int c = 0; c < 256; ++c, ++checked) bad += residual((float)c, 255.0f, 1.0f / 255.0f) != (float)c / 255.0f;
  printf("%ld %ld\n", checked, bad);
  return 0;
}
"""


def _has_fma():
    try:
        with open("/proc/cpuinfo") as fh:
            return any(line.startswith("flags") and " fma " in line + " " for line in fh)
    except OSError:
        return False


def test_residual_step_rounds_as_the_division(tmp_path):
    if not shutil.which("gcc") or not _has_fma():
        pytest.skip("needs gcc and a CPU with a fused multiply-add (libm's emulation takes minutes)")
    src, exe = tmp_path / "q.c", tmp_path / "q"
    src.write_text(SOURCE)
    subprocess.run(["gcc", "-O3", "-mavx2", "-mfma", "-fopenmp", "-ffp-contract=off", "-o", str(exe), str(src), "-lm"], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True, timeout=300).stdout.split()
    assert int(out[0]) == sum(range(2, (1 << 18) + 1, 2)) + 256 and int(out[1]) == 0, (out, os.cpu_count())
