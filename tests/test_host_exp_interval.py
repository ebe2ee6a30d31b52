"""Interval of the Chebyshev series of exp(-t T) (host code built with g++): projections with their
spectrum from 0 on, below 0, and far above it, with and without deflated columns."""

import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import krylov

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2601_11338_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include <vector>
#include "wl_internal.h"
int main() {
  int K, b;
  double hi, tmax, lo;
  while (std::scanf("%d %d %lf %lf %lf", &K, &b, &hi, &tmax, &lo) == 5) {
    std::vector<double> A((size_t)K * b * b), B((size_t)K * b * b);
    for (double& v : A)
      if (std::scanf("%lf", &v) != 1) return 1;
    for (double& v : B)
      if (std::scanf("%lf", &v) != 1) return 1;
    const int r = exp_interval(K, b, A, B, hi, tmax, 4.0, &lo);
    std::printf("%d %.17g\n", r, lo);
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("g++ or the ROCm headers are not available")
    d = tmp_path_factory.mktemp("interval")
    src, exe = d / "main.cpp", str(d / "main")
    src.write_text(MAIN)
    b = subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, str(src),
                        os.path.join(CSRC, "dense_host.cpp"), "-o", exe, "-lpthread"], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr[-3000:]
    return exe


@pytest.mark.parametrize("dependent", [0, 2])  # start columns that repeat others: zero rows of T
@pytest.mark.parametrize("low,expect", [(0.0, 0), (1e-14, 0), (0.02, 0), (-0.04, 0), (-0.5, 2), (3.0, 1), (40.0, 1)])
def test_interval(program, low, expect, dependent):
    n, b, K, hi_eig, tmax = 200, 6, 12, 50.0, 10.0
    rng = np.random.default_rng(3)
    lam = np.r_[low, low + (hi_eig - low) * np.sort(rng.random(n - 1))]
    X = rng.normal(size=(n, b))
    X[0] += 3.0  # the lowest eigenvector is resolved
    X[:, b - dependent:] = X[:, :dependent]
    _, A, B, _ = krylov.block_lanczos(lambda V: lam[:, None] * V, X, K, reorth="full")
    T = krylov.block_tridiagonal(A, B)
    kept = np.any(T != 0.0, axis=1)
    assert kept.sum() == K * (b - dependent)
    lmin = np.linalg.eigvalsh(T[np.ix_(kept, kept)])[0]
    hi = float(np.abs(T).sum(axis=1).max())
    lo = -min(0.01 * hi, 1.0 / tmax)
    text = f"{K} {b} {hi!r} {tmax!r} {lo!r} " + " ".join(repr(float(v)) for M in (A, B) for Z in M for v in Z.ravel())
    out = subprocess.run([program], input=text, capture_output=True, text=True, timeout=60)
    assert out.returncode == 0
    status, got = out.stdout.split()
    assert int(status) == expect
    if expect == 0:
        assert float(got) == lo and lo < lmin <= lo + 4.0 / tmax
    elif expect == 1:
        assert lmin - 2.0 / tmax <= float(got) < lmin
