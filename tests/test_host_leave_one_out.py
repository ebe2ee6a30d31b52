"""Leave-one-out Nystrom traces of ill-conditioned cores (host code built with g++) against exact
fractions."""

import os
import shutil
import subprocess
from fractions import Fraction

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2601_11338_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include <vector>
#include "wl_internal.h"
int main() {
  int M;
  while (std::scanf("%d", &M) == 1) {
    std::vector<double> S((size_t)M * M), G((size_t)M * M, 0.0);
    for (double& v : S)
      if (std::scanf("%lf", &v) != 1) return 1;
    for (int i = 0; i < M; ++i)
      for (int j = 0; j < M; ++j)
        for (int k = 0; k < M; ++k) G[(size_t)i * M + j] += S[(size_t)i * M + k] * S[(size_t)k * M + j];
    double t = 0.0, e = 0.0;
    if (xnys_trace_host(M, S, G, 1e-10, &t, &e)) return 2;
    std::printf("%a %a\n", t, e);
  }
  return 0;
}
"""


def exact_values(S):
    """tr(P_j G) + S_jj - s_j^T P_j s_j for every j, G = S^2, P_j the inverse of S without j."""
    M = len(S)
    S = [[Fraction(int(v)) for v in row] for row in S]
    G = [[sum(S[i][k] * S[k][j] for k in range(M)) for j in range(M)] for i in range(M)]
    values = []
    for j in range(M):
        rest, n = [a for a in range(M) if a != j], M - 1
        A = [[S[a][c] for c in rest] + [Fraction(int(i == k)) for k in range(n)] for i, a in enumerate(rest)]
        for k in range(n):  # (positive definite: no pivot is zero)
            A[k] = [v / A[k][k] for v in A[k]]
            for r in range(n):
                if r != k:
                    A[r] = [v - A[r][k] * w for v, w in zip(A[r], A[k])]
        P = [row[n:] for row in A]
        values.append(S[j][j] + sum(P[a][c] * (G[rest[c]][rest[a]] - S[j][rest[a]] * S[j][rest[c]])
                                    for a in range(n) for c in range(n)))
    return values


def cores():
    """Integer cores of condition 2e5 to 8e5 (their products are exact in 64 bits)."""
    for M in (3, 5, 8, 12):
        found, seed = 0, 0
        while found < 6:
            seed += 1
            A = np.random.default_rng(seed).integers(-9, 10, (M, M))
            S = A.T @ A
            cond = np.linalg.cond(S.astype(float))
            if 2e5 < cond < 8e5:
                found += 1
                yield S, cond


def test_ill_conditioned_cores(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("g++ or the ROCm headers are not available")
    src, exe = tmp_path / "main.cpp", str(tmp_path / "main")
    src.write_text(MAIN)
    b = subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, str(src),
                        os.path.join(CSRC, "dense_host.cpp"), "-o", exe, "-lpthread"], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr[-3000:]
    items = list(cores())
    text = "\n".join(f"{len(S)} " + " ".join(str(int(v)) for v in S.ravel()) for S, _ in items)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=60)
    assert out.returncode == 0
    for (S, cond), line in zip(items, out.stdout.splitlines()):
        t, e = (float.fromhex(x) for x in line.split())
        values = exact_values(S)
        M, mean = len(S), sum(values) / len(S)
        bound = M * 2.0 ** -52 * np.sqrt(cond)  # triangular solves
        err = abs(float((Fraction(t) - mean) / mean))
        print(M, f"condition {cond:.1e} error {err:.1e} bound {bound:.1e}")
        assert err <= bound
        spread = np.sqrt(float(sum((v - mean) ** 2 for v in values) / (M - 1) / M))
        assert abs(e - spread) <= 4 * bound * float(mean)
