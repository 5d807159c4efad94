"""The refit's eigenvector of the smallest eigenvalue, run on the host: random
positive semi-definite 3 x 3 matrices with known eigenvectors, eigenvalue ratios
from 1e-13 to just below 1 (where the Jacobi rotations take over) and exact rank
two. The bar is 256 eps l3 / (l2 - l1): the adjugate's rounding is a few eps l3^2
against its gap l3 (l2 - l1), and each of at most 12 squarings adds a few eps
over the remaining gap."""
import os
import subprocess

import pytest

from paper_2402_18008_amd import build

PROGRAM = r"""
#include "refit.hip"
#include <cmath>
#include <cstdio>
#include <random>

int main() {
  std::mt19937_64 g(3);
  std::normal_distribution<double> N(0, 1);
  std::uniform_real_distribution<double> U(0, 1);
  double worst = 0.0;
  for (int trial = 0; trial < 40000; ++trial) {
    long double Q[3][3];
    for (int i = 0; i < 3; ++i) {
      for (int k = 0; k < 3; ++k) Q[i][k] = N(g);
      for (int pass = 0; pass < 3; ++pass) {
        for (int j = 0; j < i; ++j) {
          long double d = 0;
          for (int k = 0; k < 3; ++k) d += Q[i][k] * Q[j][k];
          for (int k = 0; k < 3; ++k) Q[i][k] -= d * Q[j][k];
        }
        long double s = 0;
        for (int k = 0; k < 3; ++k) s += Q[i][k] * Q[i][k];
        for (int k = 0; k < 3; ++k) Q[i][k] /= sqrtl(s);
      }
    }
    const long double l3 = powl(10, 6 * U(g) - 3), l2 = l3 * powl(10, -6 * U(g));
    const long double l1 = trial % 50 ? l2 * powl(10, -0.0005 - 13 * U(g) * U(g)) : 0.0L;
    double C[3][3], v[3];
    for (int i = 0; i < 3; ++i)
      for (int j = i; j < 3; ++j)
        C[i][j] = C[j][i] = (double)(l1 * Q[0][i] * Q[0][j] + l2 * Q[1][i] * Q[1][j] +
                                     l3 * Q[2][i] * Q[2][j]);
    hg::smallest_eigvec3_adj(C, v);
    double dot = 0, e = 0;
    for (int k = 0; k < 3; ++k) dot += v[k] * (double)Q[0][k];
    for (int k = 0; k < 3; ++k) e = fmax(e, fabs(v[k] - (dot < 0 ? -1 : 1) * (double)Q[0][k]));
    const double bar = 256 * 2.220446049250313e-16 * (double)(l3 / (l2 - l1));
    worst = fmax(worst, e / bar);
    if (!(e <= bar)) {
      printf("trial %d: l1/l2 %.4Lg l2/l3 %.3Lg error %.3g bar %.3g\n", trial, l1 / l2, l2 / l3, e, bar);
      return 1;
    }
  }
  // zero, and not finite: a unit vector or nan, and an end
  const double Z[3][3] = {}, F[3][3] = {{INFINITY, 0, 0}, {0, NAN, 0}, {0, 0, 1}};
  double v[3];
  hg::smallest_eigvec3_adj(Z, v);
  if (v[0] * v[0] + v[1] * v[1] + v[2] * v[2] != 1.0) return 1;
  hg::smallest_eigvec3_adj(F, v);
  printf("worst error over bar %.3g\n", worst);
  return 0;
}
"""


def test_smallest_eigenvector(tmp_path):
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")
    csrc = os.path.join(build.ROOT, "paper_2402_18008_amd", "csrc")
    src = tmp_path / "eigvec_check.hip"
    src.write_text(PROGRAM)
    exe = tmp_path / "eigvec_check"
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", "-I",
                        os.path.join(build.ROOT, "include"), "-I", csrc, str(src),
                        os.path.join(csrc, "status.hip"), "-o", str(exe)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    print(r.stdout)
    assert r.returncode == 0, (r.stdout, r.stderr)
