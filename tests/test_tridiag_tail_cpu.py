"""tridiag_sqrt_tail (csrc/tridiag.hpp): the last entries and the norm of T^{1/2} e1 from parts of the
eigenvectors, against the whole vector."""
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_25161_amd", "csrc")

HARNESS = r"""
#include <cstdio>
#include <vector>
#include "tridiag.hpp"
int main() {
  int k, t;
  while (std::scanf("%d %d", &k, &t) == 2) {
    std::vector<double> a(k), b(k - 1);
    for (auto& x : a) std::scanf("%lf", &x);
    for (auto& x : b) std::scanf("%lf", &x);
    double tail, nrm;
    fsd::tridiag_sqrt_tail(a, b, t, tail, nrm);
    std::printf("%.17g %.17g\n", tail, nrm);
  }
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_tail_and_norm(tmp_path):
    src, exe = tmp_path / "h.cpp", tmp_path / "h"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    rng = np.random.default_rng(3)
    cases = []
    for k, t in [(2, 1), (4, 4), (5, 1), (8, 4), (33, 4), (100, 4)]:
        G = rng.normal(size=(k, k + (0 if k % 2 else 2)))  # also singular ones
        lam, Q = np.linalg.eigh(G @ G.T if k % 2 == 0 else G[:, :-1] @ G[:, :-1].T)
        V = [np.ones(k) / np.sqrt(k)]  # Lanczos on diag(lam), fully reorthogonalised
        a, b = [], []
        for j in range(k):
            w = lam * V[-1]
            a.append(V[-1] @ w)
            for _ in range(2):
                w = w - np.array(V).T @ (np.array(V) @ w)
            b.append(np.linalg.norm(w))
            V.append(w / b[-1] if b[-1] > 0 else 0 * w)
        cases.append((np.array(a), np.array(b[:k - 1]), t))
    text = "".join(f"{len(a)} {t} " + " ".join(map(repr, map(float, np.concatenate([a, b])))) + "\n" for a, b, t in cases)
    out = subprocess.run([str(exe)], input=text, check=True, capture_output=True, text=True).stdout.split("\n")
    for (a, b, t), line in zip(cases, out):
        tail, nrm = map(float, line.split())
        lam, Q = np.linalg.eigh(np.diag(a) + np.diag(b, 1) + np.diag(b, -1))
        x = Q @ (np.sqrt(np.clip(lam, 0, None)) * Q[0])
        # sqrt of eigenvalues that rounding leaves near zero: sqrt(eps) of the largest
        assert abs(tail - (x[-t:] ** 2).sum()) < 1e-7 * (x ** 2).sum()
        assert abs(nrm - (x ** 2).sum()) < 1e-12 * (x ** 2).sum()
