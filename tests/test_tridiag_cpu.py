"""The ground state's small eigenproblem (tridiag_lowest) against numpy's
dense solver: random matrices, Lanczos-like ones with a converged lowest
vector (its last components far below 1), nearly degenerate pairs and m = 1.
Eigenvalue within 8 eps |T|; residual |T s - l s| likewise times sqrt(m)."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2005_13498_amd", "csrc")


@pytest.fixture(scope="module")
def solve(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("tridiag") / "check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, os.path.join(ROOT, "tests", "native", "tridiag_check.cpp"),
                    os.path.join(CSRC, "host_eig.cpp"), "-o", exe], check=True)

    def f(a, b):
        text = " ".join([str(len(a))] + [repr(float(x)) for x in list(a) + list(b)])
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=30).stdout.split()
        v = np.array([float(x) for x in out])
        return v[0], v[1:]
    return f


def _cases():
    rng = np.random.default_rng(5)
    yield [3.5], []
    for m in (2, 3, 8, 60, 100):
        yield rng.normal(size=m), rng.uniform(0.1, 2.0, m - 1)
    for m in (16, 60):  # Lanczos on a diagonal with a gap below the rest
        d = np.concatenate([[-9.0], rng.uniform(-8.0, 40.0, 2000)])
        q, qp, b, al, be = np.ones(2001) / np.sqrt(2001), 0.0, 0.0, [], []
        Q = []
        for _ in range(m):
            Q.append(q)
            w = d * q
            al.append(w @ q)
            for _ in range(2):
                for u in Q:
                    w = w - (u @ w) * u
            b = np.linalg.norm(w)
            be.append(b)
            q = w / b
        yield al, be[:-1]
    yield [1.0, 50.0, 1.0], [1e-6, 1e-6]  # two eigenvalues 2e-14 apart from 1
    yield [2.0] * 40, [1e-9] * 39


@pytest.mark.parametrize("k", range(10))
def test_lowest_eigenpair(solve, k):
    a, b = list(_cases())[k]
    T = np.diag(np.asarray(a, float)) + np.diag(b, 1) + np.diag(b, -1)
    norm = np.max(np.sum(np.abs(T), axis=1))
    e = np.linalg.eigvalsh(T)
    lam, s = solve(a, b)
    eps = np.finfo(float).eps
    assert abs(lam - e[0]) <= 8 * eps * norm
    assert abs(np.linalg.norm(s) - 1.0) <= 4 * eps
    assert np.linalg.norm(T @ s - lam * s) <= 8 * eps * norm * np.sqrt(len(a))
