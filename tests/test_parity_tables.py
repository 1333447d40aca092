"""The parity split of the absorbing layers' eigen tables (csrc/parity.hpp), host code: compiled
here by itself and called through ctypes."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import stencil
from paper_2410_17446_amd import build, inputs, tables

from helpers import unsplit_tables

HARNESS = r"""
#include "parity.hpp"
#include <atomic>
#include <cstdlib>
#include <cstring>
using cd = std::complex<double>;
static std::atomic<long> allowed{1L << 40};  // allocations until the next ones fail
void* operator new(std::size_t n) {
  if (allowed.fetch_sub(1) <= 0) throw std::bad_alloc();
  if (void* p = std::malloc(n)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
extern "C" int t_invert(cd* a, int n, int ld, int threads) { return parity::invert(a, n, ld, threads); }
extern "C" int t_as_good(double halves, double whole) { return parity_as_good(halves, whole); }
// 1: split, 0: does not split, -1: bad_alloc
extern "C" int t_tables(const cd* q, const cd* l, int N, cd* hq, cd* hqi, cd* hl, long limit) {
  allowed = limit;
  int rc = 0;
  try {
    const ParityTables t = parity_tables(q, l, N);
    if (!t.lam.empty()) {
      std::memcpy(hq, t.q.data(), t.q.size() * sizeof(cd));
      std::memcpy(hqi, t.qi.data(), t.qi.size() * sizeof(cd));
      std::memcpy(hl, t.lam.data(), t.lam.size() * sizeof(cd));
      rc = 1;
    }
  } catch (const std::bad_alloc&) {
    rc = -1;
  }
  const long used = limit - allowed;
  allowed = 1L << 40;
  return rc < 1 ? rc : (int)used;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("parity")
    src, out = d / "h.cpp", d / "h.so"
    src.write_text(HARNESS)
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/bin/amdclang++"
    subprocess.run([cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-pthread", "-I", build.CSRC, str(src), "-o", str(out)],
                   check=True)
    return ctypes.CDLL(str(out))


def _ptr(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def _layer(N, W, sigma):
    c, d = stencil.stencils()
    A = tables.pml_stretched_d2(N, 0.25, inputs.K0, 1.0, W, sigma, c, d)
    Q, Qi, lam = tables.pml_eigen(N, 0.25, inputs.K0, 1.0, W, sigma, c, d)
    return A, np.ascontiguousarray(Q), Qi, lam


def _split(lib, Q, lam, N, limit=1 << 40):
    h = N // 2
    q, qi, l = np.zeros((2, h, h), complex), np.zeros((2, h, h), complex), np.zeros((2, h), complex)
    rc = lib.t_tables(_ptr(Q), _ptr(np.ascontiguousarray(lam)), N, _ptr(q), _ptr(qi), _ptr(l), ctypes.c_long(limit))
    return rc, q, qi, l


@pytest.mark.parametrize("n,ld", [(1, 1), (2, 5), (31, 32), (32, 32), (33, 33), (63, 64), (64, 64), (65, 65), (127, 128),
                                  (200, 201), (257, 257)])
def test_inverse_at_the_edges_of_panels_and_strips(lib, n, ld):
    """Against numpy, within 100 eps n kappa; the same bits on one and on four threads; what lies
    beyond the n columns is left alone."""
    rng = np.random.default_rng(n)
    a = rng.standard_normal((n, ld)) + 1j * rng.standard_normal((n, ld))
    one, four = a.copy(), a.copy()
    assert lib.t_invert(_ptr(one), n, ld, 1) == 1 and lib.t_invert(_ptr(four), n, ld, 4) == 1
    assert np.array_equal(one, four) and np.array_equal(one[:, n:], a[:, n:])
    ref = np.linalg.inv(a[:, :n])
    kappa = np.linalg.cond(a[:, :n])
    assert np.linalg.norm(one[:, :n] - ref) <= 100 * 2.2e-16 * n * kappa * np.linalg.norm(ref)


def test_singular_and_non_finite_matrices_are_refused(lib):
    a = np.ones((40, 40), complex)
    assert lib.t_invert(_ptr(a), 40, 40, 2) == 0
    b = np.eye(40, dtype=complex)
    b[3, 3] = np.nan
    assert lib.t_invert(_ptr(b), 40, 40, 2) == 0


@pytest.mark.parametrize("N,W,sigma", [(64, 8, 10.0), (128, 16, 10.0)])
def test_halves_invert_and_hold_every_eigenvalue(lib, N, W, sigma):
    A, Q, Qi, lam = _layer(N, W, sigma)
    rc, q, qi, l = _split(lib, Q, lam, N)
    assert rc > 0
    h = N // 2
    for r in range(2):
        n = h - r
        kappa = np.linalg.cond(q[r, :n, :n])
        assert np.abs(qi[r, :n, :n] @ q[r, :n, :n] - np.eye(n)).max() <= 100 * 2.2e-16 * n * kappa
    assert not q[1, -1].any() and not q[1, :, -1].any() and not qi[1, -1].any() and not qi[1, :, -1].any()
    both = np.concatenate([l[0], l[1, :-1]])
    assert np.array_equal(np.sort_complex(both), np.sort_complex(lam))


def test_columns_of_mixed_parity_do_not_split(lib):
    A, Q, Qi, lam = _layer(64, 12, 1.0)
    Q, Qi, lam = unsplit_tables(A, Q, Qi, lam)
    assert _split(lib, Q, lam, 64)[0] == 0


def test_an_allocation_that_fails_is_reported(lib):
    """Whichever allocation fails, in this thread or in one that inverts a half, the call ends with
    bad_alloc and not with the process."""
    A, Q, Qi, lam = _layer(64, 8, 10.0)
    used, *_ = _split(lib, Q, lam, 64)
    assert used > 8
    for limit in range(used):
        rc = _split(lib, Q, lam, 64, limit)[0]
        assert rc == -1 or rc > 0, limit
    assert _split(lib, Q, lam, 64, 4)[0] == -1


def test_halves_serve_within_the_scatter_of_rounding_only(lib):
    lib.t_as_good.argtypes = [ctypes.c_double, ctypes.c_double]
    for whole in (1e-13, 1e-9, 1e-4):
        assert lib.t_as_good(2.4 * whole, whole) and not lib.t_as_good(2.6 * whole + 1e-13, whole)
    assert lib.t_as_good(1e-14, 0.0) and not lib.t_as_good(2e-14, 0.0) and not lib.t_as_good(np.nan, 1e-9)


def _fold(x):
    h = (x.shape[0] + 1) // 2
    return 0.5 * (x + x[::-1])[:h], 0.5 * (x - x[::-1])[:h]


def _unfold(e, o):
    h = e.shape[0]
    out = np.empty((2 * h - 1,) + e.shape[1:], complex)
    out[:h] = e + o
    out[::-1][:h - 1] = (e - o)[:h - 1]
    return out


@pytest.mark.parametrize("N,W,sigma", [(64, 8, 1.0), (64, 8, 10.0), (128, 16, 10.0), (128, 16, 3.0), (192, 24, 10.0)])
def test_solves_by_halves_are_as_good_as_whole(lib, N, W, sigma):
    """(A Z + Z A^T - b Z = x) by the halves and by the whole planes against Bartels-Stewart, refined:
    over four right-hand sides and poles the halves' errors are no larger in the geometric mean and
    none is over twice the other's (both are rounding times the same condition)."""
    from oracle import fit
    from scipy.linalg import solve_sylvester
    A, Q, Qi, lam = _layer(N, W, sigma)
    rc, q, qi, l = _split(lib, Q, lam, N)
    assert rc > 0
    poles = fit.fit_exp_sqrt(inputs.K0, 8)["poles"]
    n, rng, ratios = N - 1, np.random.default_rng(N), []
    X = (np.arange(1, N) - N / 2) / 32.0
    beam = np.exp(-X[:, None] ** 2 - X[None] ** 2).astype(complex)
    for b in (poles[np.argmin(abs(poles.imag))], poles[3]):
        for x in (rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)), beam):
            S = A - b * np.eye(n)
            z = solve_sylvester(S, A.T, x)
            for _ in range(2):
                z = z + solve_sylvester(S, A.T, x - (S @ z + z @ A.T))
            whole = Q @ ((Qi @ x @ Qi.T) / (lam[:, None] + lam[None] - b)) @ Q.T
            rows = []
            for i, xi in enumerate(_fold(x)):
                cols = []
                for j, xij in enumerate(_fold(xi.T)):
                    den = l[i][:, None] + l[j][None] - b
                    cols.append((q[i] @ ((qi[i] @ xij.T @ qi[j].T) / np.where(den == 0, 1, den)) @ q[j].T).T)
                rows.append(_unfold(*cols).T)
            halves = _unfold(*rows)
            ratios.append(np.linalg.norm(halves - z) / np.linalg.norm(whole - z))
    assert np.exp(np.mean(np.log(ratios))) <= 1.0 and max(ratios) <= 2.0, ratios
