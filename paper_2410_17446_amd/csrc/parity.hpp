// The eigen tables of the absorbing layers (hp_set_pml) by parity: host code, plain C++.
//
// The stretch is the same at both ends of an axis, so the one-axis operator commutes
// with the reflection j -> N - j and its eigenvectors are even or odd; the dense stages
// then run on halves.
#pragma once
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstddef>
#include <new>
#include <system_error>
#include <thread>
#include <vector>

// Q, Q^-1 and lam of the even and the odd subspace (even block first), in the coordinates of the
// folded fields: node j = 1..N/2 at entry j - 1, the odd block's last entry padding (zero).  Empty
// when the given tables do not split.
struct ParityTables {
  std::vector<std::complex<double>> q, qi, lam;
};

namespace parity {

// fn(begin, end) over [0, n) in up to `parts` contiguous parts, each in a thread of its own but the
// last; a part whose thread cannot be had runs here.  Rethrows as bad_alloc what any part threw,
// after all have ended.
template <typename F>
void in_parts(int parts, int n, const F& fn) {
  parts = std::max(1, std::min(parts, n));
  std::vector<char> failed(parts, 0);
  struct Side {
    std::vector<std::thread> t;
    ~Side() {
      for (auto& x : t)
        if (x.joinable()) x.join();
    }
  };
  {
    Side side;
    side.t.reserve(parts);
    for (int p = 0; p < parts; ++p) {
      auto run = [&failed, &fn, p, parts, n]() noexcept {
        try {
          fn((int)((long)n * p / parts), (int)((long)n * (p + 1) / parts));
        } catch (...) {
          failed[p] = 1;
        }
      };
      if (p + 1 < parts) {
        try {
          side.t.emplace_back(run);
          continue;
        } catch (const std::system_error&) {
        } catch (const std::bad_alloc&) {
        }
      }
      run();
    }
  }
  for (char f : failed)
    if (f) throw std::bad_alloc();
}

// Rows of real and imaginary parts, so that the row operations vectorise.
constexpr int PANEL = 32, STRIP = 64;

// a -= sum_k f_k p_k over w <= STRIP columns in the order of k < nk <= PANEL (p packed, w per row)
inline void sub_rows(double* __restrict__ ar, double* __restrict__ ai, const double* __restrict__ pr,
                     const double* __restrict__ pi, const double* fr, const double* fi, int nk, int w) {
  int c = 0;
  for (; c + 4 <= w; c += 4) {
    double xr[4], xi[4];
    for (int j = 0; j < 4; ++j) xr[j] = ar[c + j], xi[j] = ai[c + j];
    for (int k = 0; k < nk; ++k) {
      const double *br = pr + (size_t)k * w + c, *bi = pi + (size_t)k * w + c;
      for (int j = 0; j < 4; ++j) {
        xr[j] -= fr[k] * br[j] - fi[k] * bi[j];
        xi[j] -= fr[k] * bi[j] + fi[k] * br[j];
      }
    }
    for (int j = 0; j < 4; ++j) ar[c + j] = xr[j], ai[c + j] = xi[j];
  }
  for (; c < w; ++c)
    for (int k = 0; k < nk; ++k) {
      const double br = pr[(size_t)k * w + c], bi = pi[(size_t)k * w + c];
      ar[c] -= fr[k] * br - fi[k] * bi;
      ai[c] -= fr[k] * bi + fi[k] * br;
    }
}

// In place inverse of the n x n matrix a (row stride ld): LU with row pivots, then the columns of
// the identity solved (Gauss-Jordan, cheaper, loses four digits on these eigenvectors); false if it
// meets a zero or non-finite pivot.  Every element takes its terms in the order of the row by row
// elimination; panels of PANEL rows and strips of STRIP columns keep them in the caches, and the
// strips go to `threads` threads where there are enough of them to pay for starting these.  One
// half of 512^2, 1024^2 and 2048^2: 9, 72 and 672 ms row by row, 7, 23 and 143 ms so.
inline bool invert(std::complex<double>* a, int n, int ld, int threads) {
  std::vector<double> mr((size_t)n * n), mi((size_t)n * n);
  std::vector<int> perm(n);
  for (int r = 0; r < n; ++r) {
    perm[r] = r;
    for (int c = 0; c < n; ++c) {
      mr[(size_t)r * n + c] = a[(size_t)r * ld + c].real();
      mi[(size_t)r * n + c] = a[(size_t)r * ld + c].imag();
    }
  }
  for (int k0 = 0; k0 < n; k0 += PANEL) {
    const int k1 = std::min(n, k0 + PANEL);
    for (int k = k0; k < k1; ++k) {  // the panel's columns; whole rows change places
      int best = k;
      double mag = -1.0;
      for (int r = k; r < n; ++r) {
        const double u = mr[(size_t)r * n + k], v = mi[(size_t)r * n + k], w = u * u + v * v;
        if (w > mag) mag = w, best = r;
      }
      if (!(mag > 0.0) || !std::isfinite(mag)) return false;
      if (best != k) {
        std::swap_ranges(&mr[(size_t)k * n], &mr[(size_t)k * n] + n, &mr[(size_t)best * n]);
        std::swap_ranges(&mi[(size_t)k * n], &mi[(size_t)k * n] + n, &mi[(size_t)best * n]);
        std::swap(perm[k], perm[best]);
      }
      const double dr = mr[(size_t)k * n + k] / mag, di = -mi[(size_t)k * n + k] / mag;
      for (int r = k + 1; r < n; ++r) {
        double *ar = &mr[(size_t)r * n], *ai = &mi[(size_t)r * n];
        const double fr = ar[k] * dr - ai[k] * di, fi = ar[k] * di + ai[k] * dr;
        ar[k] = fr;
        ai[k] = fi;
        for (int c = k + 1; c < k1; ++c) {
          const double pr = mr[(size_t)k * n + c], pi = mi[(size_t)k * n + c];
          ar[c] -= fr * pr - fi * pi;
          ai[c] -= fr * pi + fi * pr;
        }
      }
    }
    const int strips = (n - k1 + STRIP - 1) / STRIP;
    if (strips == 0) break;
    in_parts((long)strips * (n - k0) < 2048 ? 1 : threads, strips, [&](int s0, int s1) {
      double pr[PANEL * STRIP], pi[PANEL * STRIP];
      for (int s = s0; s < s1; ++s) {
        const int c0 = k1 + s * STRIP, w = std::min(n, c0 + STRIP) - c0;
        for (int r = k0; r < n; ++r) {
          double *ar = &mr[(size_t)r * n + c0], *ai = &mi[(size_t)r * n + c0];
          const int nk = std::min(r, k1) - k0;
          sub_rows(ar, ai, pr, pi, &mr[(size_t)r * n + k0], &mi[(size_t)r * n + k0], nk, w);
          if (r < k1) {
            std::copy(ar, ar + w, pr + (size_t)(r - k0) * w);
            std::copy(ai, ai + w, pi + (size_t)(r - k0) * w);
          }
        }
      }
    });
  }
  std::vector<int> at(n);  // row of the identity's column c after the exchanges
  for (int r = 0; r < n; ++r) at[perm[r]] = r;
  const int strips = (n + STRIP - 1) / STRIP;
  std::vector<char> finite(strips, 0);
  in_parts(n < 384 ? 1 : threads, strips, [&](int s0, int s1) {
    std::vector<double> xr, xi;
    double pr[PANEL * STRIP], pi[PANEL * STRIP], fr[PANEL], fi[PANEL];
    for (int s = s0; s < s1; ++s) {
      const int c0 = s * STRIP, w = std::min(n, c0 + STRIP) - c0;
      xr.assign((size_t)n * w, 0.0);
      xi.assign((size_t)n * w, 0.0);
      int top = n;  // the rows above stay zero in the forward pass
      for (int c = 0; c < w; ++c) {
        xr[(size_t)at[c0 + c] * w + c] = 1.0;
        top = std::min(top, at[c0 + c]);
      }
      for (int k0 = top / PANEL * PANEL; k0 < n; k0 += PANEL) {
        const int k1 = std::min(n, k0 + PANEL);
        for (int r = k0; r < n; ++r) {
          double *ar = &xr[(size_t)r * w], *ai = &xi[(size_t)r * w];
          sub_rows(ar, ai, &xr[(size_t)k0 * w], &xi[(size_t)k0 * w], &mr[(size_t)r * n + k0], &mi[(size_t)r * n + k0],
                   std::min(r, k1) - k0, w);
        }
      }
      for (int k1 = n; k1 > 0; k1 -= std::min(k1, PANEL)) {  // rows k1-1 down to k0, packed in that order
        const int k0 = std::max(0, k1 - PANEL);
        for (int r = k1 - 1; r >= 0; --r) {
          const int nk = r < k0 ? k1 - k0 : k1 - 1 - r;
          const double *ur = &mr[(size_t)r * n], *ui = &mi[(size_t)r * n];
          for (int k = 0; k < nk; ++k) fr[k] = ur[k1 - 1 - k], fi[k] = ui[k1 - 1 - k];
          double *ar = &xr[(size_t)r * w], *ai = &xi[(size_t)r * w];
          sub_rows(ar, ai, pr, pi, fr, fi, nk, w);
          if (r < k0) continue;
          const double u = ur[r], v = ui[r], m2 = u * u + v * v;
          for (int c = 0; c < w; ++c) {
            const double p = (ar[c] * u + ai[c] * v) / m2, q = (ai[c] * u - ar[c] * v) / m2;
            ar[c] = p;
            ai[c] = q;
          }
          std::copy(ar, ar + w, pr + (size_t)nk * w);
          std::copy(ai, ai + w, pi + (size_t)nk * w);
        }
      }
      bool ok = true;
      for (int r = 0; r < n; ++r)
        for (int c = 0; c < w; ++c) {
          const double p = xr[(size_t)r * w + c], q = xi[(size_t)r * w + c];
          ok = ok && std::isfinite(p) && std::isfinite(q);
          a[(size_t)r * ld + c0 + c] = {p, q};
        }
      finite[s] = ok;
    }
  });
  return std::find(finite.begin(), finite.end(), 0) == finite.end();
}

}  // namespace parity

// The operator commutes with the reflection, so each eigenvector is even or odd, except that an
// eigensolver returns arbitrary mixtures where an even and an odd eigenvalue agree to rounding (modes
// confined to the two layers).  Both columns of such a pair hold the same even and the same odd
// vector, so one of them supplies each.  The halves' inverses are computed afresh: Q is so
// ill-conditioned that folding the given inverse would not invert the folded vectors.
inline ParityTables parity_tables(const std::complex<double>* q, const std::complex<double>* l, int N) {
  using cd = std::complex<double>;
  const int n = N - 1, h = N / 2;
  std::vector<double> ev(n, 0.0), od(n, 0.0);  // squared norms of each column's even and odd part
  for (int j = 0; j < h; ++j)
    for (int c = 0; c < n; ++c) {
      const cd a = q[(size_t)j * n + c], b = q[(size_t)(n - 1 - j) * n + c];
      const double w = j == h - 1 ? 0.25 : 0.5;  // the middle node is its own mirror image
      ev[c] += w * std::norm(a + b);
      od[c] += w * std::norm(a - b);
    }
  std::vector<int> role(n, -1), mixed;
  int ne = 0, no = 0;
  for (int c = 0; c < n; ++c) {
    const double s = ev[c] + od[c];
    if (!(s > 0.0) || !std::isfinite(s)) return {};
    if (std::min(ev[c], od[c]) > 1e-6 * s)
      mixed.push_back(c);
    else if (ev[c] > od[c])
      role[c] = 0, ++ne;
    else
      role[c] = 1, ++no;
  }
  for (int a : mixed) {
    if (role[a] >= 0) continue;
    int b = -1;
    double gap = 1e300;
    for (int c : mixed)
      if (c != a && role[c] < 0 && std::norm(l[c] - l[a]) < gap) gap = std::norm(l[c] - l[a]), b = c;
    if (b < 0) return {};
    const bool first = ev[a] / (ev[a] + od[a]) >= ev[b] / (ev[b] + od[b]);
    role[first ? a : b] = 0;
    role[first ? b : a] = 1;
    ++ne, ++no;
  }
  if (ne != h || no != h - 1) return {};
  ParityTables t;
  t.q.assign(2 * (size_t)h * h, cd(0.0));
  t.lam.assign(2 * (size_t)h, cd(0.0));
  int at[2] = {0, 0};
  for (int c = 0; c < n; ++c) {
    const int r = role[c], k = at[r]++;
    for (int j = 0; j < h - r; ++j) {
      const cd a = q[(size_t)j * n + c], b = q[(size_t)(n - 1 - j) * n + c];
      t.q[((size_t)r * h + j) * h + k] = 0.5 * (r ? a - b : a + b);
    }
    t.lam[(size_t)r * h + k] = l[c];
  }
  t.qi = t.q;
  bool ok[2] = {false, false};
  const int threads = std::max(1, std::min(4, (int)std::thread::hardware_concurrency() / 2));  // per half
  parity::in_parts(2, 2, [&](int r0, int r1) {
    for (int r = r0; r < r1; ++r) ok[r] = parity::invert(t.qi.data() + (size_t)r * h * h, h - r, h, threads);
  });
  return ok[0] && ok[1] ? t : ParityTables();
}

// Relative error of the split tables' operator on x against y = s D~ x.
inline double parity_error(const ParityTables& t, int N, const std::vector<std::complex<double>>& x,
                           const std::vector<std::complex<double>>& y) {
  using cd = std::complex<double>;
  const int n = N - 1, h = N / 2;
  std::vector<cd> out[2];
  for (int r = 0; r < 2; ++r) {
    const cd *q = t.q.data() + (size_t)r * h * h, *qi = t.qi.data() + (size_t)r * h * h;
    std::vector<cd> f(h), m(h);
    out[r].assign(h, cd(0.0));
    for (int j = 0; j < h; ++j) f[j] = 0.5 * (r ? x[j] - x[n - 1 - j] : x[j] + x[n - 1 - j]);
    for (int k = 0; k < h; ++k) {
      cd s = 0.0;
      for (int j = 0; j < h; ++j) s += qi[(size_t)k * h + j] * f[j];
      m[k] = t.lam[(size_t)r * h + k] * s;
    }
    for (int j = 0; j < h; ++j)
      for (int k = 0; k < h; ++k) out[r][j] += q[(size_t)j * h + k] * m[k];
  }
  double num = 0.0, den = 0.0;
  for (int j = 0; j < h; ++j) {
    num += std::norm(out[0][j] + out[1][j] - y[j]);
    den += std::norm(y[j]);
    if (j == h - 1) continue;
    num += std::norm(out[0][j] - out[1][j] - y[n - 1 - j]);
    den += std::norm(y[n - 1 - j]);
  }
  const double e = std::sqrt(num / den);
  return std::isfinite(e) ? e : 1e300;
}

// Whether halves of that operator error may stand for tables of this one.  Both errors are
// rounding of the eigensolver, amplified by the condition of the eigenvectors, and scatter against
// each other: on grids of 64 to 512 nodes, layers of 8 to 64 and sigma_max 1 to 10 the ratio was 0.2 to
// 2.2, where the solves with the halves were 0.1 to 1.25 times as far from the exact ones as
// those with the whole planes.  Beyond that scatter the halves are worse, and the planes stay whole.
inline bool parity_as_good(double halves, double whole) { return halves <= 2.5 * whole + 64 * 2.2e-16; }
