// HIP kernels of one propagation step (gfx950).
//
// The step solves (Zbar - b_k I) x_k = w for every pole b_k by GMRES with the
// right preconditioner M_k = Zbar_fs - b_k I (Sec. 4.2).  Zbar = Zbar_fs + P
// where P holds the medium terms (V and, for the vector operator, the psi
// terms of eq. Z_bar_eq), so A_k M_k^{-1} v = v + P M_k^{-1} v exactly: the
// Laplacian stencil never runs inside the Arnoldi loop, only the medium part.
//
// Krylov vectors live in the row-transformed domain (DST-I along x applied,
// "R-domain"): the transform is orthonormal, so inner products and GMRES
// iterates are unchanged, and one Arnoldi step needs two passes over HBM:
//   column pass  z = S_y [(S_y u) / (mu_y + mu_x - b)]   (R-domain in, out)
//   row pass     p = S_x P S_x z  (+ the inner products with the basis)
// plus the Gram-Schmidt update.  All dot products, Givens rotations and the
// residue-weighted sum accumulate in FP64.
//
// R-domain fields are stored column-tiled, [nx/TW][ny][TW] with TW elements =
// 128 bytes, so the row pass reads whole 128-byte lines of each tile and the
// column pass reads each tile as one contiguous block.  Physical fields (the
// caller's E, n^2 and the coefficient planes) are row-major [ny][nx].
#include <math.h>

#include "fft.hpp"
#include "kernels.hpp"

namespace {

template <typename T>
struct Tile {
  static constexpr int W = 128 / (int)sizeof(cx<T>);  // elements per 128-byte tile row
};

// offset of element (row i, column q) of a tiled field with ny rows
template <int TW>
__device__ __forceinline__ size_t tix(int i, int q, int ny) {
  return ((size_t)(q / TW) * ny + i) * TW + (q % TW);
}

// Tiled offsets of the points q = t + s * NT (s = 0, 1, ...) of row i: when NT
// is a multiple of TW they step by a uniform stride (kept in a scalar
// register instead of one address per point).
template <int TW, int NT>
struct RowWalk {
  size_t o0, step;
  int i, t, ny;
  __device__ __forceinline__ RowWalk(size_t base, int i_, int t_, int ny_) : i(i_), t(t_), ny(ny_) {
    o0 = base + tix<TW>(i_, t_, ny_);
    step = (size_t)(NT / TW) * ny_ * TW;
  }
  __device__ __forceinline__ size_t at(int s) const {
    if constexpr (NT % TW == 0)
      return o0 + (size_t)s * step;
    else
      return o0 - tix<TW>(i, t, ny) + tix<TW>(i, t + s * NT, ny);
  }
};

template <int N>
struct RowCfg {
  static constexpr int NT = N / 8;                           // threads per transform
  static constexpr int RPW = (256 / NT) > 0 ? 256 / NT : 1;  // transforms per workgroup
  static constexpr int WG = RPW * NT;
  static constexpr int PT = N / NT;                          // values per thread per row (8)
  static constexpr int SCR = ScanScratch<NT>::SIZE;          // scan scratch per transform
};

// LDS budget of a column workgroup's transform buffers, which sets how many
// columns it transforms at once.  Three budgets are built; the plan uses the
// middle one (two complex128 columns of 1024 per workgroup, four workgroups per
// CU; the largest for long complex128 vector columns, see launch_col) unless
// hp_autotune measured another to be faster for its shape.
constexpr int kColLds[3] = {20480, 40960, 81920};

template <typename T, typename C, int N, int LB = 40960>
struct ColCfg {
  static constexpr int TW = Tile<T>::W;
  static constexpr int NT = N / 8;
  static constexpr int PB = plen<C>(N) * (int)sizeof(cx<C>);
  static constexpr int G0 = LB / PB;
  static constexpr int G1 = G0 < 1 ? 1 : (G0 > TW ? TW : G0);
  static constexpr int G2 = (G1 * NT > 1024) ? 1024 / NT : G1;
  // columns transformed at once: a power of two, so that it divides the tile width
  static constexpr int GC = G2 >= 16 ? 16 : G2 >= 8 ? 8 : G2 >= 4 ? 4 : G2 >= 2 ? 2 : 1;
  static_assert(TW % GC == 0, "column groups tile the 128-byte row");
  static constexpr int WG = GC * NT;
  static constexpr int SCR = ScanScratch<NT>::SIZE;
  // LDS stride between the GC column buffers: plen<C>(N) (a multiple of 256
  // bytes) plus 256/GC bytes, so that neighbouring threads, which alternate
  // columns in the load, divide and store loops, hit different banks
  static constexpr int SHIFT = (256 / GC) / (int)sizeof(cx<C>) > 0 ? (256 / GC) / (int)sizeof(cx<C>) : 1;
  static constexpr int PLC = plen<C>(N) + SHIFT;
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

// Sum over the workgroup in a fixed order; result valid in thread 0.
template <int WG>
__device__ __forceinline__ double block_sum(double v, double* red) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[w] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < (WG + 63) / 64; ++i) r += red[i];
  }
  return r;
}

template <typename T>
__device__ __forceinline__ cx<T> czero() {
  return mk<T>((T)0, (T)0);
}

__device__ __forceinline__ double edge_loss(int i, int j, int nx, int ny, int W, double eta, double coef) {
  int d = min(min(i, ny - i), min(j, nx - j));
  if (d < 1 || d > W) return 1.0;
  double f = (double)(W + 1 - d) / (double)W;
  return exp(-coef * eta * f * f);
}

// ------------------------------------------------------------------ row forward (physical -> R-domain)

template <typename T, typename C, int N, int TW>
__global__ __launch_bounds__(RowCfg<N>::WG) void k_row_fwd(const c128* __restrict__ in, cx<T>* __restrict__ out,
                                                           double* __restrict__ part, const cx<C>* __restrict__ tw,
                                                           int ny, size_t fsz, int nblk, const PoleList isel,
                                                           const PoleList osel, size_t in_bs, size_t out_bs,
                                                           size_t part_bs) {
  // batch entry z = blockIdx.z: input isel.k[z], output osel.k[z], partial sums z
  in += (size_t)isel.k[blockIdx.z] * in_bs;
  out += (size_t)osel.k[blockIdx.z] * out_bs;
  part += (size_t)blockIdx.z * part_bs;
  using RC = RowCfg<N>;
  constexpr int NT = RC::NT, RPW = RC::RPW, WG = RC::WG, PT = RC::PT;
  __shared__ cx<C> lds[RPW * plen<C>(N)];
  __shared__ cx<C> scr[RPW * RC::SCR];
  __shared__ double red[(WG + 63) / 64];
  const int g = threadIdx.x / NT, t = threadIdx.x % NT;
  const int row = 1 + blockIdx.x * RPW + g;
  const int comp = blockIdx.y;
  const bool valid = row < ny;
  cx<C>* buf = lds + g * plen<C>(N);
  const c128* src = in + comp * fsz + (size_t)row * N;
  const PStep<C, NT> at(t);  // LDS index of element t + s NT
  double nrm = 0.0;
#pragma unroll
  for (int s = 0; s < PT; ++s) {
    const int m = t + s * NT;
    cx<C> v = czero<C>();
    if (valid && m > 0) {
      const c128 a = src[m];
      nrm += abs2(a);
      v = cvt<C>(a);
    }
    buf[at(s)] = v;
  }
  __syncthreads();
  dst1<C, N>(buf, tw, scr + g * RC::SCR, t);
  const C scale = (C)sqrt(2.0 / N);
  if (valid) {
    cx<T>* dst = out + comp * fsz;
#pragma unroll
    for (int s = 0; s < PT; ++s) {
      const int p = t + s * NT;
      dst[tix<TW>(row, p, ny)] = (p == 0) ? czero<T>() : cvt<T>(scale * buf[at(s)]);
    }
  }
  double sum = block_sum<WG>(nrm, red);
  if (threadIdx.x == 0) part[comp * nblk + blockIdx.x] = sum;
}

// ------------------------------------------------------------------ row inverse (R-domain -> physical complex128)

template <typename T, typename C, int N, int TW>
__global__ __launch_bounds__(RowCfg<N>::WG) void k_row_inv(const cx<T>* __restrict__ in, c128* __restrict__ out,
                                                           const cx<C>* __restrict__ tw, int ny, size_t fsz,
                                                           const PoleList sel, size_t in_bs, size_t out_bs) {
  // batch entry z = blockIdx.z: input entry sel.k[z], output z
  in += (size_t)sel.k[blockIdx.z] * in_bs;
  out += (size_t)blockIdx.z * out_bs;
  using RC = RowCfg<N>;
  constexpr int NT = RC::NT, RPW = RC::RPW, PT = RC::PT;
  __shared__ cx<C> lds[RPW * plen<C>(N)];
  __shared__ cx<C> scr[RPW * RC::SCR];
  const int g = threadIdx.x / NT, t = threadIdx.x % NT;
  const int row = blockIdx.x * RPW + g;  // all rows, row 0 -> zeros
  const int comp = blockIdx.y;
  const bool valid = row < ny && row > 0;
  cx<C>* buf = lds + g * plen<C>(N);
  const cx<T>* src = in + comp * fsz;
  const PStep<C, NT> at(t);  // LDS index of element t + s NT
#pragma unroll
  for (int s = 0; s < PT; ++s) {
    const int m = t + s * NT;
    buf[at(s)] = (valid && m > 0) ? cvt<C>(src[tix<TW>(row, m, ny)]) : czero<C>();
  }
  __syncthreads();
  dst1<C, N>(buf, tw, scr + g * RC::SCR, t);
  const C scale = (C)sqrt(2.0 / N);
  if (row < ny) {
    c128* dst = out + comp * fsz + (size_t)row * N;
#pragma unroll
    for (int s = 0; s < PT; ++s) {
      const int p = t + s * NT;
      dst[p] = (!valid || p == 0) ? mk(0.0, 0.0) : cvt<double>(scale * buf[at(s)]);
    }
  }
}

// ------------------------------------------------------------------ column pass (preconditioner)
//
// One workgroup per group of GC columns of a tile (a tile row is one 128-byte
// line, TW columns).  Workgroups are dealt to the 8 XCDs round-robin; the
// TW/GC sibling groups of a tile get block indices with the same value mod 8,
// consecutive in dispatch order: they run at the
// same time on one XCD, so each line comes from HBM once and from that XCD's
// L2 for the siblings (one workgroup walking the groups in turn lost the
// lines from L2 between groups and read the tile about three times).
__device__ __forceinline__ void col_block(int bid, int ntiles, int S, int& tile, int& sub) {
  if (ntiles % 8 == 0) {
    tile = (bid / (8 * S)) * 8 + bid % 8;
    sub = (bid / 8) % S;
  } else {
    tile = bid / S;
    sub = bid % S;
  }
}

// Waves per SIMD for the column pass (as for the row pass: the most that
// compile without spilling, but for 12 bytes at n = 128).
template <typename C, int N>
struct ColWaves {
  static constexpr bool POW2 = (N & (N - 1)) == 0;
  static constexpr int V = (N <= 1024 && POW2) ? 4 : 2;
};

// MODE: the whole pass (COL_WHOLE), or its two halves for a round whose poles all
// start from the shared first basis vector: S_y u_0 once (COL_FORWARD, left in z's
// place as transformed), then each pole's divide and inverse from it (COL_INVERSE,
// u being that field).
enum { COL_WHOLE = 0, COL_FORWARD = 1, COL_INVERSE = 2 };

template <typename T, typename C, int N, int NC, int LB, int MODE>
__global__ __launch_bounds__((ColCfg<T, C, N, LB>::WG), (ColWaves<C, N>::V)) void k_col(
    const Basis<cx<T>> basis, cx<T>* __restrict__ zbase, size_t zsp, size_t zsi, cx<T>* __restrict__ dzbase,
    size_t dzsp, const PoleState* __restrict__ st, const RoundList list, const double* __restrict__ mu_x,
    const double* __restrict__ mu_y, const cx<C>* __restrict__ tw, size_t fsz, StencilCoef sc) {
  using CC = ColCfg<T, C, N, LB>;
  constexpr int NT = CC::NT, TW = CC::TW, GC = CC::GC, WG = CC::WG, S = TW / GC;
  constexpr int PL = CC::PLC;  // padded per-column stride
  __shared__ cx<C> lds[GC * PL];
  __shared__ cx<C> scr[GC * CC::SCR];
  int tile, sub;
  col_block(blockIdx.x, gridDim.x / S, S, tile, sub);
  const int col0 = tile * TW;
  const int c0 = sub * GC;
  const int comp = blockIdx.y % NC;
  const int tid = threadIdx.x;
  const int g = tid / NT, t = tid % NT;
  const C scale = (C)sqrt(2.0 / N);
  const int e = list.e[blockIdx.y / NC], k = round_pole(e), m = round_m(e);
  const c128 b = st[k].bk;
  if (st[k].flag) return;
  const C sc2 = (C)st[k].sigma[m] * scale;
  const size_t tbase = comp * fsz + (size_t)tile * N * TW;  // this tile, component comp (ny == N)
  const cx<T>* __restrict__ u = basis.at(e, m) + tbase;
  cx<T>* z = zbase + k * zsp + m * zsi + tbase;
  cx<T>* dz = (NC == 2) ? dzbase + k * dzsp + tbase : nullptr;
  // The loops below give consecutive threads the columns of a row in turn,
  // from row 0, so that every 16 threads touch one aligned run of rows:
  // thread tid takes column c = tid % GC, rows r0 + i NT (i = 0..7).
  const int c = tid % GC, r0 = tid / GC, q = col0 + c0 + c;
  const double mq = mu_x[q] - b.re, li = -b.im;
  cx<C>* bc = lds + c * PL;
  const PStep<C, NT> at(r0);
  const cx<C>* sintab = tw + N;
  // divide by mu_y[p] + mu_x[q] - b (one FP64 division)
  auto divide = [&](cx<C> X, int p) {
    const double lr = mu_y[p] + mq, inv = 1.0 / (lr * lr + li * li);
    return (scale * X) * mk<C>((C)(lr * inv), (C)(-li * inv));
  };
  {
    if constexpr (MODE != COL_INVERSE) {
      // load fused with the first transform's pre-processing: thread (c, r0) takes the
      // row pairs (j, N - j), j = r0 + i NT < N/2, of its column, and row N/2 when r0 = 0
#pragma unroll 2
      for (int i = 0; i < N / (2 * NT); ++i) {
        const int j = r0 + i * NT;
        if (j == 0) {
          bc[pidx<C>(0)] = czero<C>();
          bc[pidx<C>(N / 2)] = (C)2 * cvt<C>(u[(size_t)(N / 2) * TW + c0 + c]);
          continue;
        }
        cx<C> ya, yb;
        dst1_pair(cvt<C>(u[(size_t)j * TW + c0 + c]), cvt<C>(u[(size_t)(N - j) * TW + c0 + c]), sintab[j].re, ya, yb);
        bc[at(i)] = ya;
        bc[pidx<C>(N - j)] = yb;
      }
      __syncthreads();
      dst1_core<C, N>(lds + g * PL, tw, scr + g * CC::SCR, t);
    }
    if constexpr (MODE == COL_FORWARD) {
#pragma unroll 2
      for (int i = 0; i < N / NT; ++i) z[(size_t)(r0 + i * NT) * TW + c0 + c] = cvt<T>(bc[at(i)]);
      return;
    }
    // the divide fused with the inverse transform's pre-processing, same pairs
    auto first = [&](int p, int at_p) {
      return MODE == COL_INVERSE ? cvt<C>(u[(size_t)p * TW + c0 + c]) : bc[at_p];
    };
#pragma unroll 1
    for (int i = 0; i < N / (2 * NT); ++i) {
      const int j = r0 + i * NT;
      if (j == 0) {
        bc[pidx<C>(0)] = czero<C>();
        bc[pidx<C>(N / 2)] = (C)2 * divide(first(N / 2, pidx<C>(N / 2)), N / 2);
        continue;
      }
      cx<C> ya, yb;
      dst1_pair(divide(first(j, at(i)), j), divide(first(N - j, pidx<C>(N - j)), N - j), sintab[j].re, ya, yb);
      bc[at(i)] = ya;
      bc[pidx<C>(N - j)] = yb;
    }
    __syncthreads();
    dst1_core<C, N>(lds + g * PL, tw, scr + g * CC::SCR, t);
#pragma unroll 2
    for (int i = 0; i < N / NT; ++i) {
      const int p = r0 + i * NT;
      if (p == 0) continue;
      z[(size_t)p * TW + c0 + c] = cvt<T>(sc2 * bc[at(i)]);
      if constexpr (NC == 2) {
        // D1y of the column, physical in y (odd reflection about rows 0 and N)
        cx<double> acc = mk(0.0, 0.0);
#pragma unroll
        for (int mm = 1; mm <= 6; ++mm)
          acc = acc + sc.d1y[mm - 1] * cvt<double>(odd_at(bc, N, p + mm) - odd_at(bc, N, p - mm));
        dz[(size_t)p * TW + c0 + c] = cvt<T>(sc2 * cvt<C>(acc));
      }
    }
  }
}

// ------------------------------------------------------------------ row pass (medium part + inner products)

// Load of one row of an R-domain field fused with the DST-I pre-processing:
// thread t takes the point pairs (j, N - j), j = t + s NT < N/2, and point N/2
// when t = 0; an invalid row loads zeros.
template <typename T, typename C, int N, int NT, int TW>
__device__ __forceinline__ void load_pre_row(cx<C>* buf, const cx<T>* __restrict__ src, const RowWalk<TW, NT>& toff,
                                             size_t rbase, int ny, bool valid, int t, const PStep<C, NT>& at,
                                             const cx<C>* __restrict__ sintab) {
#pragma unroll 2
  for (int s = 0; s < N / (2 * NT); ++s) {
    const int j = t + s * NT;
    if (j == 0) {
      buf[pidx<C>(0)] = czero<C>();
      buf[pidx<C>(N / 2)] = valid ? (C)2 * cvt<C>(src[rbase + tix<TW>(0, N / 2, ny)]) : czero<C>();
      continue;
    }
    cx<C> ya = czero<C>(), yb = czero<C>();
    if (valid) dst1_pair(cvt<C>(src[toff.at(s)]), cvt<C>(src[rbase + tix<TW>(0, N - j, ny)]), sintab[j].re, ya, yb);
    buf[at(s)] = ya;
    buf[pidx<C>(N - j)] = yb;
  }
}

// The same value, which the compiler must take as new: the LDS addresses of a
// transform derive from the thread index alone, and without this the
// compiler keeps those of every transform in a kernel live from the first to
// the last (registers the vector row pass cannot spare).
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// D1x at point j of a row held (unscaled) in the transform buffer b: the
// 13-point first-difference stencil, with the odd reflection about points 0
// and N taken only where the caller says the stencil may reach them.
template <typename C, int N, bool INTERIOR>
__device__ __forceinline__ cx<C> row_d1x(const cx<C>* b, int j, const StencilCoef& sc) {
  cx<C> acc = czero<C>();
#pragma unroll
  for (int mm = 1; mm <= 6; ++mm) {
    if constexpr (INTERIOR)
      acc = acc + (C)sc.d1x[mm - 1] * (b[pidx<C>(j + mm)] - b[pidx<C>(j - mm)]);
    else
      acc = acc + (C)sc.d1x[mm - 1] * (odd_at(b, N, j + mm) - odd_at(b, N, j - mm));
  }
  return acc;
}

// Inner products a row workgroup collects in LDS between two barriers.
constexpr int DOT_B = 16;

// Threads of a row workgroup: 256, but 64 (one wave, no waits between waves) for
// n <= 384, where one pole's rows in workgroups of 256 reach a third of the CUs (77 of
// them at 384).  At 512 and above the smaller workgroup lost 2-4 % (1024^2 16
// poles 6.41 -> 6.70 ms).
constexpr int apply_threads(int n) { return n <= 384 ? 64 : 256; }

template <int N, int NC>
struct ApplyCfg {
  static constexpr int NT = N / 8;
  static constexpr int G0 = (apply_threads(N) / NT) / NC * NC;
  static constexpr int GROUPS = G0 < NC ? NC : G0;  // transforms per workgroup (NC per row)
  static constexpr int ROWS = GROUPS / NC;
  static constexpr int WG = GROUPS * NT;
  static constexpr int WAVES = (WG + 63) / 64;
  static constexpr int SCR = ScanScratch<NT>::SIZE;
  static_assert(NT >= 8, "the stencil's interior points assume at least 8 threads per row");
};

// Lengths whose row pass is also built with a basis vector's loads in flight ahead (AHEAD), for
// rounds whose workgroups leave the SIMDs a wave each at most.
constexpr bool apply_ahead(int n) { return n <= 384; }

// Waves per SIMD the register allocation must allow: two where a round has no more of them to
// offer and the basis vectors' loads want the registers (AHEAD); else
// scalar fields four (128 VGPRs) for 2^k up to 1024, else three (complex128
// at 2048: two); vector fields four, which lets two 512-thread workgroups share
// a CU at 2048 (their LDS, one buffer per component, fits twice).
template <typename C, int N, int NC, bool AHEAD>
struct ApplyWaves {
  static constexpr bool POW2 = (N & (N - 1)) == 0;
  static constexpr int V = AHEAD     ? 2
                           : NC == 2 ? 4
                                     : ((N <= 1024 && POW2) ? 4 : (sizeof(C) == 4 || N < 2048 ? 3 : 2));
};

template <typename T, typename C, int N, int NC, bool AHEAD>
__global__ __launch_bounds__((ApplyCfg<N, NC>::WG), (ApplyWaves<C, N, NC, AHEAD>::V)) void k_row_apply(
    const cx<T>* __restrict__ zbase, size_t zsp, size_t zsi, const cx<T>* __restrict__ dzbase, size_t dzsp,
    cx<T>* __restrict__ pbase, size_t psp, const Basis<cx<T>> basis, const C* __restrict__ coef,
    const PoleState* __restrict__ st, const RoundList list, int nrb, double2* __restrict__ part,
    const cx<C>* __restrict__ tw, int ny, size_t fsz, StencilCoef sc) {
  using AC = ApplyCfg<N, NC>;
  constexpr int NT = AC::NT, GROUPS = AC::GROUPS, ROWS = AC::ROWS, TW = Tile<T>::W;
  constexpr int PT = N / NT;  // values per thread per row
  constexpr int PL = plen<C>(N);
  __shared__ cx<C> lds[GROUPS * PL];
  __shared__ cx<C> scr[GROUPS * AC::SCR];
  __shared__ double dsum[AC::WAVES > 1 ? DOT_B : 1][AC::WAVES][4];
  const int g = threadIdx.x / NT, t = threadIdx.x % NT;
  const int comp = g % NC;
  // XCD-aware order (workgroups go round-robin to the eight XCDs): the
  // workgroups of one XCD take its row blocks in turn with every pole's
  // workgroup for a block next to the others, so the block's medium
  // coefficients (and, in a first cycle, the shared basis vector) come from
  // that XCD's L2 for all but the first pole
  const int xcd = blockIdx.x % 8, q = blockIdx.x / 8;
  const int rb = (q / list.n) * 8 + xcd;
  if (rb >= nrb) return;
  const int row = 1 + rb * ROWS + g / NC;
  const bool valid = row < ny;
  const int e = list.e[q % list.n], k = round_pole(e), m = round_m(e);
  if (st[k].flag) return;
  cx<C>* buf = lds + g * PL;
  cx<C>* sg = scr + g * AC::SCR;
  const C scale = (C)sqrt(2.0 / N);
  const size_t cbase = comp * fsz;
  const size_t ci0 = (size_t)row * N;  // physical row offset
  const RowWalk<TW, NT> toff(cbase, valid ? row : 0, t, ny);  // tiled offsets of the thread's points
  const PStep<C, NT> at(t);                                    // LDS index of point t + s NT

  const cx<T>* z = zbase + k * zsp + m * zsi;
  cx<C> pz[PT];  // P z at the thread's points j = t + s * NT (vector fields)
  if constexpr (NC == 1) {
    // load fused with the inverse transform's pre-processing: thread t takes the point
    // pairs (j, N - j), j = t + s NT < N/2, of its row, and point N/2 when t = 0
    const cx<C>* sintab = tw + N;
    const size_t rbase = cbase + tix<TW>(valid ? row : 0, 0, ny);
#pragma unroll 2
    for (int s = 0; s < PT / 2; ++s) {
      const int j = t + s * NT;
      if (j == 0) {
        buf[pidx<C>(0)] = czero<C>();
        buf[pidx<C>(N / 2)] = valid ? (C)2 * cvt<C>(z[rbase + tix<TW>(0, N / 2, ny)]) : czero<C>();
        continue;
      }
      cx<C> ya = czero<C>(), yb = czero<C>();
      if (valid) dst1_pair(cvt<C>(z[toff.at(s)]), cvt<C>(z[rbase + tix<TW>(0, N - j, ny)]), sintab[j].re, ya, yb);
      buf[at(s)] = ya;
      buf[pidx<C>(N - j)] = yb;
    }
    __syncthreads();
    // the inverse transform's outputs leave multiplied by the medium: P z = V z
    dst1_core_op<C, N>(buf, tw, sg, t, [&](int p, cx<C> X) {
      return (valid ? coef[ci0 + p] : (C)0) * (scale * X);
    });
  } else {
    // eq. Z_bar_eq, medium part (coefficient planes carry s = 1/(k0 n0)^2):
    //   (P w)_1 = psi_xx w1 + psi_x D1x w1 + psi_xy w2 + psi_y D1x w2 + V w1
    //   (P w)_2 = psi_xy w1 + psi_x D1y w1 + psi_yy w2 + psi_y D1y w2 + V w2
    // A workgroup holds one transform buffer per component (two workgroups fit
    // a CU) and no partial product stays in registers across a transform: the
    // D1y rows (the column pass's second output) are transformed first, and
    // the D1y part of (P w)_2 waits in the component's own output row of p (in
    // the storage precision), which the final store overwrites.  Each group
    // reads its partner's buffer directly, and each takes one x-derivative
    // stencil.  Both loads are fused with their transforms' pre-processing, as
    // for scalar fields.
    const size_t rbase = cbase + tix<TW>(valid ? row : 0, 0, ny);
    const cx<C>* ob = lds + (g ^ 1) * PL;
    cx<T>* pk = pbase + k * psp;
    load_pre_row<T, C, N, NT, TW>(buf, dzbase + k * dzsp, toff, rbase, ny, valid, t, at, tw + N);
    __syncthreads();
    dst1_core<C, N>(buf, tw, sg, fresh(t));
    if (comp == 1 && valid) {
#pragma unroll
      for (int s = 0; s < PT; ++s) {
        const int j = t + s * NT;
        if (j == 0) continue;
        const size_t ci = ci0 + j;
        pk[toff.at(s)] = cvt<T>(coef[2 * fsz + ci] * (scale * buf[at(s)]) + coef[fsz + ci] * (scale * ob[at(s)]));
      }
    }
    __syncthreads();
    load_pre_row<T, C, N, NT, TW>(buf, z, toff, rbase, ny, valid, t, at, tw + N);
    __syncthreads();
    dst1_core<C, N>(buf, tw, sg, fresh(t));
    // component 1 takes psi_y D1x w2 of component 0's product from its own
    // buffer and leaves it (storage precision) in component 0's output row of
    // p, where component 0 picks it up after the barrier
    cx<T>* pk0 = pk - cbase;  // component 0's rows of p
    if (comp == 1 && valid) {
#pragma unroll
      for (int s = 0; s < PT; ++s) {
        const int j = t + s * NT;
        if (j == 0) continue;
        // the thread's middle points never reach the reflections at 0 and N
        const bool inner = s > 0 && s < PT - 1;
        const cx<C> dx = inner ? row_d1x<C, N, true>(buf, j, sc) : row_d1x<C, N, false>(buf, j, sc);
        pk0[toff.at(s)] = cvt<T>(coef[2 * fsz + ci0 + j] * (scale * dx));
        // one point at a time: hoisting every point's loads would spill
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int s = 0; s < PT; ++s) {
      const int j = t + s * NT;
      pz[s] = czero<C>();
      if (!valid || j == 0) continue;
      const size_t ci = ci0 + j;
      const cx<C> zc = scale * buf[at(s)], zo = scale * ob[at(s)];
      const C v = coef[ci], pxy = coef[5 * fsz + ci];
      if (comp == 0) {
        const bool inner = s > 0 && s < PT - 1;
        const cx<C> dx = inner ? row_d1x<C, N, true>(buf, j, sc) : row_d1x<C, N, false>(buf, j, sc);
        pz[s] = (coef[3 * fsz + ci] + v) * zc + coef[fsz + ci] * (scale * dx) + pxy * zo;
      } else {
        pz[s] = (coef[4 * fsz + ci] + v) * zc + pxy * zo + cvt<C>(pk[toff.at(s)]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    if (comp == 0 && valid) {
#pragma unroll
      for (int s = 0; s < PT; ++s)
        if (t + s * NT > 0) pz[s] = pz[s] + cvt<C>(pk0[toff.at(s)]);
    }
  }
  // forward transform of P z (already in buf for scalar fields)
  if constexpr (NC == 2) {
#pragma unroll
    for (int s = 0; s < PT; ++s) {
      const int j = t + s * NT;
      buf[at(s)] = (j == 0) ? czero<C>() : pz[s];
    }
    __syncthreads();
  }
  dst1<C, N>(buf, tw, sg, NC == 1 ? t : fresh(t));
  // p as stored: the inner products use exactly what the update reads (vector
  // fields re-read it from LDS in each product, to keep fewer values live)
  auto pval = [&](int s) {
    const int j = t + s * NT;
    return (j == 0 || !valid) ? czero<T>() : cvt<T>(scale * buf[at(s)]);
  };
  cx<T> pv[NC == 1 ? PT : 1];
  cx<T>* p = pbase + k * psp;
#pragma unroll
  for (int s = 0; s < PT; ++s) {
    const cx<T> ps = pval(s);
    if constexpr (NC == 1) pv[s] = ps;
    if (valid) p[toff.at(s)] = ps;
  }
  // <u_i, p> and <u_i, u_m>, i = 0..m: the new direction's projections and
  // the reorthogonalisation of the provisional u_m, from the same reads of the
  // basis, u_m itself read once (read again in its turn, it came from the fabric in part:
  // without, 1024^2 scalar 6.03 -> 5.90 ms a step, 512 x 768 vector 2.13 -> 2.05).  The
  // loads are unconditional (a row beyond the field reads row 0, and its p and u_m are
  // zero; a vector beyond u_m reads u_m), so nothing waits for them
  // before their products; with AHEAD the next vector's are in flight during the current one's (one
  // 384^2 pole, average over the cycle: 26.6 -> 18.7 us with the smaller workgroups).  The waves' sums
  // meet in LDS once per DOT_B vectors, so a workgroup leaves one partial sum per
  // product.
  auto load_u = [&](int i, cx<T>* v) {
    const cx<T>* __restrict__ u = basis.at(e, min(i, m));
#pragma unroll
    for (int s = 0; s < PT; ++s) v[s] = u[toff.at(s)];
  };
  cx<T> um[PT], ua[PT], ub[AHEAD ? PT : 1];
  load_u(m, um);
  if (AHEAD) load_u(0, ua);
#pragma unroll
  for (int s = 0; s < PT; ++s) um[s] = valid ? um[s] : czero<T>();
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double* out = reinterpret_cast<double*>(part) + ((size_t)k * (HP_MAXM + 1) * 2 * nrb + rb) * 2;
  for (int i0 = 0; i0 <= m; i0 += DOT_B) {
    const int ie = min(m + 1, i0 + DOT_B);
    auto products = [&](int i, const cx<T>* uc) {
      double pr = 0.0, pi = 0.0, qr = 0.0, qi = 0.0;
#pragma unroll
      for (int s = 0; s < PT; ++s) {
        const cx<double> a = cvt<double>(uc[s]);
        const cx<double> bp = cvt<double>(NC == 1 ? pv[s] : pval(s));
        const cx<double> bq = cvt<double>(um[s]);
        pr = fma(a.re, bp.re, fma(a.im, bp.im, pr));
        pi = fma(a.re, bp.im, fma(-a.im, bp.re, pi));
        qr = fma(a.re, bq.re, fma(a.im, bq.im, qr));
        qi = fma(a.re, bq.im, fma(-a.im, bq.re, qi));
      }
      const double r = wave_sum4(pr, pi, qr, qi);
      if (lane < 4) {
        if constexpr (AC::WAVES == 1)
          out[((size_t)(2 * i + (lane >> 1)) * nrb) * 2 + (lane & 1)] = r;
        else
          dsum[i - i0][wave][lane] = r;
      }
    };
    if (ie > m) products(m, um);
    const int il = min(ie, m);
    if constexpr (AHEAD) {
      for (int i = i0; i < il; i += 2) {
        load_u(i + 1, ub);
        products(i, ua);
        load_u(i + 2, ua);
        if (i + 1 < il) products(i + 1, ub);
      }
    } else {
      for (int i = i0; i < il; ++i) {
        load_u(i, ua);
        products(i, ua);
      }
    }
    if constexpr (AC::WAVES > 1) {
      __syncthreads();
      for (int x = threadIdx.x; x < 4 * (ie - i0); x += AC::WG) {
        double r = dsum[x >> 2][0][x & 3];
#pragma unroll
        for (int w = 1; w < AC::WAVES; ++w) r += dsum[x >> 2][w][x & 3];
        out[((size_t)(2 * (i0 + (x >> 2)) + ((x >> 1) & 1)) * nrb) * 2 + (x & 1)] = r;
      }
      __syncthreads();
    }
  }
}

// ------------------------------------------------------------------ Gram-Schmidt update

constexpr int UPD_WG = 256;

// u_{m+1} = cu_{m+1} p + sum_{i<=m} cu_i u_i and partial |u_{m+1}|^2.  Bound by
// the copy rate (m + 3 fields; the stored vectors stay as they are, their
// reorthogonalisation is in the coefficients).  E elements per thread, UPD_WG apart,
// and two basis vectors at a time, so that their loads are in flight together.
template <typename T, int E>
__global__ __launch_bounds__(UPD_WG) void k_update(const cx<T>* __restrict__ pbase, size_t psp,
                                                   const Basis<cx<T>> basis, const PoleState* __restrict__ st,
                                                   const RoundList list, double* __restrict__ part, int nblk,
                                                   size_t total) {
  __shared__ c128 cf[HP_MAXM + 2];
  __shared__ double red[UPD_WG / 64];
  const int en = list.e[blockIdx.y], k = round_pole(en), m = round_m(en);
  if (st[k].flag) return;
  if ((int)threadIdx.x <= m + 1) cf[threadIdx.x] = st[k].cu[threadIdx.x];
  __syncthreads();
  const cx<T>* p = pbase + k * psp;
  cx<T>* out = basis.at(en, m + 1);
  double nrm = 0.0;
  const size_t chunk = (size_t)UPD_WG * E;
  for (size_t base = (size_t)blockIdx.x * chunk + threadIdx.x; base < total; base += (size_t)gridDim.x * chunk) {
    cx<double> v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const size_t idx = base + (size_t)e * UPD_WG;
      v[e] = (idx < total) ? cf[m + 1] * cvt<double>(p[idx]) : mk(0.0, 0.0);
    }
    auto add = [&](int i, const cx<T>* a) {
      const c128 fi = cf[i];
#pragma unroll
      for (int e = 0; e < E; ++e) v[e] = cfma(fi, cvt<double>(a[e]), v[e]);
    };
    auto load = [&](int i, cx<T>* a) {
      const cx<T>* ui = basis.at(en, i);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const size_t idx = base + (size_t)e * UPD_WG;
        a[e] = (idx < total) ? ui[idx] : czero<T>();
      }
    };
    int i = 0;
    for (; i + 1 <= m; i += 2) {
      cx<T> a[E], b[E];
      load(i, a);
      load(i + 1, b);
      add(i, a);
      add(i + 1, b);
    }
    if (i <= m) {
      cx<T> a[E];
      load(i, a);
      add(i, a);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const size_t idx = base + (size_t)e * UPD_WG;
      if (idx >= total) continue;
      const cx<T> r = cvt<T>(v[e]);
      out[idx] = r;
      nrm += abs2(cvt<double>(r));
    }
  }
  double s = block_sum<UPD_WG>(nrm, red);
  if (threadIdx.x == 0) part[(size_t)k * nblk + blockIdx.x] = s;
}

// ------------------------------------------------------------------ reductions / small FP64 kernels

// Upper triangle of an n x n matrix packed by columns: (r, c), r <= c.
__device__ __forceinline__ int pk(int r, int c) { return c * (c + 1) / 2 + r; }

// v of lane l of the wave (l uniform)
__device__ __forceinline__ double lane_get(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}
__device__ __forceinline__ c128 lane_get(c128 v, int l) { return mk(lane_get(v.re, l), lane_get(v.im, l)); }

// Sum the partial inner products of one pole, then the delayed
// reorthogonalisation algebra of its step m in FP64.  The stored vectors are the
// provisional ones and are never rewritten: with ~v_l the stored vector l scaled to
// diagonal 1 (sigma_l u_l), ~v_l = v_l + sum_{i<l} R_il v_i, so <v, x> = R^-H <~v, x>
// and sum_l c_l v_l = ~V R^-1 c; R^-1 grows by the column -R^-1 r_m per step, so both
// are matrix-vector products.  (Rewriting u_m in place cost the update a write of a
// field in every step: 1024^2 16 poles 6.45 -> 6.11 ms, 2048^2 vector 14.2 -> 13.5.)
//   s_i = <v_i, ~v_m>, t = <~v_m, ~v_m>, rho^2 = t - sum |s_i|^2,
//   v_m = (~v_m - sum s_i v_i) / rho,  R_im = s_i / rho,
//   column m-1:  H[i][m-1] += h~ s_i,  H[m][m-1] = h~ rho  (h~ = old H[m][m-1]),
//   c_i = <v_i, p>, c_m = (<~v_m, p> - sum conj(s_i) c_i) / rho,
//   A M^-1 v_m = (~v_m + p - sum_i s_i A M^-1 v_i) / rho   (A M^-1 ~v_m = ~v_m + p),
//   H[l][m] = <v_l, A M^-1 v_m>, u_{m+1} = A M^-1 v_m - sum_l H[l][m] v_l,
// expressed as coefficients of the stored vectors for the update kernel.
//
// One workgroup per pole (the row pass leaves one partial per workgroup, so a
// wave sums a product of 1024^2 in eight loads a lane).  Wave w takes the products
// i = w, w + 16, ..., and the same rows of each matrix-vector product as wave sums
// (lane l entry l), so the chain has three barriers and no loop over the basis in one
// thread (substitutions with R took 5 % of a 384^2 solve of 30-vector cycles).
// Latency-bound: 9.5 us at 64^2 and 11.5 us at 1024^2 when 2 (m + 1) workgroups a pole
// met in an atomic counter and one thread ran the sums, 4.3 and 5.9 us now.
constexpr int RED_WG = 1024;
__global__ __launch_bounds__(RED_WG) void k_reduce_dots(const double2* __restrict__ part, int nparts,
                                                        PoleState* __restrict__ st, const RoundList list) {
  constexpr int LD = HP_MAXM + 1, NW = RED_WG / 64;
  __shared__ c128 PQ[HP_MAXM + 1][2];
  __shared__ c128 SC[HP_MAXM][2];
  __shared__ c128 G[HP_MAXM + 1];
  // H (entries 0..c+1 of column c) and the strict upper part of R^-1, packed by columns:
  // columns come in whole lines, rows are read here (64 lines a row from memory)
  __shared__ c128 Hs[HP_MAXM * (HP_MAXM + 3) / 2], Rs[HP_MAXM * (HP_MAXM - 1) / 2];
  auto hx = [](int r, int c) { return c * (c + 3) / 2 + r; };
  auto rx = [](int r, int c) { return c * (c - 1) / 2 + r; };
  const int e = list.e[blockIdx.x], k = round_pole(e), m = round_m(e);
  PoleState& S = st[k];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // what the algebra needs of the state, in flight during the sums
  const double sig = lane <= m ? S.sigma[lane] : 0.0;
  const c128 *Hr = S.Hraw, *Ri = S.Ri;
  const c128 zero = mk(0.0, 0.0);
  auto h_at = [&](int l) { return (lane < m && l <= lane + 1) ? Hs[hx(l, lane)] : zero; };
  auto ri_at = [&](int i) { return (lane > i && lane < m) ? Rs[rx(i, lane)] : lane == i ? mk(1.0, 0.0) : zero; };
  auto rh_at = [&](int i) { return lane < i ? Rs[rx(lane, i)] : lane == i ? mk(1.0, 0.0) : zero; };
  const double hsub = m > 0 ? Hr[m + (m - 1) * LD].re : 0.0;
  const c128 g0 = S.g[0];
  if (S.flag) return;
  // columns from the last wave down, products from the first up: a short cycle's waves have one each
  for (int c = NW - 1 - wave; c < m; c += NW) {
    if (lane <= c + 1) Hs[hx(lane, c)] = Hr[lane + c * LD];
    if (lane < c) Rs[rx(lane, c)] = Ri[lane + c * LD];
  }
  for (int i = wave; i <= m; i += NW) {
    const double2* src = part + (((size_t)k * LD + i) * 2) * nparts;
    double a[4][4] = {};
    int b = lane;
    for (; b + 3 * 64 < nparts; b += 4 * 64) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double2 p = src[b + u * 64], q = src[nparts + b + u * 64];
        a[u][0] += p.x;
        a[u][1] += p.y;
        a[u][2] += q.x;
        a[u][3] += q.y;
      }
    }
    for (; b < nparts; b += 64) {
      const double2 p = src[b], q = src[nparts + b];
      a[0][0] += p.x;
      a[0][1] += p.y;
      a[0][2] += q.x;
      a[0][3] += q.y;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) a[0][v] += a[1][v] + (a[2][v] + a[3][v]);
    const double r = wave_sum4(a[0][0], a[0][1], a[0][2], a[0][3]);
    if (lane < 4) reinterpret_cast<double*>(&PQ[i][lane >> 1])[lane & 1] = r;
  }
  __syncthreads();
  const double sm = lane_get(sig, m);
  const c128 Pm = PQ[m][0], Qm = PQ[m][1];
  {
    // s and c: R^-H of the products with the stored vectors
    const c128 q = lane < m ? (sig * sm) * PQ[lane][1] : zero, p = lane < m ? sig * PQ[lane][0] : zero;
    for (int i = wave; i < m; i += NW) {
      const c128 r = rh_at(i), x = cmulc(r, q), y = cmulc(r, p);
      const double t = wave_sum4(x.re, x.im, y.re, y.im);
      if (lane < 4) reinterpret_cast<double*>(&SC[i][lane >> 1])[lane & 1] = t;
    }
  }
  __syncthreads();
  // lane i: s_i, c_i (i < m); every wave
  const c128 sv = lane < m ? SC[lane][0] : zero, cc = lane < m ? SC[lane][1] : zero;
  const c128 sc = cmulc(sv, cc);
  const double t = wave_sum4(abs2(sv), sc.re, sc.im, 0.0);
  double rho2 = sm * sm * Qm.re - lane_get(t, 0);
  if (!(rho2 > 1e-300)) rho2 = 1e-300;
  const double rho = sqrt(rho2), irho = 1.0 / rho;
  const c128 cm = irho * (sm * Pm - mk(lane_get(t, 1), lane_get(t, 2)));
  // column m: h_l = (<v_l, ~v_m> + <v_l, p> - A_l) / rho, A_l = sum_{i<m, i>=l-1} s_i H[l][i],
  // with column m-1 of H as corrected
  for (int l = wave; l <= m; l += NW) {
    c128 hv = h_at(l);
    const c128 sl = l < m ? lane_get(sv, l) : mk(rho, 0.0);
    if (lane == m - 1) hv = l < m ? hv + hsub * sl : mk(hsub * rho, 0.0);
    const c128 a = (lane < m && lane >= l - 1) ? sv * hv : zero;
    const double r = wave_sum4(a.re, a.im, 0.0, 0.0);
    const c128 A = mk(lane_get(r, 0), lane_get(r, 1));
    const c128 h = irho * (sl + (l < m ? lane_get(cc, l) : cm) - A);
    if (lane == 0) {
      S.Hraw[l + m * LD] = h;
      G[l] = irho * A + h;
    }
  }
  __syncthreads();
  const c128 gam = G[m];
  // u_{m+1} = (1/rho) p + (1 - gam)/rho ~v_m + sum_{l<m} (gam s_l / rho - A_l / rho - h_l) v_l,
  // the v_l's coefficients taken to the stored vectors by R^-1, and R^-1's column m
  const c128 rm = irho * sv, d = lane < m ? gam * rm - G[lane] : zero;
  for (int i = wave; i < m; i += NW) {
    const c128 r = ri_at(i), x = r * d, y = r * rm;
    const double w = wave_sum4(x.re, x.im, y.re, y.im);
    const c128 ci = mk(lane_get(w, 0), lane_get(w, 1)), col = mk(lane_get(w, 2), lane_get(w, 3));
    if (lane == i) {
      S.cu[i] = sig * ci;
      S.Ri[i + m * LD] = -col;
    }
  }
  if (wave != 0) return;
  if (lane < m) {
    S.Rc[lane + m * LD] = sv;
    S.Hraw[lane + (m - 1) * LD] = Hr[lane + (m - 1) * LD] + hsub * sv;
  }
  if (lane == 0) {
    S.Rc[m + m * LD] = mk(rho, 0.0);
    S.cu[m] = (sm * irho) * (mk(1.0, 0.0) - gam);
    S.cu[m + 1] = mk(irho, 0.0);
    S.sigma[m] = sm * irho;  // ~v_m with diagonal 1
    if (m == 0)
      S.g[0] = rho * g0;
    else
      S.Hraw[m + (m - 1) * LD] = mk(hsub * rho, 0.0);
  }
}

__device__ __forceinline__ void givens(c128 a, double b, double& c, c128& sn, c128& r) {
  const double aa = sqrt(abs2(a));
  const double rho = sqrt(aa * aa + b * b);
  if (rho == 0.0) {
    c = 1.0;
    sn = mk(0.0, 0.0);
  } else if (aa == 0.0) {
    c = 0.0;
    sn = mk(1.0, 0.0);
  } else {
    c = aa / rho;
    sn = (b / (rho * aa)) * a;  // (a/|a|) conj(b)/rho with b real
  }
  r = c * a + b * sn;
}

// Back substitution R x = rhs (R packed upper triangular, n <= 64) by the first
// wave of the block: lane l keeps rhs[l] in a register and x[i] reaches it by a
// lane read; x is written to LDS.  rhs is not modified.
__device__ void upper_solve(const c128* __restrict__ R, const c128* rhs, c128* x, int n) {
  const int l = threadIdx.x;
  if (l < 64) {
    c128 r = (l < n) ? rhs[l] : mk(0.0, 0.0);
    // lane l divides by its own diagonal entry; the inverse is ready before the chain
    const c128 d = (l < n) ? R[pk(l, l)] : mk(1.0, 0.0);
    c128 col = (l < n) ? R[pk(l, n - 1)] : mk(0.0, 0.0);  // entry l of column i, one step ahead
    for (int i = n - 1; i >= 0; --i) {
      const c128 di = lane_get(d, i), ri = lane_get(r, i);
      const c128 xi = (abs2(di) > 0.0) ? cdiv(ri, di) : mk(0.0, 0.0);
      const c128 ci = col;
      if (l < i) col = R[pk(l, i - 1)];
      if (l == i) x[i] = xi;
      if (l < i) r = r - ci * xi;
    }
  }
  __syncthreads();
}

// Hessenberg column m, its rotations, the estimate and the flag of one pole.
// Wave 0 keeps the columns, cosines and sines in registers (lane i entry i) and
// walks the rotations with lane reads, columns m-1 and m together; the other
// waves only help to sum the partial norms and to load the triangles at a
// cycle's end.
constexpr int ARN_WG = 256;
__global__ __launch_bounds__(ARN_WG) void k_arnoldi(PoleState* __restrict__ st, const RoundList list,
                                                    const double* __restrict__ part, int nblk, int restart,
                                                    unsigned long long* __restrict__ ftag, unsigned long long seq,
                                                    double* __restrict__ ests) {
  __shared__ c128 c1[HP_MAXM + 1], c2[HP_MAXM + 1], rhs[HP_MAXM + 1], y[HP_MAXM];
  __shared__ double red[ARN_WG / 64];
  __shared__ int flag_s;
  const int en = list.e[blockIdx.x], k = round_pole(en), m = round_m(en);
  const int tid = threadIdx.x;
  PoleState& S = st[k];
  constexpr int LD = HP_MAXM + 1;
  // the columns and scalars, in flight during the sum (lane i < 64; entry 64 of a
  // column is its subdiagonal, set here)
  c128 x1 = mk(0.0, 0.0), x2 = x1, xs = x1, g_m1 = x1, g_m = x1;
  double xc = 0.0;
  if (tid < 64) {
    if (tid <= m) {
      x2 = S.Hraw[tid + m * LD];
      if (m >= 1) x1 = S.Hraw[tid + (m - 1) * LD];
    }
    if (tid < m) {
      xc = S.cs[tid];
      xs = S.sn[tid];
    }
    if (m >= 1) g_m1 = S.gpre[m - 1];
    g_m = S.g[m];
  }
  const int fixed = S.fixed, total = S.total;
  const double tol = S.tol;
  if (S.flag) return;
  double s = 0.0;
  {
    double acc[4] = {0, 0, 0, 0};
    const double* src = part + (size_t)k * nblk;
    int b = tid;
    for (; b + 3 * ARN_WG < nblk; b += 4 * ARN_WG) {
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] += src[b + u * ARN_WG];
    }
    for (; b < nblk; b += ARN_WG) acc[0] += src[b];
    s = wave_sum((acc[0] + acc[1]) + (acc[2] + acc[3]));
  }
  if ((tid & 63) == 0) red[tid >> 6] = s;
  __syncthreads();
  if (tid < 64) {
    const double h = sqrt((red[0] + red[1]) + (red[2] + red[3]));
    c128 a1 = lane_get(x1, 0), a2 = lane_get(x2, 0);  // the running entry i of each column
    for (int i = 0; i + 1 < m; ++i) {
      const double c = lane_get(xc, i);
      const c128 sn = lane_get(xs, i), b1 = lane_get(x1, i + 1), b2 = lane_get(x2, i + 1);
      const c128 r1 = c * a1 + sn * b1, r2 = c * a2 + sn * b2;
      a1 = -1.0 * cmulc(sn, a1) + c * b1;
      a2 = -1.0 * cmulc(sn, a2) + c * b2;
      if (tid == i) {
        x1 = r1;
        x2 = r2;
      }
    }
    c128 gm = g_m;  // g[m] as it stands after column m-1
    if (m >= 1) {
      // column m-1 was corrected by the reorthogonalisation: redo its rotation
      double c;
      c128 sn, r;
      givens(a1, lane_get(x1, m).re, c, sn, r);
      const c128 b2 = lane_get(x2, m);
      const c128 r2 = c * a2 + sn * b2;
      a2 = -1.0 * cmulc(sn, a2) + c * b2;
      gm = -1.0 * cmulc(sn, g_m1);
      if (tid == m - 1) {
        x1 = r;
        x2 = r2;
        S.cs[m - 1] = c;
        S.sn[m - 1] = sn;
        S.g[m - 1] = c * g_m1;
      }
      if (tid == m) x1 = mk(0.0, 0.0);
    }
    double c;
    c128 sn, r;
    givens(a2, h, c, sn, r);
    const c128 gnext = -1.0 * cmulc(sn, gm);
    const double est = sqrt(abs2(gnext));
    int flag = 0;
    if (!isfinite(h) || !isfinite(est)) {
      flag = 4;  // a NaN or Inf reached the Krylov space (n^2 or the right-hand side): stop the pole
    } else if (fixed > 0) {
      if (m + 1 >= fixed) flag = 1;
    } else if (est <= tol || h == 0.0) {
      flag = 1;
    } else if (m + 1 >= restart) {
      flag = 2;
    }
    if (tid == m) {
      x2 = r;
      S.cs[m] = c;
      S.sn[m] = sn;
      S.Hraw[m + 1 + m * LD] = mk(h, 0.0);
      S.H[m + 1 + m * LD] = mk(0.0, 0.0);
      S.gpre[m] = gm;
      S.g[m] = c * gm;
      S.g[m + 1] = gnext;
      S.sigma[m + 1] = (h > 0.0) ? 1.0 / h : 0.0;
      S.est = est;
      S.m = m + 1;
      S.total = total + 1;
      rhs[m] = c * gm;
      flag_s = flag;
    }
    if (tid <= m) {
      S.H[tid + m * LD] = x2;
      c2[tid] = x2;
      if (m >= 1) {
        S.H[tid + (m - 1) * LD] = x1;
        c1[tid] = x1;
      }
    }
    if (m >= 1 && tid == m - 1) rhs[m - 1] = S.g[m - 1];
    if (tid + 1 < m) rhs[tid] = S.g[tid];
  }
  __syncthreads();
  int flag = flag_s;
  if (flag && flag != 4) {
    // least squares R y = g, then y~ = Rc^{-1} y (the coefficients of the stored Z~);
    // both triangles go through LDS, packed (one parallel load each)
    __shared__ c128 tri[HP_MAXM * (HP_MAXM + 1) / 2];
    const int n = m + 1, npk = n * (n + 1) / 2;
    // packed index e = c (c + 1)/2 + r: every thread loads entries of its own, all at once
    auto unpack = [](int e, int& r, int& c) {
      c = (int)((sqrt(8.0 * e + 1.0) - 1.0) * 0.5);
      if ((c + 1) * (c + 2) / 2 <= e) ++c;
      if (c * (c + 1) / 2 > e) --c;
      r = e - c * (c + 1) / 2;
    };
    for (int e = tid; e < npk; e += ARN_WG) {
      int r, c;
      unpack(e, r, c);
      tri[e] = (c == m) ? c2[r] : (c == m - 1 ? c1[r] : S.H[r + c * LD]);
    }
    __syncthreads();
    upper_solve(tri, rhs, y, n);
    for (int e = tid; e < npk; e += ARN_WG) {
      int r, c;
      unpack(e, r, c);
      tri[e] = S.Rc[r + c * LD];
    }
    for (int i = tid; i < n; i += ARN_WG) rhs[i] = y[i];  // the least-squares solution
    __syncthreads();
    upper_solve(tri, rhs, y, n);
    for (int i = tid; i < n; i += ARN_WG) S.y[i] = y[i];
    // The estimate measures the split operator I + P M~^-1; it differs from
    // A M~^-1 by about eps kappa(M_k) ||y|| (y the least-squares solution, so
    // ||y|| = ||M x||).  When that is not well below tol, the true residual decides.
    if (tid == 0 && flag == 1 && fixed == 0) {
      double yn = 0.0;
      for (int i = 0; i < n; ++i) yn += abs2(rhs[i]);
      if (S.incons * sqrt(yn) > 0.1 * S.tol) flag = 3;
    }
  }
  if (tid == 0) {
    S.flag = flag;
    ests[k] = S.est;
    // the round's tag and the flag in one 8-byte system-scope store to host
    // memory, which the host polls (no event per round); the host reads
    // nothing else of this round before a synchronisation, so no release
    __hip_atomic_store(&ftag[k], (seq << 8) | (unsigned long long)flag, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

__global__ __launch_bounds__(64) void k_cycle_init(PoleState* __restrict__ st, const PoleList poles,
                                                   const double* __restrict__ part, int nblk, int first, double tol,
                                                   double rtol_cycle, size_t part_bs, int set_has_x) {
  const int k = poles.k[blockIdx.x];
  part += (size_t)blockIdx.x * part_bs;
  double s = 0.0;
  for (int b = threadIdx.x; b < nblk; b += 64) s += part[b];
  s = wave_sum(s);
  if (threadIdx.x != 0) return;
  PoleState& S = st[k];
  const double beta = sqrt(s);
  if (first) {  // 1: a step's first solve; 2: a later solve of the same step (the count runs on)
    S.beta0 = beta;
    if (first == 1) S.total = 0;
    S.cycle = 0;
    S.has_x = 0;
  } else {
    S.cycle += 1;
  }
  S.beta = beta;
  S.tol = fmax(tol * S.beta0, rtol_cycle * beta);
  S.m = 0;
  S.flag = 0;
  S.est = beta;
  S.g[0] = mk(beta, 0.0);
  S.sigma[0] = (beta > 0.0) ? 1.0 / beta : 0.0;
  if (set_has_x) S.has_x = 1;
}

// ------------------------------------------------------------------ residue-weighted sum and output

// One row per workgroup; its RPW thread groups take the terms (pole, basis
// index) in turn and meet in LDS in a fixed order, then the first group runs the
// transform.  (With a row per group 256^2 had 32 workgroups and every thread a
// chain of all terms: 37 us, latency-bound; large fields run at the copy rate.)
// A term's loads are all in flight before its first product; FULL: one at a time, where the
// workgroups fill the chip evenly (see launch_final).
template <typename T, int N, bool FULL>
__global__ __launch_bounds__(RowCfg<N>::WG) void k_final(const c128* __restrict__ w, c128* __restrict__ out,
                                                         const cx<T>* __restrict__ zbase, size_t zsp, size_t zsi,
                                                         const c128* __restrict__ xacc, size_t xsp,
                                                         const PoleState* __restrict__ st, int npoles, c128 phase,
                                                         c128 rinf_phase, double loss_coef, double eta, int W,
                                                         const c128* __restrict__ tw, int nx, int ny, size_t fsz) {
  using RC = RowCfg<N>;
  constexpr int NT = RC::NT, RPW = RC::RPW, PT = RC::PT, TW = Tile<T>::W;
  __shared__ c128 lds[RPW * plen<double>(N)];
  __shared__ c128 scr[RPW * RC::SCR];
  const int g = threadIdx.x / NT, t = threadIdx.x % NT;
  const int row = blockIdx.x;  // rows 0..ny-1
  const int comp = blockIdx.y;
  const size_t roff = comp * fsz + (size_t)row * N;
  if (row == 0) {
    if (g == 0)
      for (int j = t; j < N; j += NT) out[roff + j] = mk(0.0, 0.0);
    return;
  }
  c128* buf = lds + g * plen<double>(N);
  const RowWalk<TW, NT> toff(comp * fsz, row, t, ny);
  c128 acc[PT];
#pragma unroll
  for (int s = 0; s < PT; ++s) acc[s] = mk(0.0, 0.0);
  // terms are numbered through all poles; group g takes every RPW-th
  int next = g;
  for (int k = 0; k < npoles; ++k) {
    const int m = st[k].m, hx = st[k].has_x, nt = m + hx;
    const c128 ak = st[k].ak;
    const cx<T>* zk = zbase + k * zsp;
    if (hx && next < nt) {  // term 0 of a pole with an accumulator
      if (next == 0) {
        const c128* xk = xacc + k * xsp;
#pragma unroll
        for (int s = 0; s < PT; ++s) acc[s] = cfma(ak, xk[toff.at(s)], acc[s]);
        next += RPW;
      }
    }
#pragma unroll 1
    for (; next < nt; next += RPW) {
      const int i = next - hx;
      const c128 y = st[k].y[i];
      const cx<T>* zi = zk + i * zsi;
      constexpr int LOADS = FULL ? 1 : PT;
#pragma unroll
      for (int h = 0; h < PT; h += LOADS) {
        cx<T> a[LOADS];
#pragma unroll
        for (int s = 0; s < LOADS; ++s) a[s] = zi[toff.at(h + s)];
        if constexpr (FULL) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < LOADS; ++s) acc[h + s] = cfma(ak * y, cvt<double>(a[s]), acc[h + s]);
        if constexpr (FULL) __builtin_amdgcn_sched_barrier(0);
      }
    }
    next -= nt;
  }
  const PStep<double, NT> at(t);  // LDS index of element t + s NT
#pragma unroll
  for (int s = 0; s < PT; ++s) buf[at(s)] = acc[s];
  __syncthreads();
  if constexpr (RPW > 1) {
    // element x of the row: the groups' sums, in the order of the groups
    for (int x = threadIdx.x; x < N; x += RC::WG) {
      const int e = pidx<double>(x);
      c128 v = lds[e];
#pragma unroll
      for (int q = 1; q < RPW; ++q) v = v + lds[q * plen<double>(N) + e];
      lds[e] = v;
    }
    __syncthreads();
  }
  // every group runs the (same) transform's barriers; only the first one's result is stored
  dst1<double, N>(buf, tw, scr + g * RC::SCR, t);
  const double scale = sqrt(2.0 / N);
  for (int j = threadIdx.x; j < N; j += RC::WG) {
    c128 v = mk(0.0, 0.0);
    if (j > 0) {
      const c128 sv = scale * lds[pidx<double>(j)];
      v = edge_loss(row, j, nx, ny, W, eta, loss_coef) * (phase * sv + rinf_phase * w[roff + j]);
    }
    out[roff + j] = v;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_accum(c128* __restrict__ xacc, const cx<T>* __restrict__ z, size_t zsi,
                                               const PoleState* __restrict__ st, const PoleList sel, size_t xsp,
                                               size_t zsp, size_t total) {
  // one pole per blockIdx.y: X_k += its cycle's terms
  const int pole = sel.k[blockIdx.y];
  xacc += (size_t)pole * xsp;
  z += (size_t)pole * zsp;
  const int m = st[pole].m;
  const int hx = st[pole].has_x;
  for (size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (size_t)gridDim.x * 256) {
    c128 acc = hx ? xacc[idx] : mk(0.0, 0.0);
    for (int i = 0; i < m; ++i) acc = cfma(st[pole].y[i], cvt<double>(z[i * zsi + idx]), acc);
    xacc[idx] = acc;
  }
}

// ------------------------------------------------------------------ explicit operator (FP64)

__device__ __forceinline__ c128 ld_odd(const c128* __restrict__ x, int i, int j, int nx, int ny) {
  double sg = 1.0;
  if (i < 0) {
    i = -i;
    sg = -sg;
  } else if (i > ny) {
    i = 2 * ny - i;
    sg = -sg;
  }
  if (j < 0) {
    j = -j;
    sg = -sg;
  } else if (j > nx) {
    j = 2 * nx - j;
    sg = -sg;
  }
  if (i == 0 || j == 0 || i == ny || j == nx) return mk(0.0, 0.0);
  return sg * x[(size_t)i * nx + j];
}

constexpr int OP_WG = 256;
constexpr int OP_TX = 64, OP_TY = 16, OP_H = 6;  // output tile, stencil half-width
constexpr int OP_LX = OP_TX + 2 * OP_H, OP_LY = OP_TY + 2 * OP_H;

// The explicit FP64 operator on LDS tiles: each workgroup stages a 64 x 16
// tile of every component with a 6-node halo (odd reflection about the
// Dirichlet nodes applied while staging), then each thread evaluates four
// pixels of a column of the tile.
template <int NC>
__global__ __launch_bounds__(OP_WG) void k_apply_op(const c128* __restrict__ x, const c128* __restrict__ rhs,
                                                    c128* __restrict__ y, const double* __restrict__ coef,
                                                    const ShiftList sh, StencilCoef sc, int nx, int ny, size_t fsz,
                                                    double* __restrict__ part, int medium_only, size_t xbs,
                                                    size_t ybs, size_t pbs) {
  // batch entry z = blockIdx.z: field z, shift sh.b[z]
  const c128 b = sh.b[blockIdx.z];
  x += (size_t)blockIdx.z * xbs;
  y += (size_t)blockIdx.z * ybs;
  if (part) part += (size_t)blockIdx.z * pbs;
  __shared__ c128 tile[NC][OP_LY * OP_LX];
  __shared__ double red[OP_WG / 64];
  const int ntx = (nx + OP_TX - 1) / OP_TX;
  const int x0 = (blockIdx.x % ntx) * OP_TX, y0 = (blockIdx.x / ntx) * OP_TY;
  for (int c = 0; c < NC; ++c)
    for (int e = threadIdx.x; e < OP_LY * OP_LX; e += OP_WG)
      tile[c][e] = ld_odd(x + c * fsz, y0 + e / OP_LX - OP_H, x0 + e % OP_LX - OP_H, nx, ny);
  __syncthreads();
  double nrm = 0.0;
  const int tx = threadIdx.x % OP_TX, tq = threadIdx.x / OP_TX;
#pragma unroll
  for (int q = 0; q < OP_TY / (OP_WG / OP_TX); ++q) {
    const int ty = tq + q * (OP_WG / OP_TX);
    const int i = y0 + ty, j = x0 + tx;
    if (i >= ny || j >= nx) continue;
    const size_t idx = (size_t)i * nx + j;
    const bool inner = i > 0 && j > 0;
    const int lc = (ty + OP_H) * OP_LX + tx + OP_H;
    c128 lap[NC], d1x[NC], d1y[NC], xc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const c128* t = tile[c];
      const c128 x0c = t[lc];
      c128 l = (sc.c2x[0] + sc.c2y[0]) * x0c, ax = mk(0.0, 0.0), ay = mk(0.0, 0.0);
#pragma unroll
      for (int mm = 1; mm <= 6; ++mm) {
        const c128 xp = t[lc + mm], xm = t[lc - mm], yp = t[lc + mm * OP_LX], ym = t[lc - mm * OP_LX];
        l = l + sc.c2x[mm] * (xp + xm) + sc.c2y[mm] * (yp + ym);
        ax = ax + sc.d1x[mm - 1] * (xp - xm);
        ay = ay + sc.d1y[mm - 1] * (yp - ym);
      }
      lap[c] = l;
      d1x[c] = ax;
      d1y[c] = ay;
      xc[c] = x0c;
    }
    const double V = coef[idx];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      c128 v = medium_only ? V * xc[c] : lap[c] + V * xc[c] - b * xc[c];
      if constexpr (NC == 2) {
        const double px = coef[fsz + idx], py = coef[2 * fsz + idx], pxx = coef[3 * fsz + idx],
                     pyy = coef[4 * fsz + idx], pxy = coef[5 * fsz + idx];
        if (c == 0)
          v = v + pxx * xc[0] + px * d1x[0] + pxy * xc[1] + py * d1x[1];
        else
          v = v + pxy * xc[0] + px * d1y[0] + pyy * xc[1] + py * d1y[1];
      }
      if (!inner) v = mk(0.0, 0.0);
      if (rhs) v = (inner ? rhs[c * fsz + idx] : mk(0.0, 0.0)) - v;
      y[c * fsz + idx] = v;
      nrm += abs2(v);
    }
  }
  double s = block_sum<OP_WG>(nrm, red);
  if (threadIdx.x == 0 && part) part[blockIdx.x] = s;
}

// ------------------------------------------------------------------ coefficient preparation

__global__ __launch_bounds__(256) void k_coef_a(const double* __restrict__ n2, double* __restrict__ coef,
                                                double* __restrict__ psi, double n0, int W, int nx, int ny,
                                                size_t fsz, int vector) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= fsz) return;
  const int i = (int)(idx / nx), j = (int)(idx % nx);
  const int d = min(min(i, ny - i), min(j, nx - j));
  const double v = n2[idx];
  coef[idx] = (d > W) ? (v - n0 * n0) / (n0 * n0) : 0.0;
  if (vector) psi[idx] = log(v);
}

// first derivative of psi along x (valid where the stencil stays inside)
__global__ __launch_bounds__(256) void k_coef_b(const double* __restrict__ psi, double* __restrict__ dpx,
                                                StencilCoef sc, int nx, int ny, size_t fsz) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= fsz) return;
  const int j = (int)(idx % nx);
  double a = 0.0;
  if (j >= 6 && j + 6 < nx)
    for (int mm = 1; mm <= 6; ++mm) a += sc.d1x[mm - 1] * (psi[idx + mm] - psi[idx - mm]);
  dpx[idx] = a;
}

__global__ __launch_bounds__(256) void k_coef_c(const double* __restrict__ psi, const double* __restrict__ dpx,
                                                double* __restrict__ coef, double s, StencilCoef sc, int W, int nx,
                                                int ny, size_t fsz) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= fsz) return;
  const int i = (int)(idx / nx), j = (int)(idx % nx);
  const int d = min(min(i, ny - i), min(j, nx - j));
  double px = 0, py = 0, pxx = 0, pyy = 0, pxy = 0;
  if (d > W) {
    // c2x, c2y already carry s; the psi terms of Zbar are multiplied by s too
    pxx = sc.c2x[0] * psi[idx];
    pyy = sc.c2y[0] * psi[idx];
    for (int mm = 1; mm <= 6; ++mm) {
      pxx += sc.c2x[mm] * (psi[idx + mm] + psi[idx - mm]);
      pyy += sc.c2y[mm] * (psi[idx + (size_t)mm * nx] + psi[idx - (size_t)mm * nx]);
      px += sc.d1x[mm - 1] * (psi[idx + mm] - psi[idx - mm]);
      py += sc.d1y[mm - 1] * (psi[idx + (size_t)mm * nx] - psi[idx - (size_t)mm * nx]);
      pxy += sc.d1y[mm - 1] * (dpx[idx + (size_t)mm * nx] - dpx[idx - (size_t)mm * nx]);
    }
    px *= s;
    py *= s;
    pxy *= s;
  }
  coef[fsz + idx] = px;
  coef[2 * fsz + idx] = py;
  coef[3 * fsz + idx] = pxx;
  coef[4 * fsz + idx] = pyy;
  coef[5 * fsz + idx] = pxy;
}

// After X_k has absorbed the cycle's Z terms: X_k is the whole solution.
__global__ void k_mark_folded(PoleState* __restrict__ st, int first, int count) {
  const int k = first + (int)threadIdx.x;
  if ((int)threadIdx.x < count) {
    st[k].has_x = 1;
    st[k].m = 0;
  }
}

__global__ void k_mark_list(PoleState* __restrict__ st, const PoleList sel) {
  if ((int)threadIdx.x < sel.n) {
    st[sel.k[threadIdx.x]].has_x = 1;
    st[sel.k[threadIdx.x]].m = 0;
  }
}


// ------------------------------------------------------------------ plan set-up

// One workgroup per pole: its state cleared, then the table's entries.
__global__ __launch_bounds__(256) void k_state_init(PoleState* __restrict__ st, const StateInit h) {
  static_assert(sizeof(PoleState) % 16 == 0, "cleared in 16-byte words");
  const int k = blockIdx.x;
  double2* w = reinterpret_cast<double2*>(st + k);
  for (int i = threadIdx.x; i < (int)(sizeof(PoleState) / 16); i += 256) w[i] = make_double2(0.0, 0.0);
  __syncthreads();
  if (threadIdx.x == 0) {
    st[k].bk = h.bk[k];
    st[k].ak = h.ak[k];
    st[k].fixed = h.fixed[k];
    st[k].incons = h.incons[k];
  }
}

__global__ __launch_bounds__(256) void k_clear_rows(char* __restrict__ base, size_t tiles, size_t tile_bytes,
                                                    int words) {
  const size_t n = tiles * words;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256)
    reinterpret_cast<double2*>(base + i / words * tile_bytes)[i % words] = make_double2(0.0, 0.0);
}

// a / b with b scaled by a power of two, so that |b|^2 neither overflows nor underflows; infinite
// for b = 0 and a neither 0 nor a NaN, 0 for b infinite and a finite (cdiv gives NaN there).
__device__ __forceinline__ c128 cdiv_scaled(c128 a, c128 b) {
  const double big = fmax(fabs(b.re), fabs(b.im));
  if (big == 0.0 && (fabs(a.re) > 0.0 || fabs(a.im) > 0.0)) return mk((double)INFINITY, 0.0);
  if (isinf(big) && isfinite(a.re) && isfinite(a.im)) return mk(0.0, 0.0);
  if (big == 0.0 || !isfinite(big)) return cdiv(a, b);
  const int e = -ilogb(big);
  return cdiv(mk(ldexp(a.re, e), ldexp(a.im, e)), mk(ldexp(b.re, e), ldexp(b.im, e)));
}

__device__ __forceinline__ bool finite2(c128 a) { return isfinite(a.re) && isfinite(a.im); }

// r(z) where a denominator or the sum leaves the range of cdiv; over: a term or the sum became
// infinite, whatever it met after.
__device__ __forceinline__ c128 rat_scaled(const SpectrumCheck& c, double z, bool& over) {
  c128 r = c.r_inf;
  over = false;
  for (int k = 0; k < c.npoles; ++k) {
    const c128 t = cdiv_scaled(c.a[k], mk(z - c.b[k].re, -c.b[k].im));
    r = r + t;
    over = over || isinf(t.re) || isinf(t.im) || isinf(r.re) || isinf(r.im);
  }
  return r;
}

// Maxima of |f| over the samples.  A NaN counts for nothing where r itself is one, and as an
// infinity where r is not (infinite terms of both signs met, or a finite r overflowed in the polynomial).
__global__ __launch_bounds__(256) void k_spectrum_max(const SpectrumCheck c, double* __restrict__ out) {
  __shared__ double red[4];
  double best = 0.0;
  for (int i = blockIdx.x * 256 + threadIdx.x; i <= 100000; i += kSpectrumBlocks * 256) {
    const double z = c.lo + (c.hi - c.lo) * i / 100000.0;
    c128 r = c.r_inf;
    bool plain = true, over = false;
    for (int k = 0; k < c.npoles; ++k) {
      const c128 q = mk(z - c.b[k].re, -c.b[k].im);
      const double d = abs2(q);
      plain = plain && d > 1e-280 && d < 1e280;
      r = r + cdiv(c.a[k], q);
    }
    if (!(plain && finite2(r))) r = rat_scaled(c, z, over);
    if (c.hk != 0.0 && !over) {
      const bool number = finite2(r);
      const c128 x = mk(-c.hk * r.im, c.hk * (r.re - 1.0));  // i hk (r - 1)
      const c128 one = mk(1.0, 0.0);
      c128 q = mk(1.0 / 6.0, 0.0) + (1.0 / 24.0) * x;
      q = mk(0.5, 0.0) + x * q;
      q = one + x * q;
      r = one + x * q;
      over = number && !finite2(r);
    }
    const double v = over ? INFINITY : sqrt(abs2(r));
    if (v > best) best = v;
  }
  for (int off = 32; off > 0; off >>= 1) best = fmax(best, __shfl_down(best, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = best;
  __syncthreads();
  if (threadIdx.x == 0) out[blockIdx.x] = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
}

// One stage of the classical fourth-order Runge-Kutta combination, over the
// fields in physical layout [ncomp][ny][nx]: acc_out = acc_in + ca L and, when
// v_out is given, v_out = u + cv L.  With loss_coef > 0, acc_out is multiplied
// by the edge layer's loss factor.  Row 0 and column 0 are written as zero.
// acc_in may alias acc_out (each element is read before it is written).
__global__ __launch_bounds__(256) void k_rk4_stage(const c128* __restrict__ L, const c128* acc_in, c128* acc_out,
                                                   const c128* __restrict__ u, c128* __restrict__ v_out, double ca,
                                                   double cv, double loss_coef, double eta, int W, int nx, int ny,
                                                   unsigned fsz, unsigned total) {
  for (unsigned idx = blockIdx.x * 256u + threadIdx.x; idx < total; idx += gridDim.x * 256u) {
    const unsigned e = idx % fsz;
    const int i = (int)(e / (unsigned)nx), j = (int)(e % (unsigned)nx);
    const bool inside = i > 0 && j > 0;
    c128 a = mk(0.0, 0.0), v = mk(0.0, 0.0);
    if (inside) {
      const c128 l = L[idx];
      a = acc_in[idx] + ca * l;
      if (loss_coef > 0.0) a = edge_loss(i, j, nx, ny, W, eta, loss_coef) * a;
      if (v_out) v = u[idx] + cv * l;
    }
    acc_out[idx] = a;
    if (v_out) v_out[idx] = v;
  }
}

}  // namespace

// ====================================================================== launchers

#define HP_DISPATCH_N(n, MACRO) \
  switch (n) {                  \
    case 64: MACRO(64); break;  \
    case 128: MACRO(128); break;  \
    case 192: MACRO(192); break;  \
    case 256: MACRO(256); break;  \
    case 384: MACRO(384); break;  \
    case 512: MACRO(512); break;  \
    case 768: MACRO(768); break;  \
    case 1024: MACRO(1024); break; \
    case 1536: MACRO(1536); break; \
    case 2048: MACRO(2048); break; \
    default: break;             \
  }

template <typename T>
int row_blocks(int nx) {
  const int NT = nx / 8;
  (void)sizeof(T);
  return (256 / NT) > 0 ? 256 / NT : 1;  // rows per workgroup
}

template <typename T, typename C>
void launch_row_fwd_batch(const c128* in, size_t in_bs, const int* isel_h, cx<T>* out, size_t out_bs,
                          const int* osel_h, int n, double* part, size_t part_bs, const cx<C>* tw, const Geo& g,
                          hipStream_t s, int tile_w) {
  const int rpw = row_blocks<T>(g.nx);
  const int nblk = (g.ny - 1 + rpw - 1) / rpw;
  dim3 grid(nblk, g.ncomp, n);
  if (tile_w <= 0) tile_w = tile_width<T>();
  PoleList isel, osel;
  isel.n = osel.n = n;
  for (int a = 0; a < HP_MAXPOLES; ++a) {
    isel.k[a] = a < n ? isel_h[a] : 0;
    osel.k[a] = a < n ? osel_h[a] : 0;
  }
#define L_(NN)                                                                                                    \
  if (tile_w == 8)                                                                                                \
    hipLaunchKernelGGL((k_row_fwd<T, C, NN, 8>), grid, dim3(RowCfg<NN>::WG), 0, s, in, out, part, tw, g.ny, g.fsz,   \
                       nblk, isel, osel, in_bs, out_bs, part_bs);                                                        \
  else                                                                                                            \
    hipLaunchKernelGGL((k_row_fwd<T, C, NN, 16>), grid, dim3(RowCfg<NN>::WG), 0, s, in, out, part, tw, g.ny, g.fsz,  \
                       nblk, isel, osel, in_bs, out_bs, part_bs);
  HP_DISPATCH_N(g.nx, L_)
#undef L_
}

template <typename T, typename C>
void launch_row_fwd(const c128* in, cx<T>* out, double* part, const cx<C>* tw, const Geo& g, hipStream_t s,
                    int tile_w) {
  const int zero = 0;
  launch_row_fwd_batch<T, C>(in, 0, &zero, out, 0, &zero, 1, part, 0, tw, g, s, tile_w);
}

template <typename T, typename C>
void launch_row_inv_batch(const cx<T>* in, size_t in_bs, const int* sel_h, int n, c128* out, size_t out_bs,
                          const cx<C>* tw, const Geo& g, int tile_w, hipStream_t s) {
  const int rpw = row_blocks<T>(g.nx);
  const int nblk = (g.ny + rpw - 1) / rpw;
  dim3 grid(nblk, g.ncomp, n);
  PoleList sel;
  sel.n = n;
  for (int a = 0; a < HP_MAXPOLES; ++a) sel.k[a] = a < n ? sel_h[a] : 0;
#define L_(NN)                                                                                                  \
  if (tile_w == 8)                                                                                              \
    hipLaunchKernelGGL((k_row_inv<T, C, NN, 8>), grid, dim3(RowCfg<NN>::WG), 0, s, in, out, tw, g.ny, g.fsz, sel,  \
                       in_bs, out_bs);                                                                          \
  else                                                                                                          \
    hipLaunchKernelGGL((k_row_inv<T, C, NN, 16>), grid, dim3(RowCfg<NN>::WG), 0, s, in, out, tw, g.ny, g.fsz, sel, \
                       in_bs, out_bs);
  HP_DISPATCH_N(g.nx, L_)
#undef L_
}

template <typename T, typename C>
void launch_row_inv(const cx<T>* in, c128* out, const cx<C>* tw, const Geo& g, int tile_w, hipStream_t s) {
  const int zero = 0;
  launch_row_inv_batch<T, C>(in, 0, &zero, 1, out, 0, tw, g, tile_w, s);
}

template <typename T, typename C>
void launch_col(const Basis<cx<T>>& basis, cx<T>* zbase, size_t zsp, size_t zsi, cx<T>* dzbase, size_t dzsp,
                const PoleState* st, const RoundList& list, const double* mu_x, const double* mu_y, const cx<C>* tw,
                const Geo& g, const StencilCoef& sc, cx<T>* scratch, hipStream_t s) {
#define COLM_(NN, LB, MODE, ENTRIES, IN, OUT, OSP, OSI)                                                         \
  {                                                                                                            \
    dim3 grid(g.nx / ColCfg<T, C, NN, LB>::GC, g.ncomp * (ENTRIES));                                           \
    if (g.ncomp == 1)                                                                                          \
      hipLaunchKernelGGL((k_col<T, C, NN, 1, LB, MODE>), grid, dim3(ColCfg<T, C, NN, LB>::WG), 0, s, IN, OUT,  \
                         OSP, OSI, dzbase, dzsp, st, list, mu_x, mu_y, tw, g.fsz, sc);                         \
    else                                                                                                       \
      hipLaunchKernelGGL((k_col<T, C, NN, 2, LB, MODE>), grid, dim3(ColCfg<T, C, NN, LB>::WG), 0, s, IN, OUT,  \
                         OSP, OSI, dzbase, dzsp, st, list, mu_x, mu_y, tw, g.fsz, sc);                         \
  }
  // The poles of a round that all start from the shared first basis vector share its
  // forward transform (scratch: one R-domain field) where the storage keeps the transform's
  // precision and n poles save more than the launch and the field written and read again
  // cost.  First rounds, us, each pole its own transform -> shared:
  //   complex128, 2 to 5 poles: 1024^2 17.3 -> 20.3, 22.5 -> 24.6, 26.9 -> 27.0, 31.5 -> 30.7; 512^2
  //     vector with 5, 21.3 -> 22.3; 2048^2 vector with 3, 4, 5: 213 -> 228, 291 -> 292, 373 -> 348
  //   from 6 on: 768^2 24.6 -> 22.2, 1024^2 36.0 -> 33.8, 512^2 vector 24.0 -> 23.5, 1024^2 vector with
  //     8, 111 -> 92; scalar columns of 1536 and more from 12 on: 2048^2 with 8, 12, 16 177 -> 183,
  //     262 -> 253, 346 -> 340; 1536^2 with 8, 16 106 -> 109, 201 -> 198
  //   complex64: 2048^2 with 2, 3 53.6 -> 55.6, 76.5 -> 69.3; 1024^2 with 3, 22.8 -> 19.5
  //   below 2^21 elements over all poles: 256^2 with 16, 14.0 -> 14.8; 512^2 with 6, 13.8 -> 14.2 (with
  //     8, 15.7 -> 15.6; with 10, 18.6 -> 17.4)
  //   fewer than 256 columns: 64 x 2048 vector, complex64, 8 poles, 26.4 -> 28.8 (256 x 1024 scalar 18.2 -> 17.0)
  const int least = sizeof(C) == sizeof(float) ? 3 : (g.ncomp == 1 && g.ny >= 1536 ? 12 : 6);
  bool shared = scratch && sizeof(T) == sizeof(C) && list.n >= least && g.nx * g.ncomp >= 256 &&
                (size_t)list.n * g.ncomp * g.fsz >= (size_t)1 << 21;
  for (int a = 0; a < list.n && shared; ++a) shared = round_shared(list.e[a]) && round_m(list.e[a]) == 0;
  const Basis<cx<T>> once{scratch, nullptr, 0, 0};
#define COLV_(NN, LB)                                                                                          \
  {                                                                                                            \
    if constexpr (sizeof(T) == sizeof(C)) {                                                                    \
      if (shared) {                                                                                            \
        COLM_(NN, kColLds[0], COL_FORWARD, 1, basis, scratch, 0, 0)                                            \
        COLM_(NN, LB, COL_INVERSE, list.n, once, zbase, zsp, zsi)                                              \
        break;                                                                                                 \
      }                                                                                                        \
    }                                                                                                          \
    COLM_(NN, LB, COL_WHOLE, list.n, basis, zbase, zsp, zsi)                                                   \
  }
  // Complex128 vector fields with columns of 1024 and more take the largest budget in the
  // middle variant too: their pass writes twice what it reads, and one or two columns at a
  // time are a small part of each line.  It has to leave every CU a workgroup, though, and columns
  // of 1536, two at a time instead of one, lose from about 1024 workgroups on.  us a launch, 40 and
  // 80 KB: 2048^2 with 1, 4 poles 140 and 127, 613 and 526; 1024^2 with 4, 8 116 and 112, 221 and 214; 64 x 1024
  // with 2, 4, 8 (64, 128, 256 workgroups) 17.8 and 20.9, 18.6 and 21.7, 23.2 and 22.9; 128 x 2048 with 1 (128)
  // 20.2 and 23.1, 256 x 2048 (256) 26.6 and 24.3; columns of 1536, 64, 384 and 512 with 4, 2, 1 (256, 768, 512)
  // 23.4 and 22.1, 49.7 and 47.8, 35.3 and 32.3, 1536^2 with 1, 4 89.8 and 98.7, 321 and 350.  Shorter columns and
  // scalar fields: a step of 768 and 384 1.63 and 1.72 ms, 0.80 and 0.84, 1024^2 1.53 and 1.55;
  // complex64 storage 2-6 % more.
  auto wide = [&](int nn, int gc) {
    const size_t wgs = (size_t)(g.nx / gc) * g.ncomp * list.n;
    return g.ncomp == 2 && sizeof(T) == sizeof(double) && nn >= 1024 && wgs >= 256 && (nn != 1536 || wgs < 1024);
  };
#define L_(NN)                                                                                                 \
  {                                                                                                            \
    if (g.col_variant == 0)                                                                                    \
      COLV_(NN, kColLds[0])                                                                                    \
    else if (g.col_variant == 2 || wide(NN, ColCfg<T, C, NN, kColLds[2]>::GC))                                 \
      COLV_(NN, kColLds[2])                                                                                    \
    else                                                                                                       \
      COLV_(NN, kColLds[1])                                                                                    \
  }
  HP_DISPATCH_N(g.ny, L_)
#undef L_
#undef COLV_
#undef COLM_
}

static int apply_groups(const Geo& g) {
  const int nt = g.nx / 8;
  int groups = (apply_threads(g.nx) / nt) / g.ncomp * g.ncomp;
  if (groups < g.ncomp) groups = g.ncomp;
  return groups;
}

template <typename T>
int row_apply_blocks(const Geo& g) {
  const int rows = apply_groups(g) / g.ncomp;
  return (g.ny - 1 + rows - 1) / rows;
}

template <typename T, typename C>
void launch_row_apply(const cx<T>* zbase, size_t zsp, size_t zsi, const cx<T>* dzbase, size_t dzsp, cx<T>* pbase,
                      size_t psp, const Basis<cx<T>>& basis, const C* coef, const PoleState* st,
                      const RoundList& list, double2* part, const cx<C>* tw, const Geo& g, const StencilCoef& sc,
                      hipStream_t s) {
  const int nblk = row_apply_blocks<T>(g);
  // one workgroup per (row block, pole), row blocks padded to a multiple of 8
  dim3 grid((unsigned)((nblk + 7) / 8 * 8) * (unsigned)list.n);
  // The next vector's loads ahead up to 1024 workgroups, one for each SIMD (2048 with complex64
  // storage, half the bytes in flight); beyond, other waves hide the latency and the registers are
  // better spent on more of those.  The form changes no sum.  us per launch over a cycle, ahead and not: one pole 256^2 17.3 and 19.6, 384^2 17.4 and 20.1;
  // 16 poles 64^2 (128 workgroups) 15.8 and 18.0, 256^2 (2048) 59.0 and 58.3, 384^2 152 and 147, vector
  // 256^2 125 and 112, 384^2 303 and 283, 256 x 1024 352 and 317, 384 x 768 429 and 381; complex64, a
  // step of 256 x 128 (1024) 477 and 485, launches of 256^2 (2048) 25.4 and 25.1.
  const bool ahead = (size_t)nblk * list.n < (sizeof(T) == sizeof(float) ? 2048 : 1024);
#define R_(NN, NC, AH)                                                                                          \
  hipLaunchKernelGGL((k_row_apply<T, C, NN, NC, AH>), grid, dim3(ApplyCfg<NN, NC>::WG), 0, s, zbase, zsp, zsi,  \
                     dzbase, dzsp, pbase, psp, basis, coef, st, list, nblk, part, tw, g.ny, g.fsz, sc)
#define L_(NN)                                                                                                  \
  if (apply_ahead(NN) && ahead) {                                                                               \
    if (g.ncomp == 1)                                                                                           \
      R_(NN, 1, apply_ahead(NN));                                                                               \
    else                                                                                                        \
      R_(NN, 2, apply_ahead(NN));                                                                               \
  } else if (g.ncomp == 1)                                                                                      \
    R_(NN, 1, false);                                                                                           \
  else                                                                                                          \
    R_(NN, 2, false);
  HP_DISPATCH_N(g.nx, L_)
#undef R_
#undef L_
}

// Elements per thread of the update: one for fields of up to 384^2 elements, whose workgroups
// of four elements a thread leave CUs without work when one pole is left (64 of them at 256^2,
// 144 at 384^2), else four.  us, four -> one element, one pole and 16 (12 at 256^2): 256^2 5.8 -> 5.3
// and 11.9 -> 12.6, 384^2 6.1 -> 5.5 and 30.9 -> 30.5, 512 x 384 6.4 -> 6.0 and 41.4 -> 41.5, 512^2
// 7.1 -> 6.8 and 57.5 -> 58.7, 768 x 512 8.8 -> 8.4 and 90.2 -> 91.3: above 384^2 many poles lose more
// than one gains.  The rule looks at the field alone, so a pole's sums are the same whatever the
// other poles do.
static int update_elems(size_t total) { return total <= 384 * 384 ? 1 : 4; }

template <typename T>
void launch_update(const cx<T>* pbase, size_t psp, const Basis<cx<T>>& basis, const PoleState* st,
                   const RoundList& list, double* part, int nblk, const Geo& g, hipStream_t s) {
  const size_t total = (size_t)g.ncomp * g.fsz;
  if (update_elems(total) == 1)
    hipLaunchKernelGGL((k_update<T, 1>), dim3(nblk, list.n), dim3(UPD_WG), 0, s, pbase, psp, basis, st, list, part,
                       nblk, total);
  else
    hipLaunchKernelGGL((k_update<T, 4>), dim3(nblk, list.n), dim3(UPD_WG), 0, s, pbase, psp, basis, st, list, part,
                       nblk, total);
}

template <typename T>
void launch_final(const c128* w, c128* out, const cx<T>* zbase, size_t zsp, size_t zsi, const c128* xacc, size_t xsp,
                  const PoleState* st, int npoles, c128 phase, c128 rinf_phase, double loss_coef, double eta, int W,
                  const c128* tw64, const Geo& g, hipStream_t s) {
  dim3 grid(g.ny, g.ncomp);
  // Complex128 rows of 512 and more whose workgroups come in multiples of 1024, four for each CU: then
  // enough waves wait for memory with one load a thread, and more of them only spread the
  // requests (all of a term's -> one at a time, us: 1024^2 with 16 poles 254 -> 203, 2048^2 with 8 504 -> 426,
  // 512^2 vector 136 -> 116).  With fewer or a part of 1024 left over the chain counts: 2048 x 64
  // 165 -> 620, 1536^2 287 -> 340, 768^2 152 -> 164, 512^2 122 -> 155; complex64 1024^2 122 -> 165; shorter rows
  // 384 x 1024 vector 108 -> 115, 64 x 2048 vector 89 -> 116.  (Both forms sum in the same order.)
  const bool full = sizeof(T) == sizeof(double) && (g.ny * g.ncomp) % 1024 == 0;
#define F_(NN, FULL)                                                                                              \
  hipLaunchKernelGGL((k_final<T, NN, FULL>), grid, dim3(RowCfg<NN>::WG), 0, s, w, out, zbase, zsp, zsi, xacc, xsp, \
                     st, npoles, phase, rinf_phase, loss_coef, eta, W, tw64, g.nx, g.ny, g.fsz)
#define L_(NN)                                                 \
  if (full && NN >= 512)                                       \
    F_(NN, (NN >= 512 && sizeof(T) == sizeof(double)));        \
  else                                                         \
    F_(NN, false);
  HP_DISPATCH_N(g.nx, L_)
#undef F_
#undef L_
}

template <typename T>
void launch_accum_batch(c128* xacc, size_t xsp, const cx<T>* z, size_t zsp, size_t zsi, const PoleState* st,
                        const int* sel_h, int n, const Geo& g, hipStream_t s) {
  const size_t total = (size_t)g.ncomp * g.fsz;
  PoleList sel;
  sel.n = n;
  for (int a = 0; a < HP_MAXPOLES; ++a) sel.k[a] = a < n ? sel_h[a] : 0;
  const int nb = std::max(1, update_blocks(total) / n);
  hipLaunchKernelGGL((k_accum<T>), dim3(nb, n), dim3(256), 0, s, xacc, z, zsi, st, sel, xsp, zsp, total);
}

template <typename T>
void launch_accum(c128* xacc, const cx<T>* z, size_t zsi, const PoleState* st, int pole, const Geo& g,
                  hipStream_t s) {
  // xacc and z are pole k's already: a one-entry list with zero strides
  launch_accum_batch<T>(xacc, 0, z, 0, zsi, st, &pole, 1, g, s);
}

// explicit instantiations
#define HP_INST(T)                                                                                                   \
  template int row_blocks<T>(int);                                                                                   \
  template int row_apply_blocks<T>(const Geo&);                                                                      \
  template void launch_update<T>(const cx<T>*, size_t, const Basis<cx<T>>&, const PoleState*, const RoundList&,      \
                                 double*, int, const Geo&, hipStream_t);                                             \
  template void launch_final<T>(const c128*, c128*, const cx<T>*, size_t, size_t, const c128*, size_t,               \
                                const PoleState*, int, c128, c128, double, double, int, const c128*, const Geo&,     \
                                hipStream_t);                                                                        \
  template void launch_accum<T>(c128*, const cx<T>*, size_t, const PoleState*, int, const Geo&, hipStream_t);      \
  template void launch_accum_batch<T>(c128*, size_t, const cx<T>*, size_t, size_t, const PoleState*, const int*,     \
                                      int, const Geo&, hipStream_t);

// storage type T, compute type C of the transforms
#define HP_INST2(T, C)                                                                                               \
  template void launch_row_fwd<T, C>(const c128*, cx<T>*, double*, const cx<C>*, const Geo&, hipStream_t, int);      \
  template void launch_row_inv<T, C>(const cx<T>*, c128*, const cx<C>*, const Geo&, int, hipStream_t);               \
  template void launch_row_fwd_batch<T, C>(const c128*, size_t, const int*, cx<T>*, size_t, const int*, int,       \
                                           double*, size_t, const cx<C>*, const Geo&, hipStream_t, int);             \
  template void launch_row_inv_batch<T, C>(const cx<T>*, size_t, const int*, int, c128*, size_t, const cx<C>*,       \
                                           const Geo&, int, hipStream_t);                                            \
  template void launch_col<T, C>(const Basis<cx<T>>&, cx<T>*, size_t, size_t, cx<T>*, size_t, const PoleState*,      \
                                 const RoundList&, const double*, const double*, const cx<C>*, const Geo&,           \
                                 const StencilCoef&, cx<T>*, hipStream_t);                                           \
  template void launch_row_apply<T, C>(const cx<T>*, size_t, size_t, const cx<T>*, size_t, cx<T>*, size_t,           \
                                       const Basis<cx<T>>&, const C*, const PoleState*, const RoundList&, double2*,  \
                                       const cx<C>*, const Geo&, const StencilCoef&, hipStream_t);

// The build compiles this file once per part (a third of the time of one
// compilation); without HP_PART it is whole.
#if !defined(HP_PART) || HP_PART == 1
HP_INST2(double, double)
#endif
#if !defined(HP_PART) || HP_PART == 2
HP_INST2(float, float)
#endif
#if !defined(HP_PART) || HP_PART == 3
HP_INST2(float, double)
#endif
#if !defined(HP_PART) || HP_PART == 0
HP_INST(double)
HP_INST(float)

void launch_reduce_dots(const double2* part, int nparts, PoleState* st, const RoundList& list, hipStream_t s) {
  hipLaunchKernelGGL(k_reduce_dots, dim3(list.n), dim3(RED_WG), 0, s, part, nparts, st, list);
}

int update_blocks(size_t total) {
  const size_t chunk = (size_t)UPD_WG * update_elems(total);
  size_t b = (total + chunk - 1) / chunk;
  if (b > 2048) b = 2048;
  if (b < 1) b = 1;
  return (int)b;
}

void launch_arnoldi(PoleState* st, const RoundList& list, const double* part, int nblk, int restart,
                    unsigned long long* ftag, unsigned long long seq, double* est, hipStream_t s) {
  hipLaunchKernelGGL(k_arnoldi, dim3(list.n), dim3(ARN_WG), 0, s, st, list, part, nblk, restart, ftag, seq, est);
}

void launch_cycle_init(PoleState* st, const int* poles, int npoles_in, const double* part, int nblk, int first,
                       double tol, double rtol_cycle, hipStream_t s, size_t part_bs, int set_has_x) {
  PoleList sel;
  sel.n = npoles_in;
  for (int a = 0; a < HP_MAXPOLES; ++a) sel.k[a] = a < npoles_in ? poles[a] : 0;
  hipLaunchKernelGGL(k_cycle_init, dim3(npoles_in), dim3(64), 0, s, st, sel, part, nblk, first, tol, rtol_cycle,
                     part_bs, set_has_x);
}

int op_blocks(const Geo& g) { return ((g.nx + OP_TX - 1) / OP_TX) * ((g.ny + OP_TY - 1) / OP_TY); }

void launch_apply_op_batch(const c128* x, size_t xbs, const c128* rhs, c128* y, size_t ybs, const double* coef,
                           const c128* shifts_h, int n, const StencilCoef& sc, const Geo& g, double* part, size_t pbs,
                           hipStream_t s, int medium_only) {
  ShiftList sh;
  for (int a = 0; a < HP_MAXPOLES; ++a) sh.b[a] = a < n ? shifts_h[a] : mk(0.0, 0.0);
  const dim3 grid(op_blocks(g), 1, n);
  if (g.ncomp == 2)
    hipLaunchKernelGGL((k_apply_op<2>), grid, dim3(OP_WG), 0, s, x, rhs, y, coef, sh, sc, g.nx, g.ny, g.fsz, part,
                       medium_only, xbs, ybs, pbs);
  else
    hipLaunchKernelGGL((k_apply_op<1>), grid, dim3(OP_WG), 0, s, x, rhs, y, coef, sh, sc, g.nx, g.ny, g.fsz, part,
                       medium_only, xbs, ybs, pbs);
}

void launch_apply_op(const c128* x, const c128* rhs, c128* y, const double* coef, c128 b, const StencilCoef& sc,
                     const Geo& g, double* part, hipStream_t s, int medium_only) {
  launch_apply_op_batch(x, 0, rhs, y, 0, coef, &b, 1, sc, g, part, 0, s, medium_only);
}

void launch_coef(const double* n2, double* coef, double* scratch, double n0, double s_scale, int W,
                 const StencilCoef& sc, const Geo& g, hipStream_t s) {
  const int nb = (int)((g.fsz + 255) / 256);
  const int vector = g.ncomp == 2;
  hipLaunchKernelGGL(k_coef_a, dim3(nb), dim3(256), 0, s, n2, coef, scratch, n0, W, g.nx, g.ny, g.fsz, vector);
  if (vector) {
    hipLaunchKernelGGL(k_coef_b, dim3(nb), dim3(256), 0, s, scratch, scratch + g.fsz, sc, g.nx, g.ny, g.fsz);
    hipLaunchKernelGGL(k_coef_c, dim3(nb), dim3(256), 0, s, scratch, scratch + g.fsz, coef, s_scale, sc, W, g.nx,
                       g.ny, g.fsz);
  }
}

void launch_mark_list(PoleState* st, const int* poles, int n, hipStream_t s) {
  PoleList sel;
  sel.n = n;
  for (int a = 0; a < HP_MAXPOLES; ++a) sel.k[a] = a < n ? poles[a] : 0;
  hipLaunchKernelGGL(k_mark_list, dim3(1), dim3(HP_MAXPOLES), 0, s, st, sel);
}

void launch_mark_folded(PoleState* st, int first, int count, hipStream_t s) {
  hipLaunchKernelGGL(k_mark_folded, dim3(1), dim3(HP_MAXPOLES), 0, s, st, first, count);
}

__global__ void k_to_float(const double* __restrict__ a, float* __restrict__ b, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    b[i] = (float)a[i];
}

void launch_to_float(const double* a, float* b, size_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_to_float, dim3(2048), dim3(256), 0, s, a, b, n);
}

void launch_state_init(PoleState* st, const StateInit& h, int npoles, hipStream_t s) {
  hipLaunchKernelGGL(k_state_init, dim3(npoles), dim3(256), 0, s, st, h);
}

void launch_clear_rows(void* base, size_t planes, size_t plane_bytes, int ny, int row_bytes, hipStream_t s) {
  const size_t tile = (size_t)ny * row_bytes, tiles = planes * (plane_bytes / tile);
  const int words = row_bytes / 16;
  const size_t nb = std::min<size_t>(4096, (tiles * words + 255) / 256);
  hipLaunchKernelGGL(k_clear_rows, dim3((unsigned)nb), dim3(256), 0, s, reinterpret_cast<char*>(base), tiles, tile,
                     words);
}

void launch_spectrum_max(const SpectrumCheck& c, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_spectrum_max, dim3(kSpectrumBlocks), dim3(256), 0, s, c, out);
}

void launch_rk4_stage(const c128* L, const c128* acc_in, c128* acc_out, const c128* u, c128* v_out, double ca,
                      double cv, double loss_coef, double eta, int W, const Geo& g, hipStream_t s) {
  const unsigned total = (unsigned)(g.ncomp * g.fsz);
  const unsigned nb = std::min(2048u, (total + 1023u) / 1024u);
  hipLaunchKernelGGL(k_rk4_stage, dim3(nb), dim3(256), 0, s, L, acc_in, acc_out, u, v_out, ca, cv, loss_coef, eta, W,
                     g.nx, g.ny, (unsigned)g.fsz, total);
}

#endif  // part 0
