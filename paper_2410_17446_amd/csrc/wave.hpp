// Wave-level (64-lane) reductions and scans of the FP64 and FP32 kernels.
//
// They move data with DPP register moves instead of __shfl (ds_bpermute): a
// move is a VALU instruction of the same wave, without the LDS round trip that
// made the shuffles the longest chain of the row pass's inner products.
#pragma once
#include "cplx.hpp"

// v of the lane the DPP control CTRL selects; lanes without a source (and rows
// masked out by RMASK) get 0.
template <int CTRL, int RMASK = 0xf>
__device__ __forceinline__ int dpp_mov(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, RMASK, 0xf, true);
}
template <int CTRL, int RMASK = 0xf>
__device__ __forceinline__ float dpp_mov(float v) {
  return __int_as_float(dpp_mov<CTRL, RMASK>(__float_as_int(v)));
}
template <int CTRL, int RMASK = 0xf>
__device__ __forceinline__ double dpp_mov(double v) {
  return __hiloint2double(dpp_mov<CTRL, RMASK>(__double2hiint(v)), dpp_mov<CTRL, RMASK>(__double2loint(v)));
}

// DPP controls
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E;         // quad_perm [1,0,3,2], [2,3,0,1]
constexpr int DPP_SHR = 0x110, DPP_ROR = 0x120;         // + n: row (16 lanes) shift right, rotate right
constexpr int DPP_BCAST15 = 0x142, DPP_BCAST31 = 0x143; // last lane of a row / of two rows to the next ones

// Sums of four values over the wave: lane l returns the sum of v[l & 3].  Two
// exchanges inside each quad leave one value per lane (a reduction of four
// separate values would take four times the steps), then rows and the wave.
__device__ __forceinline__ double wave_sum4(double v0, double v1, double v2, double v3) {
  const int lane = threadIdx.x & 63;
  const bool b0 = lane & 1, b1 = lane & 2;
  double a = b0 ? v1 : v0, b = b0 ? v0 : v1;
  double c = b0 ? v3 : v2, d = b0 ? v2 : v3;
  a += dpp_mov<DPP_XOR1>(b);
  c += dpp_mov<DPP_XOR1>(d);
  double r = b1 ? c : a, s = b1 ? a : c;
  r += dpp_mov<DPP_XOR2>(s);
  r += dpp_mov<DPP_ROR + 4>(r);
  r += dpp_mov<DPP_ROR + 8>(r);
  r += __shfl_xor(r, 16, 64);
  r += __shfl_xor(r, 32, 64);
  return r;
}

// Inclusive prefix sum over aligned groups of W lanes (8, 16, 32 or 64).
template <typename T, int W>
__device__ __forceinline__ T lane_scan(T v) {
  static_assert(W == 8 || W == 16 || W == 32 || W == 64, "scan width");
  const int l = threadIdx.x & 15;
  // the row shifts fill with 0 at the start of a row; groups of 8 need the mask
  T x = dpp_mov<DPP_SHR + 1>(v);
  v += (W == 8 && (l & 7) < 1) ? (T)0 : x;
  x = dpp_mov<DPP_SHR + 2>(v);
  v += (W == 8 && (l & 7) < 2) ? (T)0 : x;
  x = dpp_mov<DPP_SHR + 4>(v);
  v += (W == 8 && (l & 7) < 4) ? (T)0 : x;
  if constexpr (W >= 16) v += dpp_mov<DPP_SHR + 8>(v);
  if constexpr (W >= 32) v += dpp_mov<DPP_BCAST15, 0xa>(v);
  if constexpr (W >= 64) v += dpp_mov<DPP_BCAST31, 0xc>(v);
  return v;
}
