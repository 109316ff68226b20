// Device helpers shared by the kernels of the immersed-boundary pass: the
// regularized delta, wave and workgroup reductions in a fixed order, lane
// groups of a marker, and global-address-space views.
#pragma once
#include "ib_lbm_internal.h"

namespace iblbm {

static __constant__ int c_exi[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
static __constant__ int c_eyi[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
// opposite direction, a compile-time function so that unrolled loops index
// register arrays with constants
__device__ __forceinline__ constexpr int opp_of(int i) {
  return i == 0 ? 0 : (i <= 4 ? ((i + 1) & 3) + 1 : ((i - 3) & 3) + 5);
}
static __constant__ double c_w[9] = {4.0 / 9.0,  1.0 / 9.0,  1.0 / 9.0,  1.0 / 9.0, 1.0 / 9.0,
                              1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0};

// Regularized delta kernels: hat (Eq. 9) and Peskin 4-point (Eq. 10).
__device__ __forceinline__ double delta1(int kernel, double r) {
  const double a = fabs(r);
  if (kernel == kHat) return a < 1.0 ? 1.0 - a : 0.0;
  if (a <= 1.0) return 0.125 * (3.0 - 2.0 * a + sqrt(1.0 + 4.0 * a - 4.0 * a * a));
  if (a <= 2.0) return 0.125 * (5.0 - 2.0 * a - sqrt(-7.0 + 12.0 * a - 4.0 * a * a));
  return 0.0;
}

// A device-memory pointer the compiler cannot place by itself (one read
// from a descriptor) makes generic (flat) accesses, and a flat access also
// counts as an LDS operation: the next LDS wait or barrier of the wave then
// waits until a flat store has reached the cache, a long round trip beside
// a chip-wide stream.  Stores on the IB pass's late path go through this
// global-address-space view instead.
template <typename T>
using gmem = __attribute__((address_space(1))) T;
template <typename T>
__device__ __forceinline__ gmem<T> *to_global(T *p) {
  return (gmem<T> *)p;
}

// ---- fixed-order block reductions (wave64 shuffles, then LDS) ----
// A double moved across lanes by a DPP pattern (both 32-bit halves).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ __forceinline__ double lane_f64(double v, int lane) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// Wave64 sum and maximum with every lane active: within each row of 16
// lanes a fixed tree of lane exchanges (pairs, pairs of pairs, half-row
// mirror, row mirror; each step leaves the same value in both partners, as
// IEEE addition commutes), then the four row totals in a fixed order.
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_f64<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_f64<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_f64<0x141>(v);  // row_half_mirror
  v += dpp_f64<0x140>(v);  // row_mirror
  return (lane_f64(v, 0) + lane_f64(v, 16)) + (lane_f64(v, 32) + lane_f64(v, 48));
}
__device__ __forceinline__ double wave_max(double v) {
  v = fmax(v, dpp_f64<0xB1>(v));
  v = fmax(v, dpp_f64<0x4E>(v));
  v = fmax(v, dpp_f64<0x141>(v));
  v = fmax(v, dpp_f64<0x140>(v));
  return fmax(fmax(lane_f64(v, 0), lane_f64(v, 16)), fmax(lane_f64(v, 32), lane_f64(v, 48)));
}
// Sums a, b, c, d and maxima m1, m2 over the workgroup, each in a fixed
// order: wave totals, then the wave totals (one lane of wave 0 each) by the
// same wave tree.  The results are valid in the threads of wave 0.
// Threads at or past `nlive` must hold a = b = c = d = +0 and maxima that are
// 0 or held by a live thread as well (all values are non-negative): a wave
// with no live thread writes those totals without reducing them, which is
// what its tree would give.  On the IB pass's one compute unit the FP64
// wave reductions of sixteen waves compete for four SIMDs.
__device__ __forceinline__ void block_reduce6(double &a, double &b, double &c, double &d, double &m1,
                                              double &m2, double *red, int nlive) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  if (wv * 64 < nlive) {
    a = wave_sum(a); b = wave_sum(b); c = wave_sum(c); d = wave_sum(d);
    m1 = wave_max(m1); m2 = wave_max(m2);
  } else {
    a = 0.0; b = 0.0; c = 0.0; d = 0.0; m1 = 0.0; m2 = 0.0;
  }
  // (red is used once per pass, so nothing earlier needs a barrier here)
  if (lane == 0) {
    red[6 * wv] = a; red[6 * wv + 1] = b; red[6 * wv + 2] = c; red[6 * wv + 3] = d;
    red[6 * wv + 4] = m1; red[6 * wv + 5] = m2;
  }
  __syncthreads();
  if (wv == 0) {
    const bool in = lane < nw;
    const double *r = red + 6 * min(lane, nw - 1);
    a = wave_sum(in ? r[0] : 0.0);
    b = wave_sum(in ? r[1] : 0.0);
    c = wave_sum(in ? r[2] : 0.0);
    d = wave_sum(in ? r[3] : 0.0);
    m1 = wave_max(in ? r[4] : -1e300);
    m2 = wave_max(in ? r[5] : -1e300);
  }
}

// Marker loops run LPM lanes per marker (2, or 4 in the 1024-thread kernel
// with Peskin 4-point): lanes m*LPM .. m*LPM+LPM-1 of a wave share marker
// k, lane h sums the stencil rows [h NS/LPM, (h+1) NS/LPM) and group_sum
// adds the partial sums of the group with DPP quad permutations (lanes
// 0<->1, 2<->3, then 0,1<->2,3 of every quad).  IEEE addition commutes, so
// every lane of a group holds the same total.  All lanes of a group are
// always active together (the loops over LPM nb entries step by a block
// size that is a multiple of LPM).
template <int LPM>
__device__ __forceinline__ double group_sum(double v) {
  if (LPM >= 2) v += dpp_f64<0xB1>(v);  // quad_perm [1,0,3,2]
  if (LPM >= 4) v += dpp_f64<0x4E>(v);  // quad_perm [2,3,0,1]
  return v;
}

}  // namespace iblbm
