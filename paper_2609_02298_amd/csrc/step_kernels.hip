// One launch per time step (gfx950): every tile, the face nodes and the
// immersed-boundary pass of all bodies (step_one_kernel).
//
// What the pass of a body reads and writes concerns only the nodes of its hold
// rectangle (CaseState::hold, left by the previous step's pass: the support of
// this step widened by two nodes, and the nodes carrying the previous force).
// Workgroups that update such nodes count themselves on the case state; the
// arcs of the body wait for that count and then run beside the other tiles.
// Consecutive steps are ordered by the stream alone, so a step costs one
// launch, with no second stream, events or gaps.  Everything a tile reads from
// the case state (hold rectangles, halt) is kept twice, by the step's input
// lattice, because the pass of the same launch already writes the next step's.
#include "arc_device.h"
#include "ib_lbm_internal.h"
#include "lbm_device.h"

namespace iblbm {

// Face closures present (the kernel instance): the usual ones with
// zero-gradient on the east face only, general zero-gradient, Zou-He walls.
enum { kFacePlain = 0, kFaceZeroGrad = 1, kFaceZou = 2 };

// A hold rectangle in tiles (empty: nx = 0).
struct TileRect {
  int tx0, ty0, nx, ny;
  __device__ bool has(int tx, int ty) const {
    return tx >= tx0 && tx < tx0 + nx && ty >= ty0 && ty < ty0 + ny;
  }
  __device__ int index(int tx, int ty) const { return (ty - ty0) * nx + tx - tx0; }
};

__device__ __forceinline__ TileRect hold_rect(const StepOneArgs &a, const int32_t *h) {
  const int x0 = ld_uniform(h), y0 = ld_uniform(h + 1), x1 = ld_uniform(h + 2), y1 = ld_uniform(h + 3);
  TileRect r;
  r.tx0 = x0 >> a.tx_shift;
  r.ty0 = y0 >> a.ty_shift;
  r.nx = max(0, (x1 >> a.tx_shift) - r.tx0 + 1);
  r.ny = max(0, (y1 >> a.ty_shift) - r.ty0 + 1);
  if (x1 < x0 || y1 < y0) r.nx = r.ny = 0;
  return r;
}

// Whether a hold rectangle reaches face nodes (columns 0, nx-2 and nx-1, rows
// 0 and ny-1): then the body's pass waits for the face nodes as well.
__device__ __forceinline__ bool hold_faces(const StepOneArgs &a, const int32_t *h) {
  return ld_uniform(h) < 1 || ld_uniform(h + 1) < 1 || ld_uniform(h + 2) > a.lean.nx - 3 ||
         ld_uniform(h + 3) > a.lean.ny - 2;
}

// This workgroup's updates are complete: count it for the bodies in mask.
// The tiles' updates are device-scope stores: once a wave's stores have
// completed (vmem_done) they are where the pass's loads look for them, so
// no release is needed.  (A release writes back every dirty line of the
// die's L2 beside the stream: from the last hold tile's end to the pass it
// took 7.6 us on the 2000 x 800 lattice.)  FENCE: for plain stores.
template <bool FENCE>
__device__ __forceinline__ void hold_count(CaseState *cs, uint32_t mask) {
  vmem_done();
  __syncthreads();
  if (threadIdx.x == 0) {
    if (FENCE) __threadfence();
    for (; mask; mask &= mask - 1)
      __hip_atomic_fetch_add(&cs->hold_done[__ffs(mask) - 1], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

template <typename T, int MODE, bool AGENT>
__device__ __forceinline__ void tile_any(const StepOneArgs &a, int tx, int ty) {
  const int lx = threadIdx.x & (a.bx - 1), ly = threadIdx.x / a.bx;
  if (a.cd.collision == kBGK) lean_tile<T, kBGK, MODE, AGENT>(a.lean, tx, ty, lx, ly, a.bx, a.by);
  else if (a.cd.collision == kTRT) lean_tile<T, kTRT, MODE, AGENT>(a.lean, tx, ty, lx, ly, a.bx, a.by);
  else lean_tile<T, kCMMRT, MODE, AGENT>(a.lean, tx, ty, lx, ly, a.bx, a.by);
}

// Tile t of the launch's order: slot `slot` of body b's rectangle (b >= 0), or
// any tile (b < 0) that no slot takes.
template <typename T, bool DFC>
__device__ __forceinline__ void step_tile(const StepOneArgs &a, int b, int slot, int t) {
  const int32_t (*hold)[4] = a.lean.state->hold[a.cur];
  int tx, ty;
  if (b >= 0) {
    const TileRect r = hold_rect(a, hold[b]);
    if (slot >= r.nx * r.ny) return;
    tx = r.tx0 + slot % r.nx;
    ty = r.ty0 + slot / r.nx;
  } else {
    if (t >= a.lean.ntiles) return;
    tx = t % a.lean.tiles_x;
    ty = t / a.lean.tiles_x;
  }
  // the bodies whose rectangle has the tile; the first one's slots take it,
  // or, past the last of them, the workgroup of the tile's own number
  uint32_t mask = 0;
  int taker = -1;
  for (int q = 0; q < a.cd.nbodies; q++) {
    const TileRect r = hold_rect(a, hold[q]);
    if (!r.has(tx, ty)) continue;
    if (!mask) taker = r.index(tx, ty) < a.hold_first[q + 1] - a.hold_first[q] ? q : -1;
    mask |= 1u << q;
  }
  if (b >= 0 ? taker != b : taker >= 0) return;
  if (!mask) tile_any<T, 2, false>(a, tx, ty);
  else tile_any<T, (DFC ? 2 : 1), true>(a, tx, ty);
  if (mask && !(ld_uniform(a.lean.halt) & kCaseHalted)) hold_count<false>((CaseState *)a.lean.state, mask);
}

template <typename T, int COL, int FACE, bool DFC>
__device__ __forceinline__ void step_face_node(const StepOneArgs &a, int m) {
  #pragma clang fp contract(off)
  const CaseDesc &c = a.cd;
  const int nx = c.nx, ny = c.ny;
  if (m >= face_nodes(nx, ny)) return;
  int x, y;
  face_node_at(nx, ny, m, x, y);
  const T *__restrict__ src = (const T *)c.f[a.cur];
  const int64_t pn = pop_node(x, y, c.nseg);
  T f[9];
#pragma unroll
  for (int i = 0; i < 9; i++) f[i] = src[pn + i * kSeg];
  if constexpr (FACE == kFaceZou) {
    if (is_zou_he_wall(c, x, y)) {
      uint8_t *const w = c.wall_closed + wall_index(nx, ny, x, y);
      if (*w) *w = 0;
      else if (a.zh_fold) zou_he_close<T>(c, src, x, y, f);
    }
  }
  T Fx = T(c.fluid_fx), Fy = T(c.fluid_fy);
  if (!DFC) {
    const int32_t (*hold)[4] = c.state->hold[a.cur];
    bool in = false;
    for (int q = 0; q < c.nbodies; q++)
      in |= x >= ld_uniform(hold[q]) && y >= ld_uniform(hold[q] + 1) && x <= ld_uniform(hold[q] + 2) &&
            y <= ld_uniform(hold[q] + 3);
    node_force<T>((T *)c.force, (uint32_t)c.plane, (uint32_t)y * nx + x, x, y, in, 0, 0, nx, ny, Fx, Fy);
  }
  collide<T, sizeof(T) == 4, COL>(f, Fx, Fy, c);
  push_boundary9<T, FACE == kFaceZeroGrad>(a.c, (T *)c.f[a.cur ^ 1], x, y, f[0], f[1], f[2], f[3], f[4],
                                           f[5], f[6], f[7], f[8]);
}

template <typename T, int FACE, bool DFC>
__device__ __forceinline__ void step_faces(const StepOneArgs &a, int blk) {
  CaseState *const cs = (CaseState *)a.lean.state;
  if (ld_uniform(a.lean.halt) & kCaseHalted) return;
  const int m = blk * (int)blockDim.x + (int)threadIdx.x;
  if (a.cd.collision == kBGK) step_face_node<T, kBGK, FACE, DFC>(a, m);
  else if (a.cd.collision == kTRT) step_face_node<T, kTRT, FACE, DFC>(a, m);
  else step_face_node<T, kCMMRT, FACE, DFC>(a, m);
  uint32_t mask = 0;
  for (int q = 0; q < a.cd.nbodies; q++)
    if (hold_faces(a, cs->hold[a.cur][q])) mask |= 1u << q;
  if (mask) hold_count<true>(cs, mask);
  if (a.cd.nbodies == 0 && blk == 0 && threadIdx.x == 0) {
    // no pass: nothing in the launch reads these
    cs->cur = a.cur ^ 1;
    cs->step = cs->step + 1;
  }
}

template <typename T, int FACE, bool DFC>
__global__ __launch_bounds__(DFC ? 512 : 1024) void step_one_kernel(const StepOneArgs a) {
  extern __shared__ double dyn[];
  __shared__ ArcShared sh;
  int b = blockIdx.x;
  if (b < a.narcs) {
    int body = 0;
    while (b >= a.arc_first[body + 1]) body++;
    const CaseState *cs = a.lean.state;
    const int64_t step = cs->step;
    if (cs->flags & kCaseHalted) {
      // every later launch leaves the lattices alone, whichever it starts from
      if (b == 0 && threadIdx.x == 0) {
        ((CaseState *)cs)->halt[0] = 1;
        ((CaseState *)cs)->halt[1] = 1;
      }
      return;
    }
    const int32_t *h = cs->hold[a.cur][body];
    const TileRect r = hold_rect(a, h);
    const int n = r.nx * r.ny + (hold_faces(a, h) ? a.nface : 0);
    arc_body<T, (DFC ? 2 : 1), FACE == kFaceZou>(a.cd, a.cd.bodies[body], step, a.cur,
                                                 b - a.arc_first[body], body, a.cd.nbodies, n, dyn, sh);
    return;
  }
  b -= a.narcs;
  if (b < a.nhold) {
    int body = 0;
    while (b >= a.hold_first[body + 1]) body++;
    step_tile<T, DFC>(a, body, b - a.hold_first[body], 0);
    return;
  }
  b -= a.nhold;
  if (b < a.nface) {
    step_faces<T, FACE, DFC>(a, b);
    return;
  }
  b -= a.nface;
  // neighbouring tiles on one XCD
  const int nfar = (int)gridDim.x - a.narcs - a.nhold - a.nface;
  step_tile<T, DFC>(a, -1, 0, (b & 7) * (nfar >> 3) + (b >> 3));
}

hipError_t launch_step_one(int precision, int face, bool dfc, const StepOneArgs &a, int threads,
                           int lds_bytes, hipStream_t stream) {
  if ((threads != 256 && threads != 512 && threads != 1024) || (dfc && threads > 512) ||
      a.bx * a.by != threads || (1 << a.tx_shift) != a.bx || (1 << a.ty_shift) != a.by * a.lean.rpt ||
      lds_bytes > 64 * 1024)
    return hipErrorInvalidValue;
  const int nfar = (a.lean.ntiles + 7) / 8 * 8;
  const dim3 grid(a.narcs + a.nhold + a.nface + nfar), block(threads);
#define IBL_ONE(TT, FF)                                                                                 \
  return dfc ? issue(step_one_kernel<TT, FF, true>, grid, block, lds_bytes, stream, nullptr, a)         \
             : issue(step_one_kernel<TT, FF, false>, grid, block, lds_bytes, stream, nullptr, a)
  if (precision == kPrecFP64) {
    if (face == kFaceZou) IBL_ONE(double, kFaceZou);
    if (face == kFaceZeroGrad) IBL_ONE(double, kFaceZeroGrad);
    IBL_ONE(double, kFacePlain);
  }
  if (face == kFaceZou) IBL_ONE(float, kFaceZou);
  if (face == kFaceZeroGrad) IBL_ONE(float, kFaceZeroGrad);
  IBL_ONE(float, kFacePlain);
#undef IBL_ONE
}

}  // namespace iblbm
