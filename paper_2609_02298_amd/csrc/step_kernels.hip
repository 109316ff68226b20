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
// What a workgroup of a batch step that runs no arc does.
enum { kWorkHold = 0, kWorkFace = 1, kWorkTile = 2 };

// A hold rectangle in tiles (empty: nx = 0).
struct TileRect {
  int tx0, ty0, nx, ny;
  __device__ bool has(int tx, int ty) const {
    return tx >= tx0 && tx < tx0 + nx && ty >= ty0 && ty < ty0 + ny;
  }
  __device__ int index(int tx, int ty) const { return (ty - ty0) * nx + tx - tx0; }
};

// What a workgroup knows of its case in this launch.
struct StepCase {
  const StepOneArgs &a;
  CaseState *cs;
  int cur;
  bool hold_all;  // no rectangles yet: every node counts (the first step of a batch's case)
  const int32_t *hold(int b) const { return cs->hold[cur][b]; }
};

__device__ __forceinline__ TileRect hold_rect(const StepCase &s, int b) {
  const StepOneArgs &a = s.a;
  TileRect r;
  if (s.hold_all) {
    r.tx0 = r.ty0 = 0;
    r.nx = a.lean.tiles_x;
    r.ny = a.lean.ntiles / a.lean.tiles_x;
    return r;
  }
  const int32_t *h = s.cs->hold[s.cur][b];
  const int x0 = ld_uniform(h), y0 = ld_uniform(h + 1), x1 = ld_uniform(h + 2), y1 = ld_uniform(h + 3);
  r.tx0 = x0 >> a.tx_shift;
  r.ty0 = y0 >> a.ty_shift;
  r.nx = max(0, (x1 >> a.tx_shift) - r.tx0 + 1);
  r.ny = max(0, (y1 >> a.ty_shift) - r.ty0 + 1);
  if (x1 < x0 || y1 < y0) r.nx = r.ny = 0;
  return r;
}

// Whether a hold rectangle reaches face nodes (columns 0, nx-2 and nx-1, rows
// 0 and ny-1): then the body's pass waits for the face nodes as well.
__device__ __forceinline__ bool hold_faces(const StepCase &s, int b) {
  const int32_t *h = s.cs->hold[s.cur][b];
  return s.hold_all || ld_uniform(h) < 1 || ld_uniform(h + 1) < 1 || ld_uniform(h + 2) > s.a.lean.nx - 3 ||
         ld_uniform(h + 3) > s.a.lean.ny - 2;
}

// This workgroup's updates are complete: count it for the bodies in mask.
// The tiles' updates are device-scope stores: once a wave's stores have
// completed (vmem_done) they are where the pass's loads look for them, so
// no release is needed.  (A release writes back every dirty line of the
// die's L2 beside the stream: from the last hold tile's end to the pass it
// took 7.6 us on the 2000 x 800 lattice, 1.8 us without.)  FENCE: for plain
// stores.
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

// A thread's nodes of tile (tx, ty): column x, rows y0, y0 + by, ... of the
// inner nodes.  Loads go through the nearest inner node where a row or column
// has none, so that they need no test.
struct TileThread {
  int x, y0;
  bool on;  // the column has inner nodes
};
__device__ __forceinline__ TileThread tile_thread(const StepOneArgs &a, int tx, int ty) {
  TileThread t;
  const int lx = threadIdx.x & (a.bx - 1), ly = threadIdx.x / a.bx;
  t.x = (tx << a.tx_shift) + lx;
  t.y0 = (ty << a.ty_shift) + ly;
  t.on = t.x >= 1 && t.x <= a.lean.nx - 3;
  t.x = max(1, min(a.lean.nx - 3, t.x));
  return t;
}
template <typename T>
__device__ __forceinline__ void load_node(const StepOneArgs &a, const T *__restrict__ src, int x, int y, T (&f)[9]) {
  const T *p = src + pop_node(x, max(1, min(a.lean.ny - 2, y)), a.lean.nseg);
#pragma unroll
  for (int i = 0; i < 9; i++) f[i] = p[i * kSeg];
}

// Collide and stream the thread's nodes; f: the populations of its first row,
// already loaded.  The next row's are loaded before this row's collision.
// MODE 1: nodes that may carry IB force, read and cleared; 2: none.
template <typename T, int COL, int MODE, bool AGENT>
__device__ __forceinline__ void tile_rows(const StepCase &s, const TileThread &t, T (&f)[9]) {
  #pragma clang fp contract(off)
  const StepOneArgs &a = s.a;
  const LeanArgs &l = a.lean;
  const T *__restrict__ src = (const T *)a.cd.f[s.cur];
  T *__restrict__ dst = (T *)a.cd.f[s.cur ^ 1];
  T *__restrict__ frc = (T *)l.force;
  const uint32_t plane = (uint32_t)l.nx * (uint32_t)l.ny;
  const int dxp = seg_dx_plus(t.x), dxm = seg_dx_minus(t.x), rs = l.nseg * kSegBlock;
  for (int r = 0; r < l.rpt; r++) {
    const int y = t.y0 + r * a.by;
    T g[9];
    if (r + 1 < l.rpt) load_node<T>(a, src, t.x, y + a.by, g);
    if (t.on && y >= 1 && y <= l.ny - 2) {
      T Fx = T(l.fluid_fx), Fy = T(l.fluid_fy);
      if (MODE == 1) {
        const uint32_t p = (uint32_t)y * l.nx + t.x;
        const T fa = frc[p], fb = frc[plane + p];
        if (fa != T(0) || fb != T(0)) {
          Fx += fa;
          Fy += fb;
          put<AGENT>(frc + p, T(0));
          put<AGENT>(frc + plane + p, T(0));
        }
      }
      collide<T, sizeof(T) == 4, COL>(f, Fx, Fy, l);
      push_inner<T, AGENT>(dst + pop_node(t.x, y, l.nseg), dxp, dxm, rs, f);
    }
    if (r + 1 < l.rpt) {
#pragma unroll
      for (int i = 0; i < 9; i++) f[i] = g[i];
    }
  }
}

template <typename T, int MODE, bool AGENT>
__device__ __forceinline__ void tile_any(const StepCase &s, const TileThread &t, T (&f)[9]) {
  const int col = s.a.cd.collision;
  if (col == kBGK) tile_rows<T, kBGK, MODE, AGENT>(s, t, f);
  else if (col == kTRT) tile_rows<T, kTRT, MODE, AGENT>(s, t, f);
  else tile_rows<T, kCMMRT, MODE, AGENT>(s, t, f);
}

// Slot `slot` of body b's rectangle (b >= 0), or tile t (b < 0) if no slot
// takes it.  FORCE: the bodies leave a force (not DFC).  The first row's
// populations are loaded before the words of the case state are looked at (a
// tile's own chain of round trips is what a launch waits for at four waves per
// SIMD).
template <typename T, bool FORCE>
__device__ __forceinline__ void step_tile(const StepCase &s, int b, int slot, int t) {
  const StepOneArgs &a = s.a;
  int tx, ty;
  if (b >= 0) {
    const TileRect r = hold_rect(s, b);
    if (slot >= r.nx * r.ny) return;
    tx = r.tx0 + slot % r.nx;
    ty = r.ty0 + slot / r.nx;
  } else {
    if (t >= a.lean.ntiles) return;
    tx = t % a.lean.tiles_x;
    ty = t / a.lean.tiles_x;
  }
  const TileThread th = tile_thread(a, tx, ty);
  T f[9];
  load_node<T>(a, (const T *)a.cd.f[s.cur], th.x, th.y0, f);
  // the bodies whose rectangle has the tile; the first one's slots take it,
  // or, past the last of them, the workgroup of the tile's own number
  uint32_t mask = 0;
  int taker = -1;
  for (int q = 0; q < a.cd.nbodies; q++) {
    const TileRect r = hold_rect(s, q);
    if (!r.has(tx, ty)) continue;
    if (!mask) taker = r.index(tx, ty) < a.hold_first[q + 1] - a.hold_first[q] ? q : -1;
    mask |= 1u << q;
  }
  if (b >= 0 ? taker != b : taker >= 0) return;
  // a halted case keeps its lattices as they are
  if (ld_uniform(&s.cs->halt[s.cur]) & kCaseHalted) return;
  if (!mask) {
    tile_any<T, 2, false>(s, th, f);
  } else {
    tile_any<T, (FORCE ? 1 : 2), true>(s, th, f);
    hold_count<false>(s.cs, mask);
  }
}

template <typename T, int COL, int FACE, bool FORCE>
__device__ __forceinline__ void step_face_node(const StepCase &s, int m) {
  #pragma clang fp contract(off)
  const CaseDesc &c = s.a.cd;
  const int nx = c.nx, ny = c.ny;
  if (m >= face_nodes(nx, ny)) return;
  int x, y;
  face_node_at(nx, ny, m, x, y);
  const T *__restrict__ src = (const T *)c.f[s.cur];
  const int64_t pn = pop_node(x, y, c.nseg);
  T f[9];
#pragma unroll
  for (int i = 0; i < 9; i++) f[i] = src[pn + i * kSeg];
  if constexpr (FACE == kFaceZou) {
    if (is_zou_he_wall(c, x, y)) {
      const int w = wall_index(nx, ny, x, y);
      if (!*wall_flag(c, s.cur, w)) zou_he_close<T>(c, src, x, y, f);
      *wall_flag(c, s.cur ^ 1, w) = 0;
    }
  }
  T Fx = T(c.fluid_fx), Fy = T(c.fluid_fy);
  if (FORCE) {
    bool in = false;
    for (int q = 0; q < c.nbodies; q++) {
      const int32_t *h = s.cs->hold[s.cur][q];
      in |= s.hold_all || (x >= ld_uniform(h) && y >= ld_uniform(h + 1) && x <= ld_uniform(h + 2) &&
                           y <= ld_uniform(h + 3));
    }
    node_force<T>((T *)c.force, (uint32_t)c.plane, (uint32_t)y * nx + x, x, y, in, 0, 0, nx, ny, Fx, Fy);
  }
  collide<T, sizeof(T) == 4, COL>(f, Fx, Fy, c);
  push_boundary9<T, FACE == kFaceZeroGrad>(s.a.c, (T *)c.f[s.cur ^ 1], x, y, f[0], f[1], f[2], f[3], f[4],
                                           f[5], f[6], f[7], f[8]);
}

template <typename T, int FACE, bool FORCE>
__device__ __forceinline__ void step_faces(const StepCase &s, int blk) {
  const StepOneArgs &a = s.a;
  if (ld_uniform(&s.cs->halt[s.cur]) & kCaseHalted) return;
  const int m = blk * (int)blockDim.x + (int)threadIdx.x;
  if (a.cd.collision == kBGK) step_face_node<T, kBGK, FACE, FORCE>(s, m);
  else if (a.cd.collision == kTRT) step_face_node<T, kTRT, FACE, FORCE>(s, m);
  else step_face_node<T, kCMMRT, FACE, FORCE>(s, m);
  uint32_t mask = 0;
  for (int q = 0; q < a.cd.nbodies; q++)
    if (hold_faces(s, q)) mask |= 1u << q;
  if (mask) hold_count<true>(s.cs, mask);
}

// Workgroups that body b's pass waits for.
__device__ __forceinline__ int hold_target(const StepCase &s, int b) {
  const TileRect r = hold_rect(s, b);
  return r.nx * r.ny + (hold_faces(s, b) ? s.a.nface : 0);
}

template <typename T, int FACE, bool DFC>
__global__ __launch_bounds__(DFC ? 512 : 1024) void step_one_kernel(const StepOneArgs a) {
  extern __shared__ double dyn[];
  __shared__ ArcShared sh;
  const StepCase s{a, (CaseState *)a.lean.state, a.cur, false};
  int b = blockIdx.x;
  if (b < a.narcs) {
    int body = 0;
    while (b >= a.arc_first[body + 1]) body++;
    CaseState *cs = s.cs;
    const int64_t step = cs->step;
    if (cs->flags & kCaseHalted) {
      // every later launch leaves the lattices alone, whichever it starts from
      if (b == 0 && threadIdx.x == 0) {
        cs->halt[0] = 1;
        cs->halt[1] = 1;
      }
      return;
    }
    arc_body<T, (DFC ? 2 : 1), FACE == kFaceZou>(a.cd, a.cd.bodies + body, step, a.cur,
                                                 b - a.arc_first[body], body, a.cd.nbodies,
                                                 hold_target(s, body), -1, dyn, sh);
    return;
  }
  b -= a.narcs;
  if (b < a.nhold) {
    int body = 0;
    while (b >= a.hold_first[body + 1]) body++;
    step_tile<T, !DFC>(s, body, b - a.hold_first[body], 0);
    return;
  }
  b -= a.nhold;
  if (b < a.nface) {
    step_faces<T, FACE, !DFC>(s, b);
    if (a.cd.nbodies == 0 && b == 0 && threadIdx.x == 0) {
      // no pass: nothing in the launch reads these
      s.cs->cur = a.cur ^ 1;
      s.cs->step = s.cs->step + 1;
    }
    return;
  }
  b -= a.nface;
  // neighbouring tiles on one XCD
  const int nfar = (int)gridDim.x - a.narcs - a.nhold - a.nface;
  step_tile<T, !DFC>(s, -1, 0, (b & 7) * (nfar >> 3) + (b >> 3));
}

// One step of every case of a batch: the arcs of all cases, then the tiles and
// face nodes as the work list orders them (hold slots, faces, tiles).  Which
// lattice a case starts from, and whether it is stepped at all, are words of
// its state that the previous launch left for this one (CaseState::ctl).
// Bound by the tiles: every workgroup starts with a chain of dependent loads
// (work entry, case, populations), which 16 waves per CU hide only in part.
// 12 cases (3.6 M nodes, all schemes and collisions, fp32): 130 us per step as
// one collide-stream and one face launch per collision model and two launches
// of the passes, 64 to 69 us so.  Large batches: see batch_tables.
template <typename T, int FACE>
__global__ __launch_bounds__(1024) void step_batch_kernel(const StepBatchArgs g) {
  extern __shared__ double dyn[];
  __shared__ ArcShared sh;
  int b = blockIdx.x;
  IbmSlot sl{-1, 0, 0, 0};
  int role = kWorkTile, ci;
  if (b < g.narcs) {
    sl = g.arcs[b];
    ci = sl.cas;
  } else {
    b -= g.narcs;
    role = b < g.nhold ? kWorkHold : (b < g.nhold + g.nface ? kWorkFace : kWorkTile);
    ci = ld_uniform(&g.work[b].cas);
    b = ld_uniform(&g.work[b].idx);
    if (ci < 0) return;
  }
  ci = __builtin_amdgcn_readfirstlane(ci);
  const StepOneArgs &a = g.cases[ci];
  CaseState *const cs = (CaseState *)a.lean.state;
  const int ctl = ld_uniform(&cs->ctl[g.par]);
  const StepCase s{a, cs, ctl & kCtlCur, !(ctl & kCtlHold)};
  // the workgroup that passes the control word of an idle or body-free case on
  const bool keeper = threadIdx.x == 0 && (sl.cas >= 0 ? sl.body == 0 && sl.arc == 0
                                                       : a.cd.nbodies == 0 && role == kWorkFace && b == 0);
  if (!(ctl & kCtlActive)) {
    if (keeper) cs->ctl[g.par ^ 1] = ctl;
    return;
  }
  if (sl.cas >= 0) {
    arc_body<T, 0, false>(a.cd, a.cd.bodies + sl.body, cs->step, s.cur, sl.arc, sl.body, sl.slots_in_case,
                          hold_target(s, sl.body), g.par, dyn, sh);
    return;
  }
  const bool force = a.cd.nbodies > 0 && a.cd.bodies[0].scheme != kDFC;
  if (role == kWorkFace) {
    if (force) step_faces<T, FACE, true>(s, b);
    else step_faces<T, FACE, false>(s, b);
    if (keeper) {
      const int64_t n = cs->step + 1;
      cs->cur = s.cur ^ 1;
      cs->step = n;
      cs->ctl[g.par ^ 1] = (s.cur ^ 1) | (n < cs->target ? kCtlActive : 0);
    }
    return;
  }
  int body = -1;
  if (role == kWorkHold) {
    body = 0;
    while (b >= a.hold_first[body + 1]) body++;
    b -= a.hold_first[body];
  }
  if (force) step_tile<T, true>(s, body, b, b);
  else step_tile<T, false>(s, body, b, b);
}

// The last case whose prefix does not exceed t.
__device__ __forceinline__ int find_case(const int32_t *prefix, int ncases, int t) {
  int lo = 0, hi = ncases - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (prefix[mid] <= t) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// The work list, once per composition of the batch.  (Searched by every
// workgroup of every step, the prefix sums' dependent loads cost 2.5 us of an
// 80 us step of 12 cases, 3.6 M nodes.)
__global__ void batch_work_kernel(const StepBatchArgs g) {
  int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= g.nwork) return;
  StepWork &w = g.work[b];
  const int32_t *prefix = g.hold_prefix;
  if (b >= g.nhold) {
    b -= g.nhold;
    prefix = g.face_prefix;
    if (b >= g.nface) {
      b -= g.nface;
      prefix = g.tile_prefix;
      // neighbouring tiles on one XCD
      const int n = g.nwork - g.nhold - g.nface;
      b = (b & 7) * (n >> 3) + (b >> 3);
      if (b >= g.ntile) {
        w.cas = -1;
        return;
      }
    }
  }
  w.cas = find_case(prefix, g.ncases, b);
  w.idx = b - prefix[w.cas];
}

__global__ void batch_control_kernel(const StepOneArgs *cases, int ncases) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ncases) return;
  CaseState *const cs = (CaseState *)cases[i].lean.state;
  cs->ctl[0] = cs->cur | (cs->step < cs->target && !(cs->flags & kCaseHalted) ? kCtlActive : 0) |
               (cs->step > 0 && cs->hold_step == cs->step ? kCtlHold : 0);
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

hipError_t launch_step_batch(int precision, int face, const StepBatchArgs &a, int threads, int lds_bytes,
                             hipStream_t stream) {
  if ((threads != 256 && threads != 512 && threads != 1024) || lds_bytes > 64 * 1024 || face == kFaceZou ||
      a.ncases <= 0 || a.nwork != a.nhold + a.nface + (a.ntile + 7) / 8 * 8)
    return hipErrorInvalidValue;
  const dim3 grid(a.narcs + a.nwork), block(threads);
#define IBL_BATCH(TT, FF) return issue(step_batch_kernel<TT, FF>, grid, block, lds_bytes, stream, nullptr, a)
  if (precision == kPrecFP64) {
    if (face == kFaceZeroGrad) IBL_BATCH(double, kFaceZeroGrad);
    IBL_BATCH(double, kFacePlain);
  }
  if (face == kFaceZeroGrad) IBL_BATCH(float, kFaceZeroGrad);
  IBL_BATCH(float, kFacePlain);
#undef IBL_BATCH
}

hipError_t launch_batch_work(const StepBatchArgs &a, hipStream_t stream) {
  return issue(batch_work_kernel, dim3((a.nwork + 255) / 256), dim3(256), 0, stream, nullptr, a);
}

hipError_t launch_batch_control(const StepOneArgs *cases, int ncases, hipStream_t stream) {
  return issue(batch_control_kernel, dim3((ncases + 255) / 256), dim3(256), 0, stream, nullptr, cases, ncases);
}

int step_max_waiting(int precision, int face, bool dfc, bool batch, int threads, int lds_bytes) {
  const void *k = nullptr;
#define IBL_PICK(TT, FF)                                                                       \
  k = batch ? (const void *)step_batch_kernel<TT, (FF == kFaceZou ? kFacePlain : FF)>           \
            : (dfc ? (const void *)step_one_kernel<TT, FF, true> : (const void *)step_one_kernel<TT, FF, false>)
  if (precision == kPrecFP64) {
    if (face == kFaceZou) IBL_PICK(double, kFaceZou);
    else if (face == kFaceZeroGrad) IBL_PICK(double, kFaceZeroGrad);
    else IBL_PICK(double, kFacePlain);
  } else {
    if (face == kFaceZou) IBL_PICK(float, kFaceZou);
    else if (face == kFaceZeroGrad) IBL_PICK(float, kFaceZeroGrad);
    else IBL_PICK(float, kFacePlain);
  }
#undef IBL_PICK
  int per = 0, dev = 0, ncu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k, threads, lds_bytes) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return per > 0 ? ncu * 3 / 4 : 0;
}

}  // namespace iblbm
