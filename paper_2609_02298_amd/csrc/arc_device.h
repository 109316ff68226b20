// The immersed-boundary pass of a body cut into arcs: one workgroup per arc
// of consecutive markers, no support tables.
//
// A marker's stencil lies on NS adjacent lanes (lane h of local marker m is
// thread m NS + h), each lane holding a strip of NS nodes in registers, a row of
// the stencil or a column (see COLS): it loads their populations, forms their moments and its strip's part of the interpolation, and
// DPP adds join the strips.  Markers whose stencils share a
// node are at most `bw` apart along the circle (plan_arcs), so an arc works on
// its own markers plus a margin on either side ("local" markers): bw for DF,
// 2 bw for DFC, N bw for N marker-space MDF passes, whose results are exact on
// all but bw more markers per pass.  Arcs therefore need nothing from each other
// while they run; only the force sums meet (arc_part / arrived), and DFC, which
// corrects the populations in place, once between its reads and its writes
// (arc_sync).  A body of few markers is one arc that wraps around.
//
// Spreading stays a gather in marker order: a lane sums, for each of its strip's
// nodes, the local markers covering it from the first along the circle to
// the last, and the lane of the first marker writes the node.  Each support
// node has exactly one such lane over all arcs.
//
// The pass is bound by latency and instruction issue, not bytes (a few hundred
// nodes per arc): the tables this form does without took most of a moving
// body's pass (their build: row intervals, scans, node lists), one workgroup per
// body the rest.  Whole steps, one workgroup with tables and now: fixed 2000 x
// 800 MDF P4 fp32 27.7 and 22.0 us, oscillating 1200 x 600 MDF P4 41 and 19.6,
// settling 400 x 2000 DFC P4 fp64 55.5 and 22.3, settling 1281 x 3841 DF P4 (a
// workspace in device memory before) 254 and 67.
#pragma once
#include "ib_lbm_internal.h"
#include "ibm_device.h"
#include "lbm_device.h"

namespace iblbm {

// A body's description as the passes read it: no kernel writes it, so it goes
// through the scalar data cache into scalar registers.  As ordinary memory it
// had to be loaded again, lane by lane, after every store that might have
// changed it: a round trip each on the pass's chain, or registers to keep it.
using ConstBody = const __attribute__((address_space(4))) BodyDesc;

// Kinematics of a body over one step.
struct Kin {
  double xc, yc, vhx, vhy, omh;  // position and (half-step) velocity of the step
  double udx, udy, udo;          // rigid velocity the markers are driven to
  double dimx, dimy;             // internal-mass force held over the step
  double vx0, vy0, om0;          // full-step velocity before the step
};

// Fixed, prescribed sine, the half-kick and drift of the Velocity-Verlet
// update (Eq. 23 / A3) or the Euler-explicit update (Eq. A1), from the state
// bs of the last completed step, for the step from time level `step`.
template <typename BODY>
__device__ __forceinline__ Kin body_kinematics(const CaseDesc &c, BODY &B,
                                               const BodyState *bs, int64_t step) {
  Kin k;
  k.xc = bs->xc;
  k.yc = bs->yc;
  k.vhx = k.vhy = k.omh = k.dimx = k.dimy = 0.0;
  k.vx0 = bs->vx;
  k.vy0 = bs->vy;
  k.om0 = bs->om;
  if (B.motion == kPrescribedSin) {
    const double t1 = (double)(step + 1);
    const double ph = 2.0 * M_PI * B.freq * t1 + B.phase;
    const double sn = sin(ph), cn = cos(ph);
    k.xc = B.xc0 + B.amp[0] * sn;
    k.yc = B.yc0 + B.amp[1] * sn;
    k.vhx = B.amp[0] * 2.0 * M_PI * B.freq * cn;
    k.vhy = B.amp[1] * 2.0 * M_PI * B.freq * cn;
  } else if (B.motion == kFree && B.integrator == kEulerA1) {
    // v^(n+1) = (1 + r) v^n - r v^(n-1) + (F^n + F_g)/m_s with r = m_f/m_s
    // (0 without internal mass); the rotation carries the rigid interior's
    // angular-momentum increment in both arms
    const double r = B.internal_mass == kImFeng ? B.mf / B.ms : 0.0;
    const double q = B.mf / B.ms;
    const double fgx = (B.ms - B.mf) * c.grav_x, fgy = (B.ms - B.mf) * c.grav_y;
    k.vhx = (1.0 + r) * bs->vx - r * bs->vpx + (bs->fhx + fgx) / B.ms;
    k.vhy = (1.0 + r) * bs->vy - r * bs->vpy + (bs->fhy + fgy) / B.ms;
    k.omh = (1.0 + q) * bs->om - q * bs->omp + bs->torque / B.Is;
    k.xc += k.vhx;
    k.yc += k.vhy;
  } else if (B.motion == kFree) {
    const double fgx = (B.ms - B.mf) * c.grav_x, fgy = (B.ms - B.mf) * c.grav_y;
    if (B.internal_mass == kImFeng) {
      k.dimx = B.mf * (bs->vx - bs->vpx);
      k.dimy = B.mf * (bs->vy - bs->vpy);
    }
    k.vhx = bs->vx + (bs->fhx + fgx + k.dimx) / (2.0 * B.ms);
    k.vhy = bs->vy + (bs->fhy + fgy + k.dimy) / (2.0 * B.ms);
    k.xc += k.vhx;
    k.yc += k.vhy;
    k.omh = bs->om + bs->torque / (2.0 * B.Is);
  }
  // under Velocity-Verlet the markers are driven to the last full-step
  // velocity (the half-step values only advance the position: with them the
  // torque-only rotation would feed back on itself near neutral buoyancy)
  const bool verlet = B.motion == kFree && B.integrator != kEulerA1;
  k.udx = verlet ? bs->vx : k.vhx;
  k.udy = verlet ? bs->vy : k.vhy;
  k.udo = verlet ? bs->om : k.omh;
  return k;
}

// 1D weights of the NS nodes around coordinate X (first node floor(X) - (NS/2
// - 1)).  With r = X - floor(X) and q = sqrt(1 + 4 r (1 - r)) the Peskin
// 4-point values at distances 1 + r, r, 1 - r, 2 - r are (3 - 2r - q)/8,
// (3 - 2r + q)/8, (1 + 2r + q)/8, (1 + 2r - q)/8: one root for the four.
template <int NS>
__device__ __forceinline__ void row_weights(double X, double (&w)[NS]) {
  const double r = X - floor(X);
  if constexpr (NS == 2) {
    w[0] = 1.0 - r;
    w[1] = r;
  } else {
    const double q = sqrt(1.0 + 4.0 * r * (1.0 - r));
    const double a = 3.0 - 2.0 * r, b = 1.0 + 2.0 * r;
    w[0] = 0.125 * (a - q);
    w[1] = 0.125 * (a + q);
    w[2] = 0.125 * (b + q);
    w[3] = 0.125 * (b - q);
  }
}

// The nine populations of the NS nodes (x0.., y): one vector load per
// population (NS values, aligned to one value) unless the row crosses a
// segment of the lattice's storage.
template <typename T, int NS>
__device__ __forceinline__ void load_pop_row(const T *__restrict__ f, int x0, int y, int nseg,
                                             T (&v)[9][NS]) {
  if ((x0 & (kSeg - 1)) <= kSeg - NS) {
    const T *p = f + pop_node(x0, y, nseg);
#pragma unroll
    for (int i = 0; i < 9; i++) __builtin_memcpy(v[i], p + i * kSeg, NS * sizeof(T));
  } else {
#pragma unroll
    for (int j = 0; j < NS; j++) {
      const T *p = f + pop_node(x0 + j, y, nseg);
#pragma unroll
      for (int i = 0; i < 9; i++) v[i][j] = p[i * kSeg];
    }
  }
}

// The 4 x 4 transpose within each group of four lanes: v[j] of lane h becomes
// v[h] of lane j.
__device__ __forceinline__ void quad_transpose(double (&v)[4], int h) {
  const bool odd = h & 1, high = h & 2;
#pragma unroll
  for (int i = 0; i < 4; i += 2) {
    const double o = dpp_f64<0xB1>(odd ? v[i] : v[i + 1]);
    v[i] = odd ? o : v[i];
    v[i + 1] = odd ? v[i + 1] : o;
  }
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const double o = dpp_f64<0x4E>(high ? v[i] : v[i + 2]);
    v[i] = high ? o : v[i];
    v[i + 2] = high ? v[i + 2] : o;
  }
}

// Waits until this wave's earlier stores (device-scope ones have then
// reached the level that all compute dies share) and loads have completed.
__device__ __forceinline__ void vmem_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ void st_agent(double *p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double ld_agent_f64(const double *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Case-level end of one body's step, by one thread: the last body of the
// case completes the step.  A body that failed (support outside the lattice,
// non-finite force) stops the case without completing it; bodies whose
// supports could meet within the next step stop it after completing this one.
// The union of the bodies' force boxes tells the next collide-stream where to
// read the IB force.
__device__ __forceinline__ void case_body_done(const CaseDesc &c, CaseState *cs, int64_t step, int cur,
                                               int nslots, int flags, int box_valid, const int (&box)[4],
                                               int par = -1) {
  // what the next one-launch step of a batch does with the case
  auto control = [&](bool done, bool halted) {
    if (par < 0) return;
    const bool on = !halted && (!done || step + 1 < cs->target);
    cs->ctl[par ^ 1] = (done ? cur ^ 1 : cur) | (on ? kCtlActive : 0) | (done ? kCtlHold : 0);
  };
  if (nslots == 1) {
    control(!flags, flags != 0);
    if (flags) {
      cs->flags |= kCaseHalted;
      cs->halt[cur ^ 1] = 1;
    } else {
      if (box_valid)
        for (int i = 0; i < 4; i++) cs->fbox[i] = box[i];
      cs->fbox_valid = box_valid;
      cs->cur = cur ^ 1;
      cs->step = step + 1;
    }
    cs->xcnt = 0;
    return;
  }
  __threadfence();
  if (atomicAdd(&cs->done, 1) != nslots - 1) return;
  __threadfence();
  int bflags = 0, bv = 0, b0 = 1 << 30, b1 = 1 << 30, b2 = -1, b3 = -1;
  for (int b = 0; b < c.nbodies; b++) {
    BodyState *st = c.bodies[b].state;
    bflags |= __hip_atomic_load(&st->flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__hip_atomic_load(&st->box_valid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
      bv = 1;
      b0 = min(b0, __hip_atomic_load(&st->box[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
      b1 = min(b1, __hip_atomic_load(&st->box[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
      b2 = max(b2, __hip_atomic_load(&st->box[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
      b3 = max(b3, __hip_atomic_load(&st->box[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
  }
  bool meet = false;
  for (int a = 0; a < c.nbodies && !bflags; a++)
    for (int b = a + 1; b < c.nbodies; b++) {
      const BodyDesc &A = c.bodies[a], &Bb = c.bodies[b];
      const double dx = __hip_atomic_load(&A.state->xc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) -
                        __hip_atomic_load(&Bb.state->xc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const double dy = __hip_atomic_load(&A.state->yc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) -
                        __hip_atomic_load(&Bb.state->yc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const double lim = A.radius + Bb.radius + A.ns + Bb.ns + 4.0;
      if (dx * dx + dy * dy <= lim * lim) {
        meet = true;
        A.state->flags |= kFlagOverlap;
      }
    }
  cs->done = 0;
  cs->xcnt = 0;
  if (bflags || meet) cs->halt[cur ^ 1] = 1;
  control(!bflags, bflags || meet);
  if (bflags) {
    cs->flags |= kCaseHalted;
  } else {
    cs->fbox[0] = b0; cs->fbox[1] = b1; cs->fbox[2] = b2; cs->fbox[3] = b3;
    cs->fbox_valid = bv;
    cs->cur ^= 1;
    cs->step = step + 1;
    if (meet) cs->flags |= kCaseHalted;
  }
  __threadfence();
}

constexpr int kArcSpins = 1 << 22;

// Shared memory of a pass besides its dynamic part.
struct ArcShared {
  unsigned long long rmax[3];  // adaptive MDF: squared residuals, as ordered bits
  Kin kin, next;  // this step's, and of a driven body the next step's
  int flags;
  int box[4], hold[4];  // force box; hold rectangle of the next step (not of a free body)
  int corner;           // the force box reaches a corner node's diagonal neighbour
  int64_t hist;         // offset of the step's history row
};

// A stencil origin that covers no node.
constexpr int kArcNowhere = 0x7fffffff;

// floor(x) for sums of node numbers: a body's next position may be any number (a
// force that blows up moves it by more than 2^31 nodes in one step), and the
// conversion saturates, so that a sum with it would wrap to the other side.
__device__ __forceinline__ int node_floor(double x) { return (int)fmax(-1e9, fmin(floor(x), 1e9)); }

// Whether the NS nodes around coordinate X (first node floor(X) - (NS / 2 - 1))
// lie in 0 .. n - 1; false for NaN.  Compared as doubles, as above.
__device__ __forceinline__ bool support_in(double X, int ns, int n) {
  const double i = floor(X);
  return i >= ns / 2 - 1 && i <= n - 1 - ns / 2;
}

// What the next step's pass waits for: the nodes whose pushes (two nodes
// around its support, with the walls it may close) or reads of this step's
// force reach its support, for a body at (x, y) now and (xn, yn) then; one
// node wider than the circle's box for rounding.
__device__ __forceinline__ void arc_hold(double x, double y, double xn, double yn, double r, int s1, int nx,
                                         int ny, int32_t *h) {
  h[0] = max(0, node_floor(fmin(xn, x) - r) - s1 - 3);
  h[1] = max(0, node_floor(fmin(yn, y) - r) - s1 - 3);
  h[2] = min(nx - 1, node_floor(fmax(xn, x) + r) + s1 + 4);
  h[3] = min(ny - 1, node_floor(fmax(yn, y) + r) + s1 + 4);
}

// Density and momentum of one node's populations (g = f - w rho0 in FP32).
template <typename T>
__device__ __forceinline__ void node_sums(const T (&v)[9], double rho0, double &sm, double &jx, double &jy) {
  double d[9];
#pragma unroll
  for (int i = 0; i < 9; i++) d[i] = (double)v[i];
  sm = ((d[1] + d[3]) + (d[2] + d[4])) + ((d[5] + d[7]) + (d[6] + d[8])) + d[0];
  if (sizeof(T) == 4) sm += rho0;
  const double a = d[5] - d[7], b = d[8] - d[6];
  jx = (d[1] - d[3]) + (a + b);
  jy = (d[2] - d[4]) + (a - b);
}

// Bounded wait (of one thread) until a device-scope counter that other
// workgroups add to reaches n.
__device__ __forceinline__ bool count_wait(const int32_t *cnt, int n) {
  int spins = 0;
  while (ld_agent(cnt) < n && spins < kArcSpins) {
    __builtin_amdgcn_s_sleep(2);
    spins++;
  }
  return spins < kArcSpins;
}

// One arc of one body.  T: stored population; NS: stencil width; KIND: the
// scheme.  body: its index in the case, of nslots bodies.  The workgroup has at
// least nl NS threads (a multiple of 64).  BU: band entries built at a time (MDF).
// wait_for >= 0 (one-launch steps): the pass runs beside the tiles of its step and first waits until that many workgroups have
// counted themselves in hold_done; OPEN: the lattice's Zou-He wall nodes are
// still open then; par: the launch's parity in a batch, or -1.
enum { kArcDF = 0, kArcMDF = 1, kArcDFC = 2 };
template <typename T, int NS, int KIND, bool OPEN, int BU, typename BODY>
__device__ __forceinline__ void arc_pass(const CaseDesc &c, BODY &B, int64_t step, int cur,
                                         int arc, int body, int nslots, int wait_for, int par, double *dyn,
                                         ArcShared &sh) {
  // A lane's strip of its marker's stencil: NS nodes along x in a row, or (COLS,
  // FP32 Peskin) along y in a column.  By columns the marker's lanes access
  // neighbouring nodes together, one line per marker and access instead of one per
  // lane, and a strip never crosses a segment of the lattice's storage; FP32 then
  // loads each population by itself where a row is one 16-byte load, and still
  // gains.  FP64 Peskin loads columns too and turns them into rows (TURN: the sums
  // keep their order, and with it the last bits of FP64 results).  Fixed disk, D =
  // 9, plain steps, row loads and now: DFC fp64 25.8 and 22.2 us, fp32 22.5 and
  // 20.3; DF fp32 19.7 and 18.4, MDF fp32 23.4 and 22.2.  One launch, DF fp64 12.8
  // and 10.2, MDF D = 30 fp64 21.5 and 17.2, oscillating 1200 x 600 MDF fp32 21.0
  // and 20.1.
  constexpr bool COLS = NS == 4 && sizeof(T) == 4;
  constexpr bool TURN = NS == 4 && sizeof(T) == 8;
  constexpr int QMAX = NS == 4 ? kArcBandRegsP4 : kArcBandRegsHat;
  const int tid = threadIdx.x;
  const double rho0 = c.rho0;
  const int nx = c.nx, ny = c.ny, nseg = c.nseg;
  const uint32_t plane = (uint32_t)c.plane;
  BodyState *const bs = B.state;
  const int nb = B.nb, narcs = B.arc_n, bw = B.arc_bw, halo = B.arc_halo;
  const bool whole = narcs == 1;
  const int k0 = arc * B.arc_own;
  const int own = min(B.arc_own, nb - k0);
  const int nl = whole ? nb : own + 2 * halo;
  if (tid == 0) {
    sh.kin = body_kinematics(c, B, bs, step);
    sh.flags = bs->flags;
  }
  if (tid == 64 && B.motion == kPrescribedSin) sh.next = body_kinematics(c, B, bs, step + 1);
  // the lane's marker and its strip
  const int mm = tid / NS, h = tid % NS;
  const bool live = mm < nl;
  const int m = live ? mm : 0;
  int k = whole ? m : k0 - halo + m;
  k = k < 0 ? k + nb : (k >= nb ? k - nb : k);
  const bool owned = live && (whole || (m >= halo && m < halo + own));
  const double ct = B.cos_t[k], st = B.sin_t[k];
  // Local markers as entries of LDS arrays, local marker m at entry m + bw:
  // the neighbour d markers further along is always entry m + bw + d, with no
  // test.  Around an arc bw entries on either side cover nothing and hold
  // zeros; a body in one arc keeps copies of its last and first markers there.
  // w_x (the weights along a strip) has NS zeros on either side and w_y (across)
  // one, so that a shifted row of weights (its shift clamped) needs no test either.
  constexpr int SW = 3 * NS, SY = NS + 2;
  const int E = arc_entries(NS, bw, nl);
  double2 *const lF = (double2 *)dyn;              // [2][E] forces
  double *const lwx = (double *)(lF + 2 * E);      // [E][SW]
  double *const lwy = lwx + E * SW;                // [E][SY]
  double *const lB = lwy + E * SY;                 // [E][bw + 1] (MDF), [E][9] (DFC)
  const int nB = KIND == kArcDFC ? 9 : (KIND == kArcMDF ? bw + 1 : 0);
  int *const lpos = (int *)(lB + E * nB);          // [E] first node of the stencil
  double *const lX = (double *)(lpos + ((E + 1) & ~1));  // [nl][3] X, Y, (sum w_x)(sum w_y)
  for (int i = tid; i < E * (4 + SW + SY + nB); i += blockDim.x) dyn[i] = 0.0;
  for (int i = tid; i < E; i += blockDim.x) lpos[i] = kArcNowhere;
  if (tid < 3) sh.rmax[tid] = 0ull;
  const int e0 = m + bw;  // the lane's own entry, and its copy in a whole circle
  const int e1 = whole ? (m < bw ? e0 + nl : (m >= nl - bw ? e0 - nl : e0)) : e0;
  __syncthreads();
  const double xc = sh.kin.xc, yc = sh.kin.yc;
  constexpr int s1 = NS / 2 - 1;
  int fail = 0;
  {
    // every support inside the lattice: certain when the box of the circle,
    // one node wider, is; else every marker of the body is looked at, so that
    // all arcs decide alike
    const double R = B.radius;
    if (!(xc - R >= s1 + 1 && yc - R >= s1 + 1 && xc + R <= nx - NS && yc + R <= ny - NS)) {
      for (int q = tid; q < nb; q += blockDim.x) {
        if (!support_in(xc + R * B.cos_t[q], NS, nx) || !support_in(yc + R * B.sin_t[q], NS, ny)) fail = 1;
      }
      fail = __syncthreads_or(fail);
    }
  }
  const double X = xc + B.radius * ct, Y = yc + B.radius * st;
  const double udx = sh.kin.udx - sh.kin.udo * (Y - yc), udy = sh.kin.udy + sh.kin.udo * (X - xc);
  const double ds = B.ds;
  // (The origins of a body that does not fit lead to no memory: they only decide
  // which markers' LDS entries cover which.  Zeroing them all the same measured,
  // us per step without and with: adaptive MDF 2001 x 1601 41.4 and 41.9, settling
  // DFC FP64 22.8 and 22.95, the pair 20.2 and 20.5, DFC hat 16.73 and 16.62.)
  const bool none = KIND == kArcDFC && NS == 2 && fail;
  const int ix0 = none ? 0 : (int)floor(X) - s1, iy0 = none ? 0 : (int)floor(Y) - s1;
  const int s0 = COLS ? iy0 : ix0;        // where the strip starts
  const int ln = (COLS ? ix0 : iy0) + h;  // the column or row it lies in
  double a1 = 0, a2 = 0, a3 = 0, a4 = 0, a5 = 0, a6 = 0;  // fx fy torque slip | residual slip_max
  int iters = KIND == kArcDFC ? 0 : 1;
  const int motion = B.motion;
  if (tid == 64) {
    // what the end of the pass writes and the position alone decides
    const double r = B.radius;
    sh.box[0] = max(0, node_floor(xc - r) - NS);
    sh.box[1] = max(0, node_floor(yc - r) - NS);
    sh.box[2] = min(nx - 1, node_floor(xc + r) + NS + 1);
    sh.box[3] = min(ny - 1, node_floor(yc + r) + NS + 1);
    if (motion != kFree) {
      const bool driven = motion == kPrescribedSin;
      arc_hold(xc, yc, driven ? sh.next.xc : xc, driven ? sh.next.yc : yc, r, s1, nx, ny, sh.hold);
    }
    if (OPEN)
      sh.corner = (sh.box[0] <= 1 || sh.box[2] >= nx - 2) && (sh.box[1] <= 1 || sh.box[3] >= ny - 2);
    sh.hist = (step % B.hist_cap) * kHistCols;
  }
  // The geometry of the step, all of it before the wait of a one-launch step:
  // weights, the markers covering the lane's strip, its nodes' first markers,
  // and DFC's correction scale.
  double wx[NS], wyv[NS], wy;
  row_weights<NS>(COLS ? Y : X, wx);
  row_weights<NS>(COLS ? X : Y, wyv);
  double wsum;  // (sum w_x) (sum w_y)
  {
    double wsx = 0, wsy = 0;
#pragma unroll
    for (int j = 0; j < NS; j++) { wsx += wx[j]; wsy += wyv[j]; }
    wsum = wsx * wsy;
  }
  {
    double wxh = wx[0];
    wy = wyv[0];
#pragma unroll
    for (int q = 1; q < NS; q++) {
      wy = h == q ? wyv[q] : wy;
      wxh = h == q ? wx[q] : wxh;
    }
    if (live) {
      lwx[e0 * SW + NS + h] = wxh;
      lwy[e0 * SY + 1 + h] = wy;
      if (e1 != e0) {
        lwx[e1 * SW + NS + h] = wxh;
        lwy[e1 * SY + 1 + h] = wy;
      }
    }
  }
  if (live && h == 0) {
    // (kept here rather than in registers: only the end of the pass reads them)
    lX[3 * m] = X;
    lX[3 * m + 1] = Y;
    lX[3 * m + 2] = wsum;
    lpos[e0] = ix0 | (iy0 << 16);
    lpos[e1] = ix0 | (iy0 << 16);
  }
  __syncthreads();
  // The marker at stencil origin p against the lane's strip: dx, the start of its
  // strips relative to this one's, and ly, the strip's line in its stencil.
  auto offsets = [&](int p, int &dx, int &ly) {
    dx = (COLS ? p >> 16 : p & 0xffff) - s0;
    ly = ln - (COLS ? p & 0xffff : p >> 16);
  };
  // cov: the markers covering nodes of the strip, one bit per entry m .. m + 2 bw
  // (origins loaded four at a time: one LDS round trip each); mine: the nodes
  // of the strip, one bit each, that no earlier marker covers.
  uint32_t cov = 0, mine = (1u << NS) - 1;
  for (int i0 = 0; i0 <= 2 * bw; i0 += 4) {
    int p[4];
#pragma unroll
    for (int u = 0; u < 4; u++) p[u] = lpos[m + min(i0 + u, 2 * bw)];
#pragma unroll
    for (int u = 0; u < 4; u++) {
      int dx, ly;
      offsets(p[u], dx, ly);
      const bool in = dx > -NS && dx < NS && i0 + u <= 2 * bw;
      const uint32_t cols = i0 + u < bw ? ((((1u << NS) - 1) << NS) >> (NS - dx)) : 0u;
      if (in && (unsigned)ly < (unsigned)NS) {
        cov |= 1u << (i0 + u);
        mine &= ~cols;
      }
    }
  }
  // Calls f(i, w, wy) for the markers of a set covering the strip in order along
  // the circle: entry m + i, its weights at the strip's nodes (w, zero where it
  // does not reach) and at the strip's line.
  auto for_cover = [&](uint32_t set, auto &&f) {
    while (set) {
      const int i = __ffs(set) - 1;
      set &= set - 1;
      int dx, ly;
      offsets(lpos[m + i], dx, ly);
      f(i, lwx + (m + i) * SW + NS - dx, lwy[(m + i) * SY + 1 + ly]);
    }
  };
  double lam = 0.0;
  if constexpr (KIND == kArcDFC) {
    if (bs->lambda_valid) {
      lam = B.lambda_cache[k];
    } else {
      // W_total interpolated to the marker (Eq. 17): sum_l sum_x D_k D_l
      double ws = 0.0;
      for_cover(cov, [&](int, const double *w, double wyl) {
        double q = 0.0;
#pragma unroll
        for (int j = 0; j < NS; j++) q += wx[j] * w[j];
        ws += q * (wy * wyl);
      });
      lam = 1.0 / (2.0 * rho0 * ds * group_sum<NS>(ws));
      if (motion == kFixed && owned && h == 0 && !fail) B.lambda_cache[k] = lam;
    }
  }
  if (wait_for >= 0) {
    if (tid == 0) {
      if (!count_wait(&c.state->hold_done[body], wait_for)) sh.flags |= kFlagExchange;
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
  }
  if (!fail) {
    const T *const fpop = (const T *)c.f[cur ^ 1];
    // The populations of the strip's nodes, or, to be turned, of the h-th column's.
    auto load_strip = [&](T (&v)[9][NS]) {
      constexpr bool cols = COLS || TURN;
      const int l = TURN ? ix0 + h : ln, a0 = TURN ? iy0 : s0;
      if constexpr (cols) {
        const T *p = fpop + pop_node(l, a0, nseg);
#pragma unroll
        for (int j = 0; j < NS; j++)
#pragma unroll
          for (int i = 0; i < 9; i++) v[i][j] = p[j * nseg * kSegBlock + i * kSeg];
      } else {
        load_pop_row<T, NS>(fpop, a0, l, nseg, v);
      }
      if constexpr (OPEN) {
        if (l == 0 || l == (cols ? nx : ny) - 1 || a0 == 0 || a0 + NS == (cols ? ny : nx)) {
#pragma unroll
          for (int j = 0; j < NS; j++) {
            const int x = cols ? l : a0 + j, y = cols ? a0 + j : l;
            if (!is_zou_he_wall(c, x, y)) continue;
            T w[9];
#pragma unroll
            for (int i = 0; i < 9; i++) w[i] = v[i][j];
            zou_he_close<T>(c, fpop, x, y, w);
#pragma unroll
            for (int i = 0; i < 9; i++) v[i][j] = w[i];
          }
        }
      }
    };
    auto put_force = [&](double2 *f, double Fx, double Fy) {
      if (live && h == 0) {
        f[e0] = make_double2(Fx, Fy);
        if (e1 != e0) f[e1] = make_double2(Fx, Fy);
      }
    };
    double Ux, Uy, Ftx = 0.0, Fty = 0.0;
    if constexpr (KIND != kArcDFC) {
      // moments of the strip's nodes, interpolated to the marker (rin, ux, uy:
      // 1/rho and the velocity, kept for DF)
      double rin[NS], ux[NS], uy[NS], t[NS];
      double ra = 0, rb = 0, rc = 0;
      double sm[NS], jx[NS], jy[NS];
      T v[9][NS];
      load_strip(v);
      // FP32: every load is issued before the first sum waits (2000 x 800 MDF 22.7
      // us per step, 23.2 without; plain FP64 passes are 1 % slower with it)
      if (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < NS; j++) {
        T q[9];
#pragma unroll
        for (int i = 0; i < 9; i++) q[i] = v[i][j];
        node_sums<T>(q, rho0, sm[j], jx[j], jy[j]);
      }
      if constexpr (TURN) {
        quad_transpose(sm, h);
        quad_transpose(jx, h);
        quad_transpose(jy, h);
      }
      double qa = 0, qb = 0, qc = 0;
#pragma unroll
      for (int j = 0; j < NS; j++) {
        const double inv = 1.0 / sm[j];
        jx[j] *= inv;
        jy[j] *= inv;
        qa += sm[j] * wx[j];
        qb += jx[j] * wx[j];
        qc += jy[j] * wx[j];
        if constexpr (KIND == kArcDF) {
          rin[j] = inv;
          ux[j] = jx[j];
          uy[j] = jy[j];
        } else {
          t[j] = wx[j] * wy * (0.5 * ds * inv);
        }
      }
      ra += qa * wy;
      rb += qb * wy;
      rc += qc * wy;
      if (sizeof(T) == 8) __builtin_amdgcn_sched_barrier(0);  // the populations end here
      const double rX = group_sum<NS>(ra);
      Ux = group_sum<NS>(rb);
      Uy = group_sum<NS>(rc);
      if constexpr (KIND == kArcDF) {
        // Eq. (11)
        Ftx = 2.0 * rX * (udx - Ux);
        Fty = 2.0 * rX * (udy - Uy);
        put_force(lF, Ftx, Fty);
        __syncthreads();
      } else {
        // MDF, Eq. (12)-(14), in marker space: interpolating the updated
        // node velocities of Eq. (14) gives U^(n+1) = U^(n) + omega B F^(n),
        // B_kl = sum_x D_h(x - X_k) D_h(x - X_l) ds / (2 rho(x)).  The lane
        // keeps its strip's terms of B's row k and, for the passes, its share of
        // the band in registers: a pass is one LDS round trip and one barrier.
        // BU entries at a time (arc_build) overlap their LDS round trips.
        for (int d0 = 0; d0 <= bw; d0 += BU) {
          double b[BU];
#pragma unroll
          for (int u = 0; u < BU; u++) {
            const int e = e0 + min(d0 + u, bw);
            int dx, ly;
            offsets(lpos[e], dx, ly);
            const double *w = lwx + e * SW + NS - max(-NS, min(NS, dx));
            double wj[NS];
#pragma unroll
            for (int j = 0; j < NS; j++) wj[j] = w[j];
            b[u] = 0.0;
            double q = 0.0;
#pragma unroll
            for (int j = 0; j < NS; j++) q += t[j] * wj[j];
            b[u] += q * lwy[e * SY + 1 + max(-1, min(NS, ly))];
          }
#pragma unroll
          for (int u = 0; u < BU; u++) {
            b[u] = group_sum<NS>(b[u]);
            const int d = d0 + u;
            if (live && d <= bw && h == (d & (NS - 1))) {
              lB[e0 * nB + d] = b[u];
              if (e1 != e0) lB[e1 * nB + d] = b[u];
            }
          }
        }
        __syncthreads();
        // the lane's entries of row k: i = h, h + NS, ... of 0 .. 2 bw; the
        // ones behind the diagonal are read from the earlier marker's row
        double bq[QMAX];
#pragma unroll
        for (int q = 0; q < QMAX; q++) {
          const int i = q * NS + h;
          bq[q] = i > 2 * bw ? 0.0 : (i >= bw ? lB[e0 * nB + i - bw] : lB[(m + i) * nB + bw - i]);
        }
        const int nq = (2 * bw + NS) / NS;  // entries of a lane, ceil((2 bw + 1) / NS)
        const int N = B.mdf_iters;
        const double om = B.omega_mdf, tol = B.mdf_tol;
        const bool adapt = tol > 0.0;
        double rprev = 0.0, res = 0.0;
        iters = N;
        for (int n = 1; n <= N; n++) {
          const double ex = udx - Ux, ey = udy - Uy;
          const double Fx = om * (2.0 * rX * ex), Fy = om * (2.0 * rX * ey);
          double2 *const fb = lF + (n & 1) * E;
          put_force(fb, Fx, Fy);
          if (adapt) {
            // the largest squared residual over the workgroup (a square root
            // keeps the order)
            double r = live ? ex * ex + ey * ey : 0.0;
            r = r == r ? r : 0.0;
            r = fmax(r, dpp_f64<0x4E>(r));
            r = fmax(r, dpp_f64<0x141>(r));
            r = fmax(r, dpp_f64<0x140>(r));
            r = fmax(fmax(lane_f64(r, 0), lane_f64(r, 16)), fmax(lane_f64(r, 32), lane_f64(r, 48)));
            if ((tid & 63) == 0) atomicMax(&sh.rmax[n % 3], (unsigned long long)__double_as_longlong(r));
          } else if (n == N) {
            res = owned ? sqrt(ex * ex + ey * ey) : 0.0;
          }
          __syncthreads();
          if (adapt) {
            const double rn = sqrt(__longlong_as_double((long long)sh.rmax[n % 3]));
            if (tid == 0) sh.rmax[(n + 2) % 3] = 0ull;  // read last before this barrier
            res = rn;
            if ((n > B.mdf_nmin && rn < tol) || (n > 1 && rn > 1.5 * rprev)) break;
            rprev = rn;
            iters = n;
          }
          Ftx += Fx;
          Fty += Fy;
          double sx = 0.0, sy = 0.0;
#pragma unroll
          for (int q = 0; q < QMAX; q++)
            if (q < nq) {
              const double2 F = fb[m + h + q * NS];
              sx += bq[q] * F.x;
              sy += bq[q] * F.y;
            }
          Ux += group_sum<NS>(sx);
          Uy += group_sum<NS>(sy);
        }
        a5 = res;
        // every lane has read the last pass's forces
        __syncthreads();
        put_force(lF, Ftx, Fty);
        __syncthreads();
      }
      // Eulerian force f(x) = sum_k F_total D_h ds (Eq. 8) on the nodes whose
      // first marker is this lane's; DF also adds f/(2 rho) to the velocity
      // for the slip, so there every lane sums every node of its strip
      auto spread = [&](double &sa, double &sb) {
        double fx[NS], fy[NS];
#pragma unroll
        for (int j = 0; j < NS; j++) fx[j] = fy[j] = 0.0;
        const uint32_t set = KIND == kArcDF ? cov : (mine ? cov & (~0u << bw) : 0u);
        for_cover(set, [&](int i, const double *w, double wyl) {
          const double2 F = lF[m + i];
          const double Fx = F.x * wyl, Fy = F.y * wyl;
#pragma unroll
          for (int j = 0; j < NS; j++) {
            fx[j] += Fx * w[j];
            fy[j] += Fy * w[j];
          }
        });
        const uint32_t sn = COLS ? nx : 1;  // to the strip's next node
        gmem<T> *const frc = to_global((T *)c.force) + (COLS ? (uint32_t)s0 * nx + ln : (uint32_t)ln * nx + s0);
#pragma unroll
        for (int j = 0; j < NS; j++)
          if (mine & (1u << j)) {
            frc[j * sn] = (T)(fx[j] * ds);
            frc[plane + j * sn] = (T)(fy[j] * ds);
          }
        if constexpr (KIND == kArcDF) {
          double qa = 0, qb = 0;
#pragma unroll
          for (int j = 0; j < NS; j++) {
            const double g = 0.5 * ds * rin[j];
            qa += (ux[j] + fx[j] * g) * wx[j];
            qb += (uy[j] + fy[j] * g) * wx[j];
          }
          sa += qa * wy;
          sb += qb * wy;
        }
      };
      if (owned) {
        double sa = 0, sb = 0;
        spread(sa, sb);
        if constexpr (KIND == kArcDF) {
          Ux = group_sum<NS>(sa);
          Uy = group_sum<NS>(sb);
        }
        if (h == 0) {
          // force on the body (Newton's third law) and torque (Sec. 2.7)
          const double ws = lX[3 * m + 2];
          a1 = -Ftx * ds * ws;
          a2 = -Fty * ds * ws;
          a3 = -((lX[3 * m] - sh.kin.xc) * Fty - (lX[3 * m + 1] - sh.kin.yc) * Ftx) * ds;
        }
      }
    } else {
      // DFC, Eq. (15)-(20)
      T v[9][NS];
      load_strip(v);
      if constexpr (TURN) {
#pragma unroll
        for (int i = 0; i < 9; i++) quad_transpose(v[i], h);
      }
      double gi[9];
#pragma unroll
      for (int i = 0; i < 9; i++) {
        double s = 0.0;
        double q = 0.0;
#pragma unroll
        for (int j = 0; j < NS; j++) q += (double)v[i][j] * wx[j];
        s += q * wy;
        gi[i] = group_sum<NS>(s);
      }
      double fsx = 0, fsy = 0;
#pragma unroll
      for (int i = 0; i < 9; i++) {
        const double eud = c_exi[i] * udx + c_eyi[i] * udy;
        const double dl = lam * (gi[opp_of(i)] - gi[i] + 6.0 * c_w[i] * rho0 * eud);
        fsx += c_exi[i] * dl;
        fsy += c_eyi[i] * dl;
        if (live && h == (i & (NS - 1))) {
          lB[e0 * 9 + i] = dl;
          if (e1 != e0) lB[e1 * 9 + i] = dl;
        }
      }
      Ftx = -ds * fsx;
      Fty = -ds * fsy;
      // every arc has read its populations before any of them is corrected
      bool met = true;
      vmem_done();
      __syncthreads();
      if (!whole) {
        if (tid == 0) {
          __hip_atomic_fetch_add(&bs->arc_sync, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (!count_wait(&bs->arc_sync, narcs)) sh.flags |= kFlagExchange;
        }
        __syncthreads();
        met = !(sh.flags & kFlagExchange);
      }
      if constexpr (OPEN) {
        // A corner of two walls is closed from the node diagonally inside it
        // as streaming left that node: whoever is about to correct the node
        // closes the corner, unless the body's support holds it (and closed it
        // as it was read).  Only a body near a corner looks for such nodes.
        if (__builtin_expect(__builtin_amdgcn_readfirstlane(sh.corner), 0) && owned && met)
          for (int j = 0; j < NS; j++)
            if (mine & (1u << j)) {
              const int x = COLS ? ln : s0 + j, y = COLS ? s0 + j : ln;
              int cx, cy;
              if (!inside_corner(c, x, y, cx, cy)) continue;
              bool held = false;
              for_cover(cov, [&](int i, const double *, double) {
                const int p = lpos[m + i];
                held |= (unsigned)(cx - (p & 0xffff)) < (unsigned)NS && (unsigned)(cy - (p >> 16)) < (unsigned)NS;
              });
              if (held) continue;
              gmem<T> *const fw = to_global((T *)c.f[cur ^ 1]) + pop_node(cx, cy, nseg);
              T q[9];
#pragma unroll
              for (int i = 0; i < 9; i++) q[i] = fw[i * kSeg];
              zou_he_close<T>(c, fpop, cx, cy, q);
#pragma unroll
              for (int i = 1; i < 9; i++) fw[i * kSeg] = q[i];
              *wall_flag(c, cur ^ 1, wall_index(nx, ny, cx, cy)) = 1;
            }
      }
      if (owned && met) {
        // Eq. (19) on every node of the lane's strip; the first marker's lane
        // writes it, and every lane takes the corrected velocity for the slip.
        // One walk over the covering markers for the whole strip: in two walks of
        // two nodes (176 VGPRs instead of 222, two waves per SIMD either way) the
        // D = 9 steps above take 21.7 us instead of 20.5 in fp32.
        double sa = 0, sb = 0;
        double qa = 0, qb = 0;
        double corr[NS][9];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < NS; j++)
#pragma unroll
          for (int i = 0; i < 9; i++) corr[j][i] = 0.0;
        for_cover(cov, [&](int i, const double *w, double wyl) {
          const double *q = lB + (m + i) * 9;
          double ww[NS];
#pragma unroll
          for (int j = 0; j < NS; j++) ww[j] = w[j] * wyl;
#pragma unroll
          for (int n = 0; n < 9; n++) {
            const double dq = q[n];
#pragma unroll
            for (int j = 0; j < NS; j++) corr[j][n] += dq * ww[j];
          }
        });
#pragma unroll
        for (int j = 0; j < NS; j++) {
          const int x = COLS ? ln : s0 + j, y = COLS ? s0 + j : ln;
          gmem<T> *const fw = to_global((T *)c.f[cur ^ 1]) + pop_node(x, y, nseg);
          const bool first = (mine & (1u << j)) != 0;
          if constexpr (OPEN)
            if (first && is_zou_he_wall(c, x, y)) *wall_flag(c, cur ^ 1, wall_index(nx, ny, x, y)) = 1;
          T q[9];
#pragma unroll
          for (int i = 0; i < 9; i++) {
            q[i] = (T)((double)v[i][j] + corr[j][i] * ds);
            if (first) fw[i * kSeg] = q[i];
          }
          double sm, jx, jy;
          node_sums<T>(q, rho0, sm, jx, jy);
          const double inv = 1.0 / sm;
          qa += jx * inv * wx[j];
          qb += jy * inv * wx[j];
        }
        sa += qa * wy;
        sb += qb * wy;
        Ux = group_sum<NS>(sa);
        Uy = group_sum<NS>(sb);
        if (h == 0) {
          a1 = Ftx;
          a2 = Fty;
          a3 = (lX[3 * m] - sh.kin.xc) * Fty - (lX[3 * m + 1] - sh.kin.yc) * Ftx;
        }
      }
    }
    if (owned) {
      gmem<double> *const mo = to_global(B.markers_out) + 8 * k;
      if (h == 0) {
        a4 = sqrt((Ux - udx) * (Ux - udx) + (Uy - udy) * (Uy - udy));
        a6 = a4;
        mo[0] = lX[3 * m]; mo[1] = lX[3 * m + 1]; mo[2] = udx; mo[3] = udy;
      }
      if (h == NS - 1) {
        mo[4] = Ftx; mo[5] = Fty; mo[6] = lam; mo[7] = ds;
      }
    }
    // The six sums of the owned markers: one value each into the (no longer
    // needed) dynamic shared memory, then eight lanes of wave 0 per quantity,
    // every eighth marker each, joined by a fixed tree.  (Reducing all six
    // over every wave by lane exchanges took 1.5 us more.)
    __syncthreads();
    if (owned && h == 0) {
      double *const r = dyn + (whole ? m : m - halo);
      r[0] = a1; r[own] = a2; r[2 * own] = a3; r[3 * own] = a4; r[4 * own] = a5; r[5 * own] = a6;
    }
  }
  __syncthreads();
  if (tid >= 64) return;
  const int qi = min(tid >> 3, 5);
  double tot = 0.0;
  if (!fail) {
    const double *r = dyn + qi * own;
    for (int i = tid & 7; i < own; i += 32) {
      double q[4];
#pragma unroll
      for (int u = 0; u < 4; u++) q[u] = i + 8 * u < own ? r[i + 8 * u] : 0.0;
#pragma unroll
      for (int u = 0; u < 4; u++) tot = qi < 4 ? tot + q[u] : fmax(tot, q[u]);
    }
    double o = dpp_f64<0xB1>(tot);
    tot = qi < 4 ? tot + o : fmax(tot, o);
    o = dpp_f64<0x4E>(tot);
    tot = qi < 4 ? tot + o : fmax(tot, o);
    o = dpp_f64<0x141>(tot);
    tot = qi < 4 ? tot + o : fmax(tot, o);
  }
  // the body's sums over its arcs, in arc order, by the last arc to arrive
  if (!whole) {
    if (tid < 48 && (tid & 7) == 0) st_agent(B.arc_part + 8 * arc + qi, tot);
    if (tid == 1) st_agent(B.arc_part + 8 * arc + 6, (double)sh.flags);
    vmem_done();
    int last = 0;
    if (tid == 0)
      last = __hip_atomic_fetch_add(&bs->arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == narcs - 1;
    if (!__builtin_amdgcn_readfirstlane(last)) return;
    tot = ld_agent_f64(B.arc_part + qi);
    int fl = (int)ld_agent_f64(B.arc_part + 6);
    for (int a0 = 1; a0 < narcs; a0 += 8) {
      double r[8], f[8];
#pragma unroll
      for (int u = 0; u < 8; u++) {
        const double *p = B.arc_part + 8 * min(a0 + u, narcs - 1);
        r[u] = ld_agent_f64(p + qi);
        f[u] = ld_agent_f64(p + 6);
      }
#pragma unroll
      for (int u = 0; u < 8; u++)
        if (a0 + u < narcs) {
          tot = qi < 4 ? tot + r[u] : fmax(tot, r[u]);
          fl |= (int)f[u];
        }
    }
    if (tid == 0) sh.flags |= fl;
  }
  a1 = lane_f64(tot, 0); a2 = lane_f64(tot, 8); a3 = lane_f64(tot, 16);
  a4 = lane_f64(tot, 24); a5 = lane_f64(tot, 32); a6 = lane_f64(tot, 40);
  if (tid != 0) return;
  const Kin kn = sh.kin;
  const bool euler = motion == kFree && B.integrator == kEulerA1;
  gmem<BodyState> *const g = to_global(bs);
  g->xc = kn.xc; g->yc = kn.yc;
  g->vhx = kn.vhx; g->vhy = kn.vhy; g->omh = kn.omh;
  if (motion == kFree) {
    g->vpx = kn.vx0; g->vpy = kn.vy0;
    g->dimx = kn.dimx; g->dimy = kn.dimy;
    if (euler) g->omp = kn.om0;
  } else if (motion == kPrescribedSin) {
    g->vx = kn.vhx; g->vy = kn.vhy;
  }
  g->arrived = 0;
  g->arc_sync = 0;
  c.state->hold_done[body] = 0;
  const int box[4] = {sh.box[0], sh.box[1], sh.box[2], sh.box[3]};
  if (fail) {
    const int f = sh.flags | kFlagRange;
    g->flags = f;
    g->box_valid = 0;
    case_body_done(c, c.state, step, cur, nslots, f, 0, box, par);
    return;
  }
  int flags = sh.flags;
  if (!isfinite(a1) || !isfinite(a2) || !isfinite(a3) || !isfinite(a4)) flags |= kFlagNonfinite;
  const int box_valid = KIND == kArcDFC ? 0 : 1;
  double vx = kn.vhx, vy = kn.vhy, om = kn.omh;
  if (motion == kFree) {
    if (!euler) {
      const double fgx = (B.ms - B.mf) * c.grav_x, fgy = (B.ms - B.mf) * c.grav_y;
      vx = kn.vhx + (a1 + fgx + kn.dimx) / (2.0 * B.ms);
      vy = kn.vhy + (a2 + fgy + kn.dimy) / (2.0 * B.ms);
      om = kn.omh + a3 / (2.0 * B.Is);
    }
    if (!isfinite(vx) || !isfinite(vy) || fabs(vx) > 0.5 || fabs(vy) > 0.5) flags |= kFlagNonfinite;
  } else if (motion == kFixed) {
    vx = 0.0; vy = 0.0; om = 0.0;
    if (KIND == kArcDFC) g->lambda_valid = 1;
  }
  const double slip_mean = a4 / nb, res = KIND == kArcMDF ? fmax(a5, 0.0) : 0.0;
  g->fhx = a1; g->fhy = a2; g->torque = a3;
  g->slip_mean = slip_mean; g->slip_max = a6; g->mdf_res = res;
  g->mdf_iters_done = iters;
  if (KIND != kArcDFC)
    for (int i = 0; i < 4; i++) g->box[i] = box[i];
  g->box_valid = box_valid;
  if (motion != kPrescribedSin) { g->vx = vx; g->vy = vy; g->om = om; }
  g->flags = flags;
  gmem<double> *const hr = to_global(B.history) + sh.hist;
  hr[0] = (double)(step + 1); hr[1] = a1; hr[2] = a2; hr[3] = a3;
  hr[4] = kn.xc; hr[5] = kn.yc; hr[6] = vx; hr[7] = vy; hr[8] = motion == kFree ? om : kn.omh;
  hr[9] = slip_mean; hr[10] = a6; hr[11] = res;
  hr[12] = iters; hr[13] = flags; hr[14] = 0; hr[15] = 0;
  {
    c.state->hold_step = step + 1;
    int32_t *const hb = c.state->hold[cur ^ 1][body];
    if (motion == kFree) {
      BodyState t;
      t.xc = kn.xc; t.yc = kn.yc;
      t.vx = vx; t.vy = vy; t.om = om;
      t.vpx = kn.vx0; t.vpy = kn.vy0; t.omp = kn.om0;
      t.fhx = a1; t.fhy = a2; t.torque = a3;
      const Kin q = body_kinematics(c, B, &t, step + 1);
      arc_hold(kn.xc, kn.yc, q.xc, q.yc, B.radius, s1, nx, ny, hb);
    } else {
      for (int i = 0; i < 4; i++) hb[i] = sh.hold[i];
    }
  }
  case_body_done(c, c.state, step, cur, nslots, flags, box_valid, box, par);
}

// Band entries that an MDF pass builds at a time.  FP32 Peskin: six, the whole
// band of markers a node apart (bw 5); 2000 x 800 takes 22.05 us per step, 22.2
// with five, 22.75 with four.  FP64: four; with six a disk of D = 9 (bw 6) takes 13.7
// us instead of 13.2, of D = 30 16.5 instead of 16.7.  Hat: three (bw 2); with four
// FP64 disks are up to 1 % slower.  A batch, whose passes have fewer registers,
// stays at two: with four a step of twelve members took 67.4 us instead of 65.2.
template <typename T>
__device__ constexpr int arc_build(int set, int ns) {
  return set != 1 ? 2 : (ns == 2 ? 3 : (sizeof(T) == 4 ? 6 : 4));
}

// The pass of one arc (see arc_pass).  SET: the schemes the instance holds, 0
// all, 1 DF and MDF, 2 DFC.
template <typename T, int SET, bool OPEN>
__device__ __forceinline__ void arc_body(const CaseDesc &c, const BodyDesc *body_desc, int64_t step, int cur,
                                         int arc, int body, int nslots, int wait_for, int par, double *dyn,
                                         ArcShared &sh) {
#define IBL_PASS(BODY, NSV, KINDV)                                                               \
  arc_pass<T, NSV, KINDV, OPEN, arc_build<T>(SET, NSV)>(c, *(BODY *)body_desc, step, cur, arc, body, \
                                                    nslots, wait_for, par, dyn, sh)
  if (SET == 2 || (SET == 0 && body_desc->scheme == kDFC)) {
    if constexpr (SET != 1) {
      if (body_desc->ns == 2) IBL_PASS(const BodyDesc, 2, kArcDFC);
      else IBL_PASS(const BodyDesc, 4, kArcDFC);
    }
  } else if constexpr (SET != 2) {
    ConstBody &B = *(ConstBody *)body_desc;
    if (B.scheme == kMDF) {
      if (B.ns == 2) IBL_PASS(ConstBody, 2, kArcMDF);
      else IBL_PASS(ConstBody, 4, kArcMDF);
    } else {
      if (B.ns == 2) IBL_PASS(ConstBody, 2, kArcDF);
      else IBL_PASS(ConstBody, 4, kArcDF);
    }
  }
#undef IBL_PASS
}

}  // namespace iblbm
