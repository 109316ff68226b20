// C ABI of the IB-LBM library: state ownership, validation, launch tables,
// graph capture and kernel timing.  Every step of the method runs in the HIP
// kernels of lbm_kernels.hip and ibm_kernels.hip; the host code here only
// allocates, validates, sizes the per-body workspaces and enqueues launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <limits>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/ib_lbm.h"
#include "host_copy.h"
#include "ib_lbm_internal.h"

using namespace iblbm;

namespace {

struct DevBuf {
  void *p = nullptr;
  size_t bytes = 0;
};

struct HostBody {
  ib_lbm_body_desc d;
  BodyDesc dev;  // host copy of the device description
  DevBuf cos_t, sin_t, ws, tab, acc, markers, lambda, history, state;
  // fused steps: the force copy and staged pushes (fixed DF/MDF bodies), and
  // the nodes the IB pass collides itself with their push map, built once
  // the device has built the body's tables
  DevBuf fprev, pstage, src;
  bool src_ready = false;
};

// The IB launches of a step, in the order of their slots: bodies cut into
// arcs by workgroup size (256, 512, 1024 threads), then bodies of one
// workgroup on the 1024-thread kernel and on the general one.
struct IbSlots {
  int arcs[3] = {0, 0, 0}, fast = 0, general = 0;
  int arc_lds[3] = {0, 0, 0}, lds = 0;  // dynamic shared memory, bytes
  int total() const { return arcs[0] + arcs[1] + arcs[2] + fast + general; }
};
constexpr int kArcThreads[3] = {256, 512, 1024};

struct EventPair {
  hipEvent_t a, b;
};

// Kernel timing kinds: 0 collide-stream, 1 IB pass.
constexpr int kTimingKinds = 2;

struct Timing {
  bool on = false;
  std::vector<EventPair> ev[kTimingKinds];
  std::vector<EventPair> pool;
  double folded_ms[kTimingKinds] = {0, 0};
  int64_t folded_n[kTimingKinds] = {0, 0};
};

}  // namespace

struct ib_lbm_sim {
  ib_lbm_config cfg;
  hipStream_t stream = nullptr;          // the caller's stream (NULL: null stream)
  hipStream_t cap_stream = nullptr;      // private stream used only for graph capture
  bool broken = false;
  bool started = false;
  bool tables_dirty = true;
  std::string err;
  CaseDesc cd;  // host copy
  DevBuf f0, f1, force, state, ticket, wall_closed;
  std::vector<HostBody> bodies;
  DevBuf d_bodies, d_case, d_prefix, d_slots, d_tmp;
  ib_lbm_launch launch = {128, 2, 1, 1};
  int spread_mode = 0;
  IbSlots ib;             // the IB launches of a step
  int graph_steps = 0;
  // captured steps, one graph per parity of the input lattice at its start
  // (the lattice of each step is a kernel argument)
  hipGraphExec_t graph_exec[2] = {nullptr, nullptr};
  int graph_len = 0;
  Timing timing;
  int64_t host_steps = 0;
  // lattice holding the input of the next enqueued step: flipped by every
  // enqueued step, reloaded from the device state by every call that reads
  // it (they differ only once a halted case stops flipping it on the device,
  // and a halted case's kernels do nothing)
  int host_cur = 0;
  int dev = 0;  // the device current at creation
  ib_lbm_batch *batch = nullptr;
  // Pipelined steps (see plan_split): the tiles of the hold rectangle and
  // the IB pass run on `iq`, all other tiles on `lq`, ordered by events.
  bool overlap = true;   // allowed by the caller
  bool split = false;    // in use for the current tables
  int32_t hold[4] = {0, 0, 0, 0};
  hipStream_t lq = nullptr, iq = nullptr;
  hipEvent_t ev_start = nullptr, ev_lq = nullptr, ev_iq = nullptr, ev_near = nullptr,
             ev_far = nullptr;
  // Fused steps (see plan_fused): one launch per step on the sim's stream.
  bool fused_allowed = true;  // allowed by the caller
  bool fused = false;         // in use for the current tables
  int32_t fhold[4] = {0, 0, 0, 0};  // hold rectangle in tiles of the fused shape
  // the fused launch's tile shape (bx x by, rows per thread): narrow tiles
  // keep the hold rectangle small; measured on the 2000x800 cylinder, FP32
  // 30.7 us per step at 64 x 16 and at 1024 x 1 x 4, FP64 37.0 us at 64 x 16
  // against 40.6 (256 x 4), 43.3 (512 x 2 x 2) and 46.5 (1024 x 1 x 4)
  int fbx = 64, fby = kFusedThreads / 64, frpt = 1;
  // One-launch steps (see plan_one).  hold_ready: the last step enqueued left
  // the hold rectangles of the next one (every pass in arcs does).
  bool one = false;
  bool hold_ready = false;
  bool halted = false;  // the case was halted when its state was last read
  // how the last step enqueued was launched (IB_LBM_STEP_*), and the steps of
  // the captured graphs
  int form = -1, graph_form = -1;
  StepOneArgs one_args;
  int one_threads = 0, one_lds = 0, one_face = 0;
  uint32_t fused_seq = 0;  // sequence number of the last fused launch (CaseState::gate)
};

struct ib_lbm_batch {
  hipStream_t stream = nullptr;
  hipStream_t cap_stream = nullptr;
  int precision = 0;
  bool dirty = true;
  bool broken = false;
  std::string err;
  std::vector<ib_lbm_sim *> sims;
  DevBuf d_cases, d_prefix, d_fprefix, d_slots;
  struct Group {
    int collision, first, count, ntiles, prefix_off, nface_blocks;
    int general_zg;  // some case has a zero-gradient face other than the east one
  };
  std::vector<Group> groups;
  IbSlots ib;
  ib_lbm_launch launch = {128, 2, 1, 1};
  int spread_mode = 0;
  // One-launch steps (see OneShape): the cases' arguments and prefix sums
  bool one = false;
  DevBuf d_one, d_one_prefix, d_work;
  StepBatchArgs one_args{};
  int form = -1;  // how the last step was launched (IB_LBM_STEP_*)
  int one_threads = 0, one_lds = 0, one_face = 0;
  int graph_steps = 0;
  hipGraphExec_t graph_exec = nullptr;
  int graph_len = 0;
};

namespace {

void set_err(std::string *e, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  *e = buf;
}

#define HIPCHK(sim, call)                                                             \
  do {                                                                                \
    hipError_t e_ = (call);                                                           \
    if (e_ != hipSuccess) {                                                           \
      set_err(&(sim)->err, "%s failed: %s", #call, hipGetErrorString(e_));            \
      (sim)->broken = true;                                                           \
      return IB_LBM_E_DEVICE;                                                         \
    }                                                                                 \
  } while (0)

ib_lbm_status dev_alloc(ib_lbm_sim *s, DevBuf *b, size_t bytes) {
  b->bytes = bytes;
  if (bytes == 0) return IB_LBM_OK;
  if (s->cfg.alloc && s->cfg.alloc->alloc) {
    b->p = s->cfg.alloc->alloc(s->cfg.alloc->ctx, bytes, (void *)s->stream);
    if (!b->p) {
      set_err(&s->err, "allocator returned NULL for %zu bytes", bytes);
      return IB_LBM_E_NOMEM;
    }
    return IB_LBM_OK;
  }
  hipError_t e = hipMalloc(&b->p, bytes);
  if (e != hipSuccess) {
    b->p = nullptr;
    set_err(&s->err, "hipMalloc(%zu) failed: %s", bytes, hipGetErrorString(e));
    return e == hipErrorOutOfMemory ? IB_LBM_E_NOMEM : IB_LBM_E_DEVICE;
  }
  return IB_LBM_OK;
}

void dev_free(ib_lbm_sim *s, DevBuf *b) {
  if (!b->p) return;
  if (s->cfg.alloc && s->cfg.alloc->free) s->cfg.alloc->free(s->cfg.alloc->ctx, b->p, (void *)s->stream);
  else (void)hipFree(b->p);
  b->p = nullptr;
  b->bytes = 0;
}

bool is_vel(int b) { return b == IB_LBM_VEL_PARABOLIC || b == IB_LBM_VEL_UNIFORM; }

// Regularized delta (Eq. 9, 10) for host-side sizing and omega_MDF.
double host_delta(int kernel, double r) {
  const double a = std::fabs(r);
  if (kernel == IB_LBM_HAT) return a < 1.0 ? 1.0 - a : 0.0;
  if (a <= 1.0) return 0.125 * (3.0 - 2.0 * a + std::sqrt(1.0 + 4.0 * a - 4.0 * a * a));
  if (a <= 2.0) return 0.125 * (5.0 - 2.0 * a - std::sqrt(-7.0 + 12.0 * a - 4.0 * a * a));
  return 0.0;
}

// Node count of the device's row-interval support description for a body
// centred at (xc, yc) (used to size the workspace).
int support_count(double xc, double yc, double R, int nb, int ns, const std::vector<double> &ct,
                  const std::vector<double> &stab, int *rows_used) {
  const int s = ns / 2;
  const int ylo = (int)std::floor(yc - R) - ns;
  const int mr = (int)std::ceil(2 * R) + 2 * ns + 4;
  std::vector<int> lmin(mr, 1 << 30), lmax(mr, -1), rmin(mr, 1 << 30), rmax(mr, -1);
  int rmx = 0;
  for (int k = 0; k < nb; k++) {
    const double X = xc + R * ct[k], Y = yc + R * stab[k];
    const int ix0 = (int)std::floor(X) - (s - 1), iy0 = (int)std::floor(Y) - (s - 1);
    for (int j = 0; j < ns; j++) {
      const int r = iy0 + j - ylo;
      if (r < 0 || r >= mr) continue;
      rmx = std::max(rmx, r);
      if (X < xc) { lmin[r] = std::min(lmin[r], ix0); lmax[r] = std::max(lmax[r], ix0 + ns - 1); }
      else { rmin[r] = std::min(rmin[r], ix0); rmax[r] = std::max(rmax[r], ix0 + ns - 1); }
    }
  }
  int total = 0;
  for (int r = 0; r < mr; r++) {
    const bool lv = lmax[r] >= 0, rv = rmax[r] >= 0;
    if (lv && rv && rmin[r] <= lmax[r] + 1) total += std::max(lmax[r], rmax[r]) - std::min(lmin[r], rmin[r]) + 1;
    else {
      if (lv) total += lmax[r] - lmin[r] + 1;
      if (rv) total += rmax[r] - rmin[r] + 1;
    }
  }
  if (rows_used) *rows_used = rmx + 1;
  return total;
}

// omega_MDF = 1 / ||A||_inf, ||A||_inf = ds max_l sum_x D_h(x-X_l) W(x),
// W(x) = sum_m D_h(x-X_m) (Sec. 2.5.2), on a dense local box.
double host_omega_mdf(double xc, double yc, double R, int nb, int kernel, double ds,
                      const std::vector<double> &ct, const std::vector<double> &stab) {
  const int ns = kernel == IB_LBM_HAT ? 2 : 4, s = ns / 2;
  const int x0 = (int)std::floor(xc - R) - ns - 1, y0 = (int)std::floor(yc - R) - ns - 1;
  const int w = (int)std::ceil(2 * R) + 2 * ns + 4;
  std::vector<double> W((size_t)w * w, 0.0);
  std::vector<double> X(nb), Y(nb);
  for (int k = 0; k < nb; k++) { X[k] = xc + R * ct[k]; Y[k] = yc + R * stab[k]; }
  for (int k = 0; k < nb; k++) {
    const int ix0 = (int)std::floor(X[k]) - (s - 1), iy0 = (int)std::floor(Y[k]) - (s - 1);
    for (int jy = 0; jy < ns; jy++)
      for (int jx = 0; jx < ns; jx++)
        W[(size_t)(iy0 + jy - y0) * w + (ix0 + jx - x0)] +=
            host_delta(kernel, ix0 + jx - X[k]) * host_delta(kernel, iy0 + jy - Y[k]);
  }
  double mx = 0.0;
  for (int k = 0; k < nb; k++) {
    const int ix0 = (int)std::floor(X[k]) - (s - 1), iy0 = (int)std::floor(Y[k]) - (s - 1);
    double acc = 0.0;
    for (int jy = 0; jy < ns; jy++)
      for (int jx = 0; jx < ns; jx++)
        acc += W[(size_t)(iy0 + jy - y0) * w + (ix0 + jx - x0)] *
               host_delta(kernel, ix0 + jx - X[k]) * host_delta(kernel, iy0 + jy - Y[k]);
    mx = std::max(mx, acc);
  }
  return 1.0 / (ds * mx);
}

int ws_doubles_for(int scheme, int nb, int ns, int mr, int mn, int pop_bytes) {
  return ws_tab_total(scheme, nb, ns, mr, mn) + ws_dyn_doubles(scheme, nb, ns, mn, pop_bytes);
}

void fill_case_tiles(CaseDesc *c, const ib_lbm_launch &l) {
  const int TX = l.block_x, TY = l.block_y * l.rows_per_thread;
  c->tiles_x = (c->nx + TX - 1) / TX;
  c->tiles_y = (c->ny + TY - 1) / TY;
}

ib_lbm_status check_launch(const ib_lbm_launch *l, std::string *err) {
  if (!l || l->block_x <= 0 || l->block_x % 64 || l->block_y <= 0 || l->rows_per_thread <= 0 ||
      l->block_x * l->block_y > 1024 || l->rows_per_thread > 64 ||
      (l->ib_threads != 0 && l->ib_threads != 256 && l->ib_threads != 512 && l->ib_threads != 1024)) {
    set_err(err, "invalid launch shape");
    return IB_LBM_E_INVALID;
  }
  return IB_LBM_OK;
}

void drop_graphs(ib_lbm_sim *s) {
  for (auto &g : s->graph_exec)
    if (g) {
      (void)hipGraphExecDestroy(g);
      g = nullptr;
    }
}

// Arguments of the inner-node collide-stream of a sim stepped on its own,
// with input lattice cur; mode as in LeanArgs.
LeanArgs lean_args(const ib_lbm_sim *s, int cur, int force_on) {
  const CaseDesc &c = s->cd;
  LeanArgs a;
  memset(&a, 0, sizeof a);
  a.src = c.f[cur];
  a.dst = c.f[cur ^ 1];
  a.force = c.force;
  a.state = c.state;
  a.halt = &c.state->flags;
  a.nx = c.nx;
  a.ny = c.ny;
  a.nseg = c.nseg;
  a.tiles_x = c.tiles_x;
  a.ntiles = c.tiles_x * c.tiles_y;
  a.rpt = s->launch.rows_per_thread;
  a.remap = s->launch.xcd_remap;
  a.force_on = force_on;
  a.htx0 = s->hold[0];
  a.hty0 = s->hold[1];
  a.hntx = s->split ? s->hold[2] : 0;
  a.hnty = s->split ? s->hold[3] : 0;
  a.omega = c.omega;
  a.s_e = c.s_e;
  a.s_o = c.s_o;
  a.s_q = c.s_q;
  a.s_eps = c.s_eps;
  a.rho0 = c.rho0;
  a.fluid_fx = c.fluid_fx;
  a.fluid_fy = c.fluid_fy;
  return a;
}

// Device tables of a sim stepped on its own: one case, its IB slots.
// Decide whether a sim's steps can be pipelined.  The collide-stream of
// the tiles away from the body (far tiles) does not read what the IB pass
// writes (its force, or its corrected populations) and is not read by it;
// only the tiles whose nodes the body's support can occupy, or that push into
// such nodes (the hold rectangle), are.  So the far tiles of step n run
// concurrently with the hold tiles and the IB pass of step n.  That needs a
// single body whose position is known in advance
// (fixed or prescribed), so that one tile rectangle covers every support of
// the run widened by two nodes (the pushes and the outlet copy that reach a
// support node start at most two nodes away), kept two nodes clear of the
// faces so that no periodic wrap or face rule reaches it from outside.
ib_lbm_status plan_split(ib_lbm_sim *s) {
  s->split = false;
  if (!s->overlap || s->bodies.size() != 1) return IB_LBM_OK;
  const ib_lbm_body_desc &d = s->bodies[0].d;
  if (d.motion == IB_LBM_FREE) return IB_LBM_OK;
  const double ax = d.motion == IB_LBM_PRESCRIBED_SIN ? std::fabs(d.amp[0]) : 0.0;
  const double ay = d.motion == IB_LBM_PRESCRIBED_SIN ? std::fabs(d.amp[1]) : 0.0;
  const double r = 0.5 * d.diameter;
  const int lo = d.kernel == IB_LBM_PESKIN4 ? 1 : 0, hi = d.kernel == IB_LBM_PESKIN4 ? 2 : 1;
  const double x0 = std::floor(d.xc - ax - r) - lo - 2, y0 = std::floor(d.yc - ay - r) - lo - 2;
  const double x1 = std::floor(d.xc + ax + r) + hi + 2, y1 = std::floor(d.yc + ay + r) + hi + 2;
  if (x0 < 2 || y0 < 2 || x1 > s->cd.nx - 3 || y1 > s->cd.ny - 3) return IB_LBM_OK;
  const int TX = s->launch.block_x, TY = s->launch.block_y * s->launch.rows_per_thread;
  const int tx0 = (int)x0 / TX, tx1 = (int)x1 / TX, ty0 = (int)y0 / TY, ty1 = (int)y1 / TY;
  const int nbox = (tx1 - tx0 + 1) * (ty1 - ty0 + 1);
  if (nbox >= s->cd.tiles_x * s->cd.tiles_y) return IB_LBM_OK;
  s->hold[0] = tx0;
  s->hold[1] = ty0;
  s->hold[2] = tx1 - tx0 + 1;
  s->hold[3] = ty1 - ty0 + 1;
  s->split = true;
  return IB_LBM_OK;
}

bool body_fast(const HostBody &hb, int spread_mode);
bool body_arcs(const HostBody &hb, int spread_mode);
static bool has_zou_he(const CaseDesc &c);

// Fused steps (one launch per step, step_fused_kernel): a pipelined sim
// (plan_split) whose single body is fixed, DF or MDF on the 1024-thread IB
// kernel, with BGK or TRT and no Zou-He wall.  The hold rectangle is the
// pipelined one, in tiles of the fused shape (fbx x fby, frpt rows per
// thread): the tiles that read the IB force.
ib_lbm_status plan_fused(ib_lbm_sim *s) {
  s->fused = false;
  if (s->one) {
    // what ib_lbm_get_fused reports; every configuration that steps in one
    // launch each does so alike
    const CaseDesc &c = s->cd;
    s->fused = s->split && s->bodies[0].d.motion == IB_LBM_FIXED && s->bodies[0].d.scheme != IB_LBM_DFC &&
               c.collision != IB_LBM_CMMRT && !has_zou_he(c);
    return IB_LBM_OK;
  }
  if (!s->fused_allowed || !s->split || s->bodies.size() != 1) return IB_LBM_OK;
  const HostBody &hb = s->bodies[0];
  const ib_lbm_body_desc &d = hb.d;
  if (d.motion != IB_LBM_FIXED || d.scheme == IB_LBM_DFC || hb.dev.mdf_coupled) return IB_LBM_OK;
  if (body_arcs(hb, s->spread_mode) || !body_fast(hb, s->spread_mode) || hb.dev.max_nodes >= 32768 || !hb.fprev.p || !hb.pstage.p)
    return IB_LBM_OK;
  if (s->cd.collision != IB_LBM_BGK && s->cd.collision != IB_LBM_TRT) return IB_LBM_OK;
  if (has_zou_he(s->cd) || pop_values(s->cd.nx, s->cd.ny) >= (int64_t)INT32_MAX) return IB_LBM_OK;
  const double r = 0.5 * d.diameter;
  const int lo = d.kernel == IB_LBM_PESKIN4 ? 1 : 0, hi = d.kernel == IB_LBM_PESKIN4 ? 2 : 1;
  const int x0 = (int)std::floor(d.xc - r) - lo - 2, y0 = (int)std::floor(d.yc - r) - lo - 2;
  const int x1 = (int)std::floor(d.xc + r) + hi + 2, y1 = (int)std::floor(d.yc + r) + hi + 2;
  const int TX = s->fbx, TY = s->fby * s->frpt;
  s->fhold[0] = x0 / TX;
  s->fhold[1] = y0 / TY;
  s->fhold[2] = x1 / TX - x0 / TX + 1;
  s->fhold[3] = y1 / TY - y0 / TY + 1;
  s->fused = true;
  return IB_LBM_OK;
}

static bool general_zero_gradient(const CaseDesc &c);
int arc_lds_bytes(const BodyDesc &B);

// The arcs of the one-launch steps that may be running: per stream, whose launches
// follow each other, those of the sim or batch with the most.
class ArcBudget {
 public:
  // Whether `who` may have narcs waiting on a stream, with at most `most` in all;
  // gives back what it had.
  bool take(int dev, hipStream_t stream, const void *who, int narcs, int most) {
    std::lock_guard<std::mutex> lk(mu_);
    drop(who);
    if (narcs == 0) return most > 0;
    int others = 0, own = narcs;
    for (auto &st : use_) {
      int n = 0;
      for (auto &o : st.second) n = std::max(n, o.second);
      if (st.first == Key(dev, stream)) own = std::max(own, n);
      else if (st.first.first == dev) others += n;
    }
    if (own + others > most) return false;
    use_[Key(dev, stream)][who] = narcs;
    return true;
  }
  void give_back(const void *who) {
    std::lock_guard<std::mutex> lk(mu_);
    drop(who);
  }

 private:
  using Key = std::pair<int, hipStream_t>;
  void drop(const void *who) {
    for (auto it = use_.begin(); it != use_.end();) {
      it->second.erase(who);
      it = it->second.empty() ? use_.erase(it) : std::next(it);
    }
  }
  std::mutex mu_;
  std::map<Key, std::map<const void *, int>> use_;
};
// (never destroyed: sims may outlive the library's static objects)
ArcBudget &arc_budget = *new ArcBudget;

// One-launch steps (step_one_kernel, step_batch_kernel): sims without bodies,
// or whose bodies are all cut into arcs.  The arcs wait for the tiles they
// depend on while they are resident, so all launches that may run at once share
// step_max_waiting of them (ArcBudget), and a sim on its own has at most kArcMax:
// beyond, one launch is no gain (8 x DF D = 200, 96 arcs, fp32 936 x 458: 105 us
// per step, 45 in several; 8 x DFC D = 130, 72 arcs, 2440 x 1210: 102 and 72; a
// batch of 56 cases, 64 arcs, 5.4 M nodes: 119 and 169).
// All workgroups have the size the arcs need (256 threads without bodies).
// Tiles are 128 nodes wide on lattices of at least 1024 columns (186 against
// 192 us per step on 7175 x 2014, 23.8 against 24.5 us on 1200 x 600) and 64
// below, where a row's last tile is mostly past its end and the hold rectangle
// is a larger share (22.0 against 23.6 us on 400 x 2000 FP64).  One row per
// thread for a sim on its own, whose pass waits for the first tiles; two in a
// batch, whose tiles outlast the passes (12 cases, 3.6 M nodes: 68 us per step
// against 76 with one row and 67 with four).
struct OneShape {
  int threads = 256, lds = 0;
  // false: the bodies do not all run in arcs
  bool add(const std::vector<HostBody> &bodies, int spread_mode) {
    for (auto &hb : bodies) {
      if (!body_arcs(hb, spread_mode)) return false;
      threads = std::max(threads, hb.dev.arc_threads);
      lds = std::max(lds, arc_lds_bytes(hb.dev));
    }
    return true;
  }
};

void fill_step_args(const ib_lbm_sim *s, int threads, int rows, StepOneArgs *out) {
  const CaseDesc &c = s->cd;
  StepOneArgs &a = *out;
  memset(&a, 0, sizeof a);
  a.bx = c.nx >= 1024 ? 128 : 64;
  a.by = threads / a.bx;
  a.lean = lean_args(s, 0, 0);
  a.lean.rpt = rows;
  a.lean.remap = 1;
  const int TX = a.bx, TY = a.by * a.lean.rpt;
  while ((1 << a.tx_shift) < TX) a.tx_shift++;
  while ((1 << a.ty_shift) < TY) a.ty_shift++;
  a.lean.tiles_x = (c.nx + TX - 1) / TX;
  a.lean.ntiles = a.lean.tiles_x * ((c.ny + TY - 1) / TY);
  a.nface = (face_nodes(c.nx, c.ny) + threads - 1) / threads;
  a.cd = c;
  a.c = (const CaseDesc *)s->d_case.p;
  const size_t nb = s->bodies.size();
  for (size_t b = 0; b < kMaxBodiesPerCase; b++) {
    a.arc_first[b + 1] = a.arc_first[b];
    a.hold_first[b + 1] = a.hold_first[b];
    if (b >= nb) continue;
    const HostBody &hb = s->bodies[b];
    // slots for the tiles of its hold rectangle at the speeds a body moves at
    // (a faster one's further tiles are updated in their turn)
    double mv = hb.d.motion == IB_LBM_FIXED ? 0.0 : 1.0;
    if (hb.d.motion == IB_LBM_PRESCRIBED_SIN)
      mv = std::min(64.0, 2.0 * M_PI * std::fabs(hb.d.freq) *
                              std::max(std::fabs(hb.d.amp[0]), std::fabs(hb.d.amp[1])));
    const int w = (int)std::ceil(2.0 * hb.dev.radius + mv) + hb.dev.ns + 8;
    a.arc_first[b + 1] += hb.dev.arc_n;
    a.hold_first[b + 1] += ((w >> a.tx_shift) + 2) * ((w >> a.ty_shift) + 2);
  }
  a.narcs = a.arc_first[kMaxBodiesPerCase];
  a.nhold = a.hold_first[kMaxBodiesPerCase];
}

void plan_one(ib_lbm_sim *s) {
  s->one = false;
  arc_budget.give_back(s);
  if (!s->overlap || !s->fused_allowed) return;
  OneShape sh;
  if (!sh.add(s->bodies, s->spread_mode)) return;
  const bool dfc = !s->bodies.empty() && s->bodies[0].dev.scheme == kDFC;
  if (dfc && sh.threads > 512) return;
  fill_step_args(s, sh.threads, 1, &s->one_args);
  s->one_threads = sh.threads;
  s->one_lds = sh.lds;
  s->one_face = has_zou_he(s->cd) ? 2 : (general_zero_gradient(s->cd) ? 1 : 0);
  s->one = s->one_args.narcs <= kArcMax &&
           arc_budget.take(s->dev, s->stream, s, s->one_args.narcs,
                           step_max_waiting(s->cd.precision, s->one_face, dfc, false, sh.threads, sh.lds));
}

// A body runs on the 1024-thread IB kernel when it is DF/MDF, its workspace
// fits in LDS and spreading is by gather; the choice depends on the body
// alone, so a body's results do not depend on its batch-mates.
bool body_fast(const HostBody &hb, int spread_mode) {
  return spread_mode == 0 && hb.dev.scheme != kDFC && hb.dev.ws_doubles * 8 <= ibm_max_lds_bytes();
}

// Whether a body's pass runs in arcs (the choice depends on the body and the
// spreading variant alone, so its results do not depend on its batch-mates).
bool body_arcs(const HostBody &hb, int spread_mode) { return spread_mode == 0 && hb.dev.arc_n > 0; }

// Cut a body's pass into arcs (arc_device.h).  Markers that share a support
// node are less than ns apart in x and in y, so less than ns sqrt 2: on the
// circle of radius R that makes |l - k| less than (n_b / pi) asin(ns sqrt 2 /
// (2 R)); the band half-width bw is the largest whole number below it (1e-6 for
// the rounding of the markers; at least 1).  One marker more on each side costs
// as much margin in every pass: 2000 x 800 MDF P4 takes 24.4 us per step, 25.2
// with it.
// A marker takes ns lanes, so a workgroup of t threads holds t / ns markers: a
// body of at most that many is one arc, else the own markers of an arc are what
// the margins on both sides leave.  The margin is bw for DF, 2 bw for DFC (whose
// correction scale sums over the markers around each one) and N bw for N
// marker-space MDF passes.  Adaptive MDF needs the residual of all markers in
// every pass, so it runs as one arc or not at all; coupled MDF, Eq. D1 bodies,
// very small circles and bodies with very dense markers keep the one-workgroup
// kernels.
// The smallest workgroup whose margins leave a quarter of its markers is
// taken: a pass is bound by instruction issue, and a wave more on each SIMD
// costs as much as the pass of the wave that is there.  At an eighth more
// bodies take many arcs of 256 threads, whose repeated margins hold up the
// tiles: 2000 x 800 MDF P4 fp32 23.9 us per step instead of 24.4, but fp64 36.5
// instead of 35.5 and a batch of twelve 68.9 instead of 66.9.
// FP32 DFC with the Peskin kernel is one arc as long as 512 threads hold its
// markers: the arcs' meeting between reads and writes costs more than the second
// wave per SIMD (free disk, D = 30, 17.8 us per step in three arcs, 16.6 in one;
// fixed, plain steps, 25.8 and 25.2).  FP64 keeps its arcs, and with them the order
// of its sums; with the hat kernel a fixed disk is slower in one (D = 78 fp32 14.5
// and 15.2).
void plan_arcs(BodyDesc *B) {
  B->arc_n = 0;
  if (B->mdf_coupled || B->udes != kUdRigid) return;
  const double q = B->ns * std::sqrt(2.0) / (2.0 * B->radius);
  if (!(q < 1.0)) return;
  const int nb = B->nb, ns = B->ns, bw = std::max((int)std::ceil(nb / M_PI * std::asin(q) + 1e-6) - 1, 1);
  if (bw > 15 || 2 * bw + 1 >= nb) return;
  const bool mdf = B->scheme == kMDF, adapt = mdf && B->mdf_tol > 0;
  const int regs = ns == 4 ? kArcBandRegsP4 : kArcBandRegsHat;
  if (mdf && 2 * bw + 1 > regs * ns) return;
  const int64_t halo = mdf ? (int64_t)B->mdf_iters * bw : (B->scheme == kDFC ? 2 * bw : bw);
  for (int t : kArcThreads) {
    const int cap = t / ns;
    int own = 0, n = 0;
    if (nb <= cap) {
      own = nb;
      n = 1;
    } else if (!adapt && cap - 2 * halo >= cap / 4 && !(B->scheme == kDFC && ns == 4 && B->pop_bytes == 4 && nb <= 512 / ns)) {
      n = (int)((nb + cap - 2 * halo - 1) / (cap - 2 * halo));
      own = (nb + n - 1) / n;
      n = (nb + own - 1) / own;
    }
    if (B->scheme == kDFC && t > 512) break;
    if (n == 0 || n > kArcMax) continue;
    const int nl = n == 1 ? nb : own + 2 * (int)halo;
    if (n > 1 && nl > nb) continue;
    if (arc_lds_doubles(B->scheme, ns, bw, nl) * 8 > 64 * 1024) continue;
    B->arc_n = n;
    B->arc_own = own;
    B->arc_halo = (int)halo;
    B->arc_bw = bw;
    B->arc_threads = t;
    return;
  }
}

int arc_lds_bytes(const BodyDesc &B) {
  const int nl = B.arc_n == 1 ? B.nb : B.arc_own + 2 * B.arc_halo;
  return arc_lds_doubles(B.scheme, B.ns, B.arc_bw, nl) * 8;
}

// The slots of `n` cases' bodies in launch order (see IbSlots).  all_fast:
// per case, whether a coupled case runs on the 1024-thread kernel.
struct SlotLists {
  std::vector<IbmSlot> arcs[3], fast, general;
  IbSlots ib;
  void add(const std::vector<HostBody> &bodies, int cas, int spread_mode) {
    const int n = std::max<int>(1, (int)bodies.size());
    if (bodies.empty()) general.push_back({cas, -1, 1, 0});
    // the bodies of a coupled MDF case meet during their passes, so they run
    // in one launch: the fast instance only if every one of them fits it
    bool all_fast = !bodies.empty();
    for (auto &hb : bodies) all_fast &= body_fast(hb, spread_mode);
    const bool coupled = !bodies.empty() && bodies[0].dev.mdf_coupled;
    for (int b = 0; b < (int)bodies.size(); b++) {
      const BodyDesc &B = bodies[b].dev;
      if (body_arcs(bodies[b], spread_mode)) {
        const int t = B.arc_threads == 256 ? 0 : (B.arc_threads == 512 ? 1 : 2);
        for (int a = 0; a < B.arc_n; a++) arcs[t].push_back({cas, b, n, a});
        ib.arc_lds[t] = std::max(ib.arc_lds[t], arc_lds_bytes(B));
        continue;
      }
      ((coupled ? all_fast : body_fast(bodies[b], spread_mode)) ? fast : general).push_back({cas, b, n, 0});
      if (B.ws_doubles * 8 <= ibm_max_lds_bytes()) ib.lds = std::max(ib.lds, B.ws_doubles * 8);
    }
  }
  std::vector<IbmSlot> finish() {
    std::vector<IbmSlot> all;
    for (int t = 0; t < 3; t++) {
      ib.arcs[t] = (int)arcs[t].size();
      all.insert(all.end(), arcs[t].begin(), arcs[t].end());
    }
    ib.fast = (int)fast.size();
    all.insert(all.end(), fast.begin(), fast.end());
    ib.general = (int)general.size();
    all.insert(all.end(), general.begin(), general.end());
    return all;
  }
};

// The IB launches of a step (bodies of one case may sit in several; the last
// body to finish, in whichever launch, completes the case).
hipError_t launch_ibm_slots(int precision, const CaseDesc *cases, const IbmSlot *slots, const IbSlots &ib,
                            int spread_mode, int threads, hipStream_t stream) {
  hipError_t e = hipSuccess;
  for (int t = 0; t < 3 && e == hipSuccess; t++) {
    e = launch_ibm_arcs(precision, cases, slots, ib.arcs[t], ib.arc_lds[t], kArcThreads[t], stream);
    slots += ib.arcs[t];
  }
  if (e == hipSuccess)
    e = launch_ibm(precision, cases, slots, ib.fast, ib.lds, spread_mode, 1, 1, nullptr, threads, stream);
  if (e == hipSuccess)
    e = launch_ibm(precision, cases, slots + ib.fast, ib.general, ib.lds, spread_mode, 0, 1, nullptr,
                   threads, stream);
  return e;
}

ib_lbm_status build_sim_tables(ib_lbm_sim *s) {
  if (!s->tables_dirty) return IB_LBM_OK;
  // steps still queued read the tables (and replay the graphs) rewritten here
  HIPCHK(s, hipStreamSynchronize(s->stream));
  ib_lbm_status st0;
  std::vector<BodyDesc> bd;
  for (auto &hb : s->bodies) bd.push_back(hb.dev);
  SlotLists lists;
  lists.add(s->bodies, 0, s->spread_mode);
  const std::vector<IbmSlot> slots = lists.finish();
  if (!bd.empty()) {
    if (!s->d_bodies.p || s->d_bodies.bytes < bd.size() * sizeof(BodyDesc)) {
      dev_free(s, &s->d_bodies);
      ib_lbm_status st = dev_alloc(s, &s->d_bodies, bd.size() * sizeof(BodyDesc));
      if (st) return st;
    }
    HIPCHK(s, hipMemcpy(s->d_bodies.p, bd.data(), bd.size() * sizeof(BodyDesc), hipMemcpyHostToDevice));
  }
  s->cd.bodies = (BodyDesc *)s->d_bodies.p;
  s->cd.nbodies = (int)bd.size();
  fill_case_tiles(&s->cd, s->launch);
  if (!s->d_case.p) {
    ib_lbm_status st = dev_alloc(s, &s->d_case, sizeof(CaseDesc));
    if (st) return st;
    st = dev_alloc(s, &s->d_prefix, sizeof(int32_t) * 4);
    if (st) return st;
  }
  if (s->d_slots.bytes < slots.size() * sizeof(IbmSlot)) {
    dev_free(s, &s->d_slots);
    ib_lbm_status st = dev_alloc(s, &s->d_slots, slots.size() * sizeof(IbmSlot));
    if (st) return st;
  }
  HIPCHK(s, hipMemcpy(s->d_case.p, &s->cd, sizeof(CaseDesc), hipMemcpyHostToDevice));
  // tile prefix {0, tiles}, then face workgroup prefix {0, face workgroups}
  int32_t pre[4] = {0, s->cd.tiles_x * s->cd.tiles_y, 0, face_blocks(s->cd.nx, s->cd.ny)};
  HIPCHK(s, hipMemcpy(s->d_prefix.p, pre, sizeof pre, hipMemcpyHostToDevice));
  HIPCHK(s, hipMemcpy(s->d_slots.p, slots.data(), slots.size() * sizeof(IbmSlot), hipMemcpyHostToDevice));
  s->ib = lists.ib;
  if ((st0 = plan_split(s))) return st0;
  plan_one(s);
  if ((st0 = plan_fused(s))) return st0;
  s->tables_dirty = false;
  drop_graphs(s);
  return IB_LBM_OK;
}

EventPair take_pair(Timing &t) {
  if (!t.pool.empty()) {
    EventPair p = t.pool.back();
    t.pool.pop_back();
    return p;
  }
  EventPair p;
  // timing events around device work: a device-scope release keeps the
  // cache writeback of a system-scope release out of the measured span
  (void)hipEventCreateWithFlags(&p.a, hipEventReleaseToDevice);
  (void)hipEventCreateWithFlags(&p.b, hipEventReleaseToDevice);
  return p;
}

// Zero-gradient faces other than the east one need the general copy rules
// of the face kernel.
static bool general_zero_gradient(const CaseDesc &c) {
  return c.bc[0] == kZeroGradient || c.bc[2] == kZeroGradient || c.bc[3] == kZeroGradient;
}

static bool has_zou_he(const CaseDesc &c) {
  return c.bc[0] == kZouHe || c.bc[1] == kZouHe || c.bc[2] == kZouHe || c.bc[3] == kZouHe;
}

// Enqueue one step of a sim on `stream` whose input lattice is cur:
// collide-stream, face nodes, Zou-He walls, then the IB pass.
ib_lbm_status enqueue_sim_step(ib_lbm_sim *s, bool timed, hipStream_t stream, int cur) {
  LaunchShape sh{s->launch.block_x, s->launch.block_y, s->launch.rows_per_thread, s->launch.xcd_remap};
  EventPair p0{}, p1{};
  if (timed) {
    p0 = take_pair(s->timing);
    HIPCHK(s, hipEventRecord(p0.a, stream));
  }
  HIPCHK(s, launch_collide_stream_lean(s->cd.precision, s->cd.collision, lean_args(s, cur, 1), 0, sh,
                                       stream));
  if (timed) {
    HIPCHK(s, hipEventRecord(p0.b, stream));
    s->timing.ev[0].push_back(p0);
  }
  HIPCHK(s, launch_collide_stream_faces(s->cd.precision, s->cd.collision, (const CaseDesc *)s->d_case.p,
                                        (const int32_t *)s->d_prefix.p + 2, 1,
                                        face_blocks(s->cd.nx, s->cd.ny), cur, 1,
                                        general_zero_gradient(s->cd), stream));
  if (has_zou_he(s->cd))
    HIPCHK(s, launch_zou_he(s->cd.precision, (const CaseDesc *)s->d_case.p, s->cd.nx, s->cd.ny, cur,
                            stream));
  if (timed) {
    p1 = take_pair(s->timing);
    HIPCHK(s, hipEventRecord(p1.a, stream));
  }
  HIPCHK(s, launch_ibm_slots(s->cd.precision, (const CaseDesc *)s->d_case.p, (const IbmSlot *)s->d_slots.p,
                             s->ib, s->spread_mode, s->launch.ib_threads, stream));
  if (timed) {
    HIPCHK(s, hipEventRecord(p1.b, stream));
    s->timing.ev[1].push_back(p1);
  }
  return IB_LBM_OK;
}

ib_lbm_status read_state(ib_lbm_sim *s, CaseState *cs);

// The two streams and the events of pipelined steps, created at the first
// pipelined step (sims stepped through a batch never need them).
ib_lbm_status ensure_pipe_streams(ib_lbm_sim *s) {
  if (!s->lq) {
    // The far-tile stream leaves one compute unit per IB workgroup to the
    // other stream, so that an IB pass never waits for a free unit behind a
    // full far-tile launch.
    int dev = 0, ncu = 0;
    HIPCHK(s, hipGetDevice(&dev));
    HIPCHK(s, hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    std::vector<uint32_t> mask((ncu + 31) / 32, 0u);
    for (int i = 0; i < ncu - 1; i++) mask[i / 32] |= 1u << (i % 32);
    if (ncu < 2 ||
        hipExtStreamCreateWithCUMask(&s->lq, (uint32_t)mask.size(), mask.data()) != hipSuccess) {
      (void)hipGetLastError();
      s->lq = nullptr;
      HIPCHK(s, hipStreamCreateWithFlags(&s->lq, hipStreamNonBlocking));
    }
  }
  if (!s->iq) HIPCHK(s, hipStreamCreateWithFlags(&s->iq, hipStreamNonBlocking));
  if (!s->ticket.p) {
    // the replicated IB workgroup's counter, advanced by every copy
    ib_lbm_status st = dev_alloc(s, &s->ticket, 256);
    if (st) return st;
    HIPCHK(s, hipMemsetAsync(s->ticket.p, 0, 256, s->stream));
  }
  // the events only order work between streams of this device: a
  // device-scope release suffices (the default system-scope release writes
  // back and invalidates the caches at every record)
  const unsigned evf = hipEventDisableTiming | hipEventReleaseToDevice;
  if (!s->ev_start) HIPCHK(s, hipEventCreateWithFlags(&s->ev_start, evf));
  if (!s->ev_lq) HIPCHK(s, hipEventCreateWithFlags(&s->ev_lq, evf));
  if (!s->ev_iq) HIPCHK(s, hipEventCreateWithFlags(&s->ev_iq, evf));
  if (!s->ev_near) HIPCHK(s, hipEventCreateWithFlags(&s->ev_near, evf));
  if (!s->ev_far) HIPCHK(s, hipEventCreateWithFlags(&s->ev_far, evf));
  return IB_LBM_OK;
}

// The IB pass of a pipelined step's single body: its arcs, or one copy of
// its workgroup per XCD, the first of which to start runs the pass (the far
// tiles on the other stream fill the chip).
hipError_t launch_ibm_pipelined(ib_lbm_sim *s, hipStream_t stream, LaunchTarget *ns) {
  const CaseDesc *dc = (const CaseDesc *)s->d_case.p;
  const IbmSlot *slots = (const IbmSlot *)s->d_slots.p;
  for (int t = 0; t < 3; t++)
    if (s->ib.arcs[t])
      return launch_ibm_arcs(s->cd.precision, dc, slots, s->ib.arcs[t], s->ib.arc_lds[t], kArcThreads[t],
                             stream, ns);
  return launch_ibm(s->cd.precision, dc, slots, 1, s->ib.lds, s->spread_mode, s->ib.fast, 8,
                    (uint32_t *)s->ticket.p, s->launch.ib_threads, stream, ns);
}

// Enqueue nsteps pipelined steps after the work already on `main`, the
// first with input lattice cur0.  Step n: the hold tiles and then the IB
// pass on iq, the far tiles, face nodes and Zou-He walls on lq.  The far
// tiles of step n follow the hold tiles of step n-1 (which push into far
// nodes and whose inputs the far tiles of step n overwrite); the hold tiles
// of step n follow the far tiles and face nodes of step n-1 for the same
// two reasons, and the IB pass of step n-1 by stream order.  The Zou-He
// wall pass of step n rebuilds wall nodes from the pushes of every node
// next to them, so it also follows the hold tiles of step n (rounded to
// whole tiles, the hold rectangle can reach row 1 or column 1).  `main`
// then waits for both streams.  Nothing here reads device state.
ib_lbm_status enqueue_pipelined(ib_lbm_sim *s, int64_t nsteps, bool timed, hipStream_t main, int cur0) {
  if (nsteps <= 0) return IB_LBM_OK;
  LaunchShape sh{s->launch.block_x, s->launch.block_y, s->launch.rows_per_thread, s->launch.xcd_remap};
  const bool zh = has_zou_he(s->cd);
  HIPCHK(s, hipEventRecord(s->ev_start, main));
  HIPCHK(s, hipStreamWaitEvent(s->lq, s->ev_start, 0));
  HIPCHK(s, hipStreamWaitEvent(s->iq, s->ev_start, 0));
  const CaseDesc *dc = (const CaseDesc *)s->d_case.p;
  for (int64_t i = 0; i < nsteps; i++) {
    const int cur = cur0 ^ (int)(i & 1);
    const bool last = i + 1 == nsteps;
    const LeanArgs la = lean_args(s, cur, 0);
    EventPair p0{}, p1{};
    // Each wait is enqueued before its event is recorded again for step i:
    // the hold tiles of step i after the face nodes (and so the far tiles)
    // of step i-1, the far tiles of step i after the hold tiles of step i-1.
    if (i > 0) {
      HIPCHK(s, hipStreamWaitEvent(s->iq, s->ev_far, 0));
      HIPCHK(s, hipStreamWaitEvent(s->lq, s->ev_near, 0));
    }
    if (timed) {
      p0 = take_pair(s->timing);
      HIPCHK(s, hipEventRecord(p0.a, s->lq));
    }
    HIPCHK(s, launch_collide_stream_lean(s->cd.precision, s->cd.collision, la, 2, sh, s->lq));
    if (timed) {
      HIPCHK(s, hipEventRecord(p0.b, s->lq));
      s->timing.ev[0].push_back(p0);
    }
    // face nodes lie outside the hold rectangle's reach (plan_split); the
    // events ride on the launches themselves
    LaunchTarget face_done, hold_done;
    face_done.done = s->ev_far;
    hold_done.done = s->ev_near;
    HIPCHK(s, launch_collide_stream_faces(s->cd.precision, s->cd.collision, dc,
                                          (const int32_t *)s->d_prefix.p + 2, 1,
                                          face_blocks(s->cd.nx, s->cd.ny), cur, 0,
                                          general_zero_gradient(s->cd), s->lq, &face_done));
    HIPCHK(s, launch_collide_stream_lean(s->cd.precision, s->cd.collision, la, 1, sh, s->iq, &hold_done));
    if (zh) {
      // every push into a wall node, hold tiles included, has landed
      LaunchTarget zou_done;
      zou_done.done = last ? s->ev_lq : nullptr;
      HIPCHK(s, hipStreamWaitEvent(s->lq, s->ev_near, 0));
      HIPCHK(s, launch_zou_he(s->cd.precision, dc, s->cd.nx, s->cd.ny, cur, s->lq, &zou_done));
    }
    if (timed) {
      p1 = take_pair(s->timing);
      HIPCHK(s, hipEventRecord(p1.a, s->iq));
    }
    LaunchTarget ib_done;
    ib_done.done = last ? s->ev_iq : nullptr;
    HIPCHK(s, launch_ibm_pipelined(s, s->iq, &ib_done));
    if (timed) {
      HIPCHK(s, hipEventRecord(p1.b, s->iq));
      s->timing.ev[1].push_back(p1);
    }
  }
  // the last launch on each stream carries the event the sim's stream waits for
  HIPCHK(s, hipStreamWaitEvent(main, zh ? s->ev_lq : s->ev_far, 0));
  HIPCHK(s, hipStreamWaitEvent(main, s->ev_iq, 0));
  return IB_LBM_OK;
}

// The pipelined steps as an explicitly built graph: the same kernels and
// arguments as enqueue_pipelined, with its event ordering as node
// dependencies.  Far tiles of step i after the face nodes (and Zou-He walls)
// of step i-1 and the hold tiles of step i-1; face nodes after the far
// tiles; hold tiles after the face nodes and the IB pass of step i-1;
// Zou-He walls after the face nodes and the hold tiles of the step; the IB
// pass after the hold tiles.  Launching the graph costs the host one call,
// where the events cost it two cross-stream hops per step (about 17 us
// each); the far tiles lose the compute-unit mask of their stream, which the
// IB pass's per-XCD copies make up for.  Stream capture is not used.
ib_lbm_status build_pipelined_graph(ib_lbm_sim *s, int64_t nsteps, int cur0, hipGraphExec_t *out) {
  LaunchShape sh{s->launch.block_x, s->launch.block_y, s->launch.rows_per_thread, s->launch.xcd_remap};
  const CaseDesc *dc = (const CaseDesc *)s->d_case.p;
  const bool zh = has_zou_he(s->cd);
  hipGraph_t g = nullptr;
  HIPCHK(s, hipGraphCreate(&g, 0));
  hipGraphNode_t prev_lq = nullptr, prev_hold = nullptr, prev_ib = nullptr;
  hipError_t e = hipSuccess;
  auto add = [&](std::initializer_list<hipGraphNode_t> deps, auto &&launch) -> hipGraphNode_t {
    hipGraphNode_t d[4];
    size_t n = 0;
    for (hipGraphNode_t x : deps)
      if (x) d[n++] = x;
    LaunchTarget ns{g, d, n, nullptr};
    if (e == hipSuccess) e = launch(&ns);
    return ns.node;
  };
  for (int64_t i = 0; i < nsteps && e == hipSuccess; i++) {
    const int cur = cur0 ^ (int)(i & 1);
    const LeanArgs la = lean_args(s, cur, 0);
    hipGraphNode_t far = add({prev_lq, prev_hold}, [&](LaunchTarget *ns) {
      return launch_collide_stream_lean(s->cd.precision, s->cd.collision, la, 2, sh, nullptr, ns);
    });
    hipGraphNode_t face = add({far ? far : prev_lq, far ? nullptr : prev_hold}, [&](LaunchTarget *ns) {
      return launch_collide_stream_faces(s->cd.precision, s->cd.collision, dc,
                                         (const int32_t *)s->d_prefix.p + 2, 1,
                                         face_blocks(s->cd.nx, s->cd.ny), cur, 0,
                                         general_zero_gradient(s->cd), nullptr, ns);
    });
    hipGraphNode_t lq_end = face ? face : far;
    hipGraphNode_t hold = add({prev_lq, prev_ib}, [&](LaunchTarget *ns) {
      return launch_collide_stream_lean(s->cd.precision, s->cd.collision, la, 1, sh, nullptr, ns);
    });
    if (zh) {
      hipGraphNode_t z = add({lq_end, hold}, [&](LaunchTarget *ns) {
        return launch_zou_he(s->cd.precision, dc, s->cd.nx, s->cd.ny, cur, nullptr, ns);
      });
      if (z) lq_end = z;
    }
    hipGraphNode_t ib = add({hold ? hold : prev_ib}, [&](LaunchTarget *ns) {
      return launch_ibm_pipelined(s, nullptr, ns);
    });
    if (lq_end) prev_lq = lq_end;
    if (hold) prev_hold = hold;
    if (ib) prev_ib = ib;
  }
  if (e == hipSuccess) e = hipGraphInstantiate(out, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  HIPCHK(s, e);
  return IB_LBM_OK;
}

// The nodes whose pushes reach the support of the fused sim's body, and
// their push map (BodyDesc::src), from the support the device
// built at the body's first IB pass (the hot part of its cached tables:
// the support node list nxy and its length S).  Sorted by row and column,
// so that the pass reads the lattice in runs.
ib_lbm_status build_fused_sources(ib_lbm_sim *s) {
  HostBody &hb = s->bodies[0];
  const BodyDesc &B = hb.dev;
  std::vector<double> hot((size_t)B.ws_tab_hot);
  HIPCHK(s, hipStreamSynchronize(s->stream));
  HIPCHK(s, hipMemcpy(hot.data(), hb.tab.p, hot.size() * 8, hipMemcpyDeviceToHost));
  const int32_t *ints = (const int32_t *)(hot.data() + ws_table_doubles(B.nb, B.ns));
  const int32_t *nxy = ints + B.nb * B.ns;
  const int S = ints[B.nb * B.ns + B.max_nodes + ell_width(B.ns) * B.max_nodes];
  if (S <= 0 || S > B.max_nodes) {
    set_err(&s->err, "fused step: the body's support table is not built");
    return IB_LBM_E_STATE;
  }
  std::map<int64_t, int> sup;  // (y, x) -> support index
  auto key = [](int x, int y) { return ((int64_t)y << 32) | (uint32_t)x; };
  for (int j = 0; j < S; j++) sup[key(nxy[j] & 0xffff, nxy[j] >> 16)] = j;
  static const int ex[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
  static const int ey[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
  std::map<int64_t, int> src;  // (y, x) of every node that pushes into the support
  for (int j = 0; j < S; j++) {
    const int x = nxy[j] & 0xffff, y = nxy[j] >> 16;
    for (int i = 0; i < 9; i++) src[key(x - ex[i], y - ey[i])] = 0;
  }
  const int n = (int)src.size();
  std::vector<SrcNode> rec(n);
  int u = 0;
  for (auto &e : src) {
    const int y = (int)(e.first >> 32), x = (int)(uint32_t)e.first;
    if (x < 1 || x > s->cd.nx - 3 || y < 1 || y > s->cd.ny - 2) {
      set_err(&s->err, "fused step: a support neighbour is not an inner node");
      return IB_LBM_E_STATE;
    }
    SrcNode &r = rec[u];
    memset(&r, 0, sizeof r);
    r.off = (int32_t)pop_node(x, y, s->cd.nseg);
    for (int i = 0; i < 9; i++) {
      auto it = sup.find(key(x + ex[i], y + ey[i]));
      r.map[i] = (int16_t)(it == sup.end() ? -1 : it->second);
    }
    u++;
  }
  dev_free(s, &hb.src);
  ib_lbm_status st = dev_alloc(s, &hb.src, (size_t)n * sizeof(SrcNode));
  if (st) return st;
  HIPCHK(s, hipMemcpy(hb.src.p, rec.data(), (size_t)n * sizeof(SrcNode), hipMemcpyHostToDevice));
  hb.dev.src = (const SrcNode *)hb.src.p;
  hb.dev.n_src = n;
  HIPCHK(s, hipMemcpy(s->d_bodies.p, &hb.dev, sizeof(BodyDesc), hipMemcpyHostToDevice));
  hb.src_ready = true;
  return IB_LBM_OK;
}

// Enqueue nsteps fused steps on `stream` from input lattice cur0: one
// launch each, ordered by the stream alone (see step_fused_kernel).
ib_lbm_status enqueue_fused(ib_lbm_sim *s, int64_t nsteps, hipStream_t stream, int cur0) {
  for (int64_t i = 0; i < nsteps; i++) {
    const int cur = cur0 ^ (int)(i & 1);
    FusedArgs fa;
    memset(&fa, 0, sizeof fa);
    fa.lean = lean_args(s, cur, 0);
    const int TX = s->fbx, TY = s->fby * s->frpt;
    fa.lean.tiles_x = (s->cd.nx + TX - 1) / TX;
    fa.lean.ntiles = fa.lean.tiles_x * ((s->cd.ny + TY - 1) / TY);
    fa.lean.rpt = s->frpt;
    fa.lean.remap = 1;
    fa.lean.htx0 = s->fhold[0];
    fa.lean.hty0 = s->fhold[1];
    fa.lean.hntx = s->fhold[2];
    fa.lean.hnty = s->fhold[3];
    fa.c = (const CaseDesc *)s->d_case.p;
    fa.face_prefix = (const int32_t *)s->d_prefix.p + 2;
    fa.nface = face_blocks(s->cd.nx, s->cd.ny);
    fa.gzg = general_zero_gradient(s->cd);
    fa.bx = s->fbx;
    fa.by = s->fby;
    fa.cur = cur;
    fa.seq = (int32_t)(++s->fused_seq);
    fa.nsrc = (s->bodies[0].dev.n_src + kFusedThreads - 1) / kFusedThreads;
    // FP32: the tiles wait for the IB pass's kinematics and tables (28.1 us
    // per step on the 2000x800 cylinder); FP64: the tiles bound the launch
    // and start at once (37.6 against 42.4 us with the same wait)
    fa.gated = s->cd.precision == IB_LBM_FP32_SHIFTED ? 1 : 0;
    fa.cd = s->cd;
    fa.bd = s->bodies[0].dev;
    HIPCHK(s, launch_step_fused(s->cd.precision, s->cd.collision, fa, s->ib.lds, stream));
  }
  return IB_LBM_OK;
}

// Enqueue nsteps one-launch steps on `stream` from input lattice cur0.  A step
// leaves its Zou-He wall nodes open: the next one closes what it reads, and
// the last one's are closed here.
ib_lbm_status enqueue_one(ib_lbm_sim *s, int64_t nsteps, hipStream_t stream, int cur0) {
  StepOneArgs a = s->one_args;
  for (int64_t i = 0; i < nsteps; i++) {
    const int cur = cur0 ^ (int)(i & 1);
    a.cur = cur;
    a.lean.src = s->cd.f[cur];
    a.lean.dst = s->cd.f[cur ^ 1];
    a.lean.halt = &s->cd.state->halt[cur];
    HIPCHK(s, launch_step_one(s->cd.precision, s->one_face, !s->bodies.empty() && s->bodies[0].dev.scheme == kDFC,
                              a, s->one_threads, s->one_lds, stream));
  }
  if (has_zou_he(s->cd) && nsteps > 0)
    HIPCHK(s, launch_zou_he(s->cd.precision, (const CaseDesc *)s->d_case.p, s->cd.nx, s->cd.ny, -2, stream));
  return IB_LBM_OK;
}

// Enqueue nsteps steps of a sim on `stream` from input lattice cur0,
// pipelined when the sim allows it and `pipelined` is set.
ib_lbm_status enqueue_steps(ib_lbm_sim *s, int64_t nsteps, bool timed, hipStream_t stream, int cur0,
                            bool pipelined) {
  const bool one = s->one && s->hold_ready && !timed;
  const bool fused = s->fused && !s->one && s->bodies[0].src_ready && !timed;
  if (nsteps > 0)
    s->form = one ? IB_LBM_STEP_ONE
                  : (fused ? IB_LBM_STEP_FUSED
                           : (s->split && pipelined ? IB_LBM_STEP_PIPELINED : IB_LBM_STEP_PLAIN));
  if (one) return enqueue_one(s, nsteps, stream, cur0);
  bool arcs = true;
  for (auto &hb : s->bodies) arcs &= body_arcs(hb, s->spread_mode);
  s->hold_ready = nsteps > 0 ? arcs : s->hold_ready;
  if (fused) return enqueue_fused(s, nsteps, stream, cur0);
  if (s->split && pipelined) return enqueue_pipelined(s, nsteps, timed, stream, cur0);
  for (int64_t i = 0; i < nsteps; i++) {
    ib_lbm_status st = enqueue_sim_step(s, timed, stream, cur0 ^ (int)(i & 1));
    if (st) return st;
  }
  return IB_LBM_OK;
}

ib_lbm_status usable(ib_lbm_sim *s) {
  if (!s) return IB_LBM_E_INVALID;
  if (s->broken) return IB_LBM_E_STATE;
  return IB_LBM_OK;
}

ib_lbm_status read_state(ib_lbm_sim *s, CaseState *cs) {
  HIPCHK(s, hipStreamSynchronize(s->stream));
  HIPCHK(s, hipMemcpy(cs, s->state.p, sizeof(CaseState), hipMemcpyDeviceToHost));
  s->host_cur = cs->cur;
  s->halted = (cs->flags & kCaseHalted) != 0;
  return IB_LBM_OK;
}

}  // namespace

extern "C" {

uint32_t ib_lbm_abi_version(void) { return IB_LBM_ABI_VERSION; }

size_t ib_lbm_footprint(const ib_lbm_config *cfg, int32_t n_bodies, const int32_t *n_markers) {
  if (!cfg) return 0;
  const size_t elem = cfg->precision == IB_LBM_FP64 ? 8 : 4;
  const size_t n = (size_t)cfg->nx * cfg->ny;
  bool has_zou = false;
  for (int f = 0; f < 4; f++) has_zou |= cfg->bc[f] == IB_LBM_ZOU_HE;
  const size_t lat = cfg->nx > 0 && cfg->ny > 0 ? (size_t)pop_values(cfg->nx, cfg->ny) : 0;
  size_t bytes = 2 * lat * elem + 2 * n * elem + sizeof(CaseState) + sizeof(CaseDesc) + 256 +
                 (has_zou ? 2 * (size_t)wall_nodes(cfg->nx, cfg->ny) : 0);
  const int hist = cfg->history_capacity > 0 ? cfg->history_capacity : 4096;
  for (int b = 0; b < n_bodies; b++) {
    const int nb = n_markers ? n_markers[b] : 256;
    // workspace upper estimate (P4), marker tables, history
    const double D = nb / M_PI;
    const int mr = (int)std::ceil(D) + 12, mn = (int)(8 * M_PI * D + 8 * mr + 64);
    // (the MDF workspace may carry the marker-space velocities, 2 n_b)
    bytes += (size_t)(std::max(ws_doubles_for(kDFC, nb, 4, mr, mn, (int)elem),
                               ws_doubles_for(kMDF, nb, 4, mr, mn, (int)elem) +
                                   std::max(2 * nb, ws_coupled_doubles(nb, mn))) +
                      ws_tab_total(kMDF, nb, 4, mr, mn) + 2 * mn) * 8 +
             (size_t)nb * (8 + 1 + 2) * 8 +
             (size_t)hist * kHistCols * 8 + sizeof(BodyState) + sizeof(BodyDesc) +
             (size_t)kArcMax * (64 + sizeof(IbmSlot));
  }
  return bytes;
}

ib_lbm_status ib_lbm_create(const ib_lbm_config *cfg, ib_lbm_sim **out) {
  if (!cfg || !out) return IB_LBM_E_INVALID;
  *out = nullptr;
  ib_lbm_sim *s = new ib_lbm_sim();
  host_copy_retain();
  s->cfg = *cfg;
  auto fail = [&](ib_lbm_status st, const char *msg) {
    fprintf(stderr, "ib_lbm_create: %s\n", msg);
    ib_lbm_destroy(s);
    return st;
  };
  if (cfg->abi_version != IB_LBM_ABI_VERSION) return fail(IB_LBM_E_INVALID, "abi_version mismatch");
  if (cfg->nx < 3 || cfg->ny < 3 || (int64_t)cfg->nx * cfg->ny >= (1ll << 31) || cfg->nx >= 65535 ||
      cfg->ny >= 32767)
    return fail(IB_LBM_E_INVALID, "lattice size out of range");
  if (!(cfg->tau > 0.5) || !std::isfinite(cfg->tau)) return fail(IB_LBM_E_INVALID, "tau must exceed 1/2");
  if (cfg->precision != IB_LBM_FP64 && cfg->precision != IB_LBM_FP32_SHIFTED)
    return fail(IB_LBM_E_INVALID, "unknown precision");
  if (cfg->collision < IB_LBM_BGK || cfg->collision > IB_LBM_CMMRT)
    return fail(IB_LBM_E_INVALID, "unknown collision");
  for (int f = 0; f < 4; f++)
    if (cfg->bc[f] < IB_LBM_PERIODIC || cfg->bc[f] > IB_LBM_ZOU_HE)
      return fail(IB_LBM_E_INVALID, "unknown face closure");
  {
    bool zh = false, other = false;
    for (int f = 0; f < 4; f++) {
      zh |= cfg->bc[f] == IB_LBM_ZOU_HE;
      other |= cfg->bc[f] != IB_LBM_ZOU_HE && cfg->bc[f] != IB_LBM_PERIODIC;
    }
    if (zh && other)
      return fail(IB_LBM_E_INVALID, "Zou-He walls combine only with other Zou-He walls or periodic faces");
  }
  if ((cfg->bc[0] == IB_LBM_PERIODIC) != (cfg->bc[1] == IB_LBM_PERIODIC) ||
      (cfg->bc[2] == IB_LBM_PERIODIC) != (cfg->bc[3] == IB_LBM_PERIODIC))
    return fail(IB_LBM_E_INVALID, "periodic faces must come in pairs");

  if (cfg->bc[2] == IB_LBM_VEL_PARABOLIC || cfg->bc[3] == IB_LBM_VEL_PARABOLIC)
    return fail(IB_LBM_E_INVALID, "parabolic profile only on the west or east face");
  if (cfg->collision == IB_LBM_TRT && !(cfg->trt_magic > 0.0))
    return fail(IB_LBM_E_INVALID, "TRT needs a positive magic parameter");
  if (!(cfg->rho0 > 0.0)) return fail(IB_LBM_E_INVALID, "rho0 must be positive");
  s->stream = (hipStream_t)cfg->stream;
  if (hipGetDevice(&s->dev) != hipSuccess) return fail(IB_LBM_E_DEVICE, "no HIP device");
  CaseDesc &c = s->cd;
  memset(&c, 0, sizeof c);
  c.nx = cfg->nx;
  c.ny = cfg->ny;
  c.collision = cfg->collision;
  c.precision = cfg->precision;
  for (int f = 0; f < 4; f++) c.bc[f] = cfg->bc[f];
  c.plane = (int64_t)cfg->nx * cfg->ny;
  c.nseg = pop_segments(cfg->nx);
  c.omega = 1.0 / cfg->tau;
  // TRT (Sec. 2.2): the even rate sets the viscosity; Lambda_o = Lambda_eo / Lambda_e.
  c.s_e = 1.0 / cfg->tau;
  {
    const double lam_e = cfg->tau - 0.5;
    const double lam_o = (cfg->trt_magic > 0 ? cfg->trt_magic : 0.25) / lam_e;
    c.s_o = 1.0 / (lam_o + 0.5);
  }
  c.s_q = cfg->cm_s_q;
  c.s_eps = cfg->cm_s_eps;
  c.rho0 = cfg->rho0;
  c.u_bc = cfg->u_bc;
  c.inv_ny2 = 1.0 / ((double)cfg->ny * cfg->ny);
  c.fluid_fx = cfg->fluid_force[0];
  c.fluid_fy = cfg->fluid_force[1];
  c.grav_x = cfg->gravity[0];
  c.grav_y = cfg->gravity[1];
  const size_t elem = cfg->precision == IB_LBM_FP64 ? 8 : 4;
  ib_lbm_status st;
  const size_t lat = (size_t)pop_values(c.nx, c.ny) * elem;
  if ((st = dev_alloc(s, &s->f0, lat))) return fail(st, s->err.c_str());
  if ((st = dev_alloc(s, &s->f1, lat))) return fail(st, s->err.c_str());
  if ((st = dev_alloc(s, &s->force, 2 * (size_t)c.plane * elem))) return fail(st, s->err.c_str());
  if ((st = dev_alloc(s, &s->state, sizeof(CaseState)))) return fail(st, s->err.c_str());
  if (has_zou_he(c)) {
    // (what a caller sets is used as it is, so it counts as closed)
    const size_t nw = 2 * (size_t)wall_nodes(c.nx, c.ny);
    if ((st = dev_alloc(s, &s->wall_closed, nw))) return fail(st, s->err.c_str());
    if (hipMemset(s->wall_closed.p, 1, nw) != hipSuccess) return fail(IB_LBM_E_DEVICE, "wall flags");
    c.wall_closed = (uint8_t *)s->wall_closed.p;
  }
  c.f[0] = s->f0.p;
  c.f[1] = s->f1.p;
  c.force = s->force.p;
  c.state = (CaseState *)s->state.p;
  CaseState cs{};
  cs.step = 0;
  cs.target = std::numeric_limits<int64_t>::max();
  cs.cur = 0;
  if (hipMemcpy(s->state.p, &cs, sizeof cs, hipMemcpyHostToDevice) != hipSuccess)
    return fail(IB_LBM_E_DEVICE, "state upload failed");
  if (launch_init_equilibrium(c, 0, s->stream) != hipSuccess ||
      launch_init_equilibrium(c, 1, s->stream) != hipSuccess ||
      hipStreamSynchronize(s->stream) != hipSuccess)
    return fail(IB_LBM_E_DEVICE, "initialisation kernel failed");
  *out = s;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_add_body(ib_lbm_sim *s, const ib_lbm_body_desc *b, int32_t *body_id) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (!b) return IB_LBM_E_INVALID;
  if (s->started || s->batch) {
    set_err(&s->err, "bodies can only be added before the first step");
    return IB_LBM_E_STATE;
  }
  if ((int)s->bodies.size() >= kMaxBodiesPerCase) {
    set_err(&s->err, "at most %d bodies per sim", kMaxBodiesPerCase);
    return IB_LBM_E_INVALID;
  }
  if (!(b->diameter > 0) || b->scheme < IB_LBM_DF || b->scheme > IB_LBM_DFC || b->kernel < 0 ||
      b->kernel > 1 || b->motion < 0 || b->motion > 2 || b->n_markers < 0 ||
      (b->scheme == IB_LBM_MDF && (b->mdf_iters < 1 || b->mdf_iters > 1000)) ||
      (b->scheme == IB_LBM_MDF && b->mdf_tol > 0 &&
       (b->mdf_nmin < 1 || b->mdf_nmin > b->mdf_iters)) ||
      (b->motion == IB_LBM_FREE && !(b->density_ratio > 0)) ||
      (b->integrator != IB_LBM_VERLET && b->integrator != IB_LBM_EULER_A1) ||
      (b->mdf_coupled != 0 && b->mdf_coupled != 1) ||
      (b->udes != IB_LBM_UD_RIGID && b->udes != IB_LBM_UD_TAYLOR_GREEN) ||
      (b->udes == IB_LBM_UD_TAYLOR_GREEN &&
       (b->motion != IB_LBM_FIXED || !(b->tg_k > 0) || !(b->tg_nu >= 0) || !std::isfinite(b->tg_u0)))) {
    set_err(&s->err, "invalid body description");
    return IB_LBM_E_INVALID;
  }
  if (!s->bodies.empty() && s->bodies[0].d.scheme != b->scheme) {
    set_err(&s->err, "all bodies of a sim must use the same scheme");
    return IB_LBM_E_INVALID;
  }
  const bool coupled = b->scheme == IB_LBM_MDF && b->mdf_coupled;
  if (b->scheme == IB_LBM_MDF && !s->bodies.empty()) {
    const ib_lbm_body_desc &o = s->bodies[0].d;
    if ((o.mdf_coupled != 0) != coupled ||
        (coupled && (o.mdf_iters != b->mdf_iters || (o.mdf_tol > 0) != (b->mdf_tol > 0) ||
                     (b->mdf_tol > 0 && (o.mdf_tol != b->mdf_tol || o.mdf_nmin != b->mdf_nmin))))) {
      set_err(&s->err, "coupled MDF: every body alike, with equal bounds and tolerance");
      return IB_LBM_E_INVALID;
    }
  }
  HostBody hb;
  hb.d = *b;
  BodyDesc &B = hb.dev;
  memset(&B, 0, sizeof B);
  const int nb = b->n_markers > 0 ? b->n_markers : (int)std::lround(M_PI * b->diameter);
  if (nb < 1 || nb > 32768) {
    set_err(&s->err, "marker count out of range");
    return IB_LBM_E_INVALID;
  }
  B.nb = nb;
  B.scheme = b->scheme;
  B.kernel = b->kernel;
  B.mdf_iters = b->scheme == IB_LBM_MDF ? b->mdf_iters : 1;
  B.mdf_tol = b->scheme == IB_LBM_MDF && b->mdf_tol > 0 ? b->mdf_tol : 0.0;
  B.mdf_nmin = B.mdf_tol > 0 ? b->mdf_nmin : B.mdf_iters;
  B.mdf_coupled = coupled ? 1 : 0;
  B.motion = b->motion;
  B.internal_mass = b->internal_mass;
  B.integrator = b->integrator;
  B.udes = b->udes;
  B.tg_u0 = b->tg_u0;
  B.tg_k = b->tg_k;
  B.tg_nu = b->tg_nu;
  B.ns = b->kernel == IB_LBM_HAT ? 2 : 4;
  B.radius = 0.5 * b->diameter;
  B.ds = M_PI * b->diameter / nb;
  B.dtheta = 2.0 * M_PI / nb;
  B.xc0 = b->xc;
  B.yc0 = b->yc;
  B.amp[0] = b->amp[0];
  B.amp[1] = b->amp[1];
  B.freq = b->freq;
  B.phase = b->phase;
  const double area = M_PI * B.radius * B.radius;
  B.ms = (b->motion == IB_LBM_FREE ? b->density_ratio : 1.0) * s->cfg.rho0 * area;
  B.mf = s->cfg.rho0 * area;
  B.Is = 0.5 * B.ms * B.radius * B.radius;
  // marker directions, theta_k = 2 pi k / N_b starting at angle 0
  std::vector<double> ct(nb), stb(nb);
  for (int k = 0; k < nb; k++) {
    const double th = 2.0 * M_PI * (double)k / (double)nb;
    ct[k] = std::cos(th);
    stb[k] = std::sin(th);
  }
  // every support inside the lattice at the start position (compared as doubles: a
  // position may be beyond every int, or NaN)
  const int sw = B.ns / 2;
  auto inside = [&](double xc, double yc) {
    for (int k = 0; k < nb; k++) {
      const double ix = std::floor(xc + B.radius * ct[k]), iy = std::floor(yc + B.radius * stb[k]);
      if (!(ix >= sw - 1 && iy >= sw - 1 && ix <= s->cfg.nx - 1 - sw && iy <= s->cfg.ny - 1 - sw)) return false;
    }
    return true;
  };
  if (!inside(b->xc, b->yc) ||
      (b->motion == IB_LBM_PRESCRIBED_SIN &&
       (!inside(b->xc + std::fabs(b->amp[0]), b->yc + std::fabs(b->amp[1])) ||
        !inside(b->xc - std::fabs(b->amp[0]), b->yc - std::fabs(b->amp[1]))))) {
    set_err(&s->err, "a marker support leaves the lattice");
    return IB_LBM_E_RANGE;
  }
  for (auto &o : s->bodies) {
    const double dx = o.d.xc - b->xc, dy = o.d.yc - b->yc;
    const double lim = o.dev.radius + B.radius + o.dev.ns + B.ns + 4.0;
    if (dx * dx + dy * dy <= lim * lim) {
      set_err(&s->err, "body supports would meet; bodies must stay apart");
      return IB_LBM_E_RANGE;
    }
  }
  // workspace sizing over sub-lattice positions of the centre, placed so
  // that every stencil lies at positive coordinates (support_count marks an
  // empty row with a negative column)
  const double c0 = std::ceil(B.radius) + 2 * B.ns + 8;
  int maxn = 0, maxr = 0;
  for (int a = 0; a < 4; a++)
    for (int q = 0; q < 4; q++) {
      int rows = 0;
      const int n = support_count(c0 + 0.25 * a + 0.0625, c0 + 0.25 * q + 0.125, B.radius, nb,
                                  B.ns, ct, stb, &rows);
      maxn = std::max(maxn, n);
      maxr = std::max(maxr, rows);
    }
  B.max_rows = (int)std::ceil(2 * B.radius) + 2 * B.ns + 4;
  B.max_nodes = maxn + maxn / 10 + 32;
  B.ws_tab = ws_tab_total(b->scheme, nb, B.ns, B.max_rows, B.max_nodes);
  B.ws_tab_hot = ws_tab_hot(b->scheme, nb, B.ns, B.max_nodes);
  B.pop_bytes = s->cfg.precision == IB_LBM_FP64 ? 8 : 4;
  B.ws_doubles = ws_doubles_for(b->scheme, nb, B.ns, B.max_rows, B.max_nodes, B.pop_bytes);
  // MDF passes in marker space (the 1024-thread instance): markers k and l
  // can share a stencil node only if they are less than ns apart in x and
  // in y, so less than ns sqrt 2 apart; on the circle of radius R that
  // bounds |l - k| by (n_b / pi) asin(ns sqrt 2 / (2 R)).  Used when the
  // band is narrow and the workspace with it still fits in LDS.
  B.mdf_band = 0;
  if (coupled) B.ws_doubles += ws_coupled_doubles(nb, B.max_nodes);
  if (b->scheme == IB_LBM_MDF && !coupled && B.ns * std::sqrt(2.0) < 2.0 * B.radius) {
    const int w = (int)std::floor(nb / M_PI * std::asin(B.ns * std::sqrt(2.0) / (2.0 * B.radius))) + 1;
    // U at the markers is new space; the band (its half, B being
    // symmetric) overlays the two node-velocity arrays
    const int extra = 2 * nb;
    if (w <= 12 && 2 * w + 1 < nb && nb * (w + 1) <= 2 * B.max_nodes &&
        (B.ws_doubles + extra) * 8 <= ibm_max_lds_bytes()) {
      B.mdf_band = w;
      B.ws_doubles += extra;
    }
  }
  plan_arcs(&B);
  // gather window: a node within s*sqrt(2) of marker k lies within angle
  // 2 asin(s / sqrt(2 R (R - s sqrt 2))) of it
  {
    const double sr = sw * std::sqrt(2.0);
    double dmax = M_PI;
    if (B.radius > sr + 0.5) dmax = 2.0 * std::asin(std::min(1.0, sw / std::sqrt(2.0 * B.radius * (B.radius - sr))));
    int w = (int)std::ceil(dmax / B.dtheta) + 2;
    if (2 * w + 1 >= nb) w = nb;
    B.window = w;
  }
  B.omega_mdf = b->scheme == IB_LBM_MDF
                    ? (b->mdf_omega > 0 ? b->mdf_omega
                                        : host_omega_mdf(b->xc, b->yc, B.radius, nb, b->kernel, B.ds, ct, stb))
                    : 1.0;
  B.hist_cap = s->cfg.history_capacity > 0 ? s->cfg.history_capacity : 4096;
  if ((st = dev_alloc(s, &hb.cos_t, nb * 8))) return st;
  if ((st = dev_alloc(s, &hb.sin_t, nb * 8))) return st;
  if ((st = dev_alloc(s, &hb.ws, (size_t)B.ws_doubles * 8))) return st;
  if ((st = dev_alloc(s, &hb.tab, (size_t)B.ws_tab * 8))) return st;
  if ((st = dev_alloc(s, &hb.acc, (size_t)B.max_nodes * 2 * 8))) return st;
  if ((st = dev_alloc(s, &hb.markers, (size_t)nb * 8 * 8))) return st;
  if ((st = dev_alloc(s, &hb.lambda, (size_t)nb * 8))) return st;
  if ((st = dev_alloc(s, &hb.history, (size_t)B.hist_cap * kHistCols * 8))) return st;
  // the state, and behind it the arcs' partial sums
  const size_t state_bytes = (sizeof(BodyState) + 63) / 64 * 64;
  if ((st = dev_alloc(s, &hb.state, state_bytes + (size_t)B.arc_n * 8 * 8))) return st;
  HIPCHK(s, hipMemcpy(hb.cos_t.p, ct.data(), nb * 8, hipMemcpyHostToDevice));
  HIPCHK(s, hipMemcpy(hb.sin_t.p, stb.data(), nb * 8, hipMemcpyHostToDevice));
  HIPCHK(s, hipMemset(hb.markers.p, 0, (size_t)nb * 64));
  HIPCHK(s, hipMemset(hb.history.p, 0, (size_t)B.hist_cap * kHistCols * 8));
  B.cos_t = (const double *)hb.cos_t.p;
  B.sin_t = (const double *)hb.sin_t.p;
  B.ws = (double *)hb.ws.p;
  B.tab_cache = (double *)hb.tab.p;
  B.acc = (double *)hb.acc.p;
  B.markers_out = (double *)hb.markers.p;
  B.lambda_cache = (double *)hb.lambda.p;
  B.history = (double *)hb.history.p;
  B.state = (BodyState *)hb.state.p;
  B.arc_part = (double *)((char *)hb.state.p + state_bytes);
  B.src = nullptr;
  B.n_src = 0;
  B.fprev = nullptr;
  B.pstage = nullptr;
  if (b->motion == IB_LBM_FIXED && b->scheme != IB_LBM_DFC && B.arc_n == 0) {
    // fused steps of a body that is not cut into arcs: the copy of the last force
    // (zero, as the force field starts) and the staged pushes of the support nodes
    if ((st = dev_alloc(s, &hb.fprev, (size_t)B.max_nodes * 2 * B.pop_bytes))) return st;
    if ((st = dev_alloc(s, &hb.pstage, (size_t)B.max_nodes * 9 * B.pop_bytes))) return st;
    HIPCHK(s, hipMemset(hb.fprev.p, 0, (size_t)B.max_nodes * 2 * B.pop_bytes));
    B.fprev = hb.fprev.p;
    B.pstage = hb.pstage.p;
  }
  BodyState bst;
  memset(&bst, 0, sizeof bst);
  bst.xc = b->xc;
  bst.yc = b->yc;
  HIPCHK(s, hipMemcpy(hb.state.p, &bst, sizeof bst, hipMemcpyHostToDevice));
  s->bodies.push_back(hb);
  s->tables_dirty = true;
  if (body_id) *body_id = (int32_t)s->bodies.size() - 1;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_step(ib_lbm_sim *s, int64_t nsteps) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (nsteps < 0) return IB_LBM_E_INVALID;
  if (s->batch) {
    set_err(&s->err, "sim is attached to a batch; step the batch");
    return IB_LBM_E_STATE;
  }
  if ((st = build_sim_tables(s))) return st;
  if (s->split && (st = ensure_pipe_streams(s))) return st;
  s->started = true;
  int64_t left = nsteps;
  if (s->halted) {
    // a halted case's kernels do nothing
    s->host_steps += nsteps;
    return IB_LBM_OK;
  }
  if (s->one && !s->hold_ready && left > 0 && !s->timing.on) {
    // one-launch steps need the hold rectangles that a pass leaves: one plain
    // step first
    if ((st = enqueue_steps(s, 1, false, s->stream, s->host_cur, false))) return st;
    s->host_cur ^= 1;
    left -= 1;
  }
  if (s->fused && !s->one && !s->bodies[0].src_ready && left > 0 && !s->timing.on) {
    // fused steps start from the support the device builds at the body's
    // first IB pass: one pipelined step first if none has run
    if (s->host_steps == 0) {
      if ((st = enqueue_steps(s, 1, false, s->stream, s->host_cur, true))) return st;
      s->host_cur ^= 1;
      left -= 1;
    }
    st = build_fused_sources(s);
    if (st == IB_LBM_E_STATE) {
      // no support table (a halted case): pipelined steps
      s->fused = false;
      st = IB_LBM_OK;
    }
    if (st) return st;
  }
  if (s->graph_steps > 0 && !s->timing.on && left >= s->graph_steps) {
    if (s->graph_len != s->graph_steps) {
      drop_graphs(s);
      s->graph_len = s->graph_steps;
    }
    // pipelined steps: an explicitly built graph per starting lattice, both
    // made at the first replay; plain steps: captured on a private stream
    // (the caller's may be the null stream); replayed on the caller's stream
    if (s->split && !s->fused && !s->one) {
      for (int p = 0; p < 2; p++)
        if (!s->graph_exec[p] && (st = build_pipelined_graph(s, s->graph_len, p, &s->graph_exec[p])))
          return st;
      s->graph_form = IB_LBM_STEP_PIPELINED;
    }
    if (!s->cap_stream) HIPCHK(s, hipStreamCreateWithFlags(&s->cap_stream, hipStreamNonBlocking));
    while (left >= s->graph_len) {
      hipGraphExec_t &ge = s->graph_exec[s->host_cur];
      if (!ge) {
        hipGraph_t g;
        HIPCHK(s, hipStreamBeginCapture(s->cap_stream, hipStreamCaptureModeThreadLocal));
        // captured steps are plain steps on the capturing stream: capturing
        // the two-stream pipelined step crashed the host process in the HIP
        // runtime (cause not identified), so pipelined graphs are built
        // explicitly above instead
        st = enqueue_steps(s, s->graph_len, false, s->cap_stream, s->host_cur, false);
        if (st) {
          hipGraph_t dummy;
          (void)hipStreamEndCapture(s->cap_stream, &dummy);
          return st;
        }
        HIPCHK(s, hipStreamEndCapture(s->cap_stream, &g));
        HIPCHK(s, hipGraphInstantiate(&ge, g, nullptr, nullptr, 0));
        (void)hipGraphDestroy(g);
        s->graph_form = s->form;
      }
      HIPCHK(s, hipGraphLaunch(ge, s->stream));
      s->form = s->graph_form;
      left -= s->graph_len;
      s->host_cur ^= s->graph_len & 1;
    }
  }
  if (left > 0) {
    if ((st = enqueue_steps(s, left, s->timing.on, s->stream, s->host_cur, true))) return st;
    s->host_cur ^= (int)(left & 1);
  }
  s->host_steps += nsteps;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_forces(ib_lbm_sim *s, int32_t body_id, ib_lbm_body_state *out) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (!out || body_id < 0 || body_id >= (int)s->bodies.size()) return IB_LBM_E_INVALID;
  CaseState cs;
  if ((st = read_state(s, &cs))) return st;
  BodyState b;
  HIPCHK(s, hipMemcpy(&b, s->bodies[body_id].state.p, sizeof b, hipMemcpyDeviceToHost));
  out->step = cs.step;
  out->fx = b.fhx;
  out->fy = b.fhy;
  out->torque = b.torque;
  out->xc = b.xc;
  out->yc = b.yc;
  const bool freeb = s->bodies[body_id].d.motion == IB_LBM_FREE;
  out->vx = freeb ? b.vx : b.vhx;
  out->vy = freeb ? b.vy : b.vhy;
  out->omega = freeb ? b.om : b.omh;
  out->slip_mean = b.slip_mean;
  out->slip_max = b.slip_max;
  out->mdf_residual = b.mdf_res;
  out->mdf_omega = s->bodies[body_id].dev.omega_mdf;
  out->mdf_iters = b.mdf_iters_done;
  out->flags = b.flags;
  if (b.flags & IB_LBM_FLAG_NONFINITE) {
    set_err(&s->err, "non-finite force or velocity at body %d", body_id);
    return IB_LBM_E_DIVERGED;
  }
  if (b.flags & kFlagExchange) {
    set_err(&s->err, s->bodies[body_id].dev.mdf_coupled
                         ? "body %d: the coupled MDF workgroups of the case did not meet (flags %d)"
                         : "body %d: the pass waited too long for other workgroups of its step (flags %d)",
            body_id, b.flags);
    return IB_LBM_E_STATE;
  }
  if (b.flags & (IB_LBM_FLAG_RANGE | IB_LBM_FLAG_OVERLAP | kFlagCapacity)) {
    if (b.flags & kFlagCapacity)
      set_err(&s->err, "body %d outgrew its support tables (flags %d): fewer markers or a smaller body",
              body_id, b.flags);
    else
      set_err(&s->err, "body %d left the lattice or met another body (flags %d)", body_id, b.flags);
    return IB_LBM_E_RANGE;
  }
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_history(ib_lbm_sim *s, int32_t body_id, int64_t first, int64_t count,
                             double *out) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (!out || body_id < 0 || body_id >= (int)s->bodies.size() || count < 0 || first < 1)
    return IB_LBM_E_INVALID;
  CaseState cs;
  if ((st = read_state(s, &cs))) return st;
  const int cap = s->bodies[body_id].dev.hist_cap;
  if (first + count - 1 > cs.step || first <= cs.step - cap) {
    set_err(&s->err, "history rows outside the kept window");
    return IB_LBM_E_RANGE;
  }
  const double *h = (const double *)s->bodies[body_id].history.p;
  // the rows lie in the ring in at most two runs (before and after the wrap)
  for (int64_t i = 0; i < count;) {
    const int64_t row = (first - 1 + i) % cap;
    const int64_t run = std::min<int64_t>(count - i, cap - row);
    HIPCHK(s, hipMemcpy(out + i * kHistCols, h + row * kHistCols, (size_t)run * kHistCols * 8,
                        hipMemcpyDeviceToHost));
    i += run;
  }
  return IB_LBM_OK;
}

static ib_lbm_status ensure_tmp(ib_lbm_sim *s, size_t bytes) {
  if (s->d_tmp.bytes >= bytes) return IB_LBM_OK;
  dev_free(s, &s->d_tmp);
  return dev_alloc(s, &s->d_tmp, bytes);
}

ib_lbm_status ib_lbm_fields(ib_lbm_sim *s, double *rho, double *ux, double *uy) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (!rho || !ux || !uy) return IB_LBM_E_INVALID;
  CaseState cs;
  if ((st = read_state(s, &cs))) return st;
  const size_t n = (size_t)s->cd.plane;
  if ((st = ensure_tmp(s, 3 * n * 8))) return st;
  double *d = (double *)s->d_tmp.p;
  HIPCHK(s, launch_fields(s->cd, cs.cur, d, d + n, d + 2 * n, s->stream));
  HIPCHK(s, hipStreamSynchronize(s->stream));
  const HostCopy out[3] = {{d, rho, n * 8}, {d + n, ux, n * 8}, {d + 2 * n, uy, n * 8}};
  HIPCHK(s, host_copy(out, 3));
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_get_populations(ib_lbm_sim *s, double *f) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (!f) return IB_LBM_E_INVALID;
  CaseState cs;
  if ((st = read_state(s, &cs))) return st;
  const size_t n = (size_t)s->cd.plane;
  if ((st = ensure_tmp(s, 9 * n * 8))) return st;
  HIPCHK(s, launch_export(s->cd, cs.cur, (double *)s->d_tmp.p, s->stream));
  HIPCHK(s, hipStreamSynchronize(s->stream));
  const HostCopy out{s->d_tmp.p, f, 9 * n * 8};
  HIPCHK(s, host_copy(&out, 1));
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_set_populations(ib_lbm_sim *s, const double *f) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (!f) return IB_LBM_E_INVALID;
  CaseState cs;
  if ((st = read_state(s, &cs))) return st;
  const size_t n = (size_t)s->cd.plane;
  if ((st = ensure_tmp(s, 9 * n * 8))) return st;
  HIPCHK(s, hipMemcpy(s->d_tmp.p, f, 9 * n * 8, hipMemcpyHostToDevice));
  HIPCHK(s, launch_import(s->cd, cs.cur, (const double *)s->d_tmp.p, s->stream));
  HIPCHK(s, hipStreamSynchronize(s->stream));
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_set_equilibrium(ib_lbm_sim *s, const double *rho, const double *ux,
                                    const double *uy) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (!ux || !uy) return IB_LBM_E_INVALID;
  CaseState cs;
  if ((st = read_state(s, &cs))) return st;
  const size_t n = (size_t)s->cd.plane;
  if ((st = ensure_tmp(s, 3 * n * 8))) return st;
  double *d = (double *)s->d_tmp.p;
  HIPCHK(s, hipMemcpy(d, ux, n * 8, hipMemcpyHostToDevice));
  HIPCHK(s, hipMemcpy(d + n, uy, n * 8, hipMemcpyHostToDevice));
  if (rho) HIPCHK(s, hipMemcpy(d + 2 * n, rho, n * 8, hipMemcpyHostToDevice));
  HIPCHK(s, launch_set_equilibrium(s->cd, cs.cur, rho ? d + 2 * n : nullptr, d, d + n, s->stream));
  HIPCHK(s, hipStreamSynchronize(s->stream));
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_force_field(ib_lbm_sim *s, double *fx, double *fy) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (!fx || !fy) return IB_LBM_E_INVALID;
  CaseState cs;
  if ((st = read_state(s, &cs))) return st;
  const size_t n = (size_t)s->cd.plane;
  if ((st = ensure_tmp(s, 2 * n * 8))) return st;
  double *d = (double *)s->d_tmp.p;
  HIPCHK(s, launch_force_export(s->cd, d, d + n, s->stream));
  HIPCHK(s, hipStreamSynchronize(s->stream));
  const HostCopy out[2] = {{d, fx, n * 8}, {d + n, fy, n * 8}};
  HIPCHK(s, host_copy(out, 2));
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_markers(ib_lbm_sim *s, int32_t body_id, double *out, int32_t *n_markers) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (body_id < 0 || body_id >= (int)s->bodies.size()) return IB_LBM_E_INVALID;
  const int nb = s->bodies[body_id].dev.nb;
  if (n_markers) *n_markers = nb;
  if (!out) return IB_LBM_OK;
  HIPCHK(s, hipStreamSynchronize(s->stream));
  HIPCHK(s, hipMemcpy(out, s->bodies[body_id].markers.p, (size_t)nb * 64, hipMemcpyDeviceToHost));
  return IB_LBM_OK;
}

}  // extern "C"

namespace {

// Diagnostics of body_id staged in device memory at d (8 + 6 n_b doubles),
// then copied to the host.  Allocates nothing.
ib_lbm_status diagnostics_into(ib_lbm_sim *s, int32_t body_id, int32_t kappa, double u_ref,
                               double *summary, double *per_marker, double *d) {
  CaseState cs;
  ib_lbm_status st;
  if ((st = read_state(s, &cs))) return st;
  if (cs.step < 1) {
    set_err(&s->err, "diagnostics need a completed step");
    return IB_LBM_E_STATE;
  }
  const HostBody &hb = s->bodies[body_id];
  BodyState b;
  HIPCHK(s, hipMemcpy(&b, hb.state.p, sizeof b, hipMemcpyDeviceToHost));
  const bool freeb = hb.d.motion == IB_LBM_FREE;
  const double vx = freeb ? b.vx : b.vhx, vy = freeb ? b.vy : b.vhy, om = freeb ? b.om : b.omh;
  if (!std::isfinite(b.xc) || !std::isfinite(b.yc) || !std::isfinite(vx) || !std::isfinite(vy) ||
      !std::isfinite(om)) {
    set_err(&s->err, "body %d has a non-finite position or velocity", body_id);
    return IB_LBM_E_DIVERGED;
  }
  const int nb = hb.dev.nb;
  HIPCHK(s, launch_diagnostics(s->cd, cs.cur, (const double *)hb.markers.p, nb, b.xc, b.yc, vx, vy,
                               om, hb.dev.radius, hb.dev.ds, kappa, u_ref, d, d + 8, s->stream));
  HIPCHK(s, hipStreamSynchronize(s->stream));
  HIPCHK(s, hipMemcpy(summary, d, 8 * 8, hipMemcpyDeviceToHost));
  if (per_marker) HIPCHK(s, hipMemcpy(per_marker, d + 8, (size_t)nb * 6 * 8, hipMemcpyDeviceToHost));
  return IB_LBM_OK;
}

}  // namespace

extern "C" {

ib_lbm_status ib_lbm_diagnostics(ib_lbm_sim *s, int32_t body_id, int32_t kappa, double u_ref,
                                 double *summary, double *per_marker) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (!summary || body_id < 0 || body_id >= (int)s->bodies.size() || kappa < 0 || !(u_ref > 0))
    return IB_LBM_E_INVALID;
  if (s->bodies[body_id].d.udes != IB_LBM_UD_RIGID) {
    set_err(&s->err, "boundary diagnostics are defined for rigid bodies");
    return IB_LBM_E_INVALID;
  }
  const int nb = s->bodies[body_id].dev.nb;
  if ((st = ensure_tmp(s, (size_t)(8 + 6 * nb) * 8))) return st;
  return diagnostics_into(s, body_id, kappa, u_ref, summary, per_marker, (double *)s->d_tmp.p);
}

ib_lbm_status ib_lbm_diagnostics_noalloc(ib_lbm_sim *s, int32_t body_id, int32_t kappa, double u_ref,
                                         double *summary, double *per_marker) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (!summary || body_id < 0 || body_id >= (int)s->bodies.size() || kappa < 0 || !(u_ref > 0))
    return IB_LBM_E_INVALID;
  if (s->bodies[body_id].d.udes != IB_LBM_UD_RIGID) {
    set_err(&s->err, "boundary diagnostics are defined for rigid bodies");
    return IB_LBM_E_INVALID;
  }
  const int nb = s->bodies[body_id].dev.nb;
  if (nb > diag_scratch_markers()) {
    set_err(&s->err, "ib_lbm_diagnostics_noalloc: %d markers exceed the static staging of %d", nb,
            diag_scratch_markers());
    return IB_LBM_E_INVALID;
  }
  // the staging of the sim's device, its address taken once per device
  int dev = 0;
  HIPCHK(s, hipGetDevice(&dev));
  if (dev != s->dev) HIPCHK(s, hipSetDevice(s->dev));
  double *d = nullptr;
  hipError_t e = diag_scratch(&d);
  if (e == hipSuccess) st = diagnostics_into(s, body_id, kappa, u_ref, summary, per_marker, d);
  if (dev != s->dev) (void)hipSetDevice(dev);
  HIPCHK(s, e);
  return st;
}

ib_lbm_status ib_lbm_steps_done(ib_lbm_sim *s, int64_t *steps) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (!steps) return IB_LBM_E_INVALID;
  CaseState cs;
  if ((st = read_state(s, &cs))) return st;
  *steps = cs.step;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_sync(ib_lbm_sim *s) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  HIPCHK(s, hipStreamSynchronize(s->stream));
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_destroy(ib_lbm_sim *s) {
  if (!s) return IB_LBM_E_INVALID;
  if (s->batch) ib_lbm_batch_detach(s->batch, s);
  if (s->stream) (void)hipStreamSynchronize(s->stream);
  arc_budget.give_back(s);
  drop_graphs(s);
  if (s->lq) (void)hipStreamSynchronize(s->lq);
  if (s->iq) (void)hipStreamSynchronize(s->iq);
  for (int k = 0; k < kTimingKinds; k++)
    for (auto &p : s->timing.ev[k]) { (void)hipEventDestroy(p.a); (void)hipEventDestroy(p.b); }
  for (auto &p : s->timing.pool) { (void)hipEventDestroy(p.a); (void)hipEventDestroy(p.b); }
  for (auto &hb : s->bodies) {
    dev_free(s, &hb.cos_t); dev_free(s, &hb.sin_t); dev_free(s, &hb.ws); dev_free(s, &hb.markers);
    dev_free(s, &hb.tab); dev_free(s, &hb.acc);
    dev_free(s, &hb.lambda); dev_free(s, &hb.history); dev_free(s, &hb.state);
    dev_free(s, &hb.fprev); dev_free(s, &hb.pstage); dev_free(s, &hb.src);
  }
  dev_free(s, &s->f0); dev_free(s, &s->f1); dev_free(s, &s->force); dev_free(s, &s->state);
  dev_free(s, &s->ticket); dev_free(s, &s->wall_closed);
  dev_free(s, &s->d_bodies); dev_free(s, &s->d_case); dev_free(s, &s->d_prefix);
  dev_free(s, &s->d_slots); dev_free(s, &s->d_tmp);
  if (s->cap_stream) (void)hipStreamDestroy(s->cap_stream);
  if (s->lq) (void)hipStreamDestroy(s->lq);
  if (s->iq) (void)hipStreamDestroy(s->iq);
  if (s->ev_start) (void)hipEventDestroy(s->ev_start);
  if (s->ev_lq) (void)hipEventDestroy(s->ev_lq);
  if (s->ev_iq) (void)hipEventDestroy(s->ev_iq);
  if (s->ev_near) (void)hipEventDestroy(s->ev_near);
  if (s->ev_far) (void)hipEventDestroy(s->ev_far);
  host_copy_release();
  delete s;
  return IB_LBM_OK;
}

const char *ib_lbm_last_error(const ib_lbm_sim *s) { return s ? s->err.c_str() : "null sim"; }

ib_lbm_status ib_lbm_set_launch(ib_lbm_sim *s, const ib_lbm_launch *l) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if ((st = check_launch(l, &s->err))) return st;
  s->launch = *l;
  s->tables_dirty = true;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_get_launch(const ib_lbm_sim *s, ib_lbm_launch *l) {
  if (!s || !l) return IB_LBM_E_INVALID;
  *l = s->launch;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_set_spread(ib_lbm_sim *s, int32_t mode) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (mode != IB_LBM_SPREAD_GATHER && mode != IB_LBM_SPREAD_ATOMIC) return IB_LBM_E_INVALID;
  s->spread_mode = mode;
  s->tables_dirty = true;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_set_overlap(ib_lbm_sim *s, int32_t on) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (on != 0 && on != 1) return IB_LBM_E_INVALID;
  HIPCHK(s, hipStreamSynchronize(s->stream));
  s->overlap = on != 0;
  s->tables_dirty = true;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_get_overlap(const ib_lbm_sim *s, int32_t *in_use, int64_t *near_nodes) {
  if (!s || !in_use) return IB_LBM_E_INVALID;
  *in_use = s->split ? 1 : 0;
  if (near_nodes) {
    int64_t n = 0;
    if (s->split) {
      const int TX = s->launch.block_x, TY = s->launch.block_y * s->launch.rows_per_thread;
      const int64_t x0 = (int64_t)s->hold[0] * TX, y0 = (int64_t)s->hold[1] * TY;
      const int64_t x1 = std::min<int64_t>(x0 + (int64_t)s->hold[2] * TX, s->cd.nx);
      const int64_t y1 = std::min<int64_t>(y0 + (int64_t)s->hold[3] * TY, s->cd.ny);
      n = (x1 - x0) * (y1 - y0);
    }
    *near_nodes = n;
  }
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_set_fused(ib_lbm_sim *s, int32_t on) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (on != 0 && on != 1) return IB_LBM_E_INVALID;
  HIPCHK(s, hipStreamSynchronize(s->stream));
  if (s->fused_allowed != (on != 0)) {
    s->fused_allowed = on != 0;
    s->tables_dirty = true;
  }
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_get_fused(const ib_lbm_sim *s, int32_t *in_use) {
  if (!s || !in_use) return IB_LBM_E_INVALID;
  *in_use = s->fused && !s->tables_dirty ? 1 : 0;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_get_step_form(const ib_lbm_sim *s, int32_t *form) {
  if (!s || !form) return IB_LBM_E_INVALID;
  *form = s->form;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_set_graph(ib_lbm_sim *s, int32_t steps_per_graph) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (steps_per_graph < 0 || steps_per_graph > 100000) return IB_LBM_E_INVALID;
  s->graph_steps = steps_per_graph;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_timing_enable(ib_lbm_sim *s, int32_t on) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  HIPCHK(s, hipStreamSynchronize(s->stream));
  for (int k = 0; k < kTimingKinds; k++) {
    for (auto &p : s->timing.ev[k]) s->timing.pool.push_back(p);
    s->timing.ev[k].clear();
    s->timing.folded_ms[k] = 0;
    s->timing.folded_n[k] = 0;
  }
  s->timing.on = on != 0;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_time_collide_stream(ib_lbm_sim *s, int32_t launches, double *avg_us,
                                         int64_t *inner_nodes) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (launches <= 0 || !avg_us) return IB_LBM_E_INVALID;
  if (s->batch) {
    set_err(&s->err, "sim is attached to a batch");
    return IB_LBM_E_STATE;
  }
  if ((st = build_sim_tables(s))) return st;
  s->started = true;
  LaunchShape sh{s->launch.block_x, s->launch.block_y, s->launch.rows_per_thread, s->launch.xcd_remap};
  const LeanArgs la = lean_args(s, s->host_cur, 1);
  hipEvent_t a, b;
  HIPCHK(s, hipEventCreate(&a));
  HIPCHK(s, hipEventCreate(&b));
  hipError_t e = hipEventRecord(a, s->stream);
  for (int i = 0; i < launches && e == hipSuccess; i++)
    e = launch_collide_stream_lean(s->cd.precision, s->cd.collision, la, 0, sh, s->stream);
  if (e == hipSuccess) e = hipEventRecord(b, s->stream);
  if (e == hipSuccess) e = hipEventSynchronize(b);
  float ms = 0;
  if (e == hipSuccess) e = hipEventElapsedTime(&ms, a, b);
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  HIPCHK(s, e);
  // the launches consumed the IB force: so does the copy fused steps read
  for (auto &hb : s->bodies)
    if (hb.fprev.p) HIPCHK(s, hipMemset(hb.fprev.p, 0, hb.fprev.bytes));
  *avg_us = ms * 1e3 / launches;
  if (inner_nodes) *inner_nodes = (int64_t)(s->cd.nx - 3) * (s->cd.ny - 2);
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_stream_copy(const void *src, void *dst, size_t bytes, int32_t workgroups,
                                 void *stream) {
  if (!src || !dst || src == dst || bytes == 0 || bytes % 16 || ((uintptr_t)src | (uintptr_t)dst) % 16 ||
      workgroups < 0 || workgroups > (1 << 20))
    return IB_LBM_E_INVALID;
  if (launch_stream_copy(src, dst, bytes / 16, workgroups ? workgroups : 256, (hipStream_t)stream) !=
      hipSuccess)
    return IB_LBM_E_DEVICE;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_timing_read(ib_lbm_sim *s, int32_t which, double *total_ms, int64_t *launches) {
  ib_lbm_status st = usable(s);
  if (st) return st;
  if (which < 0 || which >= kTimingKinds || !total_ms || !launches) return IB_LBM_E_INVALID;
  HIPCHK(s, hipStreamSynchronize(s->stream));
  double ms = s->timing.folded_ms[which];
  for (auto &p : s->timing.ev[which]) {
    float t = 0;
    HIPCHK(s, hipEventElapsedTime(&t, p.a, p.b));
    ms += t;
  }
  *total_ms = ms;
  *launches = s->timing.folded_n[which] + (int64_t)s->timing.ev[which].size();
  return IB_LBM_OK;
}

// ------------------------------------------------------------------ batches
#define BHIPCHK(b, call)                                                              \
  do {                                                                                \
    hipError_t e_ = (call);                                                           \
    if (e_ != hipSuccess) {                                                           \
      set_err(&(b)->err, "%s failed: %s", #call, hipGetErrorString(e_));              \
      (b)->broken = true;                                                             \
      return IB_LBM_E_DEVICE;                                                         \
    }                                                                                 \
  } while (0)

ib_lbm_status ib_lbm_batch_create(void *stream, int32_t precision, ib_lbm_batch **out) {
  if (!out || (precision != IB_LBM_FP64 && precision != IB_LBM_FP32_SHIFTED)) return IB_LBM_E_INVALID;
  ib_lbm_batch *b = new ib_lbm_batch();
  b->stream = (hipStream_t)stream;
  b->precision = precision;
  *out = b;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_batch_attach(ib_lbm_batch *b, ib_lbm_sim *s) {
  if (!b || !s) return IB_LBM_E_INVALID;
  if (b->broken || s->broken) return IB_LBM_E_STATE;
  if (s->batch) {
    set_err(&b->err, "sim already attached to a batch");
    return IB_LBM_E_STATE;
  }
  if (s->cd.precision != b->precision || s->stream != b->stream) {
    set_err(&b->err, "sim precision or stream differs from the batch");
    return IB_LBM_E_INVALID;
  }
  if (has_zou_he(s->cd)) {
    set_err(&b->err, "sims with Zou-He walls are stepped on their own, not in a batch");
    return IB_LBM_E_INVALID;
  }
  if (!s->bodies.empty() && s->bodies[0].dev.mdf_coupled) {
    set_err(&b->err, "sims with coupled MDF bodies are stepped on their own, not in a batch");
    return IB_LBM_E_INVALID;
  }
  ib_lbm_status st = build_sim_tables(s);
  if (st) return st;
  s->batch = b;
  s->started = true;
  b->sims.push_back(s);
  b->dirty = true;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_batch_detach(ib_lbm_batch *b, ib_lbm_sim *s) {
  if (!b || !s) return IB_LBM_E_INVALID;
  auto it = std::find(b->sims.begin(), b->sims.end(), s);
  if (it == b->sims.end()) return IB_LBM_E_INVALID;
  if (b->stream) (void)hipStreamSynchronize(b->stream);
  b->sims.erase(it);
  if (b->sims.empty()) arc_budget.give_back(b);
  s->batch = nullptr;
  b->dirty = true;
  // stepped on its own again: no target, and the lattice index the batch
  // launches left in the device state
  CaseState cs;
  BHIPCHK(b, hipMemcpy(&cs, s->state.p, sizeof cs, hipMemcpyDeviceToHost));
  cs.target = std::numeric_limits<int64_t>::max();
  BHIPCHK(b, hipMemcpy(s->state.p, &cs, sizeof cs, hipMemcpyHostToDevice));
  s->host_cur = cs.cur;
  s->halted = (cs.flags & kCaseHalted) != 0;
  s->hold_ready = false;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_batch_set_target(ib_lbm_batch *b, ib_lbm_sim *s, int64_t target) {
  if (!b || !s || s->batch != b || target < 0) return IB_LBM_E_INVALID;
  CaseState cs;
  BHIPCHK(b, hipStreamSynchronize(b->stream));
  BHIPCHK(b, hipMemcpy(&cs, s->state.p, sizeof cs, hipMemcpyDeviceToHost));
  cs.target = target;
  BHIPCHK(b, hipMemcpy(s->state.p, &cs, sizeof cs, hipMemcpyHostToDevice));
  return IB_LBM_OK;
}

static ib_lbm_status batch_tables(ib_lbm_batch *b) {
  if (!b->dirty) return IB_LBM_OK;
  // steps still queued read the tables (and replay the graph) rewritten here:
  // uploads are not ordered after the work of a non-blocking stream
  BHIPCHK(b, hipStreamSynchronize(b->stream));
  if (b->graph_exec) {
    (void)hipGraphExecDestroy(b->graph_exec);
    b->graph_exec = nullptr;
  }
  std::vector<CaseDesc> cases;
  std::vector<int32_t> prefix;
  std::vector<IbmSlot> slots;
  std::vector<ib_lbm_sim *> case_sims;  // the sim of each case entry
  std::vector<int32_t> fprefix;
  b->groups.clear();
  for (int col = 0; col < 3; col++) {
    ib_lbm_batch::Group g{col, (int)cases.size(), 0, 0, (int)prefix.size(), 0, 0};
    int tiles = 0, faces = 0;
    for (auto *s : b->sims) {
      if (s->cd.collision != col) continue;
      CaseDesc c = s->cd;
      fill_case_tiles(&c, b->launch);
      prefix.push_back(tiles);
      tiles += c.tiles_x * c.tiles_y;
      fprefix.push_back(faces);
      faces += face_blocks(c.nx, c.ny);
      cases.push_back(c);
      case_sims.push_back(s);
      g.count++;
      g.general_zg |= general_zero_gradient(c) ? 1 : 0;
    }
    prefix.push_back(tiles);
    fprefix.push_back(faces);
    g.ntiles = tiles;
    g.nface_blocks = faces;
    if (g.count) b->groups.push_back(g);
  }
  SlotLists lists;
  for (int ci = 0; ci < (int)cases.size(); ci++) lists.add(case_sims[ci]->bodies, ci, b->spread_mode);
  slots = lists.finish();
  auto reserve = [&](DevBuf *d, size_t bytes) -> ib_lbm_status {
    if (d->bytes >= bytes) return IB_LBM_OK;
    if (d->p) (void)hipFree(d->p);
    d->p = nullptr;
    d->bytes = 0;
    if (hipMalloc(&d->p, bytes) != hipSuccess) {
      set_err(&b->err, "batch table allocation failed");
      return IB_LBM_E_NOMEM;
    }
    d->bytes = bytes;
    return IB_LBM_OK;
  };
  auto upload = [&](DevBuf *d, const void *src, size_t bytes) -> ib_lbm_status {
    ib_lbm_status rs = reserve(d, bytes);
    if (rs) return rs;
    BHIPCHK(b, hipMemcpy(d->p, src, bytes, hipMemcpyHostToDevice));
    return IB_LBM_OK;
  };
  ib_lbm_status st;
  if (!cases.empty()) {
    if ((st = upload(&b->d_cases, cases.data(), cases.size() * sizeof(CaseDesc)))) return st;
    if ((st = upload(&b->d_prefix, prefix.data(), prefix.size() * sizeof(int32_t)))) return st;
    if ((st = upload(&b->d_fprefix, fprefix.data(), fprefix.size() * sizeof(int32_t)))) return st;
    if ((st = upload(&b->d_slots, slots.data(), slots.size() * sizeof(IbmSlot)))) return st;
  }
  b->ib = lists.ib;
  arc_budget.give_back(b);
  OneShape sh;
  // One launch per step saves a batch the launches per collision model and
  // their gaps; its tiles, compiled with the passes, have fewer waves per SIMD
  // than collide_stream_kernel's, which costs more the larger the batch.  us per
  // step in one launch and in several: FP32 5.5 M nodes 109 and 167, 17.5 M 341
  // and 366, 22 M 418 and 379, 131 M 2277 and 1923; FP64 5.5 M 181 and 248, 30 M
  // 888 and 912, 47 M 1374 and 1362, 131 M 3782 and 3579.
  int64_t nodes = 0;
  for (auto *s : case_sims) nodes += (int64_t)s->cd.nx * s->cd.ny;
  b->one = !cases.empty() && nodes <= (b->precision == IB_LBM_FP64 ? 40000000 : 20000000);
  b->one_face = 0;
  for (auto *s : case_sims) {
    b->one = b->one && sh.add(s->bodies, b->spread_mode);
    if (general_zero_gradient(s->cd)) b->one_face = 1;
  }
  if (b->one) {
    std::vector<StepOneArgs> one(cases.size());
    std::vector<int32_t> pre[3];
    StepBatchArgs &g = b->one_args;
    memset(&g, 0, sizeof g);
    for (size_t i = 0; i < cases.size(); i++) {
      fill_step_args(case_sims[i], sh.threads, 2, &one[i]);
      pre[0].push_back(g.nhold);
      pre[1].push_back(g.nface);
      pre[2].push_back(g.ntile);
      g.narcs += one[i].narcs;
      g.nhold += one[i].nhold;
      g.nface += one[i].nface;
      g.ntile += one[i].lean.ntiles;
    }
    b->one = arc_budget.take(case_sims[0]->dev, b->stream, b, g.narcs,
                             step_max_waiting(b->precision, b->one_face, false, true, sh.threads, sh.lds));
    if (b->one) {
      if ((st = upload(&b->d_one, one.data(), one.size() * sizeof(StepOneArgs)))) return st;
      std::vector<int32_t> all;
      for (auto &p : pre) all.insert(all.end(), p.begin(), p.end());
      if ((st = upload(&b->d_one_prefix, all.data(), all.size() * sizeof(int32_t)))) return st;
      const size_t n = cases.size();
      g.cases = (const StepOneArgs *)b->d_one.p;
      g.arcs = (const IbmSlot *)b->d_slots.p;
      g.hold_prefix = (const int32_t *)b->d_one_prefix.p;
      g.face_prefix = g.hold_prefix + n;
      g.tile_prefix = g.hold_prefix + 2 * n;
      g.ncases = (int)n;
      g.nwork = g.nhold + g.nface + (g.ntile + 7) / 8 * 8;
      if ((st = reserve(&b->d_work, (size_t)g.nwork * sizeof(StepWork)))) return st;
      g.work = (StepWork *)b->d_work.p;
      BHIPCHK(b, launch_batch_work(g, b->stream));
      b->one_threads = sh.threads;
      b->one_lds = sh.lds;
    }
  }

  b->dirty = false;
  return IB_LBM_OK;
}

static ib_lbm_status batch_enqueue_step(ib_lbm_batch *b, hipStream_t stream);

// Enqueue nsteps steps of the batch: one launch each where it can, after the
// control words are set from the cases' states, so that the parity of the
// launches always starts at 0.
static ib_lbm_status batch_enqueue(ib_lbm_batch *b, int64_t nsteps, hipStream_t stream) {
  if (nsteps <= 0) return IB_LBM_OK;
  if (!b->one) {
    for (int64_t i = 0; i < nsteps; i++) {
      ib_lbm_status st = batch_enqueue_step(b, stream);
      if (st) return st;
    }
    return IB_LBM_OK;
  }
  StepBatchArgs g = b->one_args;
  BHIPCHK(b, launch_batch_control(g.cases, g.ncases, stream));
  for (int64_t i = 0; i < nsteps; i++) {
    g.par = (int)(i & 1);
    BHIPCHK(b, launch_step_batch(b->precision, b->one_face, g, b->one_threads, b->one_lds, stream));
  }
  return IB_LBM_OK;
}

static ib_lbm_status batch_enqueue_step(ib_lbm_batch *b, hipStream_t stream) {
  LaunchShape sh{b->launch.block_x, b->launch.block_y, b->launch.rows_per_thread, b->launch.xcd_remap};
  for (auto &g : b->groups) {
    BHIPCHK(b, launch_collide_stream(b->precision, g.collision, (const CaseDesc *)b->d_cases.p + g.first,
                                     (const int32_t *)b->d_prefix.p + g.prefix_off, g.count, g.ntiles,
                                     sh, stream));
    BHIPCHK(b, launch_collide_stream_faces(b->precision, g.collision,
                                           (const CaseDesc *)b->d_cases.p + g.first,
                                           (const int32_t *)b->d_fprefix.p + g.prefix_off, g.count,
                                           g.nface_blocks, -1, 1, g.general_zg, stream));
  }
  BHIPCHK(b, launch_ibm_slots(b->precision, (const CaseDesc *)b->d_cases.p, (const IbmSlot *)b->d_slots.p,
                              b->ib, b->spread_mode, b->launch.ib_threads, stream));
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_batch_step(ib_lbm_batch *b, int64_t nsteps) {
  if (!b || nsteps < 0) return IB_LBM_E_INVALID;
  if (b->broken) return IB_LBM_E_STATE;
  ib_lbm_status st = batch_tables(b);
  if (st) return st;
  if (b->sims.empty()) return IB_LBM_OK;
  if (nsteps > 0) b->form = b->one ? IB_LBM_STEP_ONE : IB_LBM_STEP_PLAIN;
  int64_t left = nsteps;
  if (b->graph_steps > 0 && left >= b->graph_steps) {
    if (!b->graph_exec || b->graph_len != b->graph_steps) {
      if (b->graph_exec) (void)hipGraphExecDestroy(b->graph_exec);
      b->graph_exec = nullptr;
      if (!b->cap_stream) BHIPCHK(b, hipStreamCreateWithFlags(&b->cap_stream, hipStreamNonBlocking));
      hipGraph_t g;
      BHIPCHK(b, hipStreamBeginCapture(b->cap_stream, hipStreamCaptureModeThreadLocal));
      if ((st = batch_enqueue(b, b->graph_steps, b->cap_stream))) {
        hipGraph_t dummy;
        (void)hipStreamEndCapture(b->cap_stream, &dummy);
        return st;
      }
      BHIPCHK(b, hipStreamEndCapture(b->cap_stream, &g));
      BHIPCHK(b, hipGraphInstantiate(&b->graph_exec, g, nullptr, nullptr, 0));
      (void)hipGraphDestroy(g);
      b->graph_len = b->graph_steps;
    }
    while (left >= b->graph_len) {
      BHIPCHK(b, hipGraphLaunch(b->graph_exec, b->stream));
      left -= b->graph_len;
    }
  }
  return batch_enqueue(b, left, b->stream);
}

ib_lbm_status ib_lbm_batch_get_step_form(const ib_lbm_batch *b, int32_t *form) {
  if (!b || !form) return IB_LBM_E_INVALID;
  *form = b->form;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_batch_set_graph(ib_lbm_batch *b, int32_t steps_per_graph) {
  if (!b || steps_per_graph < 0 || steps_per_graph > 100000) return IB_LBM_E_INVALID;
  b->graph_steps = steps_per_graph;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_batch_set_launch(ib_lbm_batch *b, const ib_lbm_launch *l) {
  if (!b) return IB_LBM_E_INVALID;
  if (b->broken) return IB_LBM_E_STATE;
  ib_lbm_status st = check_launch(l, &b->err);
  if (st) return st;
  b->launch = *l;
  b->dirty = true;
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_batch_set_spread(ib_lbm_batch *b, int32_t mode) {
  if (!b) return IB_LBM_E_INVALID;
  if (mode != IB_LBM_SPREAD_GATHER && mode != IB_LBM_SPREAD_ATOMIC) return IB_LBM_E_INVALID;
  b->spread_mode = mode;
  b->dirty = true;
  if (b->graph_exec) {
    (void)hipGraphExecDestroy(b->graph_exec);
    b->graph_exec = nullptr;
  }
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_batch_sync(ib_lbm_batch *b) {
  if (!b) return IB_LBM_E_INVALID;
  if (b->broken) return IB_LBM_E_STATE;
  BHIPCHK(b, hipStreamSynchronize(b->stream));
  return IB_LBM_OK;
}

ib_lbm_status ib_lbm_batch_destroy(ib_lbm_batch *b) {
  if (!b) return IB_LBM_E_INVALID;
  if (b->stream) (void)hipStreamSynchronize(b->stream);
  for (auto *s : b->sims) s->batch = nullptr;
  arc_budget.give_back(b);
  if (b->graph_exec) (void)hipGraphExecDestroy(b->graph_exec);
  if (b->cap_stream) (void)hipStreamDestroy(b->cap_stream);
  if (b->d_cases.p) (void)hipFree(b->d_cases.p);
  if (b->d_prefix.p) (void)hipFree(b->d_prefix.p);
  if (b->d_fprefix.p) (void)hipFree(b->d_fprefix.p);
  if (b->d_slots.p) (void)hipFree(b->d_slots.p);
  if (b->d_one.p) (void)hipFree(b->d_one.p);
  if (b->d_one_prefix.p) (void)hipFree(b->d_one_prefix.p);
  if (b->d_work.p) (void)hipFree(b->d_work.p);
  delete b;
  return IB_LBM_OK;
}

const char *ib_lbm_batch_last_error(const ib_lbm_batch *b) { return b ? b->err.c_str() : "null batch"; }

}  // extern "C"
