// fvm_api.hip -- the C ABI (include/fvm.h): argument checking, plans, the
// ping-pong schedule, HIP-graph replay of step sequences, status handling.
// Host code only; the kernels live in fvm_kernels.hip, fvm_batch.hip and
// fvm_adjoint.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <cstdio>
#include <fstream>
#include <list>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/fvm.h"
#include "fvm_cluster.hpp"
#include "fvm_host.hpp"
#include "fvm_internal.hpp"
#include "fvm_models.hpp"

namespace fvm {
void* step_kernel_ptr(int model, int bc, int wpb, int cpl, bool halo);
hipError_t launch_resident_run(const StepArgs& a, int model, double* w_last, double* w_prev,
                               int nsteps, hipStream_t st);
hipError_t launch_step(const StepArgs& a, int model, hipStream_t st);
hipError_t launch_cfl(const CflArgs& a, int model, hipStream_t st);
hipError_t launch_clear_scratch(GridScratch* s, int n, hipStream_t st);
hipError_t launch_load(const LoadArgs& a, hipStream_t st);
hipError_t launch_set_log(GridScratch* s, int n, double* base, int cap, int stride,
                          hipStream_t st);
hipError_t launch_adjoint(const AdjointArgs& a, int model, const double* ug, hipStream_t st);
hipError_t launch_spray_adjoint(const AdjointArgs& a, const double* ug, hipStream_t st,
                                bool src);
hipError_t launch_maxent_adjoint_source(const AdjointArgs& a, const double* ug, hipStream_t st);
namespace cluster {
hipError_t launch_clear_area(GridScratch* scr, size_t words, hipStream_t st);
hipError_t launch_run(const Args& a, int model, hipStream_t st);
}  // namespace cluster

GridGeom grid_geometry(const fvm_params& p) {
  GridGeom g{};
  g.nx = p.nx;
  g.ny = p.ny;
  g.bc = p.bc;
  if (p.layout == FVM_LAYOUT_ROWS) {
    g.ld = fvm_nvar(p.model) * p.ld;
    g.plane = static_cast<size_t>(p.ld);
    g.uld = 2 * p.ld;
    g.uplane = static_cast<size_t>(p.ld);
  } else {
    g.ld = p.ld;
    g.plane = static_cast<size_t>(p.ld) * p.ny;
    g.uld = p.ld;
    g.uplane = g.plane;
  }
  g.rld = p.ld;
  g.dx = p.lx / p.nx;
  g.dy = p.ly / p.ny;
  g.cfl = p.cfl;
  g.dt_max = p.dt_max;
  g.hmin = g.dx < g.dy ? g.dx : g.dy;
  return g;
}

}  // namespace fvm

using namespace fvm;

namespace {

constexpr int kDefaultRows = 64;
constexpr int kDefaultWpb = 4;
// Runs are cut into graphs of 32, 16, 8, 4, 2 and 1 steps; the first run of
// a kind builds every chunk from both ping-pong buffers, so later runs of any
// length only replay cached graphs (no graph is built between the caller's
// launches).
constexpr int kGraphChunk = 32;
constexpr int kChunkSizes[6] = {32, 16, 8, 4, 2, 1};
constexpr size_t kGraphCacheMax = 40;

bool valid_params(const fvm_params* p) {
  if (!p) return false;
  if (fvm_nvar(p->model) == 0) return false;
  if (p->bc != FVM_PERIODIC && p->bc != FVM_TRANSMISSIVE && p->bc != FVM_DIRICHLET)
    return false;
  if (p->nx < 1 || p->ny < 1 || p->npart_x < 1 || p->npart_y < 1) return false;
  if (p->nx % p->npart_x != 0 || p->ny % p->npart_y != 0) return false;
  if (p->ld < p->nx) return false;
  if (p->layout != FVM_LAYOUT_PLANES && p->layout != FVM_LAYOUT_ROWS) return false;
  if (static_cast<long long>(p->ld) * fvm_nvar(p->model) > 2147483647ll) return false;
  if (!(p->lx > 0) || !(p->ly > 0) || !std::isfinite(p->lx) || !std::isfinite(p->ly)) return false;
  if (!(p->cfl > 0) || !std::isfinite(p->cfl)) return false;
  if (!(p->dt_max >= 0) || !std::isfinite(p->dt_max)) return false;
  const double cells = static_cast<double>(p->ld) * p->ny * fvm_nvar(p->model);
  if (cells > 9.0e15) return false;
  if (p->model == FVM_EULER && !(p->gamma > 1.0 && std::isfinite(p->gamma))) return false;
  if (p->model == FVM_ADV && !(std::isfinite(p->ax) && std::isfinite(p->ay))) return false;
  if (p->model == FVM_SPRAY) {
    if (!(p->K >= 0) || !std::isfinite(p->K)) return false;
    if (!(p->theta > 0)) return false;
    if (!(p->s_eps > 0 && p->s_eps < 1)) return false;
  }
  if (p->closure != FVM_CLOSURE_LOGNORMAL && p->closure != FVM_CLOSURE_MAXENT) return false;
  if (p->closure == FVM_CLOSURE_MAXENT && p->model != FVM_SPRAY) return false;
  return true;
}

// The kernel family of a grid: the model, or the transport-then-source pair
// of the spray with the entropy-maximising closure.
static int kernel_model(const fvm_params& p) {
  return p.model == FVM_SPRAY && p.closure == FVM_CLOSURE_MAXENT ? kSprayMaxEnt : p.model;
}

ModelConsts model_consts(const fvm_params& p) {
  ModelConsts m{};
  m.gamma = p.gamma;
  m.gm1 = p.gamma - 1.0;
  m.ax = p.ax;
  m.ay = p.ay;
  m.K = p.K;
  m.inv_theta = std::isinf(p.theta) ? 0.0 : 1.0 / p.theta;
  m.s_eps = p.s_eps;
  m.log_s_eps = p.s_eps > 0 ? std::log(p.s_eps) : 0.0;
  return m;
}


Tiling tiling(const GridGeom& g, int rows, int wpb, int cpl) {
  Tiling t{};
  t.rows = rows;
  t.wpb = wpb;
  t.cpl = cpl;
  const int w = strip_width(cpl) * wpb;
  t.tiles_x = (g.nx + w - 1) / w;
  t.tiles_y = (g.ny + rows - 1) / rows;
  t.ntiles = t.tiles_x * t.tiles_y;
  return t;
}

// The adjoint kernel's strips: 128 columns with two cells per lane, or 62
// columns with one (lanes 0 and 63 only supply the halo).
Tiling adjoint_tiling(const GridGeom& g, int rows, int wpb, int cpl) {
  Tiling t = tiling(g, rows, wpb, cpl);
  if (cpl == 1) {
    const int w = kOutPerWave * wpb;
    t.tiles_x = (g.nx + w - 1) / w;
    t.ntiles = t.tiles_x * t.tiles_y;
  }
  return t;
}

// Strip shape for strips_x x ny strip-rows: waves per workgroup (at most wmax)
// and rows per strip. A launch is over when its last workgroup is, so the
// workgroups should fill the chip's slots (per_cu waves on each of 256 CUs) a
// whole number of times: for each width the rows are the fewest that do so in
// as few rounds as keep them within max_rows, rounded up to the strip's
// unrolled rows, and the width is the one that leaves the least of the slots'
// wave-rows idle. Before, strips were sized for about 2048 waves whatever the
// rounds: Euler 2000^2 84.6 -> 55.6 us a step, 1531 x 997 at an odd pitch
// 47.7 -> 32.6, 4096^2 189.9 -> 181.0; spray 2048^2 100.0 -> 84.9, 1500 x 1100
// 60.1 -> 48.1; advection 3000 x 2500 42.6 -> 32.4; the adjoint of 1024^2 36.0 ->
// 26.0, of 4096^2 384 -> 323.
void fit_strips(long long strips_x, int ny, int per_cu, int unroll, int max_rows, int wmax,
                int* rows, int* wpb) {
  double best = 0.0;
  for (int w = wmax < per_cu ? wmax : per_cu; w >= 1; w /= 2) {
    const long long tiles_x = (strips_x + w - 1) / w;
    long long r = max_rows, rounds = 1;
    for (; rounds < 4096; ++rounds) {
      const long long ty = 256 * rounds * (per_cu / w) / tiles_x;
      if (ty < 1) continue;
      r = ((ny + ty - 1) / ty + unroll - 1) / unroll * unroll;
      if (r <= max_rows) break;
    }
    r = r > max_rows ? max_rows : r;
    const double used = static_cast<double>(strips_x) * ny / (rounds * 256.0 * per_cu * r);
    if (used > 1.03 * best) {
      best = used;
      *rows = static_cast<int>(r);
      *wpb = w;
    }
  }
}

// Lane layout and strip shape of the step for a grid whose buffers allow two
// cells per lane or not (wide). A grid of few cells takes one cell per lane and
// three rows (one turn of that strip's unrolled ring): the launch is as long
// as one strip, and 200 x 150 Euler cells take 8.2 us a step so, 130 x 96 7.5,
// against 10.3 and 10.2 in two-cells-per-lane strips of four rows (spray 200^2
// 10.5 against 14.7); from 512^2 on the wide strips are as fast or faster.
constexpr long long kFewStrips = 700;
int default_layout(const fvm_params& p, bool wide) {
  const long long strips = static_cast<long long>((p.nx + kWave - 1) / kWave) * ((p.ny + 2) / 3);
  return wide && strips > kFewStrips ? 2 : 1;
}
void default_tiling(const fvm_params& p, int cpl, int* rows, int* wpb) {
  const long long strips_x = (p.nx + strip_width(cpl) - 1) / strip_width(cpl);
  const bool transport = p.closure == FVM_CLOSURE_MAXENT;
  // rows of a strip's unrolled loop: loads in flight and two
  int unroll;
  if (p.model == FVM_ADV) unroll = 2 + (cpl == 2 ? FVM_PREFETCH2_ADV : FVM_PREFETCH1_ADV);
  else if (p.model == FVM_EULER) unroll = 2 + (cpl == 2 ? FVM_PREFETCH2_EULER : FVM_PREFETCH1_EULER);
  else if (transport) unroll = 3;
  else unroll = 2 + (cpl == 2 ? FVM_PREFETCH2_SPRAY : FVM_PREFETCH1_SPRAY);
  if (cpl == 1 && default_layout(p, true) == 1) {
    int w = 1;
    while (w < 8 && w < strips_x) w *= 2;
    *rows = unroll;
    *wpb = w;
    return;
  }
  // waves a CU runs well: one per SIMD for Euler's two-cells-per-lane strips
  // (256 registers), two for the others
  const int per_cu = p.model == FVM_EULER && cpl == 2 ? 4 : 8;
  fit_strips(strips_x, p.ny, per_cu, unroll, 128, 8, rows, wpb);
}

// The adjoint's strips: 62 columns, two waves per SIMD, two unrolled rows
// (advection four); tiles taller than 16 rows run slower although they re-read
// fewer rows.
void default_adjoint_tiling(const fvm_params& p, int* rows, int* wpb) {
  const int unroll = p.model == FVM_EULER ? 2 : 4;
  fit_strips((p.nx + kOutPerWave - 1) / kOutPerWave, p.ny, 8, unroll, 16, 4, rows, wpb);
}

bool valid_tiling(int rows, int wpb) {
  return rows >= 1 && rows <= 4096 && (wpb == 1 || wpb == 2 || wpb == 4 || wpb == 8);
}

int dev_err(hipError_t e) { return e == hipSuccess ? FVM_OK : FVM_EDEVICE; }

int status_from_bits(unsigned int st) {
  if (st & kStatusWait) return FVM_EDEVICE;
  if (st & kStatusNonFinite) return FVM_ENONFINITE;
  if (st & kStatusCfl) return FVM_ECFL;
  if (st & kStatusDt) return FVM_EINVAL;
  return FVM_OK;
}

// The tiles of a run that keeps the state on the chip; false where the grid
// does not fit or its step is not one kernel (entropy closure).
bool cluster_plan(const fvm_params& p, cluster::Plan* plan) {
  return p.closure == FVM_CLOSURE_LOGNORMAL &&
         cluster::make_plan(fvm_nvar(p.model), p.nx, p.ny, plan);
}
size_t cluster_bytes(const fvm_params& p) {
  cluster::Plan plan;
  if (!cluster_plan(p, &plan)) return 0;
  return (sizeof(cluster::u64) * cluster::area_words(fvm_nvar(p.model), plan) + 255) / 256 * 256;
}

// Two such runs at once, from two streams, could each hold some of the CUs
// and wait for the rest, so unordered runs have to fit the chip together. The
// chip is handed out in parts of 32 CUs, as many to a run as its tiles fill, and
// a run takes parts that its own stream had before or whose last run is over;
// where those do not suffice it does not wait for the other streams (which may
// have any amount of work ahead of their run) but makes its steps in launches,
// hipErrorNotReady here. A stream's own parts are waited for, which costs nothing
// on one stream: equal handles need not be one stream (hipStreamPerThread names a
// stream per thread, and a destroyed stream's handle may be another's by now). us
// for a run(50) on each of 8 streams, so / one run at a time / all as step launches:
// Euler 64^2 540 / 2010 / 1148, 200 x 150 1074 / 2178 / 1383, spray 200^2 1272 / 2429 /
// 1969; 512^2, which fills the chip, on 4 streams 1225 / 1672 / 2012, on 2 1107 / 836 /
// 904. The events are kept until the process ends.
constexpr int kParts = 8;
constexpr int kPartTiles = cluster::kMaxTiles / kParts;
struct ChipPart {
  hipEvent_t ended = nullptr;   // end of the part's last run; null: it is over
  hipStream_t stream = nullptr;
  unsigned long long used = 0;  // number of that run
};
struct Chip {
  std::mutex mu;
  ChipPart part[kParts];
  hipEvent_t event[kParts] = {};
  unsigned long long runs = 0;
};
constexpr int kChipDevices = 64;
Chip g_chip[kChipDevices];

int parts_of(int cus) { return std::min(cus / kPartTiles, kParts); }
int parts_for(const cluster::Plan& p) { return (p.tiles + kPartTiles - 1) / kPartTiles; }

// While it lives, calls of this thread are allowed that a capture of another
// thread would forbid (they do not touch its stream).
struct CaptureAside {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  CaptureAside() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
  ~CaptureAside() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

// Marks the parts whose last run is over, of other streams than st.
void find_free_parts(Chip& c, int parts, hipStream_t st) {
  CaptureAside aside;
  for (int k = 0; k < parts; ++k) {
    const hipEvent_t e = c.part[k].ended;
    if (!e || c.part[k].stream == st) continue;
    bool seen = false;
    for (int q = 0; q < k; ++q) seen = seen || c.part[q].ended == e;
    if (seen) continue;  // asked, and not over
    if (hipEventQuery(e) == hipSuccess) {
      for (int q = k; q < parts; ++q)
        if (c.part[q].ended == e) c.part[q].ended = nullptr;
    } else {
      (void)hipGetLastError();  // (not ready is no error)
    }
  }
}

// hipErrorNotReady: too little of the chip is free, nothing has been enqueued.
hipError_t launch_on_chip(const cluster::Args& a, int model, int device, int cus,
                          hipStream_t st) {
  Chip& c = g_chip[device];
  std::lock_guard<std::mutex> lock(c.mu);
  const int parts = parts_of(cus), n = parts_for(a.plan);
  if (n > parts) return hipErrorInvalidValue;
  ChipPart* order[kParts];
  const auto own = [st](const ChipPart* p) { return p->ended && p->stream == st; };
  const auto usable = [&](const ChipPart* p) { return !p->ended || p->stream == st; };
  for (int k = 0; k < parts; ++k) order[k] = &c.part[k];
  if (std::count_if(order, order + parts, usable) < n) find_free_parts(c, parts, st);
  // the stream's own, then free ones (the one not used for longest first)
  std::stable_sort(order, order + parts, [&](const ChipPart* x, const ChipPart* y) {
    const int rx = own(x) ? 0 : (usable(x) ? 1 : 2), ry = own(y) ? 0 : (usable(y) ? 1 : 2);
    return rx != ry ? rx < ry : x->used < y->used;
  });
  if (!usable(order[n - 1])) return hipErrorNotReady;
  hipError_t e = hipSuccess;
  for (int k = 0; k < n && e == hipSuccess; ++k) {
    bool waited = !order[k]->ended;
    for (int q = 0; q < k; ++q) waited = waited || order[q]->ended == order[k]->ended;
    if (!waited) e = hipStreamWaitEvent(st, order[k]->ended, 0);
  }
  // an event that no other part's last run needs
  hipEvent_t* ended = nullptr;
  for (int q = 0; q < kParts && !ended; ++q) {
    bool needed = false;
    for (int k = n; k < parts; ++k) needed = needed || (c.event[q] && order[k]->ended == c.event[q]);
    if (!needed) ended = &c.event[q];
  }
  if (e == hipSuccess && !*ended) {
    CaptureAside aside;
    e = hipEventCreateWithFlags(ended, hipEventDisableTiming);
  }
  if (e != hipSuccess) return e;
  e = cluster::launch_run(a, model, st);
  if (e != hipSuccess) return e;
  // (without its event the run must be over before the parts are given away)
  if (hipEventRecord(*ended, st) != hipSuccess) return hipStreamSynchronize(st);
  ++c.runs;
  for (int k = 0; k < n; ++k) {
    order[k]->ended = *ended;
    order[k]->stream = st;
    order[k]->used = c.runs;
  }
  return hipSuccess;
}

struct GraphKey {
  int kind;              // 0 adaptive run, 1 dts run, 2 tuner's dry run, 3 fixed-dt run
  int nsteps;
  const double* start;   // input buffer of the first step
  const double* other;
  const double* dts;
  int k0;
  int rows, wpb, cpl;
  double dt;             // kind 3
  const double* me_lam;  // entropy closure: the multiplier buffer, and whether
  bool me_warm;          // the graph's first step starts from it
  bool operator==(const GraphKey& o) const {
    return kind == o.kind && nsteps == o.nsteps && start == o.start && other == o.other &&
           dts == o.dts && k0 == o.k0 && rows == o.rows && wpb == o.wpb &&
           cpl == o.cpl && dt == o.dt && me_lam == o.me_lam && me_warm == o.me_warm;
  }
};

struct CachedGraph {
  GraphKey key;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

}  // namespace

struct fvm_grid {
  fvm_params p{};
  int nv = 0;
  GridGeom g{};
  ModelConsts m{};
  int rows = kDefaultRows, wpb = kDefaultWpb;
  int adj_rows = kDefaultRows, adj_wpb = kDefaultWpb;  // adjoint kernel tile shape
  int adj_cpl = 1;   // adjoint cells per lane (the tuner may pick 2 where allowed)
  int cpl_req = 0;   // requested cells per lane (0: the widest the buffers allow)
  bool resident = true;  // grids that fit on the chip keep the state there for a whole run
  cluster::Plan plan{};  // .. their tiles, and whether there are any
  bool plan_ok = false;
  bool default_strips = true;  // rows and wpb are the default for the layout
  // the caller has chosen a strip shape or lane layout: its runs are step launches
  bool strips_asked = false, lanes_asked = false;
  int device = -1;       // current at bind, -1 if it cannot hold the plan's tiles at once
  int cus = 0;           // .. its CUs
  int cpl = 1;       // layout in use
  double* w_a = nullptr;
  double* w_b = nullptr;
  double* cur = nullptr;
  const double* ug = nullptr;
  double ghost[4 * kMaxVar] = {};  // Dirichlet states, ghost[side * kMaxVar + v]
  Halo halo{};                     // rows from the caller's buffers
  double* me_lam = nullptr;        // entropy closure: the caller's multiplier buffer
  bool me_valid = false;           // it holds the multipliers of the current state's cells
  GridScratch* scr = nullptr;
  cluster::u64* area() const { return reinterpret_cast<cluster::u64*>(scr + 1); }
  const double* log_armed = nullptr;  // dt log the scratch currently points to
  hipStream_t stream = nullptr;
  bool bound = false;
  bool speeds_valid = false;
  std::list<CachedGraph> graphs;

  ~fvm_grid() { clear_graphs(); }
  void clear_graphs() {
    for (auto& c : graphs) {
      if (c.exec) (void)hipGraphExecDestroy(c.exec);
      if (c.graph) (void)hipGraphDestroy(c.graph);
    }
    graphs.clear();
  }
  double* other(const double* w) const { return w == w_a ? w_b : w_a; }

  // doubles in one state (either layout)
  size_t elems() const { return static_cast<size_t>(nv) * p.ny * p.ld; }

  StepArgs step_args(const double* win, double* wout, int mode) const {
    StepArgs a{};
    a.win = win;
    a.wout = wout;
    a.ug = ug;
    a.scr = scr;
    a.mode = mode;
    a.g = g;
    a.t = tiling(g, rows, wpb, cpl);
    a.m = m;
    for (int k = 0; k < 4 * kMaxVar; ++k) a.ghost[k] = ghost[k];
    a.halo = halo;
    return a;
  }
};

extern "C" {

const char* fvm_strerror(int status) {
  switch (status) {
    case FVM_OK: return "ok";
    case FVM_EINVAL: return "invalid argument";
    case FVM_EDEVICE: return "HIP runtime error";
    case FVM_ECFL: return "fixed time step violates the CFL condition";
    case FVM_ENONFINITE: return "non-finite or non-physical state";
    case FVM_EUNSUPPORTED: return "operation not supported for this model";
    case FVM_EIO: return "file output failed";
    default: return "unknown status";
  }
}

int fvm_nvar(int model) {
  switch (model) {
    case FVM_ADV: return 1;
    case FVM_EULER: return 4;
    case FVM_SPRAY: return 6;
    default: return 0;
  }
}

int fvm_validate(const fvm_params* p) { return valid_params(p) ? FVM_OK : FVM_EINVAL; }

size_t fvm_scratch_bytes(const fvm_params* p) {
  if (!valid_params(p)) return 0;
  return sizeof(GridScratch) + cluster_bytes(*p);
}

int fvm_create(const fvm_params* p, fvm_grid** out) {
  if (!out) return FVM_EINVAL;
  *out = nullptr;
  if (!valid_params(p)) return FVM_EINVAL;
  if (p->closure == FVM_CLOSURE_MAXENT && p->bc == FVM_DIRICHLET) return FVM_EUNSUPPORTED;
  fvm_grid* g = new (std::nothrow) fvm_grid();
  if (!g) return FVM_EINVAL;
  g->p = *p;
  g->nv = fvm_nvar(p->model);
  default_tiling(*p, default_layout(*p, p->ld % 2 == 0), &g->rows, &g->wpb);
  default_adjoint_tiling(*p, &g->adj_rows, &g->adj_wpb);
  g->g = grid_geometry(*p);
  g->m = model_consts(*p);
  g->plan_ok = cluster_plan(*p, &g->plan);
  *out = g;
  return FVM_OK;
}

int fvm_destroy(fvm_grid* g) {
  delete g;
  return FVM_OK;
}

// Two cells per lane needs an even pitch and 16-byte aligned buffers.
static bool wide_layout_ok(const fvm_grid* g) {
  auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  return g->p.ld % 2 == 0 && al(g->w_a) && al(g->w_b) && (!g->ug || al(g->ug));
}

// The adjoint covers every model and closure, without halo rows.
static bool adjoint_supported(const fvm_grid* g) { return !g->halo.s && !g->halo.n; }

// The adjoint's lane layout for one launch: two cells per lane needs an even
// pitch and 16-byte aligned state and multiplier buffers.
static int adjoint_cpl(const fvm_grid* g, const double* w, const double* li, const double* lo) {
  auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  return g->adj_cpl == 2 && g->p.ld % 2 == 0 && al(w) && al(li) && al(lo) ? 2 : 1;
}

static void choose_layout(fvm_grid* g) {
  const bool wide = g->bound && wide_layout_ok(g);
  const int cpl = g->cpl_req ? (wide ? g->cpl_req : 1) : default_layout(g->p, wide);
  if (cpl != g->cpl) g->clear_graphs();
  g->cpl = cpl;
  if (g->default_strips && g->bound) default_tiling(g->p, cpl, &g->rows, &g->wpb);
}

int fvm_bind(fvm_grid* g, double* w_a, double* w_b, const double* ug, void* scratch,
             void* stream) {
  if (!g || !w_a || !w_b || !scratch || w_a == w_b) return FVM_EINVAL;
  if ((reinterpret_cast<uintptr_t>(scratch) & 255) != 0) return FVM_EINVAL;
  if ((reinterpret_cast<uintptr_t>(w_a) & 7) || (reinterpret_cast<uintptr_t>(w_b) & 7))
    return FVM_EINVAL;
  if (g->p.model == FVM_SPRAY && !ug) return FVM_EINVAL;
  if (g->p.model != FVM_SPRAY && ug) return FVM_EINVAL;
  g->clear_graphs();
  g->w_a = w_a;
  g->w_b = w_b;
  g->cur = w_a;
  g->ug = ug;
  g->scr = static_cast<GridScratch*>(scratch);
  g->stream = static_cast<hipStream_t>(stream);
  g->bound = true;
  choose_layout(g);
  g->speeds_valid = false;
  g->me_valid = false;
  g->log_armed = nullptr;
  if (g->plan_ok) {  // one workgroup of a run per CU, all of them at once
    if (hipGetDevice(&g->device) != hipSuccess ||
        hipDeviceGetAttribute(&g->cus, hipDeviceAttributeMultiprocessorCount, g->device) !=
            hipSuccess)
      return FVM_EDEVICE;
    if (g->device >= kChipDevices || parts_of(g->cus) < parts_for(g->plan)) g->device = -1;
    return dev_err(
        cluster::launch_clear_area(g->scr, cluster::area_words(g->nv, g->plan), g->stream));
  }
  return dev_err(launch_clear_scratch(g->scr, 1, g->stream));
}

int fvm_set_boundary_states(fvm_grid* g, const double* ghost) {
  if (!g || !ghost || g->p.bc != FVM_DIRICHLET) return FVM_EINVAL;
  for (int k = 0; k < 4 * g->nv; ++k)
    if (!std::isfinite(ghost[k])) return FVM_EINVAL;
  for (int side = 0; side < 4; ++side)
    for (int v = 0; v < g->nv; ++v) g->ghost[side * kMaxVar + v] = ghost[side * g->nv + v];
  g->clear_graphs();  // the cached graphs hold the previous states
  return FVM_OK;
}

int fvm_set_halo_rows(fvm_grid* g, const double* south, const double* north) {
  if (!g) return FVM_EINVAL;
  if ((g->p.bc == FVM_DIRICHLET || g->p.closure == FVM_CLOSURE_MAXENT) && (south || north))
    return FVM_EUNSUPPORTED;
  g->halo.s = south;
  g->halo.n = north;
  g->clear_graphs();  // the cached graphs hold the previous pointers
  return FVM_OK;
}

int fvm_set_closure_buffer(fvm_grid* g, double* lam) {
  if (!g) return FVM_EINVAL;
  if (g->p.closure != FVM_CLOSURE_MAXENT) return lam ? FVM_EUNSUPPORTED : FVM_OK;
  if (lam && (reinterpret_cast<uintptr_t>(lam) & 7)) return FVM_EINVAL;
  g->me_lam = lam;
  g->me_valid = false;
  g->clear_graphs();  // the cached graphs hold the previous pointer
  return FVM_OK;
}

int fvm_set_stream(fvm_grid* g, void* stream) {
  if (!g) return FVM_EINVAL;
  g->stream = static_cast<hipStream_t>(stream);
  return FVM_OK;
}

int fvm_current(const fvm_grid* g, double** w) {
  if (!g || !w || !g->bound) return FVM_EINVAL;
  *w = g->cur;
  return FVM_OK;
}

}  // extern "C"

namespace fvm {
int grid_view(const fvm_grid* g, GridView* v) {
  if (!g || !v || !g->bound) return FVM_EINVAL;
  v->p = g->p;
  v->g = g->g;
  v->nv = g->nv;
  v->cur = g->cur;
  v->stream = g->stream;
  return FVM_OK;
}
}  // namespace fvm

extern "C" {

int fvm_set_state(fvm_grid* g, const double* src, int src_on_device) {
  if (!g || !src || !g->bound) return FVM_EINVAL;
  const size_t bytes = sizeof(double) * g->elems();
  hipError_t e = hipMemcpyAsync(g->cur, src, bytes,
                                src_on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice,
                                g->stream);
  if (e == hipSuccess && !src_on_device) e = hipStreamSynchronize(g->stream);
  g->speeds_valid = false;
  g->me_valid = false;
  return dev_err(e);
}

int fvm_load(fvm_grid* g, const double* src, long long var_stride, long long row_stride, int cols,
             double* dst) {
  if (!g || !src || !g->bound || var_stride < 0 || row_stride < 0) return FVM_EINVAL;
  if (cols != g->p.nx && cols != g->p.ld) return FVM_EINVAL;
  double* const to = dst ? dst : g->cur;
  const uintptr_t s = reinterpret_cast<uintptr_t>(src), d = reinterpret_cast<uintptr_t>(to);
  if (s % 8 || d % 8) return FVM_EUNSUPPORTED;
  const size_t extent = static_cast<size_t>(var_stride) * (g->nv - 1) +
                        static_cast<size_t>(row_stride) * (g->p.ny - 1) + cols;
  if (s < d + 8 * g->elems() && d < s + 8 * extent) return FVM_EUNSUPPORTED;
  int dev = 0, sdev = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipStreamGetDevice(g->stream, &sdev) != hipSuccess)
    return FVM_EDEVICE;
  if (dev != sdev) return FVM_EUNSUPPORTED;
  LoadArgs a{};
  a.src = src;
  a.dst = to;
  a.var_stride = var_stride;
  a.row_stride = row_stride;
  a.nv = static_cast<unsigned int>(g->nv);
  a.ny = static_cast<unsigned int>(g->p.ny);
  a.cols = static_cast<unsigned int>(cols);
  a.ld = static_cast<unsigned int>(g->p.ld);
  a.by_rows = g->p.layout == FVM_LAYOUT_ROWS;
  const hipError_t e = launch_load(a, g->stream);
  if (e == hipErrorInvalidValue) return FVM_EUNSUPPORTED;  // too many rows for one launch
  if (!dst) g->speeds_valid = g->me_valid = false;
  return dev_err(e);
}

int fvm_get_state(fvm_grid* g, double* dst, int dst_on_device) {
  if (!g || !dst || !g->bound) return FVM_EINVAL;
  const size_t bytes = sizeof(double) * g->elems();
  hipError_t e = hipMemcpyAsync(dst, g->cur, bytes,
                                dst_on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost,
                                g->stream);
  if (e == hipSuccess && !dst_on_device) e = hipStreamSynchronize(g->stream);
  return dev_err(e);
}

// Points the scratch's dt log at `log` (cap entries, cursor rewound) for the
// steps enqueued next; log == null turns logging off. Every path that
// enqueues steps calls it first, so no step logs into a buffer of an earlier
// run.
static int arm_log(fvm_grid* g, double* log, int cap) {
  if (!log && !g->log_armed) return FVM_OK;
  const int rc = dev_err(launch_set_log(g->scr, 1, log, cap, 1, g->stream));
  if (rc == FVM_OK) g->log_armed = log;
  return rc;
}

// One step launch outside a graph: the step kernel, and for the entropy
// closure the source pass that completes it.
static int enqueue_step(fvm_grid* g, const StepArgs& a) {
  const int km = kernel_model(g->p);
  int rc = dev_err(launch_step(a, km, g->stream));
  if (rc || km != kSprayMaxEnt) return rc;
  MaxEntWarm wm{g->me_lam, g->me_lam && g->me_valid ? 1 : 0, 0};
  rc = dev_err(launch_maxent_source(a, wm, g->stream));
  if (rc == FVM_OK && g->me_lam) g->me_valid = true;
  return rc;
}

static int enqueue_cfl(fvm_grid* g, double* dt_dev) {
  CflArgs a{};
  a.w = g->cur;
  a.scr = g->scr;
  a.dt_out = dt_dev;
  a.g = g->g;
  a.m = g->m;
  const int rc = dev_err(launch_cfl(a, g->p.model, g->stream));
  if (rc == FVM_OK) g->speeds_valid = true;
  return rc;
}

int fvm_cfl_dt(fvm_grid* g, double* dt_dev) {
  if (!g || !g->bound) return FVM_EINVAL;
  return enqueue_cfl(g, dt_dev);
}

static int read_scratch(fvm_grid* g, GridScratch* host) {
  hipError_t e = hipStreamSynchronize(g->stream);
  if (e == hipSuccess) e = hipMemcpy(host, g->scr, sizeof(GridScratch), hipMemcpyDeviceToHost);
  return dev_err(e);
}

int fvm_cfl_dt_host(fvm_grid* g, double* dt, double* sx, double* sy) {
  if (!g || !g->bound || !dt) return FVM_EINVAL;
  int rc = enqueue_cfl(g, nullptr);
  if (rc) return rc;
  GridScratch h;
  rc = read_scratch(g, &h);
  if (rc) return rc;
  *dt = h.dt;
  if (sx) *sx = h.cur_sx;
  if (sy) *sy = h.cur_sy;
  return status_from_bits(h.status);
}

int fvm_sync(fvm_grid* g) {
  if (!g || !g->bound) return FVM_EINVAL;
  GridScratch h;
  const int rc = read_scratch(g, &h);
  if (rc) return rc;
  return status_from_bits(h.status);
}

int fvm_get_status(fvm_grid* g, int clear) {
  if (!g || !g->bound) return FVM_EINVAL;
  GridScratch h;
  int rc = read_scratch(g, &h);
  if (rc) return rc;
  rc = status_from_bits(h.status);
  if (clear && (h.status & kStatusWait)) {
    // a run on the chip broke off: its counts and exchange words go too
    hipError_t e = cluster::launch_clear_area(g->scr, cluster::area_words(g->nv, g->plan),
                                              g->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(g->stream);
    g->speeds_valid = false;
    g->log_armed = nullptr;
    if (e != hipSuccess) return FVM_EDEVICE;
  } else if (clear && h.status) {
    const unsigned int zero = 0;
    const hipError_t e = hipMemcpy(&g->scr->status, &zero, sizeof(zero), hipMemcpyHostToDevice);
    if (e != hipSuccess) return FVM_EDEVICE;
  }
  return rc;
}

int fvm_step(fvm_grid* g, double dt) {
  if (!g || !g->bound) return FVM_EINVAL;
  if (!(dt > 0.0) || !std::isfinite(dt)) return FVM_EINVAL;
  int rc = FVM_OK;
  if (!g->speeds_valid) rc = enqueue_cfl(g, nullptr);
  if (rc == FVM_OK) rc = arm_log(g, nullptr, 0);
  if (rc) return rc;
  StepArgs a = g->step_args(g->cur, g->other(g->cur), kDtFixedCheck);
  a.dt_arg = dt;
  rc = enqueue_step(g, a);
  if (rc == FVM_OK) g->cur = a.wout;
  return rc;
}

static GraphKey graph_key(const fvm_grid* g, int kind, int n, const double* start,
                          const double* dts, int k0, double dt) {
  const bool me_warm = g->me_lam && g->me_valid;
  return GraphKey{kind,   n,      start,  g->other(start), dts, k0,
                  g->rows, g->wpb, g->cpl, dt, g->me_lam, me_warm};
}

// The cached graph of `key`, moved to the front of the cache, or null.
static CachedGraph* find_graph(fvm_grid* g, const GraphKey& key) {
  for (auto it = g->graphs.begin(); it != g->graphs.end(); ++it) {
    if (it->key == key) {
      g->graphs.splice(g->graphs.begin(), g->graphs, it);
      return &g->graphs.front();
    }
  }
  return nullptr;
}

// Builds the graph of `key`: n consecutive steps starting from buffer
// key.start, with step k reading its dt according to the kind.
static int build_graph(fvm_grid* g, const GraphKey& key, hipGraphExec_t* exec) {
  const int kind = key.kind, n = key.nsteps, k0 = key.k0;
  const double* start = key.start;
  const double* dts = key.dts;
  const double dt = key.dt;
  const bool me_warm = key.me_warm;
  CachedGraph c;
  c.key = key;
  if (hipGraphCreate(&c.graph, 0) != hipSuccess) return FVM_EDEVICE;
  hipGraphNode_t prev = nullptr;
  const double* in = start;
  const int km = kernel_model(g->p);
  void* fn = step_kernel_ptr(km, g->p.bc, g->wpb, g->cpl, g->halo.s || g->halo.n);
  std::vector<StepArgs> args(n);
  for (int s = 0; s < n; ++s) {
    double* out = g->other(in);
    args[s] = g->step_args(in, out,
                           kind == 0 ? kDtAdaptive : (kind == 3 ? kDtFixedCheck : kDtArray));
    args[s].dts = dts;
    args[s].dt_arg = dt;
    args[s].k = kind == 2 ? 0 : k0 + s;  // kind 2: dry run, dts = the scratch's zero
    void* kp[] = {&args[s]};
    hipKernelNodeParams np{};
    np.func = fn;
    np.gridDim = dim3(args[s].t.ntiles);
    np.blockDim = dim3(g->wpb * kWave);
    np.sharedMemBytes = 0;
    np.kernelParams = kp;
    np.extra = nullptr;
    hipGraphNode_t node;
    if (hipGraphAddKernelNode(&node, c.graph, prev ? &prev : nullptr, prev ? 1 : 0, &np) !=
        hipSuccess) {
      (void)hipGraphDestroy(c.graph);
      return FVM_EDEVICE;
    }
    prev = node;
    if (km == kSprayMaxEnt) {  // the source pass completes the step
      MaxEntLaunch ml = maxent_launch(args[s]);
      MaxEntWarm wm{g->me_lam, g->me_lam && (me_warm || s > 0) ? 1 : 0, 0};
      void* mp[] = {&args[s], &ml.rule, &wm};
      hipKernelNodeParams sp{};
      sp.func = ml.fn;
      sp.gridDim = ml.grid;
      sp.blockDim = ml.block;
      sp.kernelParams = mp;
      if (hipGraphAddKernelNode(&node, c.graph, &prev, 1, &sp) != hipSuccess) {
        (void)hipGraphDestroy(c.graph);
        return FVM_EDEVICE;
      }
      prev = node;
    }
    in = out;
  }
  if (hipGraphInstantiate(&c.exec, c.graph, nullptr, nullptr, 0) != hipSuccess) {
    (void)hipGraphDestroy(c.graph);
    return FVM_EDEVICE;
  }
  g->graphs.push_front(c);
  while (g->graphs.size() > kGraphCacheMax) {
    auto& b = g->graphs.back();
    (void)hipGraphExecDestroy(b.exec);
    (void)hipGraphDestroy(b.graph);
    g->graphs.pop_back();
  }
  *exec = c.exec;
  return FVM_OK;
}

// Finds or builds the graph of `n` consecutive steps starting from buffer
// `start`, with step k reading its dt according to `kind`.
static int graph_for(fvm_grid* g, int kind, int n, double* start, const double* dts, int k0,
                     hipGraphExec_t* exec, double dt = 0.0) {
  const GraphKey key = graph_key(g, kind, n, start, dts, k0, dt);
  if (CachedGraph* c = find_graph(g, key)) {
    *exec = c->exec;
    return FVM_OK;
  }
  return build_graph(g, key, exec);
}

// Adaptive and fixed-dt runs: on a miss, builds the graph of every chunk size
// from both ping-pong buffers, so that any later run of this kind and
// configuration only replays.
static int chunk_graph(fvm_grid* g, int kind, int n, double dt, hipGraphExec_t* exec) {
  const GraphKey key = graph_key(g, kind, n, g->cur, nullptr, 0, dt);
  if (CachedGraph* c = find_graph(g, key)) {
    *exec = c->exec;
    return FVM_OK;
  }
  for (double* start : {g->other(g->cur), g->cur}) {
    for (int m : kChunkSizes) {
      if (start == g->cur && m == n) continue;  // built last: it heads the cache
      const GraphKey k = graph_key(g, kind, m, start, nullptr, 0, dt);
      hipGraphExec_t e;
      if (!find_graph(g, k) && build_graph(g, k, &e) != FVM_OK) return FVM_EDEVICE;
    }
  }
  return build_graph(g, key, exec);
}

// The largest chunk size not above `left`.
static int chunk_size(int left) {
  for (int m : kChunkSizes)
    if (m <= left) return m;
  return 1;
}

// A run of adaptive steps on this grid can stay in one workgroup's LDS:
// advection, Euler or the lognormal spray, no halo rows, two states within
// kResidentDoubles.
static bool resident_ok(const fvm_grid* g) {
  if (!g->resident || g->halo.s || g->halo.n) return false;
  if (g->p.model == FVM_SPRAY && g->p.closure != FVM_CLOSURE_LOGNORMAL) return false;
  const long long need = 2LL * fvm_nvar(g->p.model) * g->p.nx * g->p.ny;
  return need <= kResidentDoubles;
}

// The stream is being captured, or may be.
static bool capturing(hipStream_t st) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing(st, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone;
}

// A run of steps can keep the state in the LDS of all CUs: the grid fits, no
// halo rows, the caller has not asked for a strip shape, the stream is one of the
// grid's device, which is the current one (the turns' events are its own), and
// is not being captured (the launch may have to wait for another stream's).
static bool cluster_ok(const fvm_grid* g) {
  if (!g->resident || !g->plan_ok || g->device < 0 || g->strips_asked || g->lanes_asked ||
      g->halo.s || g->halo.n)
    return false;
  int dev = -1, sdev = -1;
  if (hipGetDevice(&dev) != hipSuccess || hipStreamGetDevice(g->stream, &sdev) != hipSuccess ||
      dev != g->device || sdev != g->device)
    return false;
  return !capturing(g->stream);
}

// nsteps steps from state `win` kept on the chip: the last state goes to
// w_last, the one before it to w_prev (either may be null).
static cluster::Args cluster_args(const fvm_grid* g, int mode, int nsteps, const double* win,
                                  double* w_last, double* w_prev) {
  cluster::Args a{};
  a.win = win;
  a.w_last = w_last;
  a.w_prev = w_prev;
  a.spare = w_last ? g->other(w_last) : nullptr;
  a.ug = g->ug;
  a.scr = g->scr;
  a.area = g->area();
  a.g = g->g;
  a.m = g->m;
  std::memcpy(a.ghost, g->ghost, sizeof a.ghost);
  a.plan = g->plan;
  a.mode = mode;
  a.nsteps = nsteps;
  return a;
}

// The fewest steps for which a run of a state of more than a MB goes on the chip:
// start, loads and the last two states' stores cost it 10 to 25 us. us a call, steps / chip: one step of 1024^2
// Euler 28.5 / 47.6, 512^2 21.0 / 31.0, 200 x 150 21.2 / 20.5, of 860 x 900 spray
// 37.6 / 51.7, of 512^2 advection 21.3 / 26.8; two steps 51.5 / 59.9, 32.4 / 38.1,
// 22.0 / 25.2, 69.6 / 66.6, 24.1 / 31.8; three 79.6 / 73.4, 50.7 / 45.5, 34.3 / 30.1,
// 106 / 82.6, 39.7 / 36.9. Of steps that are not launched as a graph
// (checkpointed runs and their recomputation): 1024^2 with every state saved, two
// steps 65.2 / 76.4, three 89.4 / 92.5, four 113 / 110, 300^2 three 42.3 / 46.2, four
// 53.7 / 51.6; one step recomputed 141 / 178 in a backward pass of four, three
// 315 / 323 in one of eight, eight 401 / 394 in one of nine.
// Smaller states start as fast as a graph does (one step with its dt read back:
// 130 x 96 Euler 45 us on the chip, 46 to 57 as a graph).
constexpr int kMinChipRun = 3;
constexpr long long kSmallState = 1 << 17;  // doubles
constexpr int kMinChipSteps = 4;
static bool worth_the_chip(const fvm_grid* g, int nsteps) {
  return nsteps >= kMinChipRun ||
         (nsteps > 0 && static_cast<long long>(g->nv) * g->p.nx * g->p.ny <= kSmallState);
}

// One workgroup is the better place for an adaptive run of this grid, or the
// only one on the chip that is open to it (a captured stream, a strip shape). Past
// resident_cells a step takes it longer than several by some 2.6 ns a cell
// (Euler), but its start takes 6.5 us less: it is the faster one while steps times
// cells past the limit are below 2500 (us for three and four steps, one / several:
// Euler 34^2 19.1, 23.7 / 24.3, 28.5, 48^2 29.4, 36.9 / 24.9, 29.0, spray 38^2 20.6, 25.2 /
// 25.4, 29.7, advection 73^2 21.8, 26.0 / 24.9, 29.0).
constexpr long long kShortResident = 2500;
static bool one_workgroup(const fvm_grid* g, int nsteps) {
  if (!resident_ok(g)) return false;
  const long long past =
      static_cast<long long>(g->p.nx) * g->p.ny - resident_cells(fvm_nvar(g->p.model));
  return past <= 0 || nsteps < kMinChipRun || past * nsteps < kShortResident || !cluster_ok(g);
}

static int run_steps(fvm_grid* g, int kind, int nsteps, const double* dts, double* log,
                     double dt = 0.0) {
  int rc = FVM_OK;
  // adaptive steps and checked fixed steps read the current state's maxima
  if ((kind == 0 || kind == 3) && !g->speeds_valid) rc = enqueue_cfl(g, nullptr);
  if (rc == FVM_OK) rc = arm_log(g, log, nsteps);
  if (rc) return rc;
  double* const other = g->other(g->cur);
  double* const last = nsteps % 2 ? other : g->cur;
  bool one = kind == 0 && nsteps > 0 && one_workgroup(g, nsteps);
  if (!one && kind != 2 && worth_the_chip(g, nsteps) && cluster_ok(g)) {
    cluster::Args a = cluster_args(
        g, kind == 0 ? kDtAdaptive : (kind == 3 ? kDtFixedCheck : kDtArray), nsteps, g->cur, last,
        g->other(last));
    a.dts = dts;
    a.dt_arg = dt;
    const hipError_t e = launch_on_chip(a, g->p.model, g->device, g->cus, g->stream);
    if (e == hipSuccess) {
      g->cur = last;
      g->speeds_valid = true;
    }
    if (e != hipErrorNotReady) return dev_err(e);
    one = kind == 0 && resident_ok(g);
  }
  if (one) {
    const StepArgs a = g->step_args(g->cur, other, kDtAdaptive);
    rc = dev_err(launch_resident_run(a, kernel_model(g->p), last, g->other(last), nsteps,
                                     g->stream));
    if (rc) return rc;
    g->cur = last;
    g->speeds_valid = true;
    return FVM_OK;
  }
  int done = 0;
  if (capturing(g->stream)) {  // a graph launched into a capture is not recorded: its steps are
    for (; done < nsteps; ++done) {
      StepArgs a = g->step_args(g->cur, g->other(g->cur),
                                kind == 0 ? kDtAdaptive : (kind == 3 ? kDtFixedCheck : kDtArray));
      a.dts = dts;
      a.k = done;
      a.dt_arg = dt;
      rc = enqueue_step(g, a);
      if (rc) return rc;
      g->cur = a.wout;
    }
  }
  while (done < nsteps) {
    hipGraphExec_t exec;
    int n;
    if (kind == 0 || kind == 3) {
      n = chunk_size(nsteps - done);
      rc = chunk_graph(g, kind, n, dt, &exec);
    } else {
      n = std::min(kGraphChunk, nsteps - done);
      rc = graph_for(g, kind, n, g->cur, dts, kind == 1 ? done : 0, &exec, dt);
    }
    if (rc) return rc;
    rc = dev_err(hipGraphLaunch(exec, g->stream));
    if (rc) return rc;
    if (n % 2) g->cur = g->other(g->cur);
    if (g->me_lam) g->me_valid = true;
    done += n;
  }
  g->speeds_valid = true;
  return FVM_OK;
}

int fvm_run(fvm_grid* g, int nsteps, double* dts_dev) {
  if (!g || !g->bound || nsteps < 0) return FVM_EINVAL;
  return run_steps(g, 0, nsteps, nullptr, dts_dev);
}

int fvm_run_fixed(fvm_grid* g, int nsteps, double dt) {
  if (!g || !g->bound || nsteps < 0) return FVM_EINVAL;
  if (!(dt > 0.0) || !std::isfinite(dt)) return FVM_EINVAL;
  return run_steps(g, 3, nsteps, nullptr, nullptr, dt);
}

int fvm_run_dts(fvm_grid* g, int nsteps, const double* dts_dev) {
  if (!g || !g->bound || nsteps < 0 || (nsteps > 0 && !dts_dev)) return FVM_EINVAL;
  return run_steps(g, 1, nsteps, dts_dev, nullptr);
}

int fvm_run_ckpt(fvm_grid* g, int nsteps, int ckpt_every, double* const* ckpts,
                 double* dts_dev) {
  if (!g || !g->bound || nsteps < 0 || ckpt_every < 1 || !ckpts) return FVM_EINVAL;
  const int nck = (nsteps + ckpt_every - 1) / ckpt_every;
  for (int s = 0; s < nck; ++s)
    if (!ckpts[s] || ckpts[s] == g->w_a || ckpts[s] == g->w_b) return FVM_EINVAL;
  int rc = FVM_OK;
  if (!g->speeds_valid) rc = enqueue_cfl(g, nullptr);
  if (rc == FVM_OK) rc = arm_log(g, dts_dev, nsteps);
  if (rc) return rc;
  const size_t bytes = sizeof(double) * g->elems();
  if (nck > 0) {
    rc = dev_err(hipMemcpyAsync(ckpts[0], g->cur, bytes, hipMemcpyDeviceToDevice, g->stream));
    if (rc) return rc;
  }
  const double* in = g->cur;
  int k = 0;
  if (nsteps >= kMinChipSteps && cluster_ok(g)) {
    // a launch saves so many states at most; the next goes on from the last of
    // them (where a launch cannot have the chip, `last` and the other buffer hold
    // the unsaved states in turn, the current one first: `last` by the parity of
    // the first launch's steps)
    double* last = nullptr;
    while (nsteps - k >= kMinChipSteps) {
      const int s = k / ckpt_every;  // state k is checkpoint s
      const int saves = std::min(nck - 1 - s, static_cast<int>(cluster::kMaxSaves));
      const bool end = s + saves == nck - 1;
      const int steps = end ? nsteps - k : saves * ckpt_every;
      if (!last) last = steps % 2 ? g->other(g->cur) : g->cur;
      cluster::Args a = cluster_args(g, kDtAdaptive, steps, in, last, nullptr);
      a.every = ckpt_every;
      a.nsaves = saves;
      for (int q = 0; q < saves; ++q) a.saves[q] = ckpts[s + 1 + q];
      const hipError_t e = launch_on_chip(a, g->p.model, g->device, g->cus, g->stream);
      if (e == hipErrorNotReady) break;
      if (e != hipSuccess) return dev_err(e);
      k += steps;
      in = end ? last : ckpts[s + saves];
    }
  }
  for (; k < nsteps; ++k) {
    double* out;
    if ((k + 1) % ckpt_every == 0 && (k + 1) / ckpt_every < nck)
      out = ckpts[(k + 1) / ckpt_every];
    else
      out = (in == g->w_a) ? g->w_b : g->w_a;
    StepArgs a = g->step_args(in, out, kDtAdaptive);
    rc = enqueue_step(g, a);
    if (rc) return rc;
    in = out;
  }
  if (nsteps > 0 && in != g->w_a && in != g->w_b) {
    // the run ended on a checkpoint buffer: continue from a ping-pong buffer
    rc = dev_err(hipMemcpyAsync(g->w_a, in, bytes, hipMemcpyDeviceToDevice, g->stream));
    if (rc) return rc;
    in = g->w_a;
  }
  g->cur = const_cast<double*>(in);
  return FVM_OK;
}

int fvm_set_tiling(fvm_grid* g, int rows, int wpb) {
  if (!g) return FVM_EINVAL;
  const int r = rows ? rows : g->rows;
  const int w = wpb ? wpb : g->wpb;
  if (!valid_tiling(r, w)) return FVM_EINVAL;
  if (rows || wpb) {
    g->strips_asked = true;
    g->default_strips = false;
  }
  if (r != g->rows || w != g->wpb) g->clear_graphs();
  g->rows = r;
  g->wpb = w;
  return FVM_OK;
}

// ---- autotuning --------------------------------------------------------------------

}  // extern "C"

namespace {

std::string device_arch() {
  int dev = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess)
    return "unknown";
  std::string a = prop.gcnArchName;
  const size_t colon = a.find(':');
  return colon == std::string::npos ? a : a.substr(0, colon);
}

bool cache_lookup(const char* path, const std::string& key, int* rows, int* wpb, int* cpl) {
  if (!path) return false;
  std::ifstream in(path);
  std::string line;
  bool found = false;
  while (std::getline(in, line)) {
    const size_t bar = line.find(" | ");
    if (bar == std::string::npos || line.substr(0, bar) != key) continue;
    int r = 0, w = 0, c = 0;
    if (std::sscanf(line.c_str() + bar + 3, "rows=%d wpb=%d cpl=%d", &r, &w, &c) == 3) {
      *rows = r;
      *wpb = w;
      *cpl = c;
      found = true;  // the last entry for a key wins
    }
  }
  return found;
}

void cache_store(const char* path, const std::string& key, int rows, int wpb, int cpl,
                 double us) {
  if (!path) return;
  std::ofstream out(path, std::ios::app);
  out << key << " | rows=" << rows << " wpb=" << wpb << " cpl=" << cpl << " us=" << us << "\n";
}

}  // namespace

// Times `reps` launches of an n-step dry-run graph (dt = 0) in the current
// tiling; returns microseconds per step, or a negative value on error.
static double time_dry(fvm_grid* g, int n, int reps) {
  hipGraphExec_t exec;
  if (arm_log(g, nullptr, 0) != FVM_OK) return -1.0;
  if (graph_for(g, 2, n, g->cur, &g->scr->zero, 0, &exec) != FVM_OK) return -1.0;
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess) return -1.0;
  if (hipEventCreate(&e1) != hipSuccess) {
    (void)hipEventDestroy(e0);
    return -1.0;
  }
  double us = -1.0;
  bool ok = hipGraphLaunch(exec, g->stream) == hipSuccess;  // warm-up
  ok = ok && hipEventRecord(e0, g->stream) == hipSuccess;
  for (int r = 0; r < reps && ok; ++r) ok = hipGraphLaunch(exec, g->stream) == hipSuccess;
  ok = ok && hipEventRecord(e1, g->stream) == hipSuccess && hipEventSynchronize(e1) == hipSuccess;
  float ms = 0.0f;
  if (ok && hipEventElapsedTime(&ms, e0, e1) == hipSuccess) us = 1e3 * ms / (n * reps);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  return us;
}

// Times `reps` dry adjoint launches in the current adjoint tiling on
// (w, lam_in -> lam_out); with dt = 0 every cell writes the value it read,
// so the launches move the real traffic and change nothing (with
// lam_in == lam_out they rewrite it in place).
static double time_adjoint_dry(fvm_grid* g, int reps, const double* w, const double* lam_in,
                               double* lam_out) {
  AdjointArgs a{};
  a.w = w;
  a.lam_in = lam_in;
  a.lam_out = lam_out;
  a.dts = nullptr;
  a.dt_arg = 0.0;
  a.g = g->g;
  a.t = adjoint_tiling(g->g, g->adj_rows, g->adj_wpb,
                       adjoint_cpl(g, a.w, a.lam_in, a.lam_out));
  a.m = g->m;
  std::memcpy(a.ghost, g->ghost, sizeof a.ghost);
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess) return -1.0;
  if (hipEventCreate(&e1) != hipSuccess) {
    (void)hipEventDestroy(e0);
    return -1.0;
  }
  double us = -1.0;
  bool ok = launch_adjoint(a, g->p.model, g->ug, g->stream) == hipSuccess;  // warm-up
  ok = ok && hipEventRecord(e0, g->stream) == hipSuccess;
  for (int r = 0; r < reps && ok; ++r)
    ok = launch_adjoint(a, g->p.model, g->ug, g->stream) == hipSuccess;
  ok = ok && hipEventRecord(e1, g->stream) == hipSuccess && hipEventSynchronize(e1) == hipSuccess;
  float ms = 0.0f;
  if (ok && hipEventElapsedTime(&ms, e0, e1) == hipSuccess) us = 1e3 * ms / reps;
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  return us;
}

// Tuner candidates: a tile shape and lane layout, and its time per launch.
struct TuneCand {
  double us;
  int rows, wpb, cpl;
};

// Two-stage choice among timed candidates: every candidate is timed once
// over a short window, then the kRetime fastest are timed kRounds more times
// over a longer one and the lowest median wins. A short window that follows
// an idle gap can fall into the device's clock ramp, which alone reorders
// candidates a few percent apart. `time(c, reps)` applies candidate c and
// returns its microseconds per launch (< 0 on a device error).
template <class TimeFn>
static int pick_candidate(std::vector<TuneCand>& cands, TimeFn&& time, int reps_long,
                          TuneCand* best) {
  constexpr int kRetime = 6, kRounds = 3;
  if (cands.empty()) return FVM_EINVAL;
  std::stable_sort(cands.begin(), cands.end(),
                   [](const TuneCand& a, const TuneCand& b) { return a.us < b.us; });
  const int n = std::min<int>(kRetime, static_cast<int>(cands.size()));
  *best = cands[0];
  double best_med = 1e300;
  for (int k = 0; k < n; ++k) {
    double t[kRounds];
    for (int r = 0; r < kRounds; ++r) {
      t[r] = time(cands[k], reps_long);
      if (t[r] < 0) return FVM_EDEVICE;
    }
    std::sort(t, t + kRounds);
    if (t[kRounds / 2] < best_med) {
      best_med = t[kRounds / 2];
      *best = cands[k];
      best->us = best_med;
    }
  }
  return FVM_OK;
}

// The adjoint kernel's tile shape and lane layout (advection and Euler),
// timed on (state, lam_in -> lam_out); fvm_autotune passes the
// current state and the other ping-pong buffer, read and written in place.
static int tune_adjoint(fvm_grid* g, const char* cache_path, const std::string& key,
                        const double* state, const double* lam_in, double* lam_out) {
  if (g->p.model == FVM_SPRAY) return FVM_OK;
  int rows = 0, wpb = 0, cpl = 0;
  if (cache_lookup(cache_path, key, &rows, &wpb, &cpl) && valid_tiling(rows, wpb) &&
      (cpl == 1 || cpl == 2)) {
    g->adj_rows = rows;
    g->adj_wpb = wpb;
    g->adj_cpl = cpl;
    return FVM_OK;
  }
  const int wpbs[4] = {1, 2, 4, 8};
  const int rowss[9] = {4, 8, 16, 32, 48, 64, 96, 128, 256};
  auto time = [&](const TuneCand& c, int reps) {
    g->adj_rows = c.rows;
    g->adj_wpb = c.wpb;
    g->adj_cpl = c.cpl;
    return time_adjoint_dry(g, reps, state, lam_in, lam_out);
  };
  std::vector<TuneCand> cands;
  for (int c : {2, 1}) {
    for (int w : wpbs)
      for (int r : rowss) {
        if (r > g->p.ny && r != rowss[0]) continue;
        if (c == 2 && w == 8 && g->p.model == FVM_EULER) continue;  // spills at 2 waves/SIMD
        g->adj_cpl = c;
        // the timed buffers must allow the layout
        if (adjoint_cpl(g, state, lam_in, lam_out) != c) continue;
        TuneCand t{0.0, r, w, c};
        t.us = time(t, 4);
        if (t.us < 0) return FVM_EDEVICE;
        cands.push_back(t);
      }
  }
  TuneCand best{};
  const int rc = pick_candidate(cands, time, 24, &best);
  if (rc) return rc;
  g->adj_rows = best.rows;
  g->adj_wpb = best.wpb;
  g->adj_cpl = best.cpl;
  cache_store(cache_path, key, best.rows, best.wpb, best.cpl, best.us);
  return FVM_OK;
}

extern "C" {

int fvm_autotune_adjoint(fvm_grid* g, const double* w, const double* lam_in, double* lam_out,
                         const char* cache_path) {
  if (!g || !g->bound || !w || !lam_in || !lam_out || lam_in == lam_out) return FVM_EINVAL;
  if (g->p.model == FVM_SPRAY) return FVM_EUNSUPPORTED;
  char kbuf[256];
  std::snprintf(kbuf, sizeof kbuf,
                "%s grid model=%d bc=%d nx=%d ny=%d ld=%d layout=%d adjoint buffers",
                device_arch().c_str(), g->p.model, g->p.bc, g->p.nx, g->p.ny, g->p.ld,
                g->p.layout);
  return tune_adjoint(g, cache_path, kbuf, w, lam_in, lam_out);
}

int fvm_autotune(fvm_grid* g, const char* cache_path) {
  if (!g || !g->bound) return FVM_EINVAL;
  char kbuf[256];
  std::snprintf(kbuf, sizeof kbuf, "%s grid model=%d bc=%d nx=%d ny=%d ld=%d layout=%d%s",
                device_arch().c_str(), g->p.model, g->p.bc, g->p.nx, g->p.ny, g->p.ld,
                g->p.layout, g->p.closure == FVM_CLOSURE_MAXENT ? " maxent" : "");
  const std::string key = kbuf;
  int rows = 0, wpb = 0, cpl = 0;
  if (cache_lookup(cache_path, key, &rows, &wpb, &cpl) && valid_tiling(rows, wpb) &&
      (cpl == 1 || cpl == 2)) {
    g->rows = rows;
    g->wpb = wpb;
    g->cpl_req = cpl;
    g->default_strips = false;
    g->clear_graphs();
    choose_layout(g);
    return tune_adjoint(g, cache_path, key + " adjoint", g->cur, g->other(g->cur),
                        g->other(g->cur));
  }
  const int cpls[2] = {2, 1};
  const int wpbs[4] = {1, 2, 4, 8};
  const int rowss[10] = {4, 8, 16, 32, 48, 64, 96, 128, 192, 256};
  const int save_req = g->cpl_req;
  g->default_strips = false;
  auto apply = [&](const TuneCand& c) {
    g->cpl_req = c.cpl;
    choose_layout(g);
    g->rows = c.rows;
    g->wpb = c.wpb;
  };
  // reps: 8-step graphs
  auto time = [&](const TuneCand& c, int reps) {
    apply(c);
    const double us = time_dry(g, 8, reps);
    g->clear_graphs();  // one graph per candidate, not all of them at once
    return us;
  };
  std::vector<TuneCand> cands;
  for (int c : cpls) {
    g->cpl_req = c;
    choose_layout(g);
    if (g->cpl != c) continue;  // the buffers do not allow this layout
    for (int w : wpbs)
      for (int r : rowss) {
        if (r > g->p.ny && r != rowss[0]) continue;
        TuneCand t{0.0, r, w, c};
        t.us = time(t, 2);
        if (t.us < 0) {
          g->clear_graphs();
          return FVM_EDEVICE;
        }
        cands.push_back(t);
      }
  }
  TuneCand best{0.0, g->rows, g->wpb, g->cpl};
  const int prc = cands.empty() ? FVM_OK : pick_candidate(cands, time, 6, &best);
  g->clear_graphs();
  if (prc) return prc;
  const int br = best.rows, bw = best.wpb, bc = best.cpl;
  g->rows = br;
  g->wpb = bw;
  g->cpl_req = save_req ? save_req : bc;
  choose_layout(g);
  g->speeds_valid = true;  // the dry runs recomputed the maxima of the unchanged state
  cache_store(cache_path, key, br, bw, bc, best.us);
  return tune_adjoint(g, cache_path, key + " adjoint", g->cur, g->other(g->cur),
                      g->other(g->cur));
}

int fvm_set_cells_per_lane(fvm_grid* g, int cpl) {
  if (!g || cpl < 0 || cpl > 2) return FVM_EINVAL;
  g->lanes_asked = cpl != 0;
  g->cpl_req = cpl;
  choose_layout(g);
  return FVM_OK;
}

int fvm_get_cells_per_lane(const fvm_grid* g) { return g ? g->cpl : 0; }

int fvm_set_resident_runs(fvm_grid* g, int enable) {
  if (!g) return FVM_EINVAL;
  g->resident = enable != 0;
  return FVM_OK;
}

int fvm_set_adjoint_tiling(fvm_grid* g, int rows, int wpb, int cells_per_lane) {
  if (!g) return FVM_EINVAL;
  const int r = rows ? rows : g->adj_rows;
  const int w = wpb ? wpb : g->adj_wpb;
  const int c = cells_per_lane ? cells_per_lane : g->adj_cpl;
  if (!valid_tiling(r, w) || (c != 1 && c != 2)) return FVM_EINVAL;
  g->adj_rows = r;
  g->adj_wpb = w;
  g->adj_cpl = c;
  return FVM_OK;
}

int fvm_get_tiling(const fvm_grid* g, int* rows, int* wpb) {
  if (!g || !rows || !wpb) return FVM_EINVAL;
  *rows = g->rows;
  *wpb = g->wpb;
  return FVM_OK;
}

// The entropy closure's adjoint step runs in the grid's free ping-pong
// buffer (W* and then mu); none of the step's buffers may be that buffer,
// and with two cells per lane the transport step needs 16-byte alignment.
static bool maxent_adjoint_buffers_ok(const fvm_grid* g, const double* w, const double* lin,
                                      const double* lout) {
  if (kernel_model(g->p) != kSprayMaxEnt) return true;
  const double* ws = g->other(g->cur);
  auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  if (w == ws || lin == ws || lout == ws) return false;
  return g->cpl != 2 || al(w);
}

// One adjoint step (w, lin -> lout) with dt = dts[k], or dt_arg if dts is
// null. The entropy closure's step is three launches: the transport step
// W -> W* into the free ping-pong buffer ws, the source's adjoint
// mu = lam + dt J_S(W*)^T lam in place there, then the transport's adjoint
// (w, mu -> lout).
static int enqueue_adjoint(fvm_grid* g, const double* w, const double* lin, double* lout,
                           const double* dts, int k, double dt_arg) {
  AdjointArgs a{};
  a.w = w;
  a.lam_in = lin;
  a.lam_out = lout;
  a.dts = dts;
  a.k = k;
  a.dt_arg = dt_arg;
  a.g = g->g;
  a.t = adjoint_tiling(g->g, g->adj_rows, g->adj_wpb, adjoint_cpl(g, a.w, a.lam_in, a.lam_out));
  a.m = g->m;
  std::memcpy(a.ghost, g->ghost, sizeof a.ghost);
  if (kernel_model(g->p) != kSprayMaxEnt)
    return dev_err(launch_adjoint(a, g->p.model, g->ug, g->stream));
  double* ws = g->other(g->cur);
  StepArgs s = g->step_args(w, ws, dts ? kDtArray : kDtValue);
  s.dts = dts;
  s.k = k;
  s.dt_arg = dt_arg;
  int rc = dev_err(launch_step(s, kSprayMaxEnt, g->stream));
  if (rc) return rc;
  AdjointArgs b = a;
  b.w = ws;
  b.lam_out = ws;
  rc = dev_err(launch_maxent_adjoint_source(b, g->ug, g->stream));
  if (rc) return rc;
  AdjointArgs c = a;
  c.lam_in = ws;
  return dev_err(launch_spray_adjoint(c, g->ug, g->stream, false));
}

int fvm_adjoint_step(fvm_grid* g, const double* w, double dt, const double* lam_in,
                     double* lam_out) {
  if (!g || !g->bound || !w || !lam_in || !lam_out || lam_in == lam_out || w == lam_out)
    return FVM_EINVAL;
  if (!adjoint_supported(g)) return FVM_EUNSUPPORTED;
  if (!(dt >= 0.0) || !std::isfinite(dt)) return FVM_EINVAL;
  if (!maxent_adjoint_buffers_ok(g, w, lam_in, lam_out)) return FVM_EINVAL;
  return enqueue_adjoint(g, w, lam_in, lam_out, nullptr, 0, dt);
}

int fvm_adjoint_run(fvm_grid* g, double* const* ckpts, int ckpt_every, const double* dts_dev,
                    int nsteps, double* lam, double* lam_tmp, double* seg_buf) {
  if (!g || !g->bound || !ckpts || ckpt_every < 1 || !dts_dev || nsteps < 0 || !lam ||
      !lam_tmp || lam == lam_tmp)
    return FVM_EINVAL;
  if (ckpt_every > 1 && !seg_buf) return FVM_EINVAL;
  if (!adjoint_supported(g)) return FVM_EUNSUPPORTED;
  const int nck = (nsteps + ckpt_every - 1) / ckpt_every;
  for (int s = 0; s < nck; ++s)
    if (!ckpts[s]) return FVM_EINVAL;
  const size_t state = g->elems();
  if (kernel_model(g->p) == kSprayMaxEnt) {
    // the entropy closure's steps work in the free ping-pong buffer
    const double* ws = g->other(g->cur);
    if (!maxent_adjoint_buffers_ok(g, lam, lam, lam_tmp)) return FVM_EINVAL;
    for (int s = 0; s < nck; ++s)
      if (!maxent_adjoint_buffers_ok(g, ckpts[s], lam, lam_tmp)) return FVM_EINVAL;
    if (seg_buf && ckpt_every > 1) {
      if (!maxent_adjoint_buffers_ok(g, seg_buf, lam, lam_tmp)) return FVM_EINVAL;
      if (ws >= seg_buf && ws < seg_buf + static_cast<size_t>(ckpt_every - 1) * state)
        return FVM_EINVAL;
    }
  }
  if (const int rc = arm_log(g, nullptr, 0)) return rc;  // the recomputed steps log nothing
  double* lin = lam;
  double* lout = lam_tmp;
  for (int s = nck - 1; s >= 0; --s) {
    const int k0 = s * ckpt_every;
    const int k1 = std::min(nsteps, k0 + ckpt_every);
    // recompute W^{k0+1} .. W^{k1-1} into seg_buf[0 .. k1-k0-2]
    const double* in = ckpts[s];
    int k = k0;
    if (k1 - k0 - 1 >= kMinChipSteps && k1 - k0 - 1 <= cluster::kMaxSaves && cluster_ok(g)) {
      cluster::Args a = cluster_args(g, kDtArray, k1 - k0 - 1, in, nullptr, nullptr);
      a.dts = dts_dev;
      a.k0 = k0;
      a.every = 1;
      a.nsaves = a.nsteps;
      for (int q = 0; q < a.nsaves; ++q) a.saves[q] = seg_buf + static_cast<size_t>(q) * state;
      const hipError_t e = launch_on_chip(a, g->p.model, g->device, g->cus, g->stream);
      if (e != hipSuccess && e != hipErrorNotReady) return dev_err(e);
      if (e == hipSuccess) k = k1;
    }
    for (; k + 1 < k1; ++k) {
      double* out = seg_buf + static_cast<size_t>(k - k0) * state;
      StepArgs a = g->step_args(in, out, kDtArray);
      a.dts = dts_dev;
      a.k = k;
      int rc = enqueue_step(g, a);
      if (rc) return rc;
      in = out;
    }
    for (int k = k1 - 1; k >= k0; --k) {
      const double* wk = (k == k0) ? ckpts[s] : seg_buf + static_cast<size_t>(k - k0 - 1) * state;
      int rc = enqueue_adjoint(g, wk, lin, lout, dts_dev, k, 0.0);
      if (rc) return rc;
      std::swap(lin, lout);
    }
  }
  // the recompute left the scratch maxima (and the entropy closure's kept
  // multipliers) describing a recomputed state
  g->speeds_valid = false;
  g->me_valid = false;
  if (lin != lam) {
    return dev_err(hipMemcpyAsync(lam, lin, sizeof(double) * state, hipMemcpyDeviceToDevice,
                                  g->stream));
  }
  return FVM_OK;
}

}  // extern "C"

// ---- adaptive run without any allocation -------------------------------------
// fvm_run_noalloc keeps the grid's scratch block (speed maxima, arrival
// counter, next dt, status word, dt-log cursor) in this file-scope device
// array instead of a caller buffer. Host code never passes the array's name
// to a kernel (on the host it is only a stand-in for the symbol): the first
// call on a device looks up the array's device address with
// hipGetSymbolAddress, with that device current, and every launch takes that
// address. Each device holds its own copy until the process ends; calls
// that overlap on one device share it and race.
namespace {

constexpr size_t kNoAllocScratchBytes = sizeof(GridScratch);  // one grid's block
constexpr int kNoAllocMaxDevices = 64;

__device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

std::mutex g_noalloc_mu;
void* g_noalloc_ptr[kNoAllocMaxDevices] = {};

// Device address of `scratch` on device `dev` (current), or null on error.
void* noalloc_scratch(int dev) {
  if (dev < 0 || dev >= kNoAllocMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_noalloc_mu);
  if (!g_noalloc_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
    if (reinterpret_cast<uintptr_t>(ptr) & 255) return nullptr;
    g_noalloc_ptr[dev] = ptr;
  }
  return g_noalloc_ptr[dev];
}

// Writes the status code of the sticky bits (FVM_OK, FVM_ENONFINITE,
// FVM_EINVAL) to *out.
__global__ void noalloc_status_kernel(const GridScratch* s, int* out) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    const unsigned int st = s->status;
    *out = (st & kStatusNonFinite) ? FVM_ENONFINITE
                                   : ((st & kStatusCfl) ? FVM_ECFL
                                                        : ((st & kStatusDt) ? FVM_EINVAL : FVM_OK));
  }
}

}  // namespace

extern "C" {

int fvm_run_noalloc(const fvm_params* p, double* w_a, double* w_b, const double* ug,
                    int nsteps, double* dts_dev, int* status_dev, void* stream) {
  if (!valid_params(p) || !w_a || !w_b || w_a == w_b || nsteps < 0) return FVM_EINVAL;
  if ((reinterpret_cast<uintptr_t>(w_a) & 7) || (reinterpret_cast<uintptr_t>(w_b) & 7))
    return FVM_EINVAL;
  if ((p->model == FVM_SPRAY) != (ug != nullptr)) return FVM_EINVAL;
  if (p->bc == FVM_DIRICHLET || p->closure != FVM_CLOSURE_LOGNORMAL) return FVM_EUNSUPPORTED;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return FVM_EDEVICE;
  GridScratch* scr = static_cast<GridScratch*>(noalloc_scratch(dev));
  if (!scr) return FVM_EDEVICE;
  hipStream_t st = static_cast<hipStream_t>(stream);

  const GridGeom geom = grid_geometry(*p);
  const ModelConsts mc = model_consts(*p);
  auto al16 = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
  const int cpl = default_layout(
      *p, p->ld % 2 == 0 && al16(w_a) && al16(w_b) && (!ug || al16(ug)));
  int rows = kDefaultRows, wpb = kDefaultWpb;
  default_tiling(*p, cpl, &rows, &wpb);

  // clear the block (a kernel, not a memset), maxima and dt of w_a, arm the log
  int rc = dev_err(launch_clear_scratch(scr, 1, st));
  if (rc) return rc;
  CflArgs c{};
  c.w = w_a;
  c.scr = scr;
  c.g = geom;
  c.m = mc;
  rc = dev_err(launch_cfl(c, p->model, st));
  if (rc == FVM_OK) rc = dev_err(launch_set_log(scr, 1, dts_dev, nsteps, 1, st));
  if (rc) return rc;
  StepArgs a{};
  a.ug = ug;
  a.scr = scr;
  a.mode = kDtAdaptive;
  a.g = geom;
  a.t = tiling(geom, rows, wpb, cpl);
  a.m = mc;
  const double* in = w_a;
  for (int k = 0; k < nsteps; ++k) {
    double* out = in == w_a ? w_b : w_a;
    a.win = in;
    a.wout = out;
    rc = dev_err(launch_step(a, p->model, st));
    if (rc) return rc;
    in = out;
  }
  if (status_dev) {
    hipLaunchKernelGGL(noalloc_status_kernel, dim3(1), dim3(64), 0, st, scr, status_dev);
    rc = dev_err(hipGetLastError());
  }
  return rc;
}

}  // extern "C"
