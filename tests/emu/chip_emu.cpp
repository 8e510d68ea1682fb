// chip_emu.cpp -- runs the kernels of a run on the chip (fvm_cluster.hip) on the
// CPU: a host thread per workgroup, its threads as fibers that change over at
// barriers, lane exchanges and looks at a word of another workgroup. Buffers
// have exactly the size of the ABI contract, so AddressSanitizer reports any
// access outside them, and the bounds check of the LDS array any outside that.
//
// Usage: chip_emu model bc nx ny pad layout nsteps every cfl room in out
//   model, bc, in, out as in resident_emu.cpp; pad: ld - nx; every > 0: states
//   every, 2 every, .. are saved; room 0: all workgroups of the first kernel are
//   resident at once, else the start is refused and so many of the second at most.
// `out`: W^n, the other ping-pong buffer's state, the saved states (each nVar *
// ny * nx, planar), the n dts, then the status word and the number of control and
// exchange words that the run has not left empty.
#define atomicExch emu_plain_exch
#define atomicOr emu_plain_or
#define atomicMax emu_plain_max
#define atomicAdd emu_plain_add
#define __syncthreads emu_no_barrier
#define __threadfence emu_no_fence
#include <hip/hip_runtime.h>
#undef atomicExch
#undef atomicOr
#undef atomicMax
#undef atomicAdd
#undef __syncthreads
#undef __threadfence
#undef __shared__
#define __shared__ static thread_local

#include <sys/mman.h>
#include <ucontext.h>

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <mutex>
#include <thread>
#include <vector>

typedef unsigned long long u64;
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
thread_local emu_dim3 emu_threadIdx;
static thread_local dim3 blockIdx, blockDim, gridDim;

// ---- one workgroup: fibers on a host thread ---------------------------------
struct Meeting {  // of the threads of a wave, or of a workgroup
  int gen = 0, here = 0, size = 0;
  u64 slot[2][64];
};
struct Fiber {
  ucontext_t at;
  void* stack = nullptr;
  const Meeting* waits = nullptr;  // for the next generation of this meeting
  int gen = 0;
  bool done = false;
};
constexpr size_t kStack = 256 << 10;
struct Group {
  std::vector<Fiber> fibers;
  std::vector<Meeting> waves;
  Meeting all;
  ucontext_t home;
  int now = 0;
  void (*kernel)(void**) = nullptr;
  void** args = nullptr;
};
static thread_local Group* t_group = nullptr;

static void yield() {
  Group* const g = t_group;
  swapcontext(&g->fibers[g->now].at, &g->home);
}
static int meet(Meeting& m) {  // the generation that this call belongs to
  Group* const g = t_group;
  const int gen = m.gen;
  if (++m.here == m.size) {
    m.here = 0;
    ++m.gen;
  } else {
    g->fibers[g->now].waits = &m;
    g->fibers[g->now].gen = gen;
    yield();
  }
  return gen;
}
static u64 exchange(u64 x, int src) {
  Group* const g = t_group;
  Meeting& m = g->waves[g->now / 64];
  const int parity = m.gen & 1;
  m.slot[parity][g->now % 64] = x;
  meet(m);
  return src < 0 || src > 63 ? 0 : m.slot[parity][src];
}
int emu_dpp(int x, int ctrl) {
  const int lane = t_group->now % 64;
  return static_cast<int>(exchange(static_cast<unsigned>(x), ctrl == 0x130 ? lane + 1 : lane - 1));
}
u64 emu_shfl_xor(u64 x, int o) { return exchange(x, (t_group->now % 64) ^ o); }
static void __syncthreads() { meet(t_group->all); }
static void __threadfence() { std::atomic_thread_fence(std::memory_order_seq_cst); }

static void fiber_main() {
  Group* const g = t_group;
  g->kernel(g->args);
  g->fibers[g->now].done = true;
  swapcontext(&g->fibers[g->now].at, &g->home);
}

static void run_group(unsigned block, dim3 grid, dim3 threads, void (*kernel)(void**), void** args) {
  blockIdx = dim3(block);
  blockDim = threads;
  gridDim = grid;
  Group g;
  t_group = &g;
  const int n = static_cast<int>(threads.x);
  g.kernel = kernel;
  g.args = args;
  g.fibers.resize(n);
  g.waves.resize(n / 64);
  for (auto& w : g.waves) w.size = 64;
  g.all.size = n;
  for (auto& f : g.fibers) {
    f.stack = mmap(nullptr, kStack, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (f.stack == MAP_FAILED) std::abort();
    getcontext(&f.at);
    f.at.uc_stack.ss_sp = f.stack;
    f.at.uc_stack.ss_size = kStack;
    f.at.uc_link = nullptr;
    makecontext(&f.at, fiber_main, 0);
  }
  for (int left = n; left > 0;) {
    bool moved = false;
    for (int k = 0; k < n; ++k) {
      Fiber& f = g.fibers[k];
      if (f.done || (f.waits && f.waits->gen == f.gen)) continue;
      f.waits = nullptr;
      g.now = k;
      emu_threadIdx = {static_cast<unsigned>(k), 0, 0};
      moved = true;
      swapcontext(&g.home, &f.at);
      if (f.done) --left;
    }
    if (!moved && left > 0) {
      std::fprintf(stderr, "workgroup %u: its threads wait for each other\n", block);
      std::abort();
    }
    std::this_thread::yield();
  }
  for (auto& f : g.fibers) munmap(f.stack, kStack);
}

// ---- words that workgroups share --------------------------------------------
template <class T>
T emu_load(const T* p) {
  yield();  // a wait lets the others on
  return __atomic_load_n(p, __ATOMIC_SEQ_CST);
}
template <class T, class U>
T emu_cas(T* p, U* expected, T v) {
  return __atomic_compare_exchange_n(p, expected, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST);
}
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) emu_load(p)
#define __hip_atomic_store(p, v, order, scope) \
  __atomic_store_n((p), static_cast<u64>(v), __ATOMIC_SEQ_CST)
#define __hip_atomic_fetch_add(p, v, order, scope) __atomic_fetch_add((p), (v), __ATOMIC_SEQ_CST)
#define __hip_atomic_compare_exchange_strong(p, e, v, o1, o2, scope) emu_cas((p), (e), (v))
template <class T, class U>
T atomicExch(T* p, U v) {
  return __atomic_exchange_n(p, static_cast<T>(v), __ATOMIC_SEQ_CST);
}
template <class T, class U>
T atomicOr(T* p, U v) {
  return __atomic_fetch_or(p, static_cast<T>(v), __ATOMIC_SEQ_CST);
}
template <class T, class U>
T atomicAdd(T* p, U v) {
  return __atomic_fetch_add(p, static_cast<T>(v), __ATOMIC_SEQ_CST);
}
template <class T, class U>
T atomicMax(T* p, U v) {
  T o = __atomic_load_n(p, __ATOMIC_SEQ_CST);
  while (o < static_cast<T>(v) &&
         !__atomic_compare_exchange_n(p, &o, static_cast<T>(v), false, __ATOMIC_SEQ_CST,
                                      __ATOMIC_SEQ_CST)) {
  }
  return o;
}
static long long wall_clock64() { return 0; }  // no wait runs out of time

// ---- launches ---------------------------------------------------------------
enum { hipSuccess = 0, hipErrorInvalidValue = 1 };
static hipError_t hipGetLastError() { return hipSuccess; }
static hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t,
                                  hipStream_t);
#define hipLaunchKernelGGL(kernel, grid, block, lds, st, ...) ((void)&kernel)

#include "../../paper_1701_05431_amd/csrc/fvm_cluster.hip"

using namespace fvm;

static int g_room = 0;
static bool g_second = false;

template <void (*K)(cluster::Args)>
static void call1(void** a) {
  K(*static_cast<cluster::Args*>(a[0]));
}
template <void (*K)(cluster::Args, cluster::Pieces)>
static void call2(void** a) {
  K(*static_cast<cluster::Args*>(a[0]), *static_cast<cluster::Pieces*>(a[1]));
}
template <class M, int BC>
static void (*entry(const void* f))(void**) {
  using namespace cluster;
  if (f == reinterpret_cast<const void*>(&cluster_run_kernel<M, BC>))
    return &call1<&cluster_run_kernel<M, BC>>;
  if (f == reinterpret_cast<const void*>(&general_run_kernel<M, BC>))
    return &call2<&general_run_kernel<M, BC>>;
  return nullptr;
}
template <class M>
static void (*entry_bc(const void* f))(void**) {
  if (auto e = entry<M, 0>(f)) return e;
  if (auto e = entry<M, 1>(f)) return e;
  return entry<M, 2>(f);
}

static hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t,
                                  hipStream_t) {
  void (*e)(void**) = entry_bc<Adv>(f);
  if (!e) e = entry_bc<Euler>(f);
  if (!e) e = entry_bc<Spray>(f);
  if (!e) std::abort();
  // all workgroups at once, or as many as there is room for, in order
  const unsigned at_once = g_second && g_room ? std::min<unsigned>(g_room, grid.x) : grid.x;
  std::atomic<unsigned> next{0};
  std::vector<std::thread> room;
  for (unsigned k = 0; k < at_once; ++k)
    room.emplace_back([&] {
      for (unsigned b; (b = next.fetch_add(1)) < grid.x;) run_group(b, grid, block, e, args);
    });
  for (auto& t : room) t.join();
  g_second = !g_second;
  return hipSuccess;
}

int main(int argc, char** argv) {
  if (argc != 13) {
    std::fprintf(stderr, "usage: model bc nx ny pad layout nsteps every cfl room in out\n");
    return 2;
  }
  const int model = std::atoi(argv[1]), bc = std::atoi(argv[2]), nx = std::atoi(argv[3]),
            ny = std::atoi(argv[4]), pad = std::atoi(argv[5]), layout = std::atoi(argv[6]),
            nsteps = std::atoi(argv[7]), every = std::atoi(argv[8]);
  const double cfl = std::atof(argv[9]);
  g_room = std::atoi(argv[10]);
  const int nv = model == 0 ? 1 : (model == 1 ? 4 : 6), ld = nx + pad;
  const size_t ncell = static_cast<size_t>(nx) * ny;
  std::vector<double> raw(nv * ncell + (model == 2 ? 2 * ncell : 0) + 4 * nv);
  std::FILE* f = std::fopen(argv[11], "rb");
  if (!f || std::fread(raw.data(), sizeof(double), raw.size(), f) != raw.size()) return 3;
  std::fclose(f);

  cluster::Args a{};
  a.g.nx = nx;
  a.g.ny = ny;
  a.g.bc = bc;
  a.g.dx = 1.0 / nx;
  a.g.dy = 1.0 / ny;
  a.g.hmin = std::min(a.g.dx, a.g.dy);
  a.g.cfl = cfl;
  a.g.rld = ld;
  a.g.ld = layout ? nv * ld : ld;
  a.g.plane = layout ? ld : static_cast<size_t>(ld) * ny;
  a.g.uld = layout ? 2 * ld : ld;
  a.g.uplane = layout ? ld : static_cast<size_t>(ld) * ny;
  a.m.ax = 1.0;
  a.m.ay = 0.5;
  a.m.gamma = 1.4;
  a.m.gm1 = 0.4;
  a.m.K = 1.0;
  a.m.inv_theta = 10.0;
  a.m.s_eps = 0.01;
  a.m.log_s_eps = std::log(0.01);
  if (!cluster::make_plan(nv, nx, ny, &a.plan)) return 4;

  // exactly sized buffers
  const size_t state = static_cast<size_t>(nv) * ny * ld;
  auto buffer = [&](size_t n) {
    std::unique_ptr<double[]> p(new double[n]);
    std::fill(p.get(), p.get() + n, NAN);
    return p;
  };
  auto at = [&](int v, int j, int i) { return v * a.g.plane + static_cast<size_t>(j) * a.g.ld + i; };
  auto wa = buffer(state), wb = buffer(state), ug = buffer(static_cast<size_t>(2) * ny * ld);
  for (int v = 0; v < nv; ++v)
    for (int j = 0; j < ny; ++j)
      for (int i = 0; i < nx; ++i) wa[at(v, j, i)] = raw[(static_cast<size_t>(v) * ny + j) * nx + i];
  if (model == 2) {
    for (int v = 0; v < 2; ++v)
      for (int j = 0; j < ny; ++j)
        for (int i = 0; i < nx; ++i)
          ug[v * a.g.uplane + static_cast<size_t>(j) * a.g.uld + i] =
              raw[nv * ncell + (static_cast<size_t>(v) * ny + j) * nx + i];
    a.ug = ug.get();
  }
  const double* gh = raw.data() + raw.size() - 4 * nv;
  for (int s = 0; s < 4; ++s)
    for (int v = 0; v < nv; ++v) a.ghost[s * kMaxVar + v] = gh[s * nv + v];

  // scratch and exchange area, as cleared at bind
  const size_t words = cluster::area_words(nv, a.plan);
  std::unique_ptr<u64[]> area(new u64[words]);
  for (size_t k = 0; k < words; ++k) area[k] = k < cluster::kControlWords ? 0 : cluster::kEmpty;
  a.area = area.get();
  GridScratch scr{};
  a.scr = &scr;
  std::vector<double> dts(nsteps, NAN);
  scr.log = dts.data();
  scr.log_cap = nsteps;
  scr.log_stride = 1;
  u64 bx = 0, by = 0;
  auto first = [&](auto m) {
    for (size_t c = 0; c < ncell; ++c) {
      double w[6], sx, sy;
      for (int v = 0; v < nv; ++v) w[v] = raw[v * ncell + c];
      m.speeds(w, sx, sy);
      bx = umax64(bx, bits(sx));
      by = umax64(by, bits(sy));
    }
  };
  if (model == 0) first(Adv(a.m));
  else if (model == 1) first(Euler(a.m));
  else first(Spray(a.m));
  scr.cur_sx = __longlong_as_double(static_cast<long long>(bx));
  scr.cur_sy = __longlong_as_double(static_cast<long long>(by));
  scr.dt = next_dt(a.g, scr.cur_sx, scr.cur_sy);

  double* const last = nsteps % 2 ? wb.get() : wa.get();
  double* const other = nsteps % 2 ? wa.get() : wb.get();
  a.win = wa.get();
  a.w_last = last;
  a.spare = other;
  a.mode = kDtAdaptive;
  a.nsteps = nsteps;
  std::vector<std::unique_ptr<double[]>> saves;
  if (every > 0) {
    a.every = every;
    a.nsaves = (nsteps - 1) / every;
    for (int q = 0; q < a.nsaves; ++q) {
      saves.push_back(buffer(state));
      a.saves[q] = saves.back().get();
    }
  } else {
    a.w_prev = other;
  }
  if (g_room) reinterpret_cast<cluster::Control*>(a.area)->decision = 2;
  if (cluster::launch_run(a, model, nullptr) != hipSuccess) return 5;

  std::vector<double> out;
  auto put = [&](const double* w) {
    for (int v = 0; v < nv; ++v)
      for (int j = 0; j < ny; ++j)
        for (int i = 0; i < nx; ++i) out.push_back(w[at(v, j, i)]);
  };
  put(last);
  put(other);
  for (auto& s : saves) put(s.get());
  out.insert(out.end(), dts.begin(), dts.end());
  out.push_back(scr.status);
  // (the last maxima and dt of a run by tickets stay)
  int full = 0;
  for (size_t k = 0; k < words; ++k)
    full += area[k] != (k < cluster::kControlWords ? 0 : cluster::kEmpty) &&
            !(k >= offsetof(cluster::Control, sx) / 8 && k < cluster::kControlWords);
  out.push_back(full);
  f = std::fopen(argv[12], "wb");
  if (!f || std::fwrite(out.data(), sizeof(double), out.size(), f) != out.size()) return 3;
  std::fclose(f);
  return 0;
}
