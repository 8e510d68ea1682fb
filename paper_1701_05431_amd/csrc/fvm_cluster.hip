// fvm_cluster.hip -- the resident run of a grid that fits on the chip
// (rationale and exchange protocol in fvm_cluster.hpp).
//
// The workgroups wait for each other, so all of them must be resident. They
// find out first: each counts itself in, and the last one decides "go"; a
// workgroup that has waited for kStartLimit decides "no go", which of the two
// comes first stands, and on "no go" everybody leaves without having touched
// anything. The general kernel launched behind it then makes the run through
// device memory, with as many workgroups as there is room for. After "go" every workgroup is resident and
// stays until the run is over, so every later wait is for something that is on
// its way; those waits are bounded all the same (kWaitLimit), and running out
// is reported as a device error. Such a run leaves its words and counts behind
// (`abort` says so): no run starts on them, each reports the error again, until
// the host has emptied them (fvm_get_status with clear, fvm_bind).
#include <hip/hip_runtime.h>

#include <cfloat>

#include "fvm_cluster.hpp"
#include "fvm_internal.hpp"
#include "fvm_models.hpp"
#include "fvm_resident.hpp"
#include "fvm_step.hpp"

namespace fvm {
namespace cluster {

namespace {

// 20 ms of the 100 MHz clock. The workgroups of a run start within some 10 us of
// each other, or when the kernel that fills the chip has ended, and waiting for
// that is better than sharing the chip with it: 50 steps of 1024^2 beside products
// of 15 ms each on another stream take 19 ms, by tickets after 2 ms of waiting 87
// (as step launches 31).
constexpr long long kStartLimit = 2000000;
constexpr long long kWaitLimit = 400000000;   // 4 s

// Words other workgroups write or read while the kernel runs: device-scope
// accesses, performed where all XCDs see them.
__device__ __forceinline__ u64 peek(const u64* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put(u64* p, u64 v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// This wave's stores so far have been performed.
__device__ __forceinline__ void stores_done() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
}

// The values of N exchange words, waited for together (all loads are in flight
// at once); false when time is up.
template <int N>
__device__ __forceinline__ bool await(const u64* const* p, Control* ctl, u64* v) {
  long long t0 = 0;
  for (int round = 0;; ++round) {
#pragma unroll
    for (int q = 0; q < N; ++q) v[q] = peek(p[q]);
    bool all = true;
#pragma unroll
    for (int q = 0; q < N; ++q) all = all && v[q] != kEmpty;
    if (all) return true;
    if ((round & 63) == 63) {
      const long long t = wall_clock64();
      t0 = t0 ? t0 : t;
      if (t - t0 > kWaitLimit || peek(&ctl->abort) != 0) {
        put(&ctl->abort, 1);
        return false;
      }
    }
  }
}

// All workgroups are resident (true), or nobody runs (false): thread 0 only.
// (`abort` cannot come from this run yet: a wait follows the last arrival.)
__device__ inline bool all_started(Control* ctl, u64 tiles, GridScratch* s) {
  if (peek(&ctl->abort) != 0) {
    atomicOr(&s->status, kStatusWait);
    return false;
  }
  const u64 n = __hip_atomic_fetch_add(&ctl->arrived, 1ull, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
  u64 open = 0;
  if (n == tiles - 1)
    __hip_atomic_compare_exchange_strong(&ctl->decision, &open, 1ull, __ATOMIC_RELAXED,
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const long long t0 = wall_clock64();
  u64 d;
  while ((d = peek(&ctl->decision)) == 0) {
    if (wall_clock64() - t0 > kStartLimit) {
      open = 0;
      __hip_atomic_compare_exchange_strong(&ctl->decision, &open, 2ull, __ATOMIC_RELAXED,
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  return d == 1;
}

// The first `steps` steps of a run by tickets are done (true), or time is up:
// thread 0 only.
__device__ inline bool steps_done(Control* ctl, u64 steps) {
  const long long t0 = wall_clock64();
  while (peek(&ctl->steps) < steps) {
    if (wall_clock64() - t0 > kWaitLimit || peek(&ctl->abort) != 0) {
      put(&ctl->abort, 1);
      return false;
    }
  }
  return true;
}
__device__ __forceinline__ double value(u64 word) {
  return __longlong_as_double(static_cast<long long>(word));
}

template <class M, int BC>
__global__ __launch_bounds__(waves(M::NV) * kWave) void cluster_run_kernel(Args a) {
  constexpr int NV = M::NV, kWaves = waves(NV), kThreads = kWaves * kWave;
  using Prim = typename M::Prim;
  constexpr int kRowDoubles = NV * kWave;
  constexpr int Q = (tile_words(NV, max_rows(NV)) + kThreads - 1) / kThreads;
  // row -1, the tile's rows, the row above them: [row + 1][variable][lane]
  __shared__ double S[(max_rows(NV) + 2) * kRowDoubles];
  __shared__ u64 s_red[2][kWaves];
  __shared__ u64 s_max[kWaves];
  __shared__ int s_ok;

  const M m(a.m);
  const GridGeom& g = a.g;
  const Plan& P = a.plan;
  Control* const ctl = reinterpret_cast<Control*>(a.area);
  const int tid = static_cast<int>(threadIdx.x);
  const int lane = tid & (kWave - 1), wave = wave_index();
  const int tile = static_cast<int>(blockIdx.x);
  if (tid == 0) s_ok = all_started(ctl, static_cast<u64>(P.tiles), a.scr) ? 1 : 0;
  __syncthreads();
  if (!s_ok) return;

  const int tx = tile % P.tiles_x, ty = tile / P.tiles_x;
  const int x0 = tx * P.cols, ncols = min(P.cols, g.nx - x0);
  const int y0 = ty * P.rows, nrows = min(P.rows, g.ny - y0);
  const int rw = (nrows + kWaves - 1) / kWaves;  // rows per wave
  const int last_wave = (nrows - 1) / rw;
  const int jr = wave * rw;                      // this wave's rows in the tile
  const int nr = max(0, min(rw, nrows - jr));
  const bool inside = lane >= 1 && lane <= ncols;
  const int col = x0 + min(max(lane - 1, 0), ncols - 1);
  const bool west = BC != kPeriodic && tx == 0, east = BC != kPeriodic && tx == P.tiles_x - 1;
  const bool south = BC != kPeriodic && ty == 0, north = BC != kPeriodic && ty == P.tiles_y - 1;
  auto at = [](int row, int v, int l) { return ((row + 1) * NV + v) * kWave + l; };

  // this thread's exchange words: index in a tile's words, the word with the
  // same place on the neighbour's facing side, the own value's place in S and
  // the neighbour's value's place in S
  const int row_words = NV * kWave, col_words = NV * P.rows;
  const int words = 2 * (row_words + col_words);
  u64* const area = a.area + kControlWords;
  const size_t set_words = static_cast<size_t>(P.tiles) * words;
  u64* const maxima = area + 3 * set_words;      // [set][x, y][tile]
  int word[Q];
  unsigned from[Q];
  unsigned place[Q];                             // own | neighbour's << 16
  const int above = (ty + 1 == P.tiles_y ? 0 : ty + 1) * P.tiles_x + tx;
  const int below = (ty == 0 ? P.tiles_y - 1 : ty - 1) * P.tiles_x + tx;
  const int right = ty * P.tiles_x + (tx + 1 == P.tiles_x ? 0 : tx + 1);
  const int left = ty * P.tiles_x + (tx == 0 ? P.tiles_x - 1 : tx - 1);
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int i = tid + q * kThreads;
    word[q] = -1;
    from[q] = place[q] = 0;
    if (i < 2 * row_words) {
      const int side = i / row_words, v = i % row_words / kWave, l = i % kWave;
      if (l >= 1 && l <= ncols && !(side == 0 ? south : north)) {
        word[q] = i;
        from[q] = static_cast<unsigned>((side == 0 ? below : above) * words +
                                        (side == 0 ? i + row_words : i - row_words));
        place[q] = static_cast<unsigned>(side == 0 ? at(0, v, l) : at(nrows - 1, v, l)) |
                   static_cast<unsigned>(side == 0 ? at(-1, v, l) : at(nrows, v, l)) << 16;
      }
    } else if (i < words) {
      const int c = i - 2 * row_words, side = c / col_words, v = c % col_words / P.rows,
                r = c % P.rows;
      if (r < nrows && !(side == 0 ? west : east)) {
        word[q] = i;
        from[q] = static_cast<unsigned>((side == 0 ? left : right) * words +
                                        (side == 0 ? i + col_words : i - col_words));
        place[q] = static_cast<unsigned>(at(r, v, side == 0 ? 1 : ncols)) |
                   static_cast<unsigned>(at(r, v, side == 0 ? 0 : ncols + 1)) << 16;
      }
    }
  }

  // the state; ghost columns and rows: Dirichlet states now and for good,
  // transmissive ones are written along with the cells they copy
  for (int r = wave - 1; r <= nrows; r += kWaves) {
    const int j = min(max(r, 0), nrows - 1);
    const size_t c = static_cast<size_t>(y0 + j) * g.ld + col;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      double x = a.win[v * g.plane + c];
      if (BC == kDirichlet) {
        if (west && lane == 0) x = a.ghost[kWest * kMaxVar + v];
        if (east && lane == ncols + 1) x = a.ghost[kEast * kMaxVar + v];
        if (south && r < 0) x = a.ghost[kSouth * kMaxVar + v];
        if (north && r == nrows) x = a.ghost[kNorth * kMaxVar + v];
      }
      S[at(r, v, lane)] = x;
    }
  }

  GridScratch* const s = a.scr;
  const Spacings h(g);
  double dtn = s->dt;  // adaptive dt of the current state
  double sx = s->cur_sx, sy = s->cur_sy;
  double* const log = s->log;
  const unsigned int log_n = s->nstep, log_cap = static_cast<unsigned int>(s->log_cap);
  const size_t log_stride = static_cast<size_t>(s->log_stride);
  unsigned int status = 0;
  u64 bx = 0, by = 0;
  int save = 0, next_save = a.every > 0 && a.nsaves > 0 ? a.every : -1;
  const bool keep = a.w_last || a.w_prev;
  // transmissive ghost columns: what the first and last columns' lanes write a
  // second time, this many lanes further
  const bool mirror_w = BC == kTransmissive && west && lane == 1;
  const bool mirror_e = BC == kTransmissive && east && lane == ncols;

  // k: steps done; publish state k, then make the step from it
  for (int k = 0;; ++k) {
    const int set = k % 3;
    const bool final = k == a.nsteps;
    if (k > 0) {
      bx = wave_max64(bx);
      by = wave_max64(by);
      if (lane == 0) {
        s_red[0][wave] = bx;
        s_red[1][wave] = by;
      }
    }
    stores_done();  // the words emptied two states ago
    __syncthreads();
    u64* const mine = area + set * set_words + static_cast<size_t>(tile) * words;
    const u64* const theirs = area + set * set_words;
    u64* const slots = maxima + static_cast<size_t>(set) * P.tiles * 2;
    if (tid < 2) {
      u64 x = 0;
      if (k > 0) {
        x = s_red[tid][0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) x = umax64(x, s_red[tid][w]);
      }
      put(slots + tid * P.tiles + tile, x == kEmpty ? bits(__builtin_nan("")) : x);
    }
    if (!final) {
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        if (word[q] >= 0) {
          const u64 b = bits(S[place[q] & 0xffffu]);
          put(mine + word[q], b == kEmpty ? bits(__builtin_nan("")) : b);
        }
      }
    }
    // the rows of other waves next to this wave's, before they change
    double B[NV], T[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      B[v] = S[at(jr - 1, v, lane)];
      T[v] = S[at(jr + nr, v, lane)];
    }
    // wait for the neighbours' edges and, one word per thread, for the maxima
    // of all tiles (threads 0 .. 255: x, 256 .. 511: y); a thread with fewer
    // words looks at its tile's own maximum instead
    const u64* p[Q + 1];
    u64 got[Q + 1];
    const int t = tid & (kMaxTiles - 1), axis = tid / kMaxTiles;
    const bool has_max = axis < 2 && t < P.tiles;
    p[Q] = slots + (has_max ? axis * P.tiles + t : tile);
#pragma unroll
    for (int q = 0; q < Q; ++q) p[q] = !final && word[q] >= 0 ? theirs + from[q] : slots + tile;
    const bool ok = await<Q + 1>(p, ctl, got);
    if (!final) {
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (word[q] >= 0) S[place[q] >> 16] = __longlong_as_double(static_cast<long long>(got[q]));
    }
    {
      const u64 mx = wave_max64(has_max ? got[Q] : 0ull);
      if (lane == 0) s_max[wave] = mx;
    }
    if (!ok) s_ok = 0;
    __syncthreads();
    if (!s_ok) {  // uniform: a wait ran out of time
      if (tid == 0) atomicOr(&s->status, kStatusWait);
      return;
    }
    if (k > 0) {
      constexpr int kHalf = kMaxTiles / kWave;  // waves that hold x maxima
      u64 mx = s_max[0], my = s_max[kHalf];
#pragma unroll
      for (int w = 1; w < kHalf; ++w) {
        mx = umax64(mx, s_max[w]);
        my = umax64(my, s_max[kHalf + w]);
      }
      sx = __longlong_as_double(static_cast<long long>(mx));
      sy = __longlong_as_double(static_cast<long long>(my));
      dtn = h.next_dt(g, sx, sy);
      status |= state_status(sx, sy, dtn);
      // every tile is done with state k - 1
      u64* const old = area + ((k - 1) % 3) * set_words + static_cast<size_t>(tile) * words;
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (word[q] >= 0) put(old + word[q], kEmpty);
      if (tid < 2)
        put(maxima + (static_cast<size_t>((k - 1) % 3) * 2 + tid) * P.tiles + tile, kEmpty);
    }
    // where state k goes: a saved state, and the run's last two
    if (k == next_save || (k >= a.nsteps - 1 && keep)) {
      double* const out[2] = {k == next_save ? a.saves[save] : nullptr,
                              final ? a.w_last : (k == a.nsteps - 1 ? a.w_prev : nullptr)};
      for (int q = 0; q < 2; ++q) {
        double* const w = q == 0 ? out[0] : out[1];
        if (!w) continue;  // uniform
        for (int r = jr; r < jr + nr; ++r) {
          const size_t c = static_cast<size_t>(y0 + r) * g.ld + col;
          if (inside) {
#pragma unroll
            for (int v = 0; v < NV; ++v) w[v * g.plane + c] = S[at(r, v, lane)];
          }
        }
      }
      if (k == next_save) next_save = ++save < a.nsaves ? next_save + a.every : -1;
    }
    if (final) break;

    // ---- the step from state k
    bool cfl_ok;
    const double dt_used = step_dt(a, k, sx, sy, dtn, cfl_ok);
    const double dt = cfl_ok ? dt_used : 0.0;
    if (!cfl_ok) status |= kStatusCfl;
    if (tile == 0 && tid == 0 && log && log_n + k < log_cap)
      log[static_cast<size_t>(log_n + k) * log_stride] = dt;
    double mux, muy;
    h.courant(dt, mux, muy);
    bx = by = 0;
    if (nr > 0) {  // uniform across the wave
      // the exchanged rows came after the read above
      if (wave == 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) B[v] = S[at(-1, v, lane)];
      }
      if (wave == last_wave) {
#pragma unroll
        for (int v = 0; v < NV; ++v) T[v] = S[at(nrows, v, lane)];
      }
      double W[NV], G[NV];
      Prim Pc;
      {
        Prim Pb;
#pragma unroll
        for (int v = 0; v < NV; ++v) W[v] = S[at(jr, v, lane)];
        m.prim(B, Pb);
        m.prim(W, Pc);
        m.template flux<1>(B, Pb, W, Pc, G);
      }
      for (int r = jr; r < jr + nr; ++r) {
        double N[NV], Gn[NV], Wr[NV], F[NV], Wo[NV], ux = 0.0, uy = 0.0;
        Prim Pn, Pr;
        if constexpr (M::kSource) {
          const size_t uc = ucell(g, y0 + r, col);
          ux = a.ug[uc];
          uy = a.ug[g.uplane + uc];
        }
        const bool top = r + 1 == jr + nr;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const double n = S[at(r + 1, v, lane)];
          N[v] = top ? T[v] : n;
        }
        m.prim(N, Pn);
        m.template flux<1>(W, Pc, N, Pn, Gn);
        m.shift_next(W, Pc, Wr, Pr);
        m.template flux<0>(W, Pc, Wr, Pr, F);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const double fw = from_prev(F[v]);
          Wo[v] = W[v] - fma(mux, F[v] - fw, muy * (Gn[v] - G[v]));
        }
        if constexpr (M::kSource) m.source(Wo, ux, uy, dt);
        if (inside) {
          double cx, cy;
          m.speeds(Wo, cx, cy);
          bx = umax64(bx, bits(cx));
          by = umax64(by, bits(cy));
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            S[at(r, v, lane)] = Wo[v];
          }
          if constexpr (BC == kTransmissive) {
            if (mirror_w || mirror_e) {
#pragma unroll
              for (int v = 0; v < NV; ++v) {
                if (mirror_w) S[at(r, v, 0)] = Wo[v];
                if (mirror_e) S[at(r, v, ncols + 1)] = Wo[v];
              }
            }
          }
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          W[v] = N[v];
          G[v] = Gn[v];
        }
        Pc = Pn;
      }
      if constexpr (BC == kTransmissive) {  // the ghost rows copy their neighbours
        if (south && wave == 0) {
#pragma unroll
          for (int v = 0; v < NV; ++v) S[at(-1, v, lane)] = S[at(0, v, lane)];
        }
        if (north && wave == last_wave) {
#pragma unroll
          for (int v = 0; v < NV; ++v) S[at(nrows, v, lane)] = S[at(nrows - 1, v, lane)];
        }
      }
    }
  }

  // the run is over: every tile has read what this one published, and the
  // last one to leave empties the last maxima and closes the books
  stores_done();
  __syncthreads();
  if (tid == 0) {
    const u64 t = __hip_atomic_fetch_add(&ctl->done, 1ull, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
    s_ok = t == static_cast<u64>(P.tiles) - 1 ? 2 : 1;
  }
  __syncthreads();
  if (s_ok == 2) {
    for (int i = tid; i < 2 * P.tiles; i += kThreads)
      put(maxima + static_cast<size_t>(a.nsteps % 3) * P.tiles * 2 + i, kEmpty);
    if (tid == 0) {
      put(&ctl->arrived, 0);
      put(&ctl->decision, 0);
      put(&ctl->done, 0);
      s->cur_sx = sx;
      s->cur_sy = sy;
      s->dt = dtn;
      if (log) s->nstep = log_n + static_cast<unsigned int>(a.nsteps);
      if (status) atomicOr(&s->status, status);
    }
  }
}

// The same run where the tiles could not all start (`decision` is 2, else it
// leaves at once), through device memory and by whatever workgroups do start. Each
// takes the next ticket, a piece of a step's cells; tickets are numbered step by
// step, so a workgroup waits only for pieces of earlier tickets, and those are
// with workgroups that run. However few of them the chip has room for, the one
// with the lowest open ticket waits for nobody. The cells of a step are seen by
// the next through fences at device scope on both sides of the count of the
// finished pieces; the last piece of a step takes its maxima and the next dt.
// us a step in runs of five with their start, this / in one workgroup, as before:
// Euler 200 x 150 22 / 124, 512^2 64 / 1179, 1024^2 80 / 4722, spray 200^2 27 / 208,
// advection 1500^2 69 / 2674.
template <class M, int BC>
__global__ __launch_bounds__(kGeneralThreads) void general_run_kernel(Args a, Pieces pieces) {
  constexpr int NV = M::NV, kThreads = kGeneralThreads, kWaves = kThreads / kWave;
  Control* const ctl = reinterpret_cast<Control*>(a.area);
  __shared__ u64 s_red[2][kWaves];
  __shared__ u64 s_ticket;
  __shared__ int s_run, s_go;
  const int tid = static_cast<int>(threadIdx.x);
  if (tid == 0) s_run = peek(&ctl->decision) == 2 && peek(&ctl->abort) == 0;
  __syncthreads();
  if (!s_run) return;
  const M m(a.m);
  const GridGeom& g = a.g;
  GridScratch* const s = a.scr;
  const long long ncell = static_cast<long long>(g.nx) * g.ny;
  const u64 per_step = static_cast<u64>(pieces.count);
  const u64 total = per_step * static_cast<u64>(a.nsteps);
  const Spacings h(g);
  double* const log = s->log;
  const unsigned int log_n = s->nstep, log_cap = static_cast<unsigned int>(s->log_cap);
  const size_t log_stride = static_cast<size_t>(s->log_stride);
  auto load = [&](const double* w, int j, int i, double* o) {
    if (BC == kDirichlet && (i < 0 || i >= g.nx || j < 0 || j >= g.ny)) {
      const int side = i < 0 ? kWest : (i >= g.nx ? kEast : (j < 0 ? kSouth : kNorth));
#pragma unroll
      for (int v = 0; v < NV; ++v) o[v] = a.ghost[side * kMaxVar + v];
      return;
    }
    const size_t at = static_cast<size_t>(row_index<BC>(j, g.ny)) * g.ld + col_index<BC>(i, g.nx);
#pragma unroll
    for (int v = 0; v < NV; ++v) o[v] = w[v * g.plane + at];
  };
  for (;;) {
    if (tid == 0) {
      s_ticket = __hip_atomic_fetch_add(&ctl->ticket, 1ull, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
      s_go = s_ticket >= total ? 0 : (steps_done(ctl, s_ticket / per_step) ? 1 : 2);
    }
    __syncthreads();
    const u64 ticket = s_ticket;
    if (s_go == 0) break;  // uniform
    if (s_go == 2) {       // uniform: a wait ran out of time
      if (tid == 0) atomicOr(&s->status, kStatusWait);
      return;
    }
    __threadfence();  // the cells of state k as their writers left them
    const int k = static_cast<int>(ticket / per_step);
    const long long piece = static_cast<long long>(ticket % per_step);
    const double sx = k == 0 ? s->cur_sx : value(peek(&ctl->sx));
    const double sy = k == 0 ? s->cur_sy : value(peek(&ctl->sy));
    const double dtn = k == 0 ? s->dt : value(peek(&ctl->dt));
    const double* const in = k == 0 ? a.win : state_buffer(a, k);
    double* const out = state_buffer(a, k + 1);
    // the last state goes to w_last, also where it is saved
    double* const copy = k + 1 == a.nsteps && a.w_last != out ? a.w_last : nullptr;
    bool cfl_ok;
    const double used = step_dt(a, k, sx, sy, dtn, cfl_ok);
    const double dt = cfl_ok ? used : 0.0;
    if (tid == 0 && piece == 0) {
      if (!cfl_ok) atomicOr(&s->status, kStatusCfl);
      if (log && log_n + k < log_cap) log[static_cast<size_t>(log_n + k) * log_stride] = dt;
    }
    double mux, muy;
    h.courant(dt, mux, muy);
    u64 bx = 0, by = 0;
    const long long end = min(ncell, (piece + 1) * pieces.cells);
    for (long long c = piece * pieces.cells + tid; c < end; c += kThreads) {
      const int j = static_cast<int>(c / g.nx), i = static_cast<int>(c % g.nx);
      typename M::Prim P, N;
      double W[NV], X[NV], Fw[NV], Fe[NV], Gs[NV], Gn[NV], Wo[NV];
      load(in, j, i, W);
      m.prim(W, P);
      load(in, j, i - 1, X);
      m.prim(X, N);
      m.template flux<0>(X, N, W, P, Fw);
      load(in, j, i + 1, X);
      m.prim(X, N);
      m.template flux<0>(W, P, X, N, Fe);
      load(in, j - 1, i, X);
      m.prim(X, N);
      m.template flux<1>(X, N, W, P, Gs);
      load(in, j + 1, i, X);
      m.prim(X, N);
      m.template flux<1>(W, P, X, N, Gn);
#pragma unroll
      for (int v = 0; v < NV; ++v) Wo[v] = W[v] - fma(mux, Fe[v] - Fw[v], muy * (Gn[v] - Gs[v]));
      if constexpr (M::kSource) {
        const size_t uc = ucell(g, j, i);
        m.source(Wo, a.ug[uc], a.ug[g.uplane + uc], dt);
      }
      const size_t at = static_cast<size_t>(j) * g.ld + i;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        out[v * g.plane + at] = Wo[v];
        if (copy) copy[v * g.plane + at] = Wo[v];
      }
      double cx, cy;
      m.speeds(Wo, cx, cy);
      bx = umax64(bx, bits(cx));
      by = umax64(by, bits(cy));
    }
    bx = wave_max64(bx);
    by = wave_max64(by);
    if ((tid & (kWave - 1)) == 0) {
      s_red[0][tid / kWave] = bx;
      s_red[1][tid / kWave] = by;
    }
    stores_done();
    __syncthreads();
    if (tid == 0) {
      u64 mx = s_red[0][0], my = s_red[1][0];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) {
        mx = umax64(mx, s_red[0][w]);
        my = umax64(my, s_red[1][w]);
      }
      atomicMax(&ctl->max_x, mx);
      atomicMax(&ctl->max_y, my);
      __threadfence();  // the maxima and the workgroup's cells, then the count
      const u64 f = __hip_atomic_fetch_add(&ctl->finished, 1ull, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
      if (f == (static_cast<u64>(k) + 1) * per_step - 1) {  // the step's last piece
        const double nx = value(atomicExch(&ctl->max_x, 0ull));
        const double ny = value(atomicExch(&ctl->max_y, 0ull));
        const double next = h.next_dt(g, nx, ny);
        const unsigned int status = state_status(nx, ny, next);
        if (status) atomicOr(&s->status, status);
        put(&ctl->sx, bits(nx));
        put(&ctl->sy, bits(ny));
        put(&ctl->dt, bits(next));
        stores_done();
        put(&ctl->steps, static_cast<u64>(k) + 1);
      }
    }
  }
  if (tid == 0) {
    stores_done();
    const u64 left = __hip_atomic_fetch_add(&ctl->left, 1ull, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
    if (left == gridDim.x - 1) {  // all are done
      s->cur_sx = value(peek(&ctl->sx));
      s->cur_sy = value(peek(&ctl->sy));
      s->dt = value(peek(&ctl->dt));
      if (log) s->nstep = log_n + static_cast<unsigned int>(a.nsteps);
      put(&ctl->ticket, 0);
      put(&ctl->finished, 0);
      put(&ctl->steps, 0);
      put(&ctl->left, 0);
      put(&ctl->arrived, 0);
      put(&ctl->decision, 0);
    }
  }
}

// A grid's scratch block and the exchange area behind it, in one launch.
__global__ void clear_area_kernel(GridScratch* scr, size_t words) {
  const size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < words) reinterpret_cast<u64*>(scr + 1)[i] = i < kControlWords ? 0ull : kEmpty;
  if (i == 0) *scr = GridScratch{};
}

template <class M>
void* run_fn(int bc) {
  if (bc == kPeriodic) return reinterpret_cast<void*>(&cluster_run_kernel<M, kPeriodic>);
  if (bc == kTransmissive) return reinterpret_cast<void*>(&cluster_run_kernel<M, kTransmissive>);
  return reinterpret_cast<void*>(&cluster_run_kernel<M, kDirichlet>);
}
template <class M>
void* general_fn(int bc) {
  if (bc == kPeriodic) return reinterpret_cast<void*>(&general_run_kernel<M, kPeriodic>);
  if (bc == kTransmissive) return reinterpret_cast<void*>(&general_run_kernel<M, kTransmissive>);
  return reinterpret_cast<void*>(&general_run_kernel<M, kDirichlet>);
}

}  // namespace

hipError_t launch_clear_area(GridScratch* scr, size_t words, hipStream_t st) {
  hipLaunchKernelGGL(clear_area_kernel, dim3(static_cast<unsigned>((words + 255) / 256)), dim3(256),
                     0, st, scr, words);
  return hipGetLastError();
}

hipError_t launch_run(const Args& a, int model, hipStream_t st) {
  void *f = nullptr, *h = nullptr;
  const int bc = a.g.bc, nv = model == 0 ? 1 : (model == 1 ? 4 : 6);
  if (a.plan.rows < 1 || a.plan.rows > max_rows(nv) || a.plan.cols < 1 || a.plan.cols > kCols ||
      a.plan.tiles < 1 || a.plan.tiles > kMaxTiles || a.nsteps < 1 || a.nsaves > kMaxSaves)
    return hipErrorInvalidValue;
  if (model == 0) {
    f = run_fn<Adv>(bc);
    h = general_fn<Adv>(bc);
  } else if (model == 1) {
    f = run_fn<Euler>(bc);
    h = general_fn<Euler>(bc);
  } else if (model == 2) {
    f = run_fn<Spray>(bc);
    h = general_fn<Spray>(bc);
  }
  if (!f) return hipErrorInvalidValue;
  // every state of the run by tickets has a buffer, the first another than win and
  // the last but one w_prev, where that is asked for
  if (a.w_prev && (a.w_prev != a.spare || a.every > 0)) return hipErrorInvalidValue;
  if (!a.w_last ? a.every != 1 || a.nsaves < a.nsteps : a.win == state_buffer(a, 1))
    return hipErrorInvalidValue;
  Args copy = a;
  Pieces pieces = make_pieces(a.g.nx, a.g.ny);
  void* args[] = {&copy, &pieces};
  const hipError_t e = hipLaunchKernel(f, dim3(a.plan.tiles), dim3(waves(nv) * kWave), args, 0, st);
  if (e != hipSuccess) return e;
  return hipLaunchKernel(h, dim3(pieces.count), dim3(kGeneralThreads), args, 0, st);
}

}  // namespace cluster
}  // namespace fvm
