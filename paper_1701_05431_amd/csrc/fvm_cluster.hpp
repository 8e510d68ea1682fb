// fvm_cluster.hpp -- a whole run of a grid that fits in the chip's LDS, in one
// launch: device code and the plan (see fvm_cluster.hip).
//
// What bounds a step of such a grid when every step is its own launch is not
// its traffic but the launch: start, first loads, the reduction's chain of
// device atomics, the next launch (8 us a step for 200 x 150 cells, 23 us for
// 1024^2 where 6 us of arithmetic are needed). Here up to 256 workgroups, one
// per CU, keep their tile of the state in LDS for the whole run:
//  - a tile is up to 62 columns wide, one column per lane, lanes 0 and
//    cols + 1 the neighbour columns; its waves march up their share of the rows
//    in place, the x-neighbours by DPP, the y-face carried, every face and
//    update with the arguments of the marching strips (bitwise the same states,
//    maxima and dts);
//  - tiles hand their edges to each other through a small exchange area in
//    device memory;
//  - one round trip through memory a step: a word of the exchange area holds
//    kEmpty until its value is there, so a reader waits on the value itself
//    and no flag follows the data. The same holds for the tiles' speed maxima,
//    which every tile reads (the global time step) and which tell it that
//    all tiles are done with the previous step's words.
// Words rotate over three sets. After a tile has seen every tile's maxima of
// state k it empties its words of state k - 1 (all have read them) and the
// emptying is complete before it publishes state k + 1, so nobody who looks for
// state k + 2 in that set can find state k - 1.
//
// Measured, us a step in runs of 20 to 100 steps, step launches / on the chip:
// advection 512^2 9.5 / 5.7, 1500^2 17.6 / 8.6; Euler 200 x 150 8.2 / 5.4, 512^2
// 13.8 / 8.8, 1024^2 23.3 / 14.9; spray 200^2 10.5 / 5.9, 512^2 18.3 / 11.7, 860 x 900
// 32.6 / 18.2. About 5 us of each are the exchange (2 us from a store to the
// neighbour's load), the rest the arithmetic: 1.0 us a row of 8 waves for Euler.
#pragma once

#include <hip/hip_runtime.h>

#include <cfloat>

#include "fvm_internal.hpp"
#include "fvm_models.hpp"
#include "fvm_step.hpp"

namespace fvm {
namespace cluster {

typedef unsigned long long u64;

constexpr int kCols = 62;       // columns of a tile
constexpr int kMaxTiles = 256;  // one workgroup per CU of the whole chip
constexpr int kMaxSaves = 64;

// An exchange word nobody has written: a NaN pattern that no arithmetic
// returns (a state value with these bits is published as another NaN).
constexpr u64 kEmpty = 0xfff8a5c35a3ce179ull;

// Control words in front of the exchange area.
struct Control {
  u64 arrived;   // workgroups that have started
  u64 decision;  // 0 open, 1 go (all have started), 2 no go
  u64 done;      // workgroups that have finished the run
  u64 abort;     // a wait ran out of time
  // of the run by tickets (after "no go"):
  u64 ticket, finished;  // pieces handed out, pieces done
  u64 steps;             // steps done
  u64 left;              // workgroups that have left
  u64 max_x, max_y;      // speed maxima of the step under way
  u64 sx, sy, dt;        // of the state after `steps` steps: maxima, next dt
};
constexpr int kControlWords = 32;

// Tiles of a run.
struct Plan {
  int cols, rows;  // of a tile (the last ones of a row or column may be smaller)
  int tiles_x, tiles_y, tiles;
};

// Exchange words of one tile: its first and last rows, its first and last
// columns, of every variable.
__host__ __device__ constexpr int tile_words(int nv, int rows) {
  return 2 * nv * (kWave + rows);
}
__host__ __device__ inline size_t area_words(int nv, const Plan& p) {
  return kControlWords +
         3 * static_cast<size_t>(p.tiles) * (static_cast<size_t>(tile_words(nv, p.rows)) + 2);
}

// The most rows of a tile: with the row below and the one above it, nv * 512
// bytes each, within 160 KB of LDS.
__host__ __device__ constexpr int max_rows(int nv) { return nv == 1 ? 300 : (nv == 4 ? 76 : 50); }
// Waves of a workgroup. Two per SIMD for Euler and the spray: with three or
// four, 1024^2 Euler cells take as long (16.8 and 17.1 us a step against 17.1 then) and
// 200 x 150, whose tiles have 8 rows, longer (7.3 and 8.1 us against 5.9 then).
__host__ __device__ constexpr int waves(int nv) { return nv == 1 ? 16 : 8; }

// The smallest tiles that kMaxTiles workgroups cover the grid with, at least
// one row per wave; false if the grid does not fit.
inline bool make_plan(int nv, int nx, int ny, Plan* p) {
  const int tx = (nx + kCols - 1) / kCols;
  if (tx > kMaxTiles) return false;
  const int ty = kMaxTiles / tx;
  const int rows = (ny + ty - 1) / ty;
  if (rows > max_rows(nv)) return false;
  p->rows = rows < waves(nv) ? (ny < waves(nv) ? ny : waves(nv)) : rows;
  p->cols = (nx + tx - 1) / tx;
  p->tiles_x = (nx + p->cols - 1) / p->cols;
  p->tiles_y = (ny + p->rows - 1) / p->rows;
  p->tiles = p->tiles_x * p->tiles_y;
  return true;
}

// Pieces of a step of a run by tickets: consecutive cells (row-major), a
// multiple of the workgroup's threads, of at most kMaxTiles workgroups.
constexpr int kGeneralThreads = 512;
struct Pieces {
  long long cells;  // of a piece
  int count;
};
inline Pieces make_pieces(int nx, int ny) {
  const long long n = static_cast<long long>(nx) * ny;
  Pieces p;
  p.cells = (n + kMaxTiles * kGeneralThreads - 1) / (kMaxTiles * kGeneralThreads) * kGeneralThreads;
  p.count = static_cast<int>((n + p.cells - 1) / p.cells);
  return p;
}

struct Args {
  const double* win;          // state 0
  double* w_last;             // receives state nsteps (null: every state is saved)
  double* w_prev;             // receives state nsteps - 1 (may be null)
  double* spare;              // run by tickets: the states an odd number of steps before
                              // the last that are not saved (w_prev, where that is given)
  const double* ug;
  GridScratch* scr;
  u64* area;                  // control words, words of the tiles, maxima
  GridGeom g;
  ModelConsts m;
  double ghost[4 * kMaxVar];
  Plan plan;
  int mode, nsteps, k0;       // dts[k0 + k] is step k's dt (kDtArray)
  double dt_arg;
  const double* dts;
  int every;                  // > 0: states every, 2 every, .. are saved
  int nsaves;                 // at most this many
  double* saves[kMaxSaves];   // saves[q]: state (q + 1) every
};

// x / d for one d and many x: the quotient from RN(1/d) with two residual
// corrections, which is the correctly rounded one (the second correction
// starts within an ulp; P. Markstein, IBM J. Res. Dev. 34, 1990) where x and the
// quotient are normal and far from the ends of the range. Five dependent
// operations instead of some thirty, three times in a row between a state's
// maxima and the step from it.
struct Divisor {
  double d, r;
  __device__ __forceinline__ explicit Divisor(double x) : d(x), r(1.0 / x) {}
  __device__ __forceinline__ double into(double x) const {
    const double q0 = x * r;
    const double q1 = fma(fma(-d, q0, x), r, q0);
    return fma(fma(-d, q1, x), r, q1);
  }
};
__device__ __forceinline__ bool middling(double x) { return x > 1e-100 && x < 1e100; }

// dt / dx and dt / dy, and the next adaptive dt (next_dt) of a state's maxima,
// with the divisors of the spacings at hand (ordinary: those are middling).
struct Spacings {
  Divisor x, y;
  bool ordinary;
  __device__ __forceinline__ explicit Spacings(const GridGeom& g)
      : x(g.dx), y(g.dy), ordinary(middling(g.dx) && middling(g.dy)) {}
  __device__ __forceinline__ double next_dt(const GridGeom& g, double sx, double sy) const {
    if (ordinary && middling(sx) && middling(sy)) return g.cfl / (x.into(sx) + y.into(sy));
    return fvm::next_dt(g, sx, sy);
  }
  __device__ __forceinline__ void courant(double dt, double& mux, double& muy) const {
    const bool fast = ordinary && middling(dt);
    mux = fast ? x.into(dt) : dt / x.d;
    muy = fast ? y.into(dt) : dt / y.d;
  }
};

// Status bits of a state with these maxima and this next dt, as finalize_grid
// sets them.
__device__ __forceinline__ unsigned int state_status(double sx, double sy, double dtn) {
  unsigned int st = 0;
  if (!(sx <= DBL_MAX) || !(sy <= DBL_MAX)) st |= kStatusNonFinite;
  if (!(dtn > 0.0)) st |= kStatusDt;
  return st;
}

// dt of the step from state k with maxima (sx, sy) and adaptive dt dtn; ok:
// false for a fixed-dt step that fails the paper's check (a copy).
__device__ __forceinline__ double step_dt(const Args& a, int k, double sx, double sy, double dtn,
                                          bool& ok) {
  ok = true;
  if (a.mode == kDtArray) return a.dts[a.k0 + k];
  if (a.mode == kDtAdaptive) return dtn;
  ok = !(a.dt_arg * (sx > sy ? sx : sy) > a.g.hmin);
  return a.dt_arg;
}

// Where state k is saved, or null.
__host__ __device__ __forceinline__ double* saved(const Args& a, int k) {
  if (a.every <= 0 || k % a.every != 0) return nullptr;
  const int q = k / a.every;
  return q >= 1 && q <= a.nsaves ? a.saves[q - 1] : nullptr;
}

// Where a run by tickets keeps state k > 0: w_last and spare in turn between
// the saved ones.
__host__ __device__ __forceinline__ double* state_buffer(const Args& a, int k) {
  if (double* const p = saved(a, k)) return p;
  return (a.nsteps - k) % 2 == 0 ? a.w_last : a.spare;
}

}  // namespace cluster
}  // namespace fvm
