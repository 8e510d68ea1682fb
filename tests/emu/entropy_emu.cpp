// entropy_emu.cpp -- runs the entropy closure's wave solver (fvm_entropy.hpp)
// on the CPU, one cell at a time (a wave of one lane: __any(x) is x).
//
// Usage: entropy_emu in out
// `in`: rows of 8 doubles, the moments m_0, m_{1/2}, m_{2/2}, m_{3/2} and a
// start (multipliers in powers of x; NaN for none). `out`: rows of 8 doubles,
// converged (1 or 0), m_{-1/2}, n(S = 0), the multipliers, and the curvature
// rule of the result.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <vector>

#define __constant__ static const
#define __any(x) (x)
using std::ldexp;
using std::rint;
thread_local emu_dim3 emu_threadIdx;
int emu_dpp(int x, int) { return x; }
unsigned long long emu_shfl_xor(unsigned long long x, int) { return x; }

#include "../../paper_1701_05431_amd/csrc/fvm_entropy.hpp"

int main(int argc, char** argv) {
  if (argc != 3) return 2;
  std::FILE* f = std::fopen(argv[1], "rb");
  std::FILE* g = std::fopen(argv[2], "wb");
  if (!f || !g) return 3;
  double row[8];
  while (std::fread(row, sizeof(double), 8, f) == 8) {
    double c[4], l[4];
    fvm::entropy::from_x(row + 4, c);
    const fvm::entropy::Result r = fvm::entropy::solve(true, row, row[4] == row[4], c);
    fvm::entropy::to_x(r.c, l);
    const int rule = fvm::entropy::rule_of(fvm::entropy::curvature(r.c, -1.0, 1.0));
    const double out[8] = {r.ok ? 1.0 : 0.0, r.mmh, r.n0, l[0], l[1], l[2], l[3],
                           static_cast<double>(rule)};
    if (std::fwrite(out, sizeof(double), 8, g) != 8) return 3;
  }
  std::fclose(f);
  std::fclose(g);
  return 0;
}
