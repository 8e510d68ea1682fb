// fvm_entropy.hpp -- the entropy maximiser of one wave's cells (Sec. 6.2):
// Newton's method on the dual, 64 cells at a time.
//
// With x = S^{1/2} and t = 2x - 1 the maximiser is n = exp(p(t)), p a cubic
// c0 + c1 t + c2 t^2 + c3 t^3 on [-1, 1]. From the plain moments
// P_j = 2 int t^j e^p dx the model's weighted ones are
// N_k = int t^k S^0 dn = (P_k + P_{k+1}) / 2 (dS = 2x dx, x = (1 + t)/2), and
// m_{-1/2} = P_0. The c minimise the dual: N_k = tau_k, the cell's moments in
// powers of t; its Hessian is the Hankel matrix N_{k+l}.
//
// What bounds it: issue of FP64 vector instructions (the matrix cores' FP64
// rate equals the vector rate and does not overlap with it: a
// v_mfma_f64_16x16x4 takes as long as 22 v_fma_f64, 16 would do its work, and
// a wave mixing the two takes the sum of both times). So the work is cut:
//  - one Gauss-Legendre rule of 40 to 96 points over the whole interval
//    instead of 16 panels of 8 (128): as accurate at half the points, chosen
//    by the curvature of p where the density has its mass (kRules). Every
//    point needs one exponential;
//  - the points +-t share their powers: with E+- = e^{p(+-t)}, even moments
//    take E+ + E-, odd ones E+ - E-, each one fma with a constant weight, and
//    p's even and odd parts are evaluated once: 49 instructions for two points
//    and eleven moments (measured before: 37 for one point and eight);
//  - p is kept in base 2, so the exponential needs no multiplication by
//    log2(e) and no two-part ln 2;
//  - steps of third order (the second-order term of the inverse map m -> c
//    needs three more moments of the same exponentials), and an accepted cell
//    takes its last step and m_{-1/2} from the expansion instead of
//    evaluating the moments once more: two evaluations per warm cell where a
//    Newton iteration with a final check takes five (7 and 13 cold);
//  - while a cell is far from its solution the coarse 40-point rule is used.
// Source pass over 1024^2 cells of the spray workload: from kept multipliers
// 0.90 -> 0.19 ms, cold 2.5 -> 0.33 ms (3,640 and 6,570 vector instructions per 64
// cells; 60 us of the pass are its loads, stores and the reduction).
#pragma once

#include <hip/hip_runtime.h>

#include "fvm_models.hpp"

namespace fvm {
namespace entropy {

constexpr int kMoments = 11;  // P_0 .. P_10
constexpr int kStride = 12;   // doubles per table row: t, then the 11 weights

// Positive nodes t and weights of the Gauss-Legendre rules on [-1, 1]
// (roots of P_n by Newton's method in 50-digit arithmetic, rounded).
struct Node {
  double t, w;
};
constexpr Node kNodes[] = {
    // 40 points
    {0.9982377097105593, 0.004521277098533191}, {0.990726238699457, 0.010498284531152813},
    {0.9772599499837743, 0.01642105838190789}, {0.9579168192137917, 0.02224584919416696},
    {0.9328128082786765, 0.0279370069800234}, {0.9020988069688743, 0.033460195282547844},
    {0.8659595032122595, 0.038782167974472016}, {0.8246122308333117, 0.04387090818567327},
    {0.7783056514265194, 0.04869580763507223}, {0.7273182551899271, 0.05322784698393682},
    {0.6719566846141796, 0.05743976909939155}, {0.6125538896679802, 0.06130624249292894},
    {0.5494671250951282, 0.06480401345660104}, {0.4830758016861787, 0.0679120458152339},
    {0.413779204371605, 0.07061164739128678}, {0.3419940908257585, 0.07288658239580406},
    {0.2681521850072537, 0.07472316905796826}, {0.1926975807013711, 0.07611036190062624},
    {0.11608407067525521, 0.07703981816424797}, {0.03877241750605082, 0.0775059479784248},
    // 64 points
    {0.9993050417357722, 0.001783280721696433}, {0.9963401167719553, 0.004147033260562468},
    {0.9910133714767443, 0.006504457968978363}, {0.983336253884626, 0.008846759826363947},
    {0.973326827789911, 0.011168139460131128}, {0.9610087996520538, 0.013463047896718643},
    {0.9464113748584028, 0.015726030476024718}, {0.9295691721319396, 0.017951715775697343},
    {0.9105221370785028, 0.02013482315353021}, {0.8893154459951141, 0.022270173808383253},
    {0.8659993981540928, 0.024352702568710874}, {0.8406292962525803, 0.02637746971505466},
    {0.8132653151227975, 0.028339672614259483}, {0.7839723589433414, 0.030234657072402478},
    {0.7528199072605319, 0.03205792835485155}, {0.7198818501716109, 0.033805161837141606},
    {0.6852363130542333, 0.035472213256882386}, {0.6489654712546573, 0.03705512854024005},
    {0.6111553551723933, 0.038550153178615626}, {0.571895646202634, 0.03995374113272034},
    {0.5312794640198946, 0.04126256324262353}, {0.48940314570705296, 0.04247351512365359},
    {0.4463660172534641, 0.04358372452932345}, {0.4022701579639916, 0.044590558163756566},
    {0.3572201583376681, 0.04549162792741814}, {0.31132287199021097, 0.046284796581314416},
    {0.2646871622087674, 0.04696818281621002}, {0.21742364374000708, 0.04754016571483031},
    {0.16964442042399283, 0.04799938859645831}, {0.12146281929612056, 0.048344762234802954},
    {0.07299312178779904, 0.04857546744150343}, {0.024350292663424433, 0.048690957009139724},
    // 80 points
    {0.9995538226516306, 0.0011449500031869414}, {0.9976498643982377, 0.0026635335895126818},
    {0.9942275409656883, 0.004180313124694896}, {0.9892913024997555, 0.005690922451403199},
    {0.982848572738629, 0.007192904768117313}, {0.9749091405857278, 0.008683945269260859},
    {0.9654850890437993, 0.010161766041103065}, {0.9545907663436349, 0.011624114120797826},
    {0.9422427613098727, 0.01306876159240134}, {0.9284598771724458, 0.014493508040509076},
    {0.9132631025717577, 0.015896183583725687}, {0.8966755794387706, 0.017274652056269307},
    {0.8787225676782139, 0.018626814208299033}, {0.8594314066631111, 0.019950610878142},
    {0.8388314735802552, 0.021244026115782005}, {0.8169541386814635, 0.022505090246332463},
    {0.7938327175046055, 0.0237318828659301}, {0.7695024201350413, 0.024922535764115492},
    {0.7440002975835973, 0.026075235767565118}, {0.7173651853620999, 0.02718822750048638},
    {0.6896376443420276, 0.028259816057276864}, {0.6608598989861199, 0.02928836958326785},
    {0.631075773046872, 0.03027232175955798}, {0.6003306228297517, 0.0312101741881147},
    {0.5686712681227097, 0.03210049867348777}, {0.536145920897132, 0.0329419393976454},
    {0.5028041118887849, 0.03373321498461152}, {0.46869661517054445, 0.03447312045175393},
    {0.4338753708317561, 0.03516052904474759}, {0.39839340588196925, 0.035794393953416055},
    {0.3623047534994873, 0.03637374990583598}, {0.32566437074770194, 0.03689771463827601},
    {0.28852805488451183, 0.03736549023873049}, {0.25095235839227215, 0.0377763643620014},
    {0.21299450285766613, 0.038129711314477635}, {0.1747122918326468, 0.038424993006959424},
    {0.1361640228091439, 0.038661759774076467}, {0.0974083984415846, 0.03883965105905197},
    {0.058504437152420666, 0.03895839596276953}, {0.019511383256793996, 0.03901781365630665},
    // 96 points
    {0.9996895038832307, 0.0007967920655520124}, {0.9983643758631817, 0.0018539607889469217},
    {0.9959818429872093, 0.0029107318179349465}, {0.9925439003237626, 0.003964554338444687},
    {0.9880541263296237, 0.005014202742927518}, {0.9825172635630147, 0.006058545504235961},
    {0.9759391745851365, 0.007096470791153865}, {0.9683268284632642, 0.008126876925698759},
    {0.9596882914487426, 0.009148671230783386}, {0.9500327177844377, 0.010160770535008416},
    {0.9393703397527552, 0.011162102099838499}, {0.9277124567223087, 0.01215160467108832},
    {0.9150714231208981, 0.013128229566961573}, {0.9014606353158523, 0.01409094177231486},
    {0.8868945174024204, 0.015038721026994937}, {0.8713885059092965, 0.015970562902562293},
    {0.8549590334346014, 0.016885479864245174}, {0.8376235112281871, 0.01778250231604526},
    {0.8194003107379316, 0.018660679627411466}, {0.8003087441391408, 0.01951908114014502},
    {0.7803690438674332, 0.020356797154333323}, {0.7596023411766475, 0.0211729398921913},
    {0.7380306437444001, 0.02196664443874435}, {0.7156768123489676, 0.022737069658329372},
    {0.6925645366421715, 0.02348339908592622}, {0.6687183100439161, 0.024204841792364692},
    {0.6441634037849671, 0.02490063322248361}, {0.6189258401254686, 0.02557003600534936},
    {0.593032364777572, 0.026212340735672413}, {0.5665104185613972, 0.02682686672559176},
    {0.5393881083243575, 0.027412962726029243}, {0.5116941771546677, 0.027970007616848334},
    {0.48345797392059636, 0.028497411065085385}, {0.454709422167743, 0.028994614150555237},
    {0.42547898840730053, 0.029461089958167905}, {0.3957976498289086, 0.029896344136328384},
    {0.3656968614723136, 0.030299915420827595}, {0.3352085228926254, 0.030671376123669148},
    {0.30436494435449635, 0.031010332586313836}, {0.27319881259104917, 0.031316425596861354},
    {0.24174315616384, 0.03158933077072717}, {0.2100313104605672, 0.03182875889441101},
    {0.17809688236761861, 0.032034456231992664}, {0.14597371465489695, 0.03220620479403025},
    {0.11369585011066592, 0.03234382256857593}, {0.08129749546442556, 0.03244716371406427},
    {0.04881298513604973, 0.032516118713868836}, {0.01627674484960297, 0.03255061449236317},
};
struct Rule {
  int first, pairs;
  double curvature;  // largest |p''(x)| (x in [0, 1]) the rule is used at
};
// The error of a moment depends on p'' where the mass lies (a density of
// width 1/sqrt(|p''|)). Over 63,000 densities (centres -0.2..1.2, widths
// 0.008..1, skewed, and the lognormal ones of the spray workload) the
// smallest curvature within three standard deviations of the mean at which a
// rule is more than 1e-12 off, and further off than 16 panels of 8 points,
// was 316, 1172, 2510 and 4283: the lines lie below those.
constexpr Rule kRules[] = {
    {0, 20, 250.0}, {20, 32, 1000.0}, {52, 40, 2000.0}, {92, 48, 3500.0}};
constexpr int kRuleCount = 4;

constexpr int kPairs = kRules[kRuleCount - 1].first + kRules[kRuleCount - 1].pairs;
static_assert(kPairs == sizeof kNodes / sizeof kNodes[0], "nodes of all rules");

struct Table {
  double v[kPairs * kStride];
  constexpr Table() : v() {
    for (int q = 0; q < kPairs; ++q) {
      v[q * kStride] = kNodes[q].t;
      // P_j = 2 int t^j e^p dx, dx = dt / 2: the rule's weight times t^j
      double c = kNodes[q].w;
      for (int j = 0; j < kMoments; ++j) {
        v[q * kStride + 1 + j] = c;
        c *= kNodes[q].t;
      }
    }
  }
};
__constant__ Table kTable{};

// 2^y: y = n + f with |f| <= 1/2, 2^f by the degree-11 polynomial that
// interpolates it at the Chebyshev points (relative error below 2e-17 before
// rounding), scaled by 2^n (0 and infinity where that leaves the range).
template <int N>
__device__ __forceinline__ void exp2d(const double* y, double* out) {
  constexpr double k[] = {4.4558179083360645e-10, 7.074194297288521e-09, 1.0178057087733941e-07,
                          1.3215432535912375e-06, 1.5252733841556773e-05, 0.00015403530463724353,
                          0.001333355814640647,   0.009618129107587256,   0.055504108664821625,
                          0.24022650695910158,    0.6931471805599453,     1.0};
  double n[N], f[N], p[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    n[u] = rint(y[u]);
    f[u] = y[u] - n[u];
    p[u] = k[0];
  }
#pragma unroll
  for (int j = 1; j < 12; ++j)
#pragma unroll
    for (int u = 0; u < N; ++u) p[u] = fma(p[u], f[u], k[j]);
#pragma unroll
  for (int u = 0; u < N; ++u) out[u] = ldexp(p[u], static_cast<int>(n[u]));
}
__device__ __forceinline__ double exp2d(double y) {
  double e;
  exp2d<1>(&y, &e);
  return e;
}

constexpr double kLog2e = 1.4426950408889634;
constexpr double kLn2 = 0.6931471805599453;

// loads_first(): what stands before it (the next row's scalar loads) is issued
// before what follows; loaded(): x has arrived, so the loop's waits are for the
// next row only.
__device__ __forceinline__ void loads_first() {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_sched_barrier(0);
#endif
}
__device__ __forceinline__ void loaded(double& x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+s"(x));
#endif
}

// P_0 .. P_10 of exp2(c0 + c1 t + c2 t^2 + c3 t^3) by rule `rule` (uniform
// across the wave: the weights are scalar operands).
__device__ __forceinline__ void moments(const double* c, int rule, double* P) {
#pragma unroll
  for (int j = 0; j < kMoments; ++j) P[j] = 0.0;
  int q = 0, n = 0;
#pragma unroll
  for (int k = 0; k < kRuleCount; ++k) {
    q = rule == k ? kRules[k].first : q;
    n = rule == k ? kRules[k].pairs : n;
  }
  const double* T = kTable.v + q * kStride;
  // the next row of the table loads (scalar loads) while this one is used
  double row[kStride];
#pragma unroll
  for (int j = 0; j < kStride; ++j) {
    row[j] = T[j];
    loaded(row[j]);
  }
  for (int i = 0; i < n; ++i) {
    T += i + 1 < n ? kStride : 0;
    double next[kStride];
#pragma unroll
    for (int j = 0; j < kStride; ++j) next[j] = T[j];
    loads_first();
    const double t = row[0], t2 = t * t;
    const double even = fma(c[2], t2, c[0]);
    const double odd = t * fma(c[3], t2, c[1]);
    const double y[2] = {even + odd, even - odd};
    double e[2];
    exp2d<2>(y, e);
    const double s = e[0] + e[1], d = e[0] - e[1];
#pragma unroll
    for (int j = 0; j < kMoments; ++j) P[j] = fma(row[1 + j], j % 2 ? d : s, P[j]);
#pragma unroll
    for (int j = 0; j < kStride; ++j) row[j] = next[j];
  }
}

// The same by the cell's own rule: the rules that cells of the wave want, one
// after the other, each for its cells.
__device__ __forceinline__ void moments_by(bool live, int rule, const double* c, double* P) {
#pragma unroll
  for (int j = 0; j < kMoments; ++j) P[j] = 0.0;
  for (int r = 0; r < kRuleCount; ++r)
    if (live && rule == r) moments(c, __builtin_amdgcn_readfirstlane(rule), P);
}

// The four weighted moments and the Hankel matrix they span, factored as
// L D L^T: solve() applies its inverse.
struct Hankel {
  double l10, l20, l30, l21, l31, l32, r0, r1, r2, r3;  // L below the diagonal, 1/D
  bool ok;                                              // positive definite
  __device__ __forceinline__ explicit Hankel(const double* N) {
    r0 = recip(N[0]);
    l10 = N[1] * r0;
    l20 = N[2] * r0;
    l30 = N[3] * r0;
    const double d1 = fma(-l10, N[1], N[2]);
    r1 = recip(d1);
    const double a21 = fma(-l10, N[2], N[3]), a31 = fma(-l10, N[3], N[4]);
    l21 = a21 * r1;
    l31 = a31 * r1;
    const double d2 = fma(-l21, a21, fma(-l20, N[2], N[4]));
    r2 = recip(d2);
    const double a32 = fma(-l21, a31, fma(-l20, N[3], N[5]));
    l32 = a32 * r2;
    const double d3 = fma(-l32, a32, fma(-l31, a31, fma(-l30, N[3], N[6])));
    r3 = recip(d3);
    ok = N[0] > 0.0 && d1 > 0.0 && d2 > 0.0 && d3 > 0.0 && finite(N[0]);
  }
  // y = H^{-1} g
  __device__ __forceinline__ void solve(const double* g, double* y) const {
    const double y0 = g[0];
    const double y1 = fma(-l10, y0, g[1]);
    const double y2 = fma(-l21, y1, fma(-l20, y0, g[2]));
    const double y3 = fma(-l32, y2, fma(-l31, y1, fma(-l30, y0, g[3])));
    y[3] = y3 * r3;
    y[2] = fma(-l32, y[3], y2 * r2);
    y[1] = fma(-l31, y[3], fma(-l21, y[2], y1 * r1));
    y[0] = fma(-l30, y[3], fma(-l20, y[2], fma(-l10, y[1], y0 * r0)));
  }
};

// Largest |p''| (in x) within three standard deviations of the mean.
__device__ __forceinline__ double curvature(const double* c, double t_lo, double t_hi) {
  const double a = fabs(fma(6.0 * c[3], t_lo, 2.0 * c[2]));
  const double b = fabs(fma(6.0 * c[3], t_hi, 2.0 * c[2]));
  return 4.0 * kLn2 * (a > b ? a : b);
}
__device__ __forceinline__ int rule_of(double curv) {
  int r = 0;
#pragma unroll
  for (int k = 0; k < kRuleCount; ++k) r += curv <= kRules[k].curvature ? 0 : 1;
  return r;  // kRuleCount: steeper than every rule
}

// What a cell ends with.
struct Result {
  bool ok;      // converged here; otherwise the caller's general solver decides
  double c[4];  // multipliers in powers of t, base 2, for the cell's own scale
  double mmh;   // m_{-1/2}
  double n0;    // n(S = 0)
};

// All lanes of the wave call this together, each with its own cell; `live`
// lanes have positive moments w[0..3]. With `warm`, c holds a start (powers of
// t, base 2). A cell is taken on only where the powers of t resolve its
// moments well: mean of x in 0.15 .. 0.84, standard deviation at least 0.02,
// |skewness| below 2, and p no steeper than the finest rule allows; the
// others, and any that does not converge in kMaxEvals evaluations, return
// ok = false.
//
// A cell's evaluations are its own, whatever the other cells of the wave: each
// is made by the rule the cell wants, and the wave takes one rule at a time, the
// coarsest any cell wants, while cells that want a finer one wait. us for ten
// steps of the spray workload, with the finest rule any cell wants for all cells /
// so: 1024^2 from kept multipliers 2123 / 2148, cold 2952 / 3027, 100^2 400 / 412 and
// 613 / 642. (With each evaluation made by every rule that is wanted 2191 at 1024^2,
// and 2406 with a further rule of 48 points, which a third of the waves want beside
// the 64.)
constexpr int kMaxEvals = 24;

__device__ __forceinline__ Result solve(bool live, const double* w, bool warm, const double* c_in) {
  Result r;
  r.ok = false;
  r.mmh = r.n0 = 0.0;
  const double w0 = live ? w[0] : 1.0;
  const double rw = recip(w0);
  const double m1 = live ? w[1] * rw : 0.5, m2 = live ? w[2] * rw : 0.35,
               m3 = live ? w[3] * rw : 0.275;
  const double a = m1, var = fma(-a, a, m2);
  const double sd = root(var > 0.0 ? var : 1.0);
  const double skew = fma(a, fma(2.0 * a, a, -3.0 * m2), m3) * recip(sd * (var > 0.0 ? var : 1.0));
  bool run = live && a > 0.15 && a < 0.84 && var > 4e-4 && fabs(skew) < 2.0;
  // the cell's moments in powers of t = 2x - 1, for unit mass
  const double tau1 = fma(2.0, m1, -1.0);
  const double tau2 = fma(4.0, m2 - m1, 1.0);
  const double tau3 = fma(8.0, m3, fma(-12.0, m2, fma(6.0, m1, -1.0)));
  double t_lo = fma(2.0, fma(-3.0, sd, a), -1.0), t_hi = fma(2.0, fma(3.0, sd, a), -1.0);
  t_lo = t_lo < -1.0 ? -1.0 : t_lo;
  t_hi = t_hi > 1.0 ? 1.0 : t_hi;
  double c[4], step[4] = {0.0, 0.0, 0.0, 0.0};
  // cold start: in z = (x - a)/sd the cubic of a density in x close to the
  // normal one with the cell's skewness (third-order term e, the shift -3e and
  // the -9e^2 that keep its mean and variance), divided by 2x to second order
  // in sd / a
  auto cold = [&](double* q) {
    const double sk = skew > 1.0 ? 1.0 : (skew < -1.0 ? -1.0 : skew);
    const double e = sk * (0.7 / 6.0);
    double s = sd * recip(a);
    s = s > 0.5 ? 0.5 : s;
    const double z1 = fma(-3.0, e, -s);
    const double z2 = fma(0.5 * s, s, fma(-9.0 * e, e, -0.5));
    const double z3 = fma(-s * s, s * (1.0 / 3.0), e);
    // z = (t - ta) / h
    const double ih = 0.5 * recip(sd), ta = tau1;
    const double k3 = z3 * ih * ih * ih * kLog2e, k2 = z2 * ih * ih * kLog2e, k1 = z1 * ih * kLog2e;
    q[3] = k3;
    q[2] = fma(-3.0 * ta, k3, k2);
    q[1] = fma(3.0 * ta * ta, k3, fma(-2.0 * ta, k2, k1));
    q[0] = -ta * fma(ta, fma(ta, k3, -k2), k1);
  };
  const bool start = warm && finite(c_in[0]) && finite(c_in[1]) && finite(c_in[2]) && finite(c_in[3]);
  cold(c);
#pragma unroll
  for (int k = 0; k < 4; ++k) c[k] = run ? (start ? c_in[k] : c[k]) : 0.0;
  bool cold_left = start;          // the cold start has not been tried yet
  bool coarse = true, have = false;
  double phi_last = 0.0, shrink = 1.0;
  int evals = 0;
  while (__any(run)) {
    const double curv = curvature(c, t_lo, t_hi);
    const int full = rule_of(curv);
    // the coarse rule resolves what a steep cell needs to about 1e-6 up to
    // a curvature of 1000; steeper ones use finer rules from the start
    int want = coarse ? (full <= 1 ? 0 : full - 1) : full;
    want = want < kRuleCount ? want : kRuleCount - 1;
    int rule = kRuleCount - 1;
#pragma unroll
    for (int k = kRuleCount - 2; k >= 0; --k) rule = __any(run && want == k) ? k : rule;
    const bool turn = run && want == rule;
    double P[kMoments], N[kMoments - 1];
    moments(c, rule, P);
#pragma unroll
    for (int k = 0; k + 1 < kMoments; ++k) N[k] = 0.5 * (P[k] + P[k + 1]);
    // d1 = H^{-1} g: the Newton step; lam2 = g.d1 for unit mass
    const Hankel H(N);
    const double g[4] = {0.0, fma(tau1, N[0], -N[1]), fma(tau2, N[0], -N[2]),
                         fma(tau3, N[0], -N[3])};
    double d[4];
    H.solve(g, d);
    const double lam2 = fma(g[1], d[1], fma(g[2], d[2], g[3] * d[3])) * H.r0;
    const bool good = H.ok && lam2 >= 0.0 && finite(lam2);
    // the dual's value, where a step may have gone too far
    double phi = 0.0;
    if (__any(turn && !(lam2 < 1e-6)))
      phi = logd(H.ok ? N[0] : 1.0) -
            kLn2 * fma(c[1], tau1, fma(c[2], tau2, fma(c[3], tau3, c[0])));
    const bool reject = !good || (have && !(lam2 < 1e-6) && !(phi <= phi_last));
    const bool accept = turn && !reject && lam2 <= 1e-10 && want >= full;
    // second order: H d2 = -1/2 sum_ij d_i d_j N_{k+i+j}
    double q[7] = {d[0] * d[0],
                   2.0 * d[0] * d[1],
                   fma(2.0 * d[0], d[2], d[1] * d[1]),
                   2.0 * fma(d[0], d[3], d[1] * d[2]),
                   fma(2.0 * d[1], d[3], d[2] * d[2]),
                   2.0 * d[2] * d[3],
                   d[3] * d[3]};
    double h[4], d2[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      double s = q[0] * N[k];
#pragma unroll
      for (int i = 1; i < 7; ++i) s = fma(q[i], N[k + i], s);
      h[k] = -0.5 * s;
    }
    H.solve(h, d2);
    // the moments reach N + f g along c + f d + f^2 d2 + ..: the whole way
    // (f = 1) where the second-order term is at most half the first in the
    // Hessian's norm, else the part of it for which it is
    const double lam22 = fma(h[0], d2[0], fma(h[1], d2[1], fma(h[2], d2[2], h[3] * d2[3]))) * H.r0;
    const bool whole = 4.0 * lam22 <= lam2;
    const double f = whole || !good ? 1.0 : 0.5 * root(lam2 * recip(lam22));
    if (turn && full >= kRuleCount && lam2 < 1e-6) {
      run = false;  // at its solution, and steeper than the rules resolve
    } else if (accept) {
      // the last step by the expansion: its third-order terms are lam^3 ~ 1e-15
      double m = P[0];
#pragma unroll
      for (int k = 0; k < 4; ++k) m = fma(d[k] + d2[k], P[k], m);
      double s = q[0] * P[0];
#pragma unroll
      for (int i = 1; i < 7; ++i) s = fma(q[i], P[i], s);
      const double scale = w0 * H.r0;
      r.mmh = scale * fma(0.5, s, m);
#pragma unroll
      for (int k = 0; k < 4; ++k) c[k] = fma(kLog2e, d[k] + d2[k], c[k]);
      r.n0 = scale * exp2d(c[0] - c[1] + c[2] - c[3]);
      c[0] = fma(kLog2e, logd(scale), c[0]);
      r.ok = finite(r.mmh) && finite(r.n0);
      run = false;
    } else if (turn && !reject) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        step[k] = kLog2e * f * fma(f, d2[k], d[k]);
        c[k] += step[k];
      }
      coarse = coarse && !(lam2 < 1e-3);
      phi_last = phi;
      have = !(lam2 < 1e-6);  // the next evaluation has a value to compare with
      shrink = 1.0;
    } else if (turn) {
      // too far: back to a quarter of the last step, or to the cold start
      shrink *= 0.25;
      if (have && shrink > 1e-4) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          c[k] = fma(-0.75, step[k], c[k]);
          step[k] *= 0.25;
        }
      } else if (cold_left) {
        cold_left = false;
        have = false;
        coarse = true;
        shrink = 1.0;
        cold(c);
      } else {
        run = false;
      }
    }
    if (turn && ++evals == kMaxEvals) run = false;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) r.c[k] = c[k];
  return r;
}

// Multipliers in powers of x, base e, to powers of t, base 2, and back.
__device__ __forceinline__ void from_x(const double* l, double* c) {
  c[0] = kLog2e * fma(0.125, l[3], fma(0.25, l[2], fma(0.5, l[1], l[0])));
  c[1] = kLog2e * fma(0.375, l[3], fma(0.5, l[2], 0.5 * l[1]));
  c[2] = kLog2e * fma(0.375, l[3], 0.25 * l[2]);
  c[3] = kLog2e * 0.125 * l[3];
}
__device__ __forceinline__ void to_x(const double* c, double* l) {
  l[0] = kLn2 * (c[0] - c[1] + c[2] - c[3]);
  l[1] = kLn2 * fma(6.0, c[3], fma(-4.0, c[2], 2.0 * c[1]));
  l[2] = kLn2 * fma(-12.0, c[3], 4.0 * c[2]);
  l[3] = kLn2 * 8.0 * c[3];
}

}  // namespace entropy
}  // namespace fvm
