// FP64 chemistry kernels for gfx950: instantaneous rates and the adaptive
// RODAS3 step of the adiabatic constant-pressure reactor.
//
// Mapping.  A cell is handled by a group of G lanes (G = 16, 32 or 64, the
// smallest power of two >= n = K + 1), so a 64-wide wavefront carries 64/G
// cells.  Lane l of a group owns component l of the state y = [T, Y..] (lane 0 is
// T, lane c >= 1 the species DevMech::order[c - 1]).  Reactions are spread over the
// lanes of the group (lane l takes l, l + G, ... of the passes' order); their rates of
// progress and Jacobian terms are added to the group's LDS slice by LDS atomics.  The
// Newton matrix M = I/(gamma h) - J is inverted in registers.  Every cross-lane
// exchange stays inside one wavefront (DPP, permlane swaps, LDS), so no workgroup
// barrier is needed and groups may diverge freely.
//
// Scheduling.  The step kernel is persistent: every group takes a cell from a
// device-wide atomic counter, integrates it with per-cell adaptive substeps,
// writes it back and takes the next one, so cells that need many substeps do
// not hold up the lanes of cheap ones.  The wave ends when the counter runs
// past the last cell; every group reaches that exit.
#include <math.h>
#include <stdlib.h>

#include <algorithm>

#include "chem_internal.h"

namespace chem {
namespace {

constexpr double RG = 8.314462618;  // J/(mol K)
constexpr double LN_PREF_RG = 9.408091968961747;  // ln(101325 Pa / RG)

// RODAS3 (Sandu et al. 1997), transformed form (Hairer & Wanner IV.7):
// (I/(gamma h) - J) K_i = f(y + sum_j a_ij K_j) + (1/h) sum_j c_ij K_j.
constexpr double GAMMA = 0.5;
constexpr double TA[4][4] = {{0, 0, 0, 0}, {0, 0, 0, 0}, {2.0, 0, 0, 0}, {2.0, 0, 1.0, 0}};
constexpr double TC[4][4] = {{0, 0, 0, 0}, {4.0, 0, 0, 0}, {1.0, -1.0, 0, 0},
                             {1.0, -1.0, -8.0 / 3.0, 0}};
constexpr bool TNEWF[4] = {true, false, true, true};
constexpr double TM[4] = {2.0, 0.0, 1.0, 1.0};
constexpr double TE[4] = {0.0, 0.0, 0.0, 1.0};

// Tableau entries for a run-time stage index (selects, no memory access).
__device__ __forceinline__ double TA_S(int s, int j) {
  return s == 2 ? (j == 0 ? TA[2][0] : (j == 1 ? TA[2][1] : TA[2][2]))
       : (s == 3 ? (j == 0 ? TA[3][0] : (j == 1 ? TA[3][1] : TA[3][2])) : 0.0);
}
__device__ __forceinline__ double TC_S(int s, int j) {
  return s == 1 ? (j == 0 ? TC[1][0] : 0.0)
       : (s == 2 ? (j == 0 ? TC[2][0] : (j == 1 ? TC[2][1] : 0.0))
                 : (s == 3 ? (j == 0 ? TC[3][0] : (j == 1 ? TC[3][1] : TC[3][2])) : 0.0));
}
__device__ __forceinline__ bool TNEWF_S(int s) { return s == 2 || s == 3; }
// stage 0's f(y_n) is evaluated once per attempt, before the stage loop
static_assert(TNEWF[0] && !TNEWF[1] && TNEWF[2] && TNEWF[3],
              "TNEWF_S: stage 1 reuses f(y_n), stages 2 and 3 evaluate f at a new point");

enum { CELL_OK = 0, CELL_MAX_STEPS = 1, CELL_H_UNDERFLOW = 2, CELL_NONFINITE = 3,
       CELL_SINGULAR = 4 };

// Orders LDS accesses between lanes of one wavefront.  DS instructions of a
// wave execute in issue order, so this only has to stop the compiler from
// moving accesses across it.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// FP64 add to LDS (ds_add_f64); no return value.
__device__ __forceinline__ void lds_add(double *p, double v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// Cross-lane exchanges inside a group of G lanes without the LDS crossbar:
// DPP patterns pair lanes within 16-lane rows (quad_perm [1,0,3,2] and
// [2,3,0,1], row_half_mirror, row_mirror), v_permlane16_swap pairs rows 0/1
// and 2/3, v_permlane32_swap the two halves of the wave.  After each stage of
// an all-reduce every lane of the merged set holds the same bits (the
// combining operations are commutative).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <int CTRL>
__device__ __forceinline__ int dpp_i32(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}
__device__ __forceinline__ double mk_f64(unsigned lo, unsigned hi) {
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// the value of the paired row (16-lane rows 0/1, 2/3) or half (32 lanes)
__device__ __forceinline__ void swap16(double v, double &a, double &b) {
  const long long x = __double_as_longlong(v);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)x, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(x >> 32),
                                                   false, false);
  a = mk_f64(lo[0], hi[0]);  // the even row's value, in both rows of the pair
  b = mk_f64(lo[1], hi[1]);  // the odd row's value
}
__device__ __forceinline__ void swap32(double v, double &a, double &b) {
  const long long x = __double_as_longlong(v);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)x, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(x >> 32),
                                                   false, false);
  a = mk_f64(lo[0], hi[0]);
  b = mk_f64(lo[1], hi[1]);
}
__device__ __forceinline__ int swap16_min(int v) {
  const auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
  return min((int)r[0], (int)r[1]);
}
__device__ __forceinline__ int swap32_min(int v) {
  const auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
  return min((int)r[0], (int)r[1]);
}

template <int G>
__device__ __forceinline__ double grp_sum(double v) {
  static_assert(G == 16 || G == 32 || G == 64, "lane groups of 16, 32 or 64");
  v += dpp_f64<0xB1>(v);
  v += dpp_f64<0x4E>(v);
  v += dpp_f64<0x141>(v);
  v += dpp_f64<0x140>(v);
  if (G >= 32) {
    double a, b;
    swap16(v, a, b);
    v = a + b;
  }
  if (G == 64) {
    double a, b;
    swap32(v, a, b);
    v = a + b;
  }
  return v;
}

template <int G>
__device__ __forceinline__ double grp_max(double v) {
  v = fmax(v, dpp_f64<0xB1>(v));
  v = fmax(v, dpp_f64<0x4E>(v));
  v = fmax(v, dpp_f64<0x141>(v));
  v = fmax(v, dpp_f64<0x140>(v));
  if (G >= 32) {
    double a, b;
    swap16(v, a, b);
    v = fmax(a, b);
  }
  if (G == 64) {
    double a, b;
    swap32(v, a, b);
    v = fmax(a, b);
  }
  return v;
}

template <int G>
__device__ __forceinline__ int grp_min(int v) {
  v = min(v, dpp_i32<0xB1>(v));
  v = min(v, dpp_i32<0x4E>(v));
  v = min(v, dpp_i32<0x141>(v));
  v = min(v, dpp_i32<0x140>(v));
  if (G >= 32) v = swap16_min(v);
  if (G == 64) v = swap32_min(v);
  return v;
}

template <int G>
__device__ __forceinline__ bool grp_any(bool b) {
  const unsigned long long m = __ballot(b);
  if (G == 64) return m != 0ull;
  const int gbase = ((int)threadIdx.x & 63) & ~(G - 1);
  return ((m >> gbase) & ((1ull << (G & 63)) - 1ull)) != 0ull;
}

__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const long long x = __double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)x, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(x >> 32), lane);
  return mk_f64(lo, hi);
}

// v of lane 0 of the caller's group.
template <int G>
__device__ __forceinline__ double grp_first(double v) {
  const int g = ((int)threadIdx.x & 63) / G;
  double out = 0.0;
#pragma unroll
  for (int gg = 0; gg < 64 / G; ++gg) {
    const double x = readlane_f64(v, gg * G);
    out = (g == gg) ? x : out;
  }
  return out;
}

// 1/x by Newton's iteration; `miss` is 1 - x/x as it came out, NaN or far from 0
// where x is zero, not finite or beyond the range of the iteration.
__device__ __forceinline__ double rcp_newton(double x, double &miss) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  r = fma(fma(-x, r, 1.0), r, r);
  miss = fma(-x, r, 1.0);
  return r;
}

// Per-group LDS scratch (doubles), indexed by component (0 = T, c >= 1 the species
// DevMech::order[c - 1]; component 0 of the first two doubles as the dummy of empty reaction slots,
// C = 1 and g = h = 0): (concentration, g/RT) pairs (one 16-byte gather per reaction
// slot), h/RT, the net production rates being accumulated, and the Jacobian /
// Newton matrix (n rows of odd stride).  In chem_rates the matrix region holds
// k_f, k_r instead (and nothing reads iw); in the solves the h slots hold the permuted right-hand side.  iw: 1/W by component (0 for T and past n), shared by the
// wave's groups.
template <int G>
struct GLds {
  double2 *cg;  // 16-byte aligned: the slice starts so
  double *h, *wa, *J, *iw;
  int js;  // row stride of J
  __device__ GLds(double *base, int g, int R, int n) {
    cg = (double2 *)(base + g * doubles(R, n));
    h = (double *)(cg + G);
    wa = h + G;
    J = wa + G;
    js = stride(n);
    iw = base + (64 / G) * doubles(R, n);
  }
  // odd row stride (2 js banks apart: lanes reading one column hit distinct
  // banks) and only the n rows of the n x n matrix
  __host__ __device__ static int stride(int n) { return n | 1; }
  // even, so that every group's slice starts 16-byte aligned; R: reactions whose
  // rate constants the slice takes (0 in the step)
  __host__ __device__ static size_t doubles(int R, int n) {
    const size_t j = (size_t)n * stride(n), k = 2 * (size_t)R;
    return (4 * G + (j > k ? j : k) + 1) & ~(size_t)1;
  }
  __device__ void fill_iw(const DevMech &M) const {
    const int t = threadIdx.x & 63;
    if (t < G) iw[t] = (t >= 1 && t < M.n) ? M.invW[M.order[t - 1]] : 0.0;
  }
};

// A reaction as the lanes load it (three 16-byte loads): its slots' components
// (reactant0, reactant1, product0, product1; the first of either side is never
// empty), {ln A, b}, and {E_a/R, bits}.
struct RxnIn {
  int4 sp;
  double2 ab, eb;
};
__device__ __forceinline__ RxnIn rxn_load(const DevMech &M, int i) {
  return RxnIn{M.xsp[i], M.xab[i], M.xeb[i]};
}

// Rate constants and one-way rates of progress of a reaction from the species
// data in LDS: ln k_f = ln A + b ln T - E_a/(R T), ln K_c = -dG/RT + dn ln(p_ref/RT),
// k_r = exp(ln k_f - ln K_c).
struct Rxn {
  int4 sp;
  double nu[4];        // coefficients, reactants' negative
  double c[4];         // concentrations of the slots
  double kf, kr, fwd, rev;
  double b, EaR, dn;
  unsigned bits;
};

// C^nu of a reaction slot (nu = 1 or 2; 1 for an empty slot, whose C is 1)
__device__ __forceinline__ double slot_fac(double nu, double c) {
  return fabs(nu) == 2.0 ? c * c : c;
}

template <int G>
__device__ __forceinline__ Rxn rxn_eval(const GLds<G> &L, const RxnIn &in, double lnT,
                                        double invT, double lnPRT) {
  Rxn x;
  x.sp = in.sp;
  x.bits = (unsigned)__double_as_longlong(in.eb.y);
  x.b = in.ab.y;
  x.EaR = in.eb.x;
  // empty slots gather the dummy (g = h = 0, coefficient 0): no branches, so the
  // LDS reads of a reaction issue together
  const double2 a0 = L.cg[x.sp.x], a1 = L.cg[x.sp.y], a2 = L.cg[x.sp.z], a3 = L.cg[x.sp.w];
  x.c[0] = a0.x;
  x.c[1] = a1.x;
  x.c[2] = a2.x;
  x.c[3] = a3.x;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const double v = (double)(int)((x.bits >> (2 * t)) & 3u);
    x.nu[t] = t < 2 ? -v : v;
  }
  x.dn = (x.nu[0] + x.nu[1]) + (x.nu[2] + x.nu[3]);
  const double dG = x.nu[0] * a0.y + x.nu[1] * a1.y + x.nu[2] * a2.y + x.nu[3] * a3.y;
  const double lnkf = in.ab.x + x.b * lnT - x.EaR * invT;
  const double lnKc = -dG + x.dn * lnPRT;
  x.kf = exp_f64(lnkf);
  x.kr = exp_f64(lnkf - lnKc);
  x.fwd = x.kf * slot_fac(x.nu[0], x.c[0]) * slot_fac(x.nu[1], x.c[1]);
  x.rev = x.kr * slot_fac(x.nu[2], x.c[2]) * slot_fac(x.nu[3], x.c[3]);
  return x;
}

// Adds reaction x's terms of the Jacobian to the LDS matrix (atomic FP64
// adds: lanes of the group process different reactions that share species).
// q = k_f prod C^nu' - k_r prod C^nu'', so dq/dC of a slot species is the
// product of the other factors times the derivative of its own factor.  Per
// slot component a (net coefficient nu_a) and slot component b: row a, column b
// gets nu_a dq/dC_b and column 0 gets nu_a dq/dT.  Only the second slots can be
// empty: three masked regions.
template <int G>
__device__ __forceinline__ void jac_scatter(const GLds<G> &L, const Rxn &x, double dqT) {
  const double f0 = slot_fac(x.nu[0], x.c[0]), f1 = slot_fac(x.nu[1], x.c[1]);
  const double f2 = slot_fac(x.nu[2], x.c[2]), f3 = slot_fac(x.nu[3], x.c[3]);
  auto dfac = [](double nu, double c) { return fabs(nu) == 2.0 ? 2.0 * c : 1.0; };
  const double q0 = x.kf * dfac(x.nu[0], x.c[0]) * f1;
  const double q1 = x.kf * f0 * dfac(x.nu[1], x.c[1]);
  const double q2 = -x.kr * dfac(x.nu[2], x.c[2]) * f3;
  const double q3 = -x.kr * f2 * dfac(x.nu[3], x.c[3]);
  const int c0 = x.sp.x, c1 = x.sp.y, c2 = x.sp.z, c3 = x.sp.w;
  double *const r0 = L.J + c0 * L.js, *const r2 = L.J + c2 * L.js;
  lds_add(r0, x.nu[0] * dqT);
  lds_add(r2, x.nu[2] * dqT);
  lds_add(r0 + c0, x.nu[0] * q0);
  lds_add(r2 + c0, x.nu[2] * q0);
  lds_add(r0 + c2, x.nu[0] * q2);
  lds_add(r2 + c2, x.nu[2] * q2);
  double *const r1 = L.J + c1 * L.js, *const r3 = L.J + c3 * L.js;
  if (c1) {
    lds_add(r1, x.nu[1] * dqT);
    lds_add(r1 + c0, x.nu[1] * q0);
    lds_add(r1 + c1, x.nu[1] * q1);
    lds_add(r1 + c2, x.nu[1] * q2);
    lds_add(r0 + c1, x.nu[0] * q1);
    lds_add(r2 + c1, x.nu[2] * q1);
  }
  if (c3) {
    lds_add(r3, x.nu[3] * dqT);
    lds_add(r3 + c0, x.nu[3] * q0);
    lds_add(r3 + c2, x.nu[3] * q2);
    lds_add(r3 + c3, x.nu[3] * q3);
    lds_add(r0 + c3, x.nu[0] * q3);
    lds_add(r2 + c3, x.nu[2] * q3);
    if (c1) {
      lds_add(r1 + c3, x.nu[1] * q3);
      lds_add(r3 + c1, x.nu[3] * q1);
    }
  }
}

// sum_j x[j] y[j] over j < n (LDS arrays), one FMA per term in index order.
// The operands are read eight at a time, so a chunk costs one LDS round trip
// instead of one per term; the last chunk reads with its indices clamped to
// n - 1 and adds only its terms below n.
template <int SX = 1, int SY = 1>
__device__ __forceinline__ double dot_lds(const double *x, const double *y, int n, int sx = SX) {
  double acc = 0.0;
  int j0 = 0;
  for (; j0 + 8 <= n; j0 += 8) {
    double a[8], c[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      a[u] = x[(j0 + u) * sx];
      c[u] = y[(j0 + u) * SY];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) acc = fma(a[u], c[u], acc);
  }
  if (j0 < n) {
    double a[8], c[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int j = min(j0 + u, n - 1);
      a[u] = x[j * sx];
      c[u] = y[j * SY];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (j0 + u < n) acc = fma(a[u], c[u], acc);
  }
  return acc;
}

// What the Newton matrix takes from an evaluation, per lane (row l).  With J the
// LDS matrix and u = wd - sum_{c >= 1} J_lc C_c (0 in row 0): entry (l, c) for c >= 1
// is [l == c] dg - (W J_lc + c2 u) iw_c, entry (l, 0) is col + cT u.
struct NewtonRow {
  double W, wd, c2, cT, col, dg;
};

// Right-hand side of one cell, and (jac, uniform over the wave) the species
// rows of its Jacobian.  Lane l holds y_l in yl (species lanes: of species k).  On return lane l holds f_l;
// species lanes hold wdot_k in wdl.  With jac, the LDS matrix holds d wdot_k/dC_j at
// the species' components, and in row 0 the temperature's entries of M times W_j, so that
// all rows of the Newton matrix M = I dg - J follow from NewtonRow.  With KOUT the rate
// constants are left in L.J (k_f at [r], k_r at [R + r]).  With RATES (chem_rates, which
// takes any state and flags none) zero, infinite and subnormal arguments take the library's
// logarithm and division, which have their limits there; in a step such a state is no
// solution, and NaN ends it as well.
template <int G, bool RATES, bool KOUT>
__device__ __forceinline__ void eval_cell(const DevMech &M, const GLds<G> &L, int l, int k,
                                          double p, double yl, double &f, double &wdl, bool jac, double dg,
                                          NewtonRow &nr) {
  const int K = M.K, R = M.R, n = M.n;
  // the first reactions' constants, under way during the thermodynamics
  const int last = max(R - 1, 0);
  RxnIn in0 = rxn_load(M, min(l, last)), in1 = rxn_load(M, min(l + G, last));
  const double T = grp_first<G>(yl);
  double miss;
  auto div = [&](double a, double x) __attribute__((always_inline)) {
    const double r = a * rcp_newton(x, miss);
    if constexpr (RATES)
      if (!(fabs(miss) <= 1e-12)) return a / x;
    return r;
  };
  double lnT = T > 0.0 ? ln_f64(T) : NAN;
  if constexpr (RATES)
    if (!(T >= 0x1p-1022 && T < INFINITY)) lnT = log(T);
  const double invT = div(1.0, T);
  const bool isSp = (l >= 1) && (l <= K);
  double cpR = 0.0, hRT = 0.0, sR = 0.0, dcpR = 0.0, Wk = 1.0, iWk = 1.0, Yk = 0.0;
  if (isSp) {
    Wk = M.W[k];
    iWk = M.invW[k];
    Yk = yl;
    // coefficient i of species k in the range T selects: [i * K] from here
    const int o = (T <= M.Tmid[k] ? 0 : 7 * K) + k;
    const double *a = M.cpT + o, *hc = M.hT + o, *sc = M.sT + o;
    cpR = a[0] + T * (a[K] + T * (a[2 * K] + T * (a[3 * K] + T * a[4 * K])));
    hRT = hc[0] + T * (hc[K] + T * (hc[2 * K] + T * (hc[3 * K] + T * hc[4 * K]))) +
          hc[5 * K] * invT;
    sR = sc[0] * lnT + T * (sc[K] + T * (sc[2 * K] + T * (sc[3 * K] + T * sc[4 * K]))) +
         sc[5 * K];
    dcpR = a[K] + T * (2.0 * a[2 * K] + T * (3.0 * a[3 * K] + T * (4.0 * a[4 * K])));
  }
  const double S = grp_sum<G>(Yk * iWk);
  const double rho = div(p, RG * T * S);
  const double Ck = rho * Yk * iWk;
  const double cp = grp_sum<G>(Yk * RG * cpR * iWk);
  // component 0 is the empty slots' dummy
  L.cg[l] = l == 0 ? make_double2(1.0, 0.0) : make_double2(Ck, hRT - sR);
  L.h[l] = hRT;
  L.wa[l] = 0.0;
  if (jac) {
    double2 *const J2 = (double2 *)L.J;
    const int m2 = (n * L.js + 1) / 2;
    for (int i = l; i < m2; i += G) J2[i] = make_double2(0.0, 0.0);
  }
  wave_sync();

  const double lnPRT = LN_PREF_RG - lnT;
  // two reactions per pass: their gathers and exponentials are independent and
  // issue together before the adds to LDS
  auto finish_rxn = [&](const Rxn &x) __attribute__((always_inline)) {
    // wdot_k = sum_r (nu''_kr - nu'_kr) q_r, added from the reaction's lane
    // (the dummy of empty slots takes the zero terms)
    const double q = x.fwd - x.rev;
    lds_add(L.wa + x.sp.x, x.nu[0] * q);
    lds_add(L.wa + x.sp.y, x.nu[1] * q);
    lds_add(L.wa + x.sp.z, x.nu[2] * q);
    lds_add(L.wa + x.sp.w, x.nu[3] * q);
    if (KOUT) {
      const int r = (int)(x.bits >> 16);
      L.J[r] = x.kf;
      L.J[R + r] = x.kr;
    }
    if (!KOUT && jac) {
      // dq/dT at fixed C: d ln kf/dT = b/T + Ea/(R T^2), d ln Kc/dT = dH_r/(R T^2) - dn/T
      const double dlnkf = x.b * invT + x.EaR * invT * invT;
      const double dH = x.nu[0] * L.h[x.sp.x] + x.nu[1] * L.h[x.sp.y] + x.nu[2] * L.h[x.sp.z] +
                        x.nu[3] * L.h[x.sp.w];
      const double dlnKc = (dH - x.dn) * invT;
      const double dqT = x.fwd * dlnkf - x.rev * (dlnkf - dlnKc);
      jac_scatter<G>(L, x, dqT);
    }
  };
  for (int b0 = 0; b0 < R; b0 += 2 * G) {
    const int r0 = b0 + l, r1 = r0 + G;
    const bool pair = b0 + G < R;  // uniform
    Rxn x0, x1;
    x0 = rxn_eval<G>(L, in0, lnT, invT, lnPRT);
    if (pair) x1 = rxn_eval<G>(L, in1, lnT, invT, lnPRT);
    if (b0 + 2 * G < R) {
      in0 = rxn_load(M, min(r0 + 2 * G, last));
      in1 = rxn_load(M, min(r1 + 2 * G, last));
    }
    if (r0 < R) finish_rxn(x0);
    if (r1 < R) finish_rxn(x1);
  }
  wave_sync();

  const double wd = isSp ? L.wa[l] : 0.0;
  wdl = wd;
  const double Hk = isSp ? RG * T * hRT : 0.0;
  const double Q = grp_sum<G>(Hk * wd);
  const double irho = div(1.0, rho), icp = div(1.0, cp);
  const double fT = -Q * irho * icp;
  f = (l == 0) ? fT : (isSp ? Wk * wd * irho : 0.0);
  if (KOUT || !jac) return;

  // ---- analytic Jacobian ----
  // chain rule through C_j(rho(T, Y), Y): dC_j/dY_i = rho d_ij/W_j - C_j/(S W_i),
  // dC_j/dT = -C_j/T; the temperature's row is -1/(rho c_p) sum_k h_k times the
  // species rows, and the terms of 1/(rho c_p), h_k(T)
  double JwT = 0.0, dwdTC = 0.0;
  if (isSp) {
    dwdTC = L.J[l * L.js];
    JwT = RG * T * dot_lds(L.J + L.js + l, L.h + 1, K, L.js);
  }
  const double dcpdT = grp_sum<G>(Yk * RG * dcpR * iWk);
  const double sumCpW = grp_sum<G>(RG * cpR * wd);
  const double sumHqT = grp_sum<G>(Hk * dwdTC);
  const double aT = grp_sum<G>(JwT * Ck);
  const double irhocp = irho * icp, iS = rcp_newton(S, miss);
  nr.dg = dg;
  nr.W = isSp ? Wk : (l == 0 ? -1.0 : 0.0);
  nr.wd = wd;
  nr.c2 = isSp ? Wk * irho * iS : 0.0;
  nr.cT = isSp ? -(Wk * irho * invT) : 0.0;
  nr.col = isSp ? -(Wk * irho * dwdTC)
                : (l == 0 ? dg - (-(sumCpW + sumHqT - aT * invT) * irhocp -
                                  fT * (-invT + dcpdT * icp))
                          : 0.0);
  if (isSp) L.J[l] = (rho * JwT - aT * iS) * irhocp + fT * (RG * cpR * icp - iS);
  wave_sync();
}

// The Newton matrix written out in LDS, row l by lane l.
template <int G>
__device__ __forceinline__ void newton_lds(const GLds<G> &L, int l, int n, const NewtonRow &nr) {
  if (l < n) {
    double *const row = L.J + l * L.js;
    const double u =
        l == 0 ? 0.0 : nr.wd - dot_lds<1, 2>(row + 1, (const double *)(L.cg + 1), n - 1);
    const double c2 = nr.c2 * u;
    // eight entries read, then eight written: one LDS round trip per chunk
    for (int c0 = 1; c0 < n; c0 += 8) {
      double jr[8], iw[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int c = min(c0 + t, n - 1);
        jr[t] = row[c];
        iw[t] = L.iw[c];
      }
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int c = c0 + t;
        if (c < n) row[c] = (c == l ? nr.dg : 0.0) - (nr.W * jr[t] + c2) * iw[t];
      }
    }
    row[0] = nr.col + nr.cT * u;
  }
  wave_sync();
}

// Gauss-Jordan elimination with partial pivoting of the n x n matrix held in
// LDS, row l owned by lane l (odd row stride).  Pivot of step k: the
// not-yet-eliminated row with the largest |a_ik| (NaN counts as largest), ties
// to the lowest row, as in an LU with partial pivoting.  Rows do not move and
// pivot rows are not scaled: with p_k the pivot row of step k and
// m_i = a_ik / a_{p_k k}, every other row i becomes a_i. - m_i a_{p_k}. and
// its column k holds -m_i, the pivot row's column k holds 1.  Afterwards row
// p_k holds a_{p_k k} times row k of the inverse with its columns in pivot
// order (column j belongs to unknown p_j): each solve is then one
// matrix-vector product instead of two triangular sweeps of n dependent
// steps.  Lane l records its step (mystep) and 1/a_{l,mystep}.  Returns false
// for a zero or non-finite pivot.
template <int G>
__device__ __forceinline__ bool gj_factor(double *A, int l, int n, int &mystep, double &invd) {
  const int JS = GLds<G>::stride(n);
  double *row = A + l * JS;
  bool done = (l >= n);
  mystep = done ? l : -1;
  invd = 1.0;
  bool ok = true;
  for (int k = 0; k < n; ++k) {
    double v = done ? -1.0 : fabs(row[k]);
    if (v != v) v = INFINITY;
    const double vmax = grp_max<G>(v);
    const int idx = grp_min<G>(v == vmax ? l : G);
    const double *prow = A + idx * JS;
    const double pv = prow[k];
    if (!(fabs(pv) > 0.0) || !isfinite(pv)) ok = false;
    const double inv = 1.0 / pv;
    const bool isp = (l == idx);
    if (isp) {
      done = true;
      mystep = k;
      invd = inv;
    }
    if (l < n) {
      // the pivot row itself takes m = 0 and stays unchanged, so lanes
      // reading it see the same values whatever the order of the stores.
      // Eight entries are loaded before any is stored (the stores may alias
      // the pivot row as far as the compiler knows, which would otherwise
      // cost one LDS round trip per entry).
      const double m = isp ? 0.0 : row[k] * inv;
      for (int j0 = 0; j0 < n; j0 += 8) {
        double pr[8], rr[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (j0 + u < n) {
            pr[u] = prow[j0 + u];
            rr[u] = row[j0 + u];
          }
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (j0 + u < n) row[j0 + u] = fma(-m, pr[u], rr[u]);
      }
      row[k] = isp ? 1.0 : -m;
    }
    wave_sync();
  }
  return ok;
}

// Largest of 32-bit integer values over the caller's group (one DPP max per
// stage, as in grp_max).
template <int G>
__device__ __forceinline__ int grp_max_i32(int v) {
  v = max(v, dpp_i32<0xB1>(v));
  v = max(v, dpp_i32<0x4E>(v));
  v = max(v, dpp_i32<0x141>(v));
  v = max(v, dpp_i32<0x140>(v));
  if (G >= 32) {
    const auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    v = max((int)r[0], (int)r[1]);
  }
  if (G == 64) {
    const auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    v = max((int)r[0], (int)r[1]);
  }
  return v;
}
template <int G>
__device__ __forceinline__ unsigned grp_max_u32(unsigned v) {
  v = max(v, (unsigned)dpp_i32<0xB1>((int)v));
  v = max(v, (unsigned)dpp_i32<0x4E>((int)v));
  v = max(v, (unsigned)dpp_i32<0x141>((int)v));
  v = max(v, (unsigned)dpp_i32<0x140>((int)v));
  if (G >= 32) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = max((unsigned)r[0], (unsigned)r[1]);
  }
  if (G == 64) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = max((unsigned)r[0], (unsigned)r[1]);
  }
  return v;
}

// Lowest lane (index within the caller's group) whose b is set; G if none.
template <int G>
__device__ __forceinline__ int grp_first_lane(bool b) {
  const unsigned long long m = __ballot(b);
  if (G == 64) return m ? __builtin_ctzll(m) : G;
  const int g = ((int)threadIdx.x & 63) / G;
  int out = G;
#pragma unroll
  for (int gg = 0; gg < 64 / G; ++gg) {
    // bit G stands in for "no lane"
    const unsigned long long part =
        ((m >> (gg * G)) & ((1ull << (G & 63)) - 1ull)) | (1ull << (G & 63));
    const int f = __builtin_ctzll(part);
    out = (g == gg) ? f : out;
  }
  return out;
}

// Pivot lane of an elimination step: the lane with the largest v in the
// group, the lowest lane among equal values.  v is +0 ... +inf (a candidate
// row's |entry|) or -1 (a row already used), never NaN; on these values the
// order of the doubles is the order of the pair (high word as a signed
// integer, low word as an unsigned one), so the search runs on 32-bit words
// and ends in a ballot of the lanes holding the maximum.
template <int G>
__device__ __forceinline__ bool grp_is_max(double v) {
  const long long b = __double_as_longlong(v);
  const int hi = (int)(b >> 32);
  const unsigned lo = (unsigned)b;
  const int mh = grp_max_i32<G>(hi);
  const unsigned ml = grp_max_u32<G>(hi == mh ? lo : 0u);
  return hi == mh && lo == ml;
}
template <int G>
__device__ __forceinline__ int grp_argmax(double v) {
  return grp_first_lane<G>(grp_is_max<G>(v));
}
// c - m a as a three-address FMA: its result may go to another register than
// c, so the rotation of the register row below costs no copies.
__device__ __forceinline__ double fma_nm(double m, double a, double c) {
  double d;
  asm("v_fma_f64 %0, -%1, %2, %3" : "=v"(d) : "v"(m), "v"(a), "v"(c));
  return d;
}

// gj_factor with each lane's row held in registers (groups of up to 32
// lanes): slot 0 always holds the column being eliminated (the row is
// rotated by one slot per step, so every index is a compile-time constant),
// and the pivot row reaches the other lanes through pbuf (G doubles of LDS)
// as one broadcast per step; the only LDS round trip left on a step's
// dependency chain.  Every lane forms the reciprocal of its own candidate
// pivot while the pivot is searched for, and the pivot lane sends its
// reciprocal in place of the pivot (slot 0): the division leaves the chain.
// Same arithmetic, in the same order, as gj_factor; the factors are written
// back to the LDS rows at the end.  pbuf: 16-byte aligned.
template <int G>
__device__ __forceinline__ bool gj_factor_reg(double *A, double *pbuf, int l, int n, int &mystep,
                                              double &invd) {
  static_assert(G <= 32, "the register row holds G doubles");
  const int JS = GLds<G>::stride(n);
  double *rowp = A + l * JS;
  const bool real = l < n;
  double r[G];
#pragma unroll
  for (int i = 0; i < G; ++i) r[i] = (real && i < n) ? rowp[i] : 0.0;
  bool done = !real;
  mystep = done ? l : -1;
  invd = 1.0;
  bool ok = true;  // this lane's pivot (if it was one) is finite and non-zero
  // the reciprocal of slot 0, formed as soon as the slot is (at the end of
  // the previous step)
  double rinv = 1.0 / r[0];
  for (int k = 0; k < n; ++k) {
    double v = done ? -1.0 : fabs(r[0]);
    if (v != v) v = INFINITY;
    const int idx = grp_argmax<G>(v);
    const bool isp = (l == idx);
    // the row moves as G / 2 pairs (b128 accesses)
    double2 *const pb2 = (double2 *)pbuf;
    if (isp) {
      pb2[0] = make_double2(rinv, r[1]);
#pragma unroll
      for (int i = 1; i < G / 2; ++i) pb2[i] = make_double2(r[2 * i], r[2 * i + 1]);
      if (!(fabs(r[0]) > 0.0) || !isfinite(r[0])) ok = false;
      done = true;
      mystep = k;
      invd = rinv;
    }
    wave_sync();
    double2 q[G / 2];
#pragma unroll
    for (int i = 0; i < G / 2; ++i) q[i] = pb2[i];
    const double inv = q[0].x;
    const double m = isp ? 0.0 : r[0] * inv;
    double pr[G];
#pragma unroll
    for (int i = 1; i < G; ++i) pr[i] = (i & 1) ? q[i / 2].y : q[i / 2].x;
    const double c0 = isp ? 1.0 : -m;
    // the next step's column first, so that its reciprocal (formed here by
    // every lane, not sunk into the pivot's branch) overlaps the other updates
    r[0] = fma_nm(m, pr[1], r[1]);
    rinv = 1.0 / r[0];
    asm volatile("" : "+v"(rinv));
#pragma unroll
    for (int i = 1; i < G - 1; ++i) r[i] = fma_nm(m, pr[i + 1], r[i + 1]);
    r[G - 1] = c0;
    wave_sync();  // every lane has read pbuf before the next pivot row goes there
  }
  // after n rotations slot i holds column (n + i) mod G: G - n more put
  // column i back in slot i, so the stores take constant offsets
  for (int t = n; t < G; ++t) {
    const double c0 = r[0];
#pragma unroll
    for (int i = 0; i < G - 1; ++i) r[i] = r[i + 1];
    r[G - 1] = c0;
  }
  if (real) {
#pragma unroll
    for (int i = 0; i < G; ++i)
      if (i < n) rowp[i] = r[i];
  }
  wave_sync();
  return !grp_any<G>(!ok);
}

// ---- elimination with the diagonal as the pivots
// The Newton matrix is I/(gamma h) - J: at the step sizes the error control
// accepts, the diagonal is nearly always the largest entry left in its column
// (with the components in DevMech::order, in all of the attempts sampled).  So the
// pivots are taken on the diagonal without a search, each step verifies off the
// chain that the search would have chosen it (ties to the lowest row are the
// diagonal's), and only a group that fails repeats the elimination with the search.
//
// With the pivot row known at compile time its broadcast needs no LDS: lane p of
// every 16-lane row reaches its row as the DPP operand of the FMAs (row_newbcast).
// A group of 16 lanes holds one matrix row per lane.  In a group of 32, 16-lane row
// h holds columns 16 h .. 16 h + 15 of all rows, two per lane: lane (h, i) has rows i
// and 16 + i; the multipliers (column k, in one half only) cross to the other half by
// v_permlane16_swap.
//
// A step is about 75 instructions (32 of them the FMAs); with the searched pivot
// and its row's way through LDS (14 16-byte writes and reads) it took 2800 cycles of a
// wave with eight others on the CU, now about 500.  30011 CH4/air cells, dt = 1e-5 s:
// 58.9 -> 40.1 ms by this, 30.3 ms with the changes around it (reactions' order and
// scatter, one copy of the evaluation, the factors kept in registers).
template <int P>
__device__ __forceinline__ double bcast16(double v) {
  const long long b = __double_as_longlong(v);
  return __longlong_as_double(__builtin_amdgcn_update_dpp(0ll, b, 0x150 + P, 0xf, 0xf, false));
}

// x[q] += m y[q](lane P of the 16-lane row), then y[q] likewise with my, for
// four columns q: FMAs whose DPP operand is the broadcast.  The wait states
// let a y[q] written just before reach the DPP read.
template <int P>
__device__ __forceinline__ void fma_bcast4(double &x0, double &x1, double &x2, double &x3,
                                           double &y0, double &y1, double &y2, double &y3,
                                           double mx, double my) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %4, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %5, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %6, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %7, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %4, %4, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %5, %5, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %6, %6, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %7, %7, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf"
      : "+v"(x0), "+v"(x1), "+v"(x2), "+v"(x3), "+v"(y0), "+v"(y1), "+v"(y2), "+v"(y3)
      : "v"(mx), "v"(my), "n"(P));
}
// the same without the x rows (one matrix row per lane)
template <int P>
__device__ __forceinline__ void fma_bcast4(double &y0, double &y1, double &y2, double &y3,
                                           double my) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %0, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %1, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %2, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %3, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
      : "+v"(y0), "+v"(y1), "+v"(y2), "+v"(y3)
      : "v"(my), "n"(P));
}

// lane i > P of each 16-lane row
constexpr unsigned long long rows_after(int P) {
  return ((0xfffeull << P) & 0xffffull) * 0x0001000100010001ull;
}

// Elimination steps K, K + 1, ...: a[x] is the lane's row 16 x + (l & 15).
template <int K, int G>
__device__ __forceinline__ void gj_diag_steps(double (&a)[2][16], int l, int n, double &invd,
                                              unsigned long long &bad) {
  if constexpr (K < G) {
    // every fourth step may be the last (past n the padding's pivots are 1): the
    // steps between are one block for the scheduler
    if (K % 4 == 0 && K >= n) return;  // uniform
    constexpr int P = K % 16, S = K / 16;
    double(&piv)[16] = a[S];
    double(&oth)[16] = a[S ^ 1];
    double c = piv[P], d = 0.0;
    if constexpr (G == 32) {
      double e, o;
      swap16(c, e, o);
      c = S == 0 ? e : o;
      swap16(oth[P], e, o);
      d = S == 0 ? e : o;
    }
    const double pv = bcast16<P>(c);
    double miss;
    const double inv = rcp_newton(pv, miss);
    // the lane compares are made here, not kept as masks across the steps (the
    // scalar registers do not hold them): l and n are made to depend on the step
    asm("" : "+v"(l), "+s"(n) : "v"(pv));
    // a larger or NaN entry in a row not yet used, or an unusable pivot
    bad |= __ballot(!(fabs(c) <= fabs(pv))) & rows_after(P);
    if constexpr (G == 32 && S == 0) bad |= __ballot(!(fabs(d) <= fabs(pv)));
    bad |= __ballot(!(fabs(miss) <= 1e-12));
    invd = l == K ? inv : invd;
    const bool isp = (l & 15) == P;
    // minus the multipliers; the pivot row itself stays as it is
    double mp = -(c * inv);
    const double mo = -(d * inv);
    const double cp = isp ? 1.0 : mp;
    mp = isp ? 0.0 : mp;
#pragma unroll
    for (int t = 0; t < 16; t += 4) {
      // the next step's column first
      const int j0 = (P + 1 + t) & 15, j1 = (P + 2 + t) & 15, j2 = (P + 3 + t) & 15,
                j3 = (P + 4 + t) & 15;
      if constexpr (G == 32)
        fma_bcast4<P>(oth[j0], oth[j1], oth[j2], oth[j3], piv[j0], piv[j1], piv[j2], piv[j3], mo,
                      mp);
      else
        fma_bcast4<P>(piv[j0], piv[j1], piv[j2], piv[j3], mp);
    }
    const bool mine = G == 16 || (l >> 4) == S;
    piv[P] = mine ? cp : piv[P];
    if constexpr (G == 32) oth[P] = mine ? mo : oth[P];
    gj_diag_steps<K + 1, G>(a, l, n, invd, bad);
  }
}

// Gauss-Jordan factors of the Newton matrix (see NewtonRow) in registers: afterwards
// a holds the rows of the inverse by unknown (laid out as in gj_diag_steps), not yet
// scaled by the reciprocal pivots (invd: lane l's unknown l), with their columns in
// pivot order: lane l's right-hand side belongs to column mystep.  They stay there
// for the four solves (parked in LDS between the solves an attempt took 6 % longer).
template <int G>
__device__ __forceinline__ bool gj_factor_diag(const GLds<G> &L, int l, int n,
                                               const NewtonRow &nr, double (&a)[2][16],
                                               int &mystep, double &invd) {
  static_assert(G <= 32, "one or two 16-lane rows");
  constexpr int NS = G / 16;
  const int i = l & 15, h = G == 32 ? (l >> 4) & 1 : 0;
  // rows and columns past n read the last one and take W = c2 = 0 or iw = 0: zero
  // off the diagonal, which is 1 there
#pragma unroll
  for (int x = 0; x < NS; ++x) {
    const double *const src = L.J + min(16 * x + i, n - 1) * L.js;
#pragma unroll
    for (int j = 0; j < 16; ++j) a[x][j] = src[min(16 * h + j, n - 1)];
  }
  // u of the lane's own row (NewtonRow): the row's sum over both halves' columns
  double u;
  {
    double e[NS];
#pragma unroll
    for (int x = 0; x < NS; ++x) e[x] = 0.0;
    const double2 *const C = L.cg + 16 * h;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      // C_0 is the empty slots' dummy, and past n nothing counts
      const int c = 16 * h + j;
      const double w = (c >= 1 && c < n) ? C[j].x : 0.0;
#pragma unroll
      for (int x = 0; x < NS; ++x) e[x] = fma(a[x][j], w, e[x]);
    }
    u = e[0];
    if constexpr (G == 32) {
      double e0, o0, e1, o1;
      swap16(e[0], e0, o0);
      swap16(e[1], e1, o1);
      u = h ? e1 + o1 : e0 + o0;
    }
    u = l == 0 ? 0.0 : nr.wd - u;
  }
  // the lane's rows' coefficients
  const double c2l = nr.c2 * u, coll = nr.col + nr.cT * u;
  double W[2], c2[2], col[2];
  if constexpr (G == 32) {
    swap16(nr.W, W[0], W[1]);
    swap16(c2l, c2[0], c2[1]);
    swap16(coll, col[0], col[1]);
  } else {
    W[0] = nr.W;
    c2[0] = c2l;
    col[0] = coll;
  }
  const double2 *const iw = (const double2 *)(L.iw + 16 * h);
#pragma unroll
  for (int x = 0; x < NS; ++x) {
    const int row = 16 * x + i;
    const double dg = h != x ? 0.0 : (row < n ? nr.dg : 1.0);
#pragma unroll
    for (int j = 0; j < 16; j += 2) {
      const double2 w = iw[j / 2];
      a[x][j] = (i == j ? dg : 0.0) - (W[x] * a[x][j] + c2[x]) * w.x;
      a[x][j + 1] = (i == j + 1 ? dg : 0.0) - (W[x] * a[x][j + 1] + c2[x]) * w.y;
    }
    a[x][0] = h == 0 ? (row < n ? col[x] : 0.0) : a[x][0];
  }
  invd = 1.0;
  mystep = l;
  unsigned long long bad = 0;
  gj_diag_steps<0, G>(a, l, n, invd, bad);
  const int gbase = ((int)threadIdx.x & 63) & ~(G - 1);
  bool ok = true;
  if ((bad >> gbase) & ((1ull << G) - 1ull)) {
    // the search's elimination leaves the rows in their places: L.h takes the row of each
    // unknown, L.wa the reciprocal pivots.  It holds the rows in registers as well: H2/air
    // with shifted enthalpies, dt = 1e-2 s, 4096 cells, where 44 % of the attempts come here,
    // 18.4 ms (searching every attempt 19.0, the repetition on rows in LDS 19.9); CH4/air
    // likewise, 1e-4 s, 8192 cells, 32 %: 22.4 ms (29.1, 28.1).  Not trying the diagonal
    // after an attempt that came here: 19.4 and 28.0 with the rows in LDS.
    newton_lds<G>(L, l, n, nr);
    double id;
    ok = gj_factor_reg<G>(L.J, L.wa, l, n, mystep, id);
    ok = ok && !grp_any<G>(mystep < 0);
    if (ok && l < n) {
      L.h[mystep] = (double)l;
      L.wa[mystep] = id;
    }
    wave_sync();
#pragma unroll
    for (int x = 0; x < NS; ++x) {
      const int row = 16 * x + i;
      const double *const src = L.J + (ok && row < n ? (int)L.h[row] : 0) * L.js;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int c = 16 * h + j;
        const double v = src[min(c, n - 1)];
        a[x][j] = (row < n && c < n) ? v : 0.0;
      }
    }
    invd = ok && l < n ? L.wa[l] : 1.0;
  }
  wave_sync();  // the matrix has been read
  return ok;
}

// Solve M x = b with these factors.  Lane l passes b_l, gets x_l.
template <int G>
__device__ __forceinline__ double gj_solve_diag(const GLds<G> &L, const double (&a)[2][16], int l, int n, int mystep,
                                                double invd, double b) {
  double *const v = L.h;  // G doubles, 16-byte aligned: b in pivot order
  v[l < n ? mystep : l] = l < n ? b : 0.0;
  wave_sync();
  const double2 *const w = (const double2 *)(v + (G == 16 ? 0 : (l & 16)));
  double acc[G / 16], odd[G / 16];
#pragma unroll
  for (int x = 0; x < G / 16; ++x) acc[x] = odd[x] = 0.0;
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const double2 q = w[t];
#pragma unroll
    for (int x = 0; x < G / 16; ++x) {
      acc[x] = fma(a[x][2 * t], q.x, acc[x]);
      odd[x] = fma(a[x][2 * t + 1], q.y, odd[x]);
    }
  }
#pragma unroll
  for (int x = 0; x < G / 16; ++x) acc[x] += odd[x];
  wave_sync();
  double x = acc[0];
  if constexpr (G == 32) {
    // the two halves' columns, rows i to the first 16 lanes, 16 + i to the others
    double e0, o0, e1, o1;
    swap16(acc[0], e0, o0);
    swap16(acc[1], e1, o1);
    x = (l & 16) ? e1 + o1 : e0 + o0;
  }
  return l < n ? x * invd : 0.0;
}

// Solve M x = b with the factors of gj_factor.  Lane l passes b_l, gets x_l.
// v (G doubles of LDS) carries b in pivot order, then x.
template <int G>
__device__ __forceinline__ double gj_solve(const double *A, double *v, int l, int n, int mystep,
                                           double invd, double b) {
  const int JS = GLds<G>::stride(n);
  const double *row = A + l * JS;
  const bool real = l < n;  // lanes past n own no row (none is stored for them)
  if (real) v[mystep] = b;
  wave_sync();
  const double acc = real ? dot_lds(row, v, n) : 0.0;
  wave_sync();
  if (real) v[mystep] = acc * invd;
  wave_sync();
  const double x = real ? v[l] : 0.0;
  wave_sync();
  return x;
}

struct StepArgs {
  int64_t n, ld;
  double dt;
  const double *dt_cell;
  double *T;
  const double *p;
  double *Y;
  double *RR;
  double *h_hint;
  int32_t *stats;
  const int32_t *index;  // optional cell index list (cell j of the call is index[j])
  StepOpts o;
  unsigned long long *counter;
  const unsigned long long *n_dev;  // optional device-side cell count (overrides n)
  uint8_t *flags;                    // optional: bit 4 set for cells that fail
  const chem_set *sets;              // optional set table (device): queue index q is cell
  const int64_t *set_off;            //   q - set_off[s] of the set s with set_off[s] <= q
  int n_sets;
};

// Arrays of the cell a group is working on.
struct CellRef {
  double *T;
  const double *p;
  double *Y;
  double *RR;
  double *hh;
  int32_t *stats;
  int64_t ld, i;
  double dt;
};

__global__ void k_reset_counter(unsigned long long *c) {
  if (threadIdx.x == 0) c[0] = 0ull;
}

template <int G>
__global__ __launch_bounds__(64) void k_rates(DevMech M, int64_t N, int64_t ld, const double *T,
                                              const double *p, const double *Y, double *wdot,
                                              double *dTdt, double *kfkr) {
  extern __shared__ double lds[];
  constexpr int CPW = 64 / G;
  const int lane = threadIdx.x;
  const int g = lane / G, l = lane % G;
  GLds<G> L(lds, g, M.R, M.n);
  const int k = (l >= 1 && l <= M.K) ? M.order[l - 1] : 0;
  NewtonRow nr;
  for (int64_t base = (int64_t)blockIdx.x * CPW; base < N; base += (int64_t)gridDim.x * CPW) {
    const int64_t cell = base + g;
    if (cell >= N) break;  // group-uniform
    double yl = 0.0;
    if (l == 0) yl = T[cell];
    else if (l <= M.K) yl = Y[(int64_t)k * ld + cell];
    const double pc = p[cell];
    double f, wd;
    if (kfkr)
      eval_cell<G, true, true>(M, L, l, k, pc, yl, f, wd, false, 0.0, nr);
    else
      eval_cell<G, true, false>(M, L, l, k, pc, yl, f, wd, false, 0.0, nr);
    if (l >= 1 && l <= M.K) wdot[(int64_t)k * ld + cell] = wd;
    if (l == 0 && dTdt) dTdt[cell] = f;
    if (kfkr) {
      for (int r = l; r < M.R; r += G) {
        kfkr[(int64_t)r * ld + cell] = L.J[r];
        kfkr[(int64_t)(M.R + r) * ld + cell] = L.J[M.R + r];
      }
    }
    wave_sync();
  }
}

template <int G>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(STEP_WAVES_EU, STEP_WAVES_EU)))
void k_step(DevMech M, StepArgs A) {
  extern __shared__ double lds[];
  const int lane = threadIdx.x;
  const int g = lane / G, l = lane % G, lane_in_group = l;
  const int n = M.n;
  GLds<G> L(lds, g, 0, M.n);
  L.fill_iw(M);
  wave_sync();
  const int k = (l >= 1 && l < n) ? M.order[l - 1] : 0;  // the lane's species
  const StepOpts &o = A.o;

  // per-cell state (group-uniform scalars are replicated in every lane)
  int64_t cell = 0, gcell = 0;
  bool active = false;
  double yl = 0.0, y0 = 0.0, p = 0.0, dt = 0.0, t = 0.0, h = 0.0, fac_max = 6.0, rho0 = 0.0;
  int nacc = 0, nrej = 0, status = CELL_OK;

  const int64_t ncell = A.n_dev ? (int64_t)*A.n_dev : A.n;
  // an empty device-side list (no cell fell back) ends every wave here,
  // without a round of atomics on the queue counter
  if (ncell <= 0) return;
  CellRef cr{};
  auto fetch = [&]() {
    unsigned long long c = 0;
    if (l == 0) c = atomicAdd(A.counter, 1ull);
    c = __shfl(c, 0, G);
    cell = (int64_t)c;
    active = cell < ncell;
    if (!active) return;
    if (A.n_sets > 0) {
      int lo = 0, hi = A.n_sets;
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (A.set_off[mid] <= cell) lo = mid;
        else hi = mid;
      }
      const chem_set &st = A.sets[lo];
      cr = CellRef{st.T, st.p, st.Y, st.RR, st.h_hint, st.stats, st.ld, cell - A.set_off[lo],
                   st.dt};
    } else {
      const int64_t gc = A.index ? (int64_t)A.index[cell] : cell;
      cr = CellRef{A.T, A.p, A.Y, A.RR, A.h_hint, A.stats, A.ld, gc,
                   A.dt_cell ? A.dt_cell[gc] : A.dt};
    }
    gcell = cr.i;
    yl = 0.0;
    if (l == 0) yl = cr.T[gcell];
    else if (l < n) yl = cr.Y[(int64_t)k * cr.ld + gcell];
    y0 = yl;
    p = cr.p[gcell];
    dt = cr.dt;
    const double hh = cr.hh ? cr.hh[gcell] : 0.0;
    h = (hh > 0.0) ? hh : o.h0;
    if (h > dt) h = dt;
    t = 0.0;
    fac_max = 6.0;
    nacc = 0;
    nrej = 0;
    status = CELL_OK;
    const bool bad = grp_any<G>(l < n && !isfinite(yl));
    const double T0 = __shfl(yl, 0, G);
    if (bad || !(T0 > 0.0) || !isfinite(p) || !(p > 0.0) || !(dt > 0.0) || !isfinite(dt))
      status = CELL_NONFINITE;
    // density at the initial state, for the rates output
    const double s = grp_sum<G>((l >= 1 && l < n) ? yl / M.W[k] : 0.0);
    rho0 = p / (RG * T0 * s);
  };

  auto finish = [&]() {
    const bool ok = (status == CELL_OK);
    if (ok && l < n) {
      if (l == 0) cr.T[gcell] = yl;
      else cr.Y[(int64_t)k * cr.ld + gcell] = yl;
    }
    if (cr.RR && l >= 1 && l < n)
      cr.RR[(int64_t)k * cr.ld + gcell] = ok ? rho0 * (yl - y0) / dt : 0.0;
    if (l == 0) {
      if (cr.hh && ok) cr.hh[gcell] = h;
      if (cr.stats) {
        cr.stats[gcell] = nacc;
        cr.stats[cr.ld + gcell] = nrej;
        cr.stats[2 * cr.ld + gcell] = status;
      }
      if (A.flags && !ok) A.flags[gcell] |= 4;
    }
  };

  bool want = true;  // the group has no cell and the queue may have one
  for (;;) {
    if (want) {
      fetch();
      want = false;
    }
    if (!__any(active)) break;
    if (active) {
      bool end = (status != CELL_OK) || !(t < dt);
      if (!end) {
        if (nacc + nrej >= o.max_steps) {
          status = CELL_MAX_STEPS;
          end = true;
        }
      }
      bool last = false;
      if (!end) {
        if (h >= dt - t) {
          h = dt - t;
          last = true;
        }
        if (h < o.h_min) {
          status = CELL_H_UNDERFLOW;
          end = true;
        }
      }
      if (!end) {
        // ---- one RODAS3 attempt of size h from yl ----
        // Stage loop kept rolled so that one copy of the right-hand side, of the
        // elimination and of the solve is emitted: an attempt walks through all of
        // the code, which has to stay in the instruction cache.  Terms with j >= s
        // add exact zeros, so the sums equal the oracle's sums over j < s.
        const double ih = 1.0 / h;
        double F = 0.0, wd, K0 = 0.0, K1 = 0.0, K2 = 0.0, K3 = 0.0;
        int mystep = l;
        double invd = 1.0;
        NewtonRow nr;
        double fa[2][16];
        bool ok = true;
#pragma nounroll
        for (int s = 0; s < 4; ++s) {
          // addresses that follow from the lane are formed anew in each stage: kept
          // across the loop they would push the reactions' values out of the registers
          int l = lane_in_group;
          asm volatile("" : "+v"(l));
          if (s != 1) {
            const double v = yl + TA_S(s, 0) * K0 + TA_S(s, 1) * K1 + TA_S(s, 2) * K2;
            eval_cell<G, false, false>(M, L, l, k, p, v, F, wd, s == 0, ih / GAMMA, nr);
          }
          if (s == 0) {
            if constexpr (G <= 32) {
              ok = gj_factor_diag<G>(L, l, n, nr, fa, mystep, invd);
            } else {
              newton_lds<G>(L, l, n, nr);
              ok = gj_factor<G>(L.J, l, n, mystep, invd);
            }
            if (!ok) break;
          }
          const double c = TC_S(s, 0) * K0 + TC_S(s, 1) * K1 + TC_S(s, 2) * K2;
          double x;
          if constexpr (G <= 32)
            x = gj_solve_diag<G>(L, fa, l, n, mystep, invd, F + c * ih);
          else
            x = gj_solve<G>(L.J, L.h, l, n, mystep, invd, F + c * ih);
          K0 = (s == 0) ? x : K0;
          K1 = (s == 1) ? x : K1;
          K2 = (s == 2) ? x : K2;
          K3 = (s == 3) ? x : K3;
        }
        if (!ok) {
          status = CELL_SINGULAR;
          end = true;
        } else {
          double ynew = yl, errv = 0.0;
          ynew += TM[0] * K0;
          errv += TE[0] * K0;
          ynew += TM[1] * K1;
          errv += TE[1] * K1;
          ynew += TM[2] * K2;
          errv += TE[2] * K2;
          ynew += TM[3] * K3;
          errv += TE[3] * K3;
          double r2 = 0.0;
          if (l < n) {
            const double atol = (l == 0) ? o.atol_T : o.atol_Y;
            const double sc = atol + o.rtol * fmax(fabs(yl), fabs(ynew));
            const double rr = errv / sc;
            r2 = rr * rr;
          }
          const double err = sqrt(grp_sum<G>(r2) / n);
          // 0.9 err^(-1/3) where it is used (err positive and finite)
          const double shrink = 0.9 * exp_f64(ln_f64(err) * (-1.0 / 3.0));
          if (isfinite(err) && err <= 1.0) {
            yl = ynew;
            t = last ? dt : t + h;
            ++nacc;
            double fac = (err > 0.0) ? shrink : fac_max;
            fac = fmin(fac_max, fmax(0.2, fac));
            h *= fac;
            fac_max = 6.0;
          } else {
            ++nrej;
            double fac = isfinite(err) ? shrink : 0.2;
            fac = fmin(1.0, fmax(0.2, fac));
            h *= fac;
            fac_max = 1.0;
          }
          end = !(t < dt);
        }
      }
      if (end) {
        if (status != CELL_OK) yl = y0;
        finish();
        active = false;
        want = true;
      }
    }
  }
}

template <int G>
size_t lds_bytes(int R, int n, int cpw) {
  return (size_t)cpw * GLds<G>::doubles(R, n) * sizeof(double);
}

// LDS of one wave of k_rates, whose slices take the rate constants of all reactions.  A
// mechanism that has too many for it is refused by chem_rates whatever the batch (the
// cell-per-lane kernel could take it) and by chem_step, which a caller pairs with it.
size_t rates_lds_bytes(const chem_mech *m, int G) {
  const int cpw = 64 / G;
  return G == 16 ? lds_bytes<16>(m->R, m->d.n, cpw)
                 : (G == 32 ? lds_bytes<32>(m->R, m->d.n, cpw) : lds_bytes<64>(m->R, m->d.n, cpw));
}

chem_status check_lds(size_t sh, int *cus) {
  int dev = 0, maxsh = 0;
  CHEM_HIP(hipGetDevice(&dev));
  CHEM_HIP(hipDeviceGetAttribute(&maxsh, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
  if (cus) {
    CHEM_HIP(hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev));
    if (*cus < 1) *cus = 1;
  }
  if (sh > (size_t)maxsh) {
    set_error("mechanism needs %zu bytes of LDS per wave, the device allows %d", sh, maxsh);
    return CHEM_EUNSUPPORTED;
  }
  return CHEM_OK;
}

}  // namespace

int group_size(int n) { return n <= 16 ? 16 : (n <= 32 ? 32 : 64); }

size_t step_lds_bytes(const chem_mech *m, int G) {
  const int cpw = 64 / G;
  return (G == 16 ? lds_bytes<16>(0, m->d.n, cpw)
                  : (G == 32 ? lds_bytes<32>(0, m->d.n, cpw) : lds_bytes<64>(0, m->d.n, cpw))) +
         G * sizeof(double);
}

int max_waves_per_cu(size_t sh) {
  const int w = (int)((160 * 1024) / (sh > 0 ? sh : 1));
  return std::clamp(w, 1, 4 * STEP_WAVES_EU);
}

chem_status launch_rates(const chem_mech *m, int64_t N, int64_t ld, const double *T,
                         const double *p, const double *Y, double *wdot, double *dTdt,
                         double *kfkr, hipStream_t s) {
  const int G = group_size(m->d.n);
  const size_t sh = rates_lds_bytes(m, G);
  chem_status st = check_lds(sh, nullptr);
  if (st != CHEM_OK) return st;
  // one cell per lane from 128 blocks of 64 cells on (16 000 CH4/air cells: 22
  // against 34 us with a lane group per cell, 2^20: 0.68 against 1.60 ms);
  // below, the groups spread a batch over more waves (1000 cells: 18 against
  // 20 us, 8000: 20 against 21), and beyond the grid's limit they walk it in strides.
  if (N >= 8192 && (N + 63) / 64 * RATES_THREADS <= GRID_THREADS)
    return launch_rates_cells(m, N, ld, T, p, Y, wdot, dTdt, kfkr, s);
  const int cpw = 64 / G;
  int64_t blocks = (N + cpw - 1) / cpw;
  if (blocks > 65536) blocks = 65536;
  ProfScope prof("chem_rates", s);
  switch (G) {
    case 16:
      hipLaunchKernelGGL(k_rates<16>, dim3((unsigned)blocks), dim3(64), sh, s, m->d, N, ld, T, p,
                         Y, wdot, dTdt, kfkr);
      break;
    case 32:
      hipLaunchKernelGGL(k_rates<32>, dim3((unsigned)blocks), dim3(64), sh, s, m->d, N, ld, T, p,
                         Y, wdot, dTdt, kfkr);
      break;
    default:
      hipLaunchKernelGGL(k_rates<64>, dim3((unsigned)blocks), dim3(64), sh, s, m->d, N, ld, T, p,
                         Y, wdot, dTdt, kfkr);
      break;
  }
  CHEM_HIP(hipGetLastError());
  return CHEM_OK;
}

// Offsets of a device set table: off[s] = cells of the valid sets before s,
// off[n_sets] and *total = all of them; a set with bad sizes, null arrays or
// a bad dt counts as empty and is counted in *n_bad.  One block: each thread
// sums a contiguous run of sets, a scan over the runs, then each thread
// writes its run's offsets.
constexpr int SETOFF_THREADS = 1024;

__device__ __forceinline__ int64_t valid_cells(const chem_set &c, int *bad) {
  const bool ok = c.n >= 0 && c.ld >= c.n &&
                  (c.n == 0 || (c.T && c.p && c.Y && c.dt > 0.0 && isfinite(c.dt)));
  *bad = ok ? 0 : 1;
  return ok ? c.n : 0;
}

__global__ __launch_bounds__(SETOFF_THREADS) void k_set_offsets(const chem_set *sets, int n_sets,
                                                                 int64_t *off,
                                                                 unsigned long long *total,
                                                                 int32_t *n_bad) {
  __shared__ int64_t run[SETOFF_THREADS];
  __shared__ int bads[SETOFF_THREADS];
  const int t = threadIdx.x;
  const int per = (n_sets + SETOFF_THREADS - 1) / SETOFF_THREADS;
  const int s0 = t * per, s1 = s0 + per < n_sets ? s0 + per : n_sets;
  int64_t sum = 0;
  int nb = 0;
  for (int i = s0; i < s1; ++i) {
    int b = 0;
    sum += valid_cells(sets[i], &b);
    nb += b;
  }
  run[t] = sum;
  bads[t] = nb;
  __syncthreads();
  if (t == 0) {  // exclusive scan of the runs, in order
    int64_t acc = 0;
    int nbad = 0;
    for (int q = 0; q < SETOFF_THREADS; ++q) {
      const int64_t v = run[q];
      run[q] = acc;
      acc += v;
      nbad += bads[q];
    }
    off[n_sets] = acc;
    *total = (unsigned long long)acc;
    if (n_bad) *n_bad = nbad;
  }
  __syncthreads();
  int64_t acc = run[t];
  for (int i = s0; i < s1; ++i) {
    off[i] = acc;
    int b = 0;
    acc += valid_cells(sets[i], &b);
  }
}

chem_status launch_set_offsets(const chem_set *sets, int n_sets, int64_t *off,
                               unsigned long long *total, int32_t *n_bad, hipStream_t s) {
  hipLaunchKernelGGL(k_set_offsets, dim3(1), dim3(SETOFF_THREADS), 0, s, sets, n_sets, off,
                     total, n_bad);
  CHEM_HIP(hipGetLastError());
  return CHEM_OK;
}

chem_status launch_step(const chem_mech *m, int64_t N, int64_t ld, double dt,
                        const double *dt_cell, double *T, const double *p, double *Y, double *RR,
                        double *h_hint, int32_t *stats, const StepOpts &o, const int32_t *index,
                        hipStream_t s, const unsigned long long *n_dev, uint8_t *flags,
                        const chem_set *sets, const int64_t *set_off, int n_sets,
                        unsigned long long *queue) {
  StepArgs A{N,     ld,    dt,    dt_cell, T,    p,       Y,      RR,
             h_hint, stats, index, o,       queue ? queue : m->counters, n_dev, flags, sets,
             set_off, n_sets};
  const int G = m->tune_G ? m->tune_G : group_size(m->d.n);
  const int cpw = 64 / G;
  const size_t sh = step_lds_bytes(m, G);
  int cus = 0;
  chem_status st = check_lds(std::max(sh, rates_lds_bytes(m, G)), &cus);
  if (st != CHEM_OK) return st;
  // persistent grid: the single-wave blocks that a CU's LDS and registers hold, or the tuned
  // number of waves per CU
  int per_cu = max_waves_per_cu(sh);
  if (m->tune_waves > 0 && m->tune_waves < per_cu) per_cu = m->tune_waves;
  int64_t want = (N + cpw - 1) / cpw;  // with n_dev, N is an upper bound
  int64_t blocks = (int64_t)cus * per_cu;
  if (blocks > want) blocks = want;
  if (blocks < 1) return CHEM_OK;
  if (!queue) hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(64), 0, s, m->counters);
  ProfScope prof(index ? "chem_step_fallback" : (sets ? "chem_step_sets" : "chem_step"), s);
  switch (G) {
    case 16:
      hipLaunchKernelGGL(k_step<16>, dim3((unsigned)blocks), dim3(64), sh, s, m->d, A);
      break;
    case 32:
      hipLaunchKernelGGL(k_step<32>, dim3((unsigned)blocks), dim3(64), sh, s, m->d, A);
      break;
    default:
      hipLaunchKernelGGL(k_step<64>, dim3((unsigned)blocks), dim3(64), sh, s, m->d, A);
      break;
  }
  CHEM_HIP(hipGetLastError());
  return CHEM_OK;
}

}  // namespace chem
