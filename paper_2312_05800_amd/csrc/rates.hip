// Instantaneous chemistry of many cells, one cell per lane.  A block of eight
// waves owns 64 consecutive cells, so every load and store instruction moves
// one row of 64 cells (512 contiguous bytes).  The waves share the work of a
// cell: wave w evaluates the thermodynamics of its species and every eighth
// reaction; concentrations and g/RT go through LDS ([species][lane], free of
// bank conflicts), and so do the rates of progress, a chunk of RATES_CHUNK
// reactions at a time, from which each wave adds the production rates of its
// own species in registers: a fixed order, no atomics.  What is uniform over
// the wave (the reaction, its species and constants) stays in scalar
// registers.
//
// Bound: the vector pipe (two exponentials and about 30 further operations
// per reaction and cell; 64 % of the cycles issue one, the rest is the
// barriers between chunks).  2^20 CH4/air cells: 0.68 ms, where one cell per
// 32-lane group (16 useful bytes per line and load, LDS atomics for the sums)
// took 1.60 ms.  Chunks of 32: four reactions per wave between barriers, and
// two chunk buffers leave two blocks per CU their LDS.
#include <math.h>

#include "chem_internal.h"

namespace chem {
namespace {

constexpr double RG = 8.314462618;
constexpr double PREF = 101325.0;
constexpr int RC_WAVES = RATES_THREADS / 64;

// constants through the scalar cache: the index is wave-uniform and nothing
// writes the tables while a kernel runs
template <typename T>
using cptr = const __attribute__((address_space(4))) T *;
template <typename T>
__device__ __forceinline__ cptr<T> uni(const T *p) {
  return (cptr<T>)(uintptr_t)p;
}

struct RatesArgs {
  int64_t n, ld;
  const double *T, *p, *Y;
  double *wdot, *dTdt, *kfkr;
};

// J: species per wave (species w J + j of wave w)
template <int J>
__global__ __launch_bounds__(RATES_THREADS) void k_rates_cells(DevMech M, RatesArgs a) {
  constexpr int KP = J * RC_WAVES, CH = RATES_CHUNK, PW = RATES_PER_WAVE;
  __shared__ double2 cg[KP + 1][64];   // (C, g/RT) of the species, then the empty slots' dummy
  __shared__ double q[2][CH + 1][64];  // rates of progress; row CH is zero
  __shared__ double red[3][RC_WAVES][64];
  const int K = M.K, R = M.R;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const int64_t c0 = (int64_t)blockIdx.x * 64;
  const bool live = c0 + lane < a.n;
  const int64_t cell = live ? c0 + lane : a.n - 1;
  const double T = a.T[cell], p = a.p[cell];
  double y[J], h[J], g[J];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int k = w * J + j;
    y[j] = k < K ? a.Y[(int64_t)k * a.ld + cell] : 0.0;
  }
  if (w < 2) q[w][CH][lane] = 0.0;
  if (w == 2) cg[K][lane] = make_double2(1.0, 0.0);
  const double lnT = log(T), invT = 1.0 / T;
  const double lnPRT = log(PREF / RG) - lnT;
  double S = 0.0, cp = 0.0;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int k = w * J + j;
    h[j] = g[j] = 0.0;
    if (k >= K) continue;
    const cptr<SpPack> t = uni(M.tp) + k;
    const bool low = T <= t->Tmid;
    double cv = 0.0;
    // the polynomials of a range; both are evaluated where the wave's cells
    // lie on either side of the species' T_mid
    auto range = [&](int o, bool mine) __attribute__((always_inline)) {
      double c[17];
#pragma unroll
      for (int i = 0; i < 17; ++i) c[i] = scalar_const(t->c[o][i]);
      const double *hc = c + 5, *sc = c + 11;
      const double cpR = c[0] + T * (c[1] + T * (c[2] + T * (c[3] + T * c[4])));
      const double hRT =
          hc[0] + T * (hc[1] + T * (hc[2] + T * (hc[3] + T * hc[4]))) + hc[5] * invT;
      const double sR =
          sc[0] * lnT + T * (sc[1] + T * (sc[2] + T * (sc[3] + T * sc[4]))) + sc[5];
      cv = mine ? cpR : cv;
      h[j] = mine ? hRT : h[j];
      g[j] = mine ? hRT - sR : g[j];
    };
    if (__any(low)) range(0, low);
    if (!__all(low)) range(1, !low);
    const double iw = t->invW;
    S += y[j] * iw;
    cp += y[j] * RG * cv * iw;
  }
  red[0][w][lane] = S;
  red[1][w][lane] = cp;
  __syncthreads();
  S = cp = 0.0;
#pragma unroll
  for (int v = 0; v < RC_WAVES; ++v) {
    S += red[0][v][lane];
    cp += red[1][v][lane];
  }
  const double rho = p / (RG * T * S);
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int k = w * J + j;
    if (k < K) cg[k][lane] = make_double2(rho * y[j] * (uni(M.tp) + k)->invW, g[j]);
  }
  __syncthreads();
  double wd[J];
#pragma unroll
  for (int j = 0; j < J; ++j) wd[j] = 0.0;
  const int nch = (R + CH - 1) / CH;
  for (int ch = 0; ch < nch; ++ch) {
    double(*const qb)[64] = q[ch & 1];
    const int r0 = ch * CH + PW * w;
    if (r0 < R) {
#pragma unroll
      for (int i = 0; i < PW; ++i) {
        const cptr<RxnPack> x = uni(M.rx) + r0 + i;
        const double2 a0 = cg[x->sp[0]][lane], a1 = cg[x->sp[1]][lane], a2 = cg[x->sp[2]][lane],
                      a3 = cg[x->sp[3]][lane];
        const double dG = x->cf[0] * a0.y + x->cf[1] * a1.y + x->cf[2] * a2.y + x->cf[3] * a3.y;
        const double lnkf = x->lnA + x->b * lnT - x->EaR * invT;
        const double kf = exp_f64(lnkf);
        const double kr = exp_f64(lnkf + dG - x->dn * lnPRT);
        auto fac = [](int n, double c) { return c * (n == 2 ? c : 1.0); };
        qb[PW * w + i][lane] = kf * fac(x->nu[0], a0.x) * fac(x->nu[1], a1.x) -
                               kr * fac(x->nu[2], a2.x) * fac(x->nu[3], a3.x);
        if (a.kfkr && live && r0 + i < R) {
          a.kfkr[(int64_t)(r0 + i) * a.ld + cell] = kf;
          a.kfkr[(int64_t)(R + r0 + i) * a.ld + cell] = kr;
        }
      }
    }
    // publishes the chunk; the buffer it will be overwritten in is two chunks
    // on, behind the next barrier
    __syncthreads();
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int k = w * J + j;
      if (k >= K) continue;
      const cptr<int> st = uni(M.rs_start) + ch * K + k;
      for (int e = st[0]; e < st[1]; e += 4) {
        const cptr<int> row = uni(M.rs_row) + e;
        const cptr<double> cf = uni(M.rs_coef) + e;
        const double q0 = qb[row[0]][lane], q1 = qb[row[1]][lane], q2 = qb[row[2]][lane],
                     q3 = qb[row[3]][lane];
        wd[j] = fma(cf[0], q0, wd[j]);
        wd[j] = fma(cf[1], q1, wd[j]);
        wd[j] = fma(cf[2], q2, wd[j]);
        wd[j] = fma(cf[3], q3, wd[j]);
      }
    }
  }
  double Q = 0.0;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int k = w * J + j;
    if (k >= K) continue;
    Q += RG * T * h[j] * wd[j];
    if (live) a.wdot[(int64_t)k * a.ld + cell] = wd[j];
  }
  if (a.dTdt) {
    red[2][w][lane] = Q;
    __syncthreads();
    if (w == 0) {
      Q = 0.0;
#pragma unroll
      for (int v = 0; v < RC_WAVES; ++v) Q += red[2][v][lane];
      if (live) a.dTdt[cell] = -Q / (rho * cp);
    }
  }
}

}  // namespace

chem_status launch_rates_cells(const chem_mech *m, int64_t N, int64_t ld, const double *T,
                               const double *p, const double *Y, double *wdot, double *dTdt,
                               double *kfkr, hipStream_t s) {
  RatesArgs a{N, ld, T, p, Y, wdot, dTdt, kfkr};
  const dim3 grid((unsigned)((N + 63) / 64)), block(RATES_THREADS);
  ProfScope prof("chem_rates", s);
  const int K = m->d.K;
  if (K <= 2 * RC_WAVES)
    hipLaunchKernelGGL(k_rates_cells<2>, grid, block, 0, s, m->d, a);
  else if (K <= 4 * RC_WAVES)
    hipLaunchKernelGGL(k_rates_cells<4>, grid, block, 0, s, m->d, a);
  else
    hipLaunchKernelGGL(k_rates_cells<8>, grid, block, 0, s, m->d, a);
  CHEM_HIP(hipGetLastError());
  return CHEM_OK;
}

}  // namespace chem
