// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <string>

#include "chemstep.h"

namespace chem {

constexpr int KMAX = 63;  // species limit: n = K + 1 <= 64 lanes per cell

// Device-resident mechanism constants (one allocation, see chem_api.hip).
struct RxnPack;
struct SpPack;
struct PostPack;
struct DevMech {
  int K, R, E, n;
  const double *W;        // [K] kg/mol
  const double *invW;     // [K]
  const double *Tmid;     // [K]
  const double *nasa_h;   // [K][7] low-range h/RT polynomial: a1, a2/2, a3/3, a4/4, a5/5, a6, 0
  const double *nasa_hh;  // [K][7] same for the high range
  const double *compd;    // [E][K] atoms of element e in species k
  const double *cpT;      // [2][7][K] the c_p/R, h/RT and s/R polynomials (divisors folded
  const double *hT;       //   in), low range then high range, coefficient-major
  const double *sT;
  // the integrator's lane groups: component c >= 1 is species order[c - 1] (see
  // species_order); the reactions in the order of their passes (see pass_order),
  // slots by component (0 = empty)
  const int *order;    // [K]
  const int4 *xsp;     // [R]
  const double2 *xab;  // [R] ln A, b
  const double2 *xeb;  // [R] E_a/R, bits: coefficients (2 bits per slot), from bit 16 the
                       //   reaction's index
  // k_rates_cells: the species (tp [K]), the reactions (rx, R rounded up to a
  // multiple of RATES_PER_WAVE by null reactions), and per chunk of RATES_CHUNK reactions and species, the
  // reactions that the species takes part in: entries rs_start[chunk K + k] ..
  // rs_start[chunk K + k + 1], a multiple of four of them (padded with the zero row),
  // each a reaction's row in the chunk and the species' net coefficient
  const SpPack *tp;
  const RxnPack *rx;
  const int *rs_start;
  const int *rs_row;
  const double *rs_coef;
  const PostPack *pp;  // [KMAX + 1], the entries past K null species
};
constexpr int RATES_CHUNK = 32, RATES_PER_WAVE = 4;
constexpr int RATES_THREADS = 64 * (RATES_CHUNK / RATES_PER_WAVE);  // for 64 cells
// threads a launch may have in the x direction of its grid
constexpr int64_t GRID_THREADS = ((int64_t)1 << 32) - 1;

// What k_rates_cells reads of a reaction, contiguous for the scalar cache.
struct RxnPack {
  // species of slots reactant0, reactant1, product0, product1 and their
  // coefficients; an empty slot names the dummy species K with coefficient 0 (C = 1
  // and h = g = 0 are kept for it, so it drops out of every product and sum without
  // a branch), a null reaction has all slots empty
  int sp[4], nu[4];
  double cf[4];      // net coefficients: minus the reactants', plus the products'
  double lnA, b, EaR, dn;
};
// The same of a species: the c_p/R (5), h/RT (6) and s/R (6) polynomials of
// the low and the high range.
struct SpPack {
  double c[2][17];
  double Tmid, invW;
};

// What the surrogate's post-processing reads of a species: h/RT of the low range, 1/W and the
// range limit; h/RT of the high range and two elements' mass per unit mass
// fraction; the other elements'.  Three cache lines; a null species is all zeros
// with Tmid = infinity.
struct PostPack {
  double lo[6], invW, Tmid;
  double hi[6], el[10];
};

// A constant kept in scalar registers: the FMA takes it as an operand
// instead of a copy of it in vector registers that each use overwrites.
__device__ __forceinline__ double scalar_const(double c) {
  asm("" : "+s"(c));
  return c;
}

// e^x: x = n ln 2 + r with |r| <= ln 2 / 2, 1 + r + r^2 P(r) with P the Chebyshev
// interpolant of degree 9 of (e^r - 1 - r) / r^2 (relative error 1.6e-17 before
// rounding), scaled by 2^n.  Above 1024 infinity, below -1075 zero, NaN stays
// NaN.  24 vector instructions where the library's exp, whose
// coefficients are copied into vector registers at every use, takes about 40.
__device__ __forceinline__ double exp_f64(double x) {
  const double n = __builtin_rint(x * scalar_const(1.4426950408889634));
  double r = __builtin_fma(n, scalar_const(-0.69314718055994529), x);
  r = __builtin_fma(n, scalar_const(-2.3190468138462996e-17), r);
  double p = __builtin_fma(r, scalar_const(2.5100375832561234e-08),
                           scalar_const(2.7620075879983367e-07));
  p = __builtin_fma(r, p, scalar_const(2.7557268480310024e-06));
  p = __builtin_fma(r, p, scalar_const(2.4801521322368692e-05));
  p = __builtin_fma(r, p, scalar_const(0.00019841269863040545));
  p = __builtin_fma(r, p, scalar_const(0.0013888888917196719));
  p = __builtin_fma(r, p, scalar_const(0.008333333333330065));
  p = __builtin_fma(r, p, scalar_const(0.041666666666624164));
  p = __builtin_fma(r, p, scalar_const(0.16666666666666669));
  p = __builtin_fma(r, p, scalar_const(0.50000000000000011));
  p = __builtin_fma(r, p, 1.0);
  p = __builtin_fma(r, p, 1.0);
  p = __builtin_amdgcn_ldexp(p, (int)n);
  p = x > scalar_const(1024.0) ? INFINITY : p;
  return x < scalar_const(-1075.0) ? 0.0 : p;
}

// ln x of a finite positive x: x = 2^e m with m in [1/sqrt 2, sqrt 2),
// ln m = 2 atanh(s) = 2 s + s z P(z) with s = (m - 1) / (m + 1), z = s^2 and P the
// Chebyshev interpolant of degree 6 (relative error 4.2e-18 before rounding).
__device__ __forceinline__ double ln_f64(double x) {
  double m = __builtin_amdgcn_frexp_mant(x);
  int e = __builtin_amdgcn_frexp_exp(x);
  const bool up = m < 0.70710678118654752;
  m = up ? 2.0 * m : m;
  e = up ? e - 1 : e;
  // the quotient by Newton's reciprocal (the divisor is in [1.7, 2.5])
  const double num = m - 1.0, den = m + 1.0;
  double r = __builtin_amdgcn_rcp(den);
  r = fma(fma(-den, r, 1.0), r, r);
  r = fma(fma(-den, r, 1.0), r, r);
  double s = num * r;
  s = fma(fma(-den, s, num), r, s);
  const double z = s * s;
  double P = fma(z, scalar_const(0.14617807153417325), scalar_const(0.15331611722055008));
  P = fma(z, P, scalar_const(0.18182892432536871));
  P = fma(z, P, scalar_const(0.22222211089379496));
  P = fma(z, P, scalar_const(0.28571428626253836));
  P = fma(z, P, scalar_const(0.39999999999898889));
  P = fma(z, P, scalar_const(0.66666666666666696));
  const double k = (double)e;
  const double lo = fma(s * z, P, k * scalar_const(2.3190468138462996e-17));
  return fma(k, scalar_const(0.69314718055994529), fma(2.0, s, lo));
}

struct StepOpts {
  double rtol, atol_Y, atol_T, h0, h_min;
  int max_steps;
};

}  // namespace chem

struct chem_mech {
  chem::DevMech d;
  void *blob;                      // device allocation behind d
  unsigned long long *counters;    // device work-queue counters
  void *set_buf = nullptr;         // device copy of the last chem_step_sets table
  size_t set_cap = 0;
  void *dset_buf = nullptr;        // offsets and count of chem_step_sets_device's table
  size_t dset_cap = 0;
  double *sample_buf = nullptr;    // training-set sampler: range partials and ranges
  int device;
  int K, R, E;
  // integrator launch shape (0 = default heuristic), set by chem_autotune or
  // chem_set_tuning
  int tune_G = 0, tune_waves = 0;
  double tune_cps = 0.0;
  uint64_t digest = 0;  // FNV-1a of the packed tables (keys the tuning cache)
};

// A captured step: the graph, its executable and the stream it was captured
// on; `release` (if set) runs at destruction (returns the model's workspace
// to growable).
struct chem_graph {
  hipGraph_t g = nullptr;
  hipGraphExec_t e = nullptr;
  hipStream_t s = nullptr;
  void (*release)(void *) = nullptr;
  void *owner = nullptr;
};

namespace chem {

// Brackets the launches issued during its lifetime with HIP events on stream
// s when launch timing is enabled (chem_profile_enable); no-op otherwise.
class ProfScope {
 public:
  ProfScope(const char *label, hipStream_t s);
  ~ProfScope();
  ProfScope(const ProfScope &) = delete;
  ProfScope &operator=(const ProfScope &) = delete;

 private:
  const char *label_;
  hipStream_t s_;
  void *a_ = nullptr, *b_ = nullptr;
  bool on_ = false;
};

void set_error(const char *fmt, ...);

// Tuning results kept between runs in the text file named by the environment
// variable CHEM_AUTOTUNE_CACHE (no file: nothing is kept): one line
// "key = value" per tuned problem, the last write of a key winning.
// The version in the keys is that of the kernels the results were measured on: raised with a
// change of k_step or of the training products, so that older results are measured again.
constexpr int TUNE_VERSION = 2;
bool tune_cache_get(const std::string &key, std::string *value);
void tune_cache_put(const std::string &key, const std::string &value);
// The current device's architecture name and compute-unit count, for keys.
std::string tune_device_key();
uint64_t fnv1a(const void *p, size_t n, uint64_t h = 1469598103934665603ull);

// ProfScope is a no-op while suspended (graph capture).
void profile_suspend(bool on);

chem_status hip_fail(hipError_t e, const char *what);

// Records body(stream) on a fresh stream (default priority) into a HIP graph
// and instantiates it; launch timing is suspended meanwhile.  On failure
// nothing is left behind.
template <typename F>
chem_status capture_graph(F &&body, chem_graph **out) {
  if (!out) {
    set_error("graph: null output handle");
    return CHEM_EINVAL;
  }
  *out = nullptr;
  chem_graph *cg = new chem_graph();
  hipError_t e = hipStreamCreateWithFlags(&cg->s, hipStreamNonBlocking);
  if (e != hipSuccess) {
    delete cg;
    return hip_fail(e, "graph: hipStreamCreateWithFlags");
  }
  chem_status st = CHEM_OK;
  profile_suspend(true);
  e = hipStreamBeginCapture(cg->s, hipStreamCaptureModeThreadLocal);
  if (e == hipSuccess) {
    st = body(cg->s);
    const hipError_t e2 = hipStreamEndCapture(cg->s, &cg->g);
    if (st == CHEM_OK && e2 != hipSuccess) st = hip_fail(e2, "graph: hipStreamEndCapture");
    if (st == CHEM_OK) {
      const hipError_t e3 = hipGraphInstantiate(&cg->e, cg->g, nullptr, nullptr, 0);
      if (e3 != hipSuccess) st = hip_fail(e3, "graph: hipGraphInstantiate");
    }
  } else {
    st = hip_fail(e, "graph: hipStreamBeginCapture");
  }
  profile_suspend(false);
  if (st != CHEM_OK) {
    if (cg->e) (void)hipGraphExecDestroy(cg->e);
    if (cg->g) (void)hipGraphDestroy(cg->g);
    (void)hipStreamDestroy(cg->s);
    delete cg;
    return st;
  }
  *out = cg;
  return CHEM_OK;
}

#define CHEM_HIP(call)                                   \
  do {                                                   \
    hipError_t e_ = (call);                              \
    if (e_ != hipSuccess) return chem::hip_fail(e_, #call); \
  } while (0)

StepOpts resolve_opts(const chem_step_opts *o);

// launchers (chem_kernels.hip)
chem_status launch_rates(const chem_mech *m, int64_t n, int64_t ld, const double *T,
                         const double *p, const double *Y, double *wdot, double *dTdt,
                         double *kfkr, hipStream_t s);
// the same, one cell per lane (rates.hip)
chem_status launch_rates_cells(const chem_mech *m, int64_t n, int64_t ld, const double *T,
                               const double *p, const double *Y, double *wdot, double *dTdt,
                               double *kfkr, hipStream_t s);
// smallest lane group (16, 32 or 64) that holds n = K + 1 components
int group_size(int n);
// LDS bytes of one integrator wavefront with G lanes per cell
size_t step_lds_bytes(const chem_mech *m, int G);
// resident integrator wavefronts per CU: what the LDS allows, at most two a SIMD (k_step is
// compiled for that many, and takes all of their registers)
constexpr int STEP_WAVES_EU = 2;
int max_waves_per_cu(size_t sh);
// queue: the cell queue's counter, cleared by the caller; null: the mechanism's own, cleared
// by a launch before the integrator's.
chem_status launch_step(const chem_mech *m, int64_t n, int64_t ld, double dt,
                        const double *dt_cell, double *T, const double *p, double *Y,
                        double *RR, double *h_hint, int32_t *stats, const StepOpts &o,
                        const int32_t *index, hipStream_t s,
                        const unsigned long long *n_dev = nullptr, uint8_t *flags = nullptr,
                        const chem_set *sets = nullptr, const int64_t *set_off = nullptr,
                        int n_sets = 0, unsigned long long *queue = nullptr);
// Offsets and total cell count of a device set table (see k_set_offsets).
chem_status launch_set_offsets(const chem_set *sets, int n_sets, int64_t *off,
                               unsigned long long *total, int32_t *n_bad, hipStream_t s);

}  // namespace chem
