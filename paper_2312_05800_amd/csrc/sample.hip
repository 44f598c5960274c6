// Training-set sampler (the random-data generation of Sec. 3.1) on the GPU:
// every seed state is perturbed by Eqs. (Trand)-(Yrand) with the seed set's
// ranges and renormalised with N2 held at its perturbed value, or replaced by
// a state on the line between two given end states; each sample is then
// tested against the temperature threshold and the element-ratio limits of
// Table 1.  One thread per sample; the ranges come from an exact min/max
// reduction over the seeds first.
#include <math.h>

#include <algorithm>

#include "chem_internal.h"

namespace chem {
namespace {

constexpr int RANGE_BLOCKS = 512;
constexpr int RANGE_THREADS = 256;

// partial min/max of T, p and y_N2 per block: part[b][6] =
// (min T, max T, min p, max p, min y_N2, max y_N2)
__global__ void k_ranges_part(int64_t n, int64_t ld, const double *T, const double *p,
                              const double *Y, int n2, double *part) {
  __shared__ double red[6][RANGE_THREADS];
  double v[6] = {INFINITY, -INFINITY, INFINITY, -INFINITY, INFINITY, -INFINITY};
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double t = T[i], q = p[i], y = Y[(int64_t)n2 * ld + i];
    v[0] = fmin(v[0], t);
    v[1] = fmax(v[1], t);
    v[2] = fmin(v[2], q);
    v[3] = fmax(v[3], q);
    v[4] = fmin(v[4], y);
    v[5] = fmax(v[5], y);
  }
  for (int q = 0; q < 6; ++q) red[q][threadIdx.x] = v[q];
  __syncthreads();
  for (int off = RANGE_THREADS / 2; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off)
      for (int q = 0; q < 6; ++q) {
        const double a = red[q][threadIdx.x], b = red[q][threadIdx.x + off];
        red[q][threadIdx.x] = (q & 1) ? fmax(a, b) : fmin(a, b);
      }
    __syncthreads();
  }
  if (threadIdx.x < 6) part[blockIdx.x * 6 + threadIdx.x] = red[threadIdx.x][0];
}

// One wave per quantity: 64 lanes take the partials in turn, then meet in
// shuffles (a single lane's loop over 512 partials took longer than the
// samples of a small batch).
__global__ __launch_bounds__(6 * 64) void k_ranges_fin(const double *part, int nparts,
                                                       double *out) {
  const int q = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double v = (q & 1) ? -INFINITY : INFINITY;
  for (int b = lane; b < nparts; b += 64) {
    const double x = part[b * 6 + q];
    v = (q & 1) ? fmax(v, x) : fmin(v, x);
  }
  for (int off = 32; off > 0; off >>= 1) {
    const double x = __shfl_xor(v, off);
    v = (q & 1) ? fmax(v, x) : fmin(v, x);
  }
  if (lane == 0) out[q] = v;
}

struct SampleArgs {
  int64_t n, ld;
  int64_t i0;  // the launch's first sample
  const double *T, *p, *Y;   // seeds
  const double *c;           // [K + 3][ld] uniform in [-1, 1]
  const double *s;           // [ld] mixing fraction (< 0: perturb), nullable
  const double *end_eq, *end_air;  // [K + 2]: T, p, Y_1..K
  const double *ranges;      // [6] from k_ranges_fin
  double *To, *po, *Yo;
  uint8_t *keep;
  chem_sample_opts o;
};

// 1 + gamma c of Eq. (Yrand), the product rounded: where |ln y| is large, the
// last bit of the exponent is most of the power's error.
__device__ __forceinline__ double exponent(double gamma, double c) {
#pragma clang fp contract(off)
  return 1.0 + gamma * c;
}

// KP >= K: species slots per sample.  One pass over the species: the chunk's
// loads (Y and c of eight species) go out together and the raw values stay in
// registers until the sum that scales them is known, so that Y and c are read
// once and Y_out is written once.  2^20 states of 30 species: 275 us, where the
// scaling read the raw values back from Y_out 604.  The power is the library's: y times
// the exponential of gamma c ln y from a plain FP64 logarithm took 250 us, and its largest
// error was past an ulp of the power (see the accuracy test; over whole samples 26.4
// units of 2^-53 instead of 24.9).
template <int KP>
__global__ __launch_bounds__(256) void k_sample(DevMech M, SampleArgs a) {
  constexpr int CHK = 8;
  const int K = M.K, n2 = a.o.n2;
  const int64_t ld = a.ld;
  const int64_t i = a.i0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const double s = a.s ? a.s[i] : -1.0;
  const bool line = s >= 0.0;  // a state on the line between the two ends
  const double cT = a.c[i], cp = a.c[ld + i], cn = a.c[2 * ld + i];
  const double T0 = a.T[i], p0 = a.p[i];
  double v[KP];
  double sum = 0.0, yn2 = 0.0;
#pragma unroll
  for (int k0 = 0; k0 < KP; k0 += CHK) {
    if (k0 >= K) break;
    double y[CHK], c[CHK];
#pragma unroll
    for (int t = 0; t < CHK; ++t) {
      const int k = min(k0 + t, K - 1);
      y[t] = a.Y[(int64_t)k * ld + i];
      c[t] = a.c[(int64_t)(3 + k) * ld + i];
    }
#pragma unroll
    for (int t = 0; t < CHK; ++t) {
      const int k = k0 + t;
      v[k] = 0.0;
      if (k < K) {
        if (k == n2) {
          yn2 = y[t];
        } else {
          // Eq. (Yrand)
          v[k] = y[t] > 0.0 ? pow(y[t], exponent(a.o.gamma, c[t])) : 0.0;
          sum += v[k];
        }
      }
    }
  }
  const double *r = a.ranges;
  // Eqs. (Trand), (Prand), (N2rand)
  double T = T0 + a.o.alpha * cT * (r[1] - r[0]);
  double p = p0 + a.o.beta * cp * (r[3] - r[2]);
  yn2 += a.o.alpha * cn * (r[5] - r[4]);
  // every species but N2 rescaled so that the mass fractions sum to one
  const double scale = (1.0 - yn2) / sum;
  if (a.s) {
    T = line ? (1.0 - s) * a.end_eq[0] + s * a.end_air[0] : T;
    p = line ? (1.0 - s) * a.end_eq[1] + s * a.end_air[1] : p;
  }
  a.To[i] = T;
  a.po[i] = p;
  // element moles per kg, the ratios of Table 1 and the equivalence ratio
  // (2 n_C + n_H / 2) / n_O
  double nC = 0.0, nH = 0.0, nO = 0.0, nN = 0.0, yn2o = 0.0;
  bool ok = isfinite(T) && T >= a.o.T_min;
#pragma unroll
  for (int k = 0; k < KP; ++k) {
    if (k < K) {
      double y = k == n2 ? yn2 : v[k] * scale;
      if (a.s) {
        const double yl = (1.0 - s) * a.end_eq[2 + k] + s * a.end_air[2 + k];
        y = line ? yl : y;
      }
      a.Yo[(int64_t)k * ld + i] = y;
      if (k == n2) yn2o = y;
      ok = ok && isfinite(y) && y >= 0.0;
      // moles per kg (a non-finite y has cleared `ok`, whatever 0 y gives)
      const double x = y * M.invW[k];
      nC = fma(M.compd[a.o.el_C * K + k], x, nC);
      nH = fma(M.compd[a.o.el_H * K + k], x, nH);
      nO = fma(M.compd[a.o.el_O * K + k], x, nO);
      nN = fma(M.compd[a.o.el_N * K + k], x, nN);
    }
  }
  ok = ok && yn2o >= 0.0 && yn2o < 1.0;
  const double hc = nH / nC, on = nO / nN, phi = (2.0 * nC + 0.5 * nH) / nO;
  ok = ok && isfinite(hc) && hc >= a.o.hc_min && hc <= a.o.hc_max;
  ok = ok && isfinite(on) && on >= a.o.on_min && on <= a.o.on_max;
  ok = ok && isfinite(phi) && phi >= a.o.phi_min && phi <= a.o.phi_max;
  a.keep[i] = ok ? 1 : 0;
}

}  // namespace
}  // namespace chem

using namespace chem;

extern "C" chem_status chem_sample_states(const chem_mech *m, chem_batch seeds, const double *T,
                                          const double *p, const double *Y, const double *c,
                                          const double *s, const double *end_eq,
                                          const double *end_air, const chem_sample_opts *opts,
                                          double *T_out, double *p_out, double *Y_out,
                                          uint8_t *keep, void *stream) {
  if (!m || !opts) {
    set_error("chem_sample_states: null mechanism or options");
    return CHEM_EINVAL;
  }
  const int64_t n = seeds.n;
  if (n < 0 || seeds.ld < n || n > ((int64_t)1 << 40)) {
    set_error("chem_sample_states: bad batch n=%lld ld=%lld", (long long)n, (long long)seeds.ld);
    return CHEM_EINVAL;
  }
  const chem_sample_opts &o = *opts;
  if (o.n2 < 0 || o.n2 >= m->K) {
    set_error("chem_sample_states: N2 index %d outside the %d species", o.n2, m->K);
    return CHEM_EINVAL;
  }
  const int el[4] = {o.el_C, o.el_H, o.el_O, o.el_N};
  for (int a = 0; a < 4; ++a) {
    if (el[a] < 0 || el[a] >= m->E) {
      set_error("chem_sample_states: element index %d outside the %d elements", el[a], m->E);
      return CHEM_EINVAL;
    }
    for (int b = 0; b < a; ++b)
      if (el[a] == el[b]) {
        set_error("chem_sample_states: the C, H, O and N element indices must differ");
        return CHEM_EINVAL;
      }
  }
  if (!(o.alpha >= 0.0) || !(o.beta >= 0.0) || !(o.gamma >= 0.0) || !isfinite(o.T_min)) {
    set_error("chem_sample_states: alpha, beta, gamma must be >= 0 and T_min finite");
    return CHEM_EINVAL;
  }
  if (n == 0) return CHEM_OK;
  if (!T || !p || !Y || !c || !T_out || !p_out || !Y_out || !keep ||
      (s && (!end_eq || !end_air))) {
    set_error("chem_sample_states: null array (the end states are needed with s)");
    return CHEM_EINVAL;
  }
  if (!m->sample_buf) {
    const hipError_t e = hipMalloc((void **)&((chem_mech *)m)->sample_buf,
                                   (size_t)(RANGE_BLOCKS * 6 + 8) * sizeof(double));
    if (e != hipSuccess) {
      set_error("chem_sample_states: cannot allocate the range buffer");
      return CHEM_ENOMEM;
    }
  }
  hipStream_t st = (hipStream_t)stream;
  double *part = m->sample_buf, *ranges = m->sample_buf + RANGE_BLOCKS * 6;
  ProfScope prof("sample_states", st);
  const int64_t rows = (n + RANGE_THREADS - 1) / RANGE_THREADS;
  const int parts = (int)(rows < RANGE_BLOCKS ? rows : RANGE_BLOCKS);
  hipLaunchKernelGGL(k_ranges_part, dim3(parts), dim3(RANGE_THREADS), 0, st, n, seeds.ld, T, p, Y,
                     o.n2, part);
  hipLaunchKernelGGL(k_ranges_fin, dim3(1), dim3(6 * 64), 0, st, part, parts, ranges);
  SampleArgs a{n, seeds.ld, 0, T, p, Y, c, s, end_eq, end_air, ranges, T_out, p_out, Y_out,
               keep, o};
  // 2^31 samples a launch, whose grid has fewer than 2^32 threads (a loop over the grid in
  // the kernel took 375 us instead of 275 at 2^20)
  constexpr int64_t LAUNCH = (int64_t)1 << 31;
  for (; a.i0 < n; a.i0 += LAUNCH) {
    const dim3 grid((unsigned)((std::min(n - a.i0, LAUNCH) + 255) / 256)), block(256);
    if (m->K <= 16)
      hipLaunchKernelGGL(k_sample<16>, grid, block, 0, st, m->d, a);
    else if (m->K <= 32)
      hipLaunchKernelGGL(k_sample<32>, grid, block, 0, st, m->d, a);
    else
      hipLaunchKernelGGL(k_sample<64>, grid, block, 0, st, m->d, a);
  }
  CHEM_HIP(hipGetLastError());
  return CHEM_OK;
}
