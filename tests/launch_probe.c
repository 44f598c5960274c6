/* Calls the library with a HIP runtime of its own that only records the launches, so that the
 * launch shapes of batches no host could hold can be checked without a GPU.  Test code only.
 *   launch_probe LIB LDS_BYTES REACTIONS {rates|sample|step|autotune|autotune_train} N...
 * prints per N a line "call N STATUS" after its launches, "KERNEL gx gy gz bx by bz" each.
 * Time, as events see it, passes by launches: LAUNCH_COSTS names parts of kernels' names and the
 * milliseconds of each ("k_a=1.5,k_b=2", 0 for the others).
 * Built with -rdynamic: the functions below stand in for the runtime's of the same names. */
#include <dlfcn.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "chemstep.h"

typedef struct { unsigned x, y, z; } dim3;
typedef int hipError_t;

static long lds_bytes;
static dim3 cfg_grid, cfg_block;
static struct { const void *host; const char *name; } kernels[1024];
static int n_kernels;
static float now_ms;

static float cost_of(const char *kernel) {
  const char *c = getenv("LAUNCH_COSTS");
  while (c && *c) {
    const char *eq = strchr(c, '='), *end = strchr(c, ',');
    char part[128] = "";
    if (!eq || eq - c >= (long)sizeof(part)) break;
    memcpy(part, c, eq - c);
    if (strstr(kernel, part)) return strtof(eq + 1, NULL);
    c = end ? end + 1 : NULL;
  }
  return 0.0f;
}

void **__hipRegisterFatBinary(const void *data) { static void *h; (void)data; return &h; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g) {
  (void)m, (void)v, (void)h, (void)d, (void)e, (void)s, (void)c, (void)g;
}
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned limit,
                           void *t, void *b, void *bd, void *gd, int *w) {
  (void)m, (void)dev, (void)limit, (void)t, (void)b, (void)bd, (void)gd, (void)w;
  if (n_kernels < 1024) {
    kernels[n_kernels].host = host;
    kernels[n_kernels++].name = strdup(name);
  }
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, void *s) {
  (void)sh, (void)s;
  cfg_grid = g;
  cfg_block = b;
  return 0;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, void **s) {
  *g = cfg_grid;
  *b = cfg_block;
  *sh = 0;
  *s = NULL;
  return 0;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t sh, void *s) {
  (void)args, (void)sh, (void)s;
  const char *name = "?";
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].host == f) name = kernels[i].name;
  now_ms += cost_of(name);
  printf("%s %u %u %u %u %u %u\n", name, g.x, g.y, g.z, b.x, b.y, b.z);
  return 0;
}
hipError_t hipGetLastError(void) { return 0; }
const char *hipGetErrorString(hipError_t e) { (void)e; return "recorded"; }
hipError_t hipGetDevice(int *d) { *d = 0; return 0; }
/* the LDS of a block, else the number of CUs */
hipError_t hipDeviceGetAttribute(int *v, int attr, int d) {
  (void)d;
  static int first = -1;
  if (first < 0) first = attr; /* the LDS is asked for first, by every caller */
  *v = attr == first ? (int)lds_bytes : 256;
  return 0;
}
hipError_t hipMalloc(void **p, size_t n) { *p = malloc(n); return *p ? 0 : 2; }
hipError_t hipFree(void *p) { free(p); return 0; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
hipError_t hipMemset(void *d, int v, size_t n) { memset(d, v, n); return 0; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, void *s) { (void)s; return hipMemset(d, v, n); }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) {
  (void)d, (void)s, (void)n, (void)k, (void)st;
  return 0;
}
hipError_t hipMemcpy2DAsync(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h, int k, void *st) {
  (void)d, (void)dp, (void)s, (void)sp, (void)w, (void)h, (void)k, (void)st;
  return 0;
}
hipError_t hipEventCreate(void **e) { *e = calloc(1, sizeof(float)); return *e ? 0 : 2; }
hipError_t hipEventDestroy(void *e) { free(e); return 0; }
hipError_t hipEventRecord(void *e, void *s) { (void)s; *(float *)e = now_ms; return 0; }
hipError_t hipEventSynchronize(void *e) { (void)e; return 0; }
hipError_t hipEventElapsedTime(float *ms, void *a, void *b) { *ms = *(float *)b - *(float *)a; return 0; }
hipError_t hipStreamSynchronize(void *s) { (void)s; return 0; }
hipError_t hipDeviceSynchronize(void) { return 0; }
hipError_t hipGetDevicePropertiesR0600(void *p, int d) { (void)p, (void)d; return 1; }

int main(int argc, char **argv) {
  if (argc < 6) return 2;
  void *lib = dlopen(argv[1], RTLD_NOW);
  if (!lib) return fprintf(stderr, "%s\n", dlerror()), 2;
  lds_bytes = atol(argv[2]);
  const int R = atoi(argv[3]);
  chem_status (*create)(const chem_mech_desc *, chem_mech **) = dlsym(lib, "chem_mech_create");
  chem_status (*rates)(const chem_mech *, chem_batch, const double *, const double *, const double *,
                       double *, double *, double *, void *) = dlsym(lib, "chem_rates");
  chem_status (*step)(const chem_mech *, chem_batch, double, const double *, double *, const double *,
                      double *, double *, double *, int32_t *, const chem_step_opts *, void *) =
      dlsym(lib, "chem_step");
  chem_status (*sample)(const chem_mech *, chem_batch, const double *, const double *, const double *,
                        const double *, const double *, const double *, const double *,
                        const chem_sample_opts *, double *, double *, double *, uint8_t *, void *) =
      dlsym(lib, "chem_sample_states");
  /* four isomers over C, H, O, N and R copies of a reaction between two and two of them */
  int32_t comp[16];
  double W[4], awt[4] = {0.012, 0.001, 0.016, 0.014}, nasa[68] = {0};
  for (int k = 0; k < 4; ++k) {
    for (int e = 0; e < 4; ++e) comp[4 * k + e] = 1;
    W[k] = 0.043;
    nasa[17 * k] = 200.0;
    nasa[17 * k + 1] = 1000.0;
    nasa[17 * k + 2] = 3000.0;
    nasa[17 * k + 3] = nasa[17 * k + 10] = 4.0;
  }
  int32_t *rsp = malloc(R * 16), *rnu = malloc(R * 16);
  double *A = malloc(R * 8), *b = calloc(R, 8), *Ea = calloc(R, 8);
  for (int r = 0; r < R; ++r) {
    const int32_t sp[4] = {0, 1, 2, 3}, nu[4] = {1, 1, 1, 1};
    memcpy(rsp + 4 * r, sp, 16);
    memcpy(rnu + 4 * r, nu, 16);
    A[r] = 1.0;
  }
  const chem_mech_desc d = {4, R, 4, W, comp, awt, nasa, rsp, rnu, A, b, Ea};
  chem_mech *m = NULL;
  if (create(&d, &m) != CHEM_OK) return 2;
  double *const x = (double *)64; /* never followed */
  const chem_sample_opts o = {0.125, 10.0, 0.1, 500.0, 0.0, 10.0, 0.0, 10.0, 0.0, 10.0, 1, 0, 1, 2, 3};
  for (int i = 5; i < argc; ++i) {
    const chem_batch n = {atoll(argv[i]), atoll(argv[i])};
    chem_status st = CHEM_EINVAL;
    if (!strcmp(argv[4], "rates")) st = rates(m, n, x, x, x, x, x, NULL, NULL);
    if (!strcmp(argv[4], "step")) st = step(m, n, 1e-6, NULL, x, x, x, NULL, NULL, NULL, NULL, NULL);
    if (!strcmp(argv[4], "autotune")) {
      chem_status (*tune)(chem_mech *, chem_batch, double, const double *, const double *,
                          const double *, const chem_step_opts *, void *, chem_tuning *) =
          dlsym(lib, "chem_autotune");
      st = tune(m, n, 1e-6, x, x, x, NULL, NULL, NULL);
    }
    if (!strcmp(argv[4], "autotune_train")) {
      chem_status (*make)(const ann_arch *, uint64_t, ann_model **) = dlsym(lib, "ann_create");
      chem_status (*tune)(ann_model *, int64_t, double *, double *, void *) =
          dlsym(lib, "ann_autotune_train");
      const ann_arch arch = {4, 2, {160, 96, 64}, 0, 1};
      ann_model *net = NULL;
      st = make(&arch, 1, &net);
      if (st == CHEM_OK) st = tune(net, n.n, NULL, NULL, NULL);
    }
    if (!strcmp(argv[4], "sample")) st = sample(m, n, x, x, x, x, NULL, NULL, NULL, &o, x, x, x, (uint8_t *)x, NULL);
    printf("call %lld %d\n", (long long)n.n, (int)st);
  }
  return 0;
}
