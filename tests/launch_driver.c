/* Launch errors of libpe's host code, without a GPU: this program defines the HIP
 * runtime functions that the library launches through, so that no kernel runs and
 * any one launch can be made to fail, and opens the library behind them.  For
 * several calls (argv[1]: the library) every launch in turn fails; the call has to
 * return PE_EHIP and to stop (two more launches at most, where the library checks a
 * group of three).  Like the runtime, the stub keeps a launch's error until it is asked for it. */
#include <dlfcn.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include "pe.h"

static int launches, fail_at, last_error;
typedef struct { unsigned x, y, z; } dim;

int __hipPushCallConfiguration(dim g, dim b, size_t sh, void* st) { (void)g; (void)b; (void)sh; (void)st; return 0; }
int __hipPopCallConfiguration(dim* g, dim* b, size_t* sh, void** st) {
  dim one = {1, 1, 1};
  *g = one; *b = one; *sh = 0; *st = NULL;
  return 0;
}
int hipLaunchKernel(const void* f, dim g, dim b, void** args, size_t sh, void* st) {
  (void)f; (void)g; (void)b; (void)args; (void)sh; (void)st;
  if (++launches != fail_at) return 0;
  return last_error = 1;
}
int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int t, size_t sh) { (void)f; (void)t; (void)sh; *n = 1; return 0; }

typedef struct { const char* name; int count; long m, n; int compute, T, tile, fp8, fast, init, force, muon; double tau, k; } call;

int main(int argc, char** argv) {
  static const call calls[] = {
    {"256 tile, full rounds", 1, 1024, 4096, PE_COMPUTE_BF16, 2, 2, 0, 0, 0, -1, 0, 0, 1},
    {"256 tile, short last round", 2, 3072, 3072, PE_COMPUTE_BF16, 3, 2, 0, 0, 0, -1, 1, 0, 1},
    {"256 tile, init step", 1, 1024, 1024, PE_COMPUTE_BF16, 2, 2, 0, 0, 3, -1, 0, 0, 1},
    {"small tiles", 1, 768, 768, PE_COMPUTE_BF16, 2, 0, 0, 0, 0, -1, 0, 0, 1},
    {"small tiles, split k", 1, 128, 8192, PE_COMPUTE_BF16, 2, 1, 0, 0, 0, -1, 1, 0, 1},
    {"one kernel", 80, 64, 700, PE_COMPUTE_BF16, 2, 0, 0, 0, 0, -1, 0, 0, 1},
    {"few rows", 1, 9, 300, PE_COMPUTE_BF16, 2, 0, 0, 0, 0, -1, 0, 0, 1},
    {"e4m3, 256", 1, 1024, 2048, PE_COMPUTE_FP8, 3, 2, 2, 0, 0, -1, 0, 0, 1},
    {"e4m3, 128", 1, 512, 1024, PE_COMPUTE_FP8, 3, 1, 2, 0, 0, -1, 0, 0, 1},
    {"fp32 planes", 2, 700, 900, PE_COMPUTE_F32, 2, 0, 0, 0, 0, -1, 0, 0, 1},
    {"fp32 planes, init step", 1, 1700, 1700, PE_COMPUTE_F32, 2, 0, 0, 0, 3, -1, 0, 0, 1},
    {"fp32 MFMA", 1, 500, 900, PE_COMPUTE_F32, 8, 0, 0, 0, 0, -1, 0, 0, 1},
    {"fast", 1, 700, 3000, PE_COMPUTE_F32, 4, 0, 0, 3, 0, -1, 0, 0, 1},
    {"fast, short last round", 1, 4096, 8192, PE_COMPUTE_F32, 4, 0, 0, 3, 0, -1, 0, 0, 1},
    {"fast, fp32 MFMA", 1, 700, 3000, PE_COMPUTE_F32, 4, 0, 0, 3, 0, -1, 0, 0, 8},
    {"fast, few rows", 1, 9, 3000, PE_COMPUTE_F32, 4, 0, 0, 3, 0, -1, 0, 0, 1},
    {"learned with fallback", 2, 300, 700, PE_COMPUTE_BF16, 3, 0, 0, 0, 0, 2, 0, 0.5, 1},
    {"learned, fp32", 2, 300, 700, PE_COMPUTE_F32, 3, 0, 0, 0, 0, 2, 0, 0.5, 1},
  };
  void* lib = argc > 1 ? dlopen(argv[1], RTLD_NOW | RTLD_GLOBAL) : NULL;
  if (!lib) { printf("%s\n", dlerror()); return 2; }
  pe_status (*coeffs)(double, int32_t, const pe_coeff_opts*, double*, double*, double*, int32_t*) =
      (pe_status (*)(double, int32_t, const pe_coeff_opts*, double*, double*, double*, int32_t*))dlsym(lib, "pe_coeffs");
  pe_status (*batched)(int32_t, const pe_matrix*, const pe_opts*, void*, size_t, void*) =
      (pe_status (*)(int32_t, const pe_matrix*, const pe_opts*, void*, size_t, void*))dlsym(lib, "pe_polar_batched");
  int bad = 0;
  for (size_t c = 0; c < sizeof calls / sizeof *calls; ++c) {
    const call* q = calls + c;
    double abc[3 * 64];
    coeffs(1e-3, q->T, NULL, abc, NULL, NULL, NULL);
    if (q->k > 1) { abc[0] = q->k; abc[1] = abc[2] = 0; }
    static pe_matrix mats[80];
    memset(mats, 0, sizeof mats);
    for (int i = 0; i < q->count; ++i) {
      pe_matrix* m = mats + i;  /* (device addresses are only handed on) */
      m->G = (void*)0x10000000; m->X = (void*)0x20000000;
      m->m = q->m; m->n = q->n; m->ldg = m->ldx = m->ldm = m->ldw = q->n;
      if (q->muon) { m->M = (float*)0x30000000; m->W = (void*)0x40000000; }
      m->g_dtype = q->compute == PE_COMPUTE_F32 ? PE_F32 : PE_BF16;
    }
    pe_opts o;
    memset(&o, 0, sizeof o);
    o.T = q->T; o.abc = abc; o.compute = q->compute; o.tile = q->tile; o.fp8_steps = q->fp8;
    o.fast_restart = q->fast; o.spectral_init = q->init; o.force_class = q->force; o.fallback_tau = (float)q->tau;
    launches = fail_at = last_error = 0;
    pe_status s = batched(q->count, mats, &o, (void*)0x100000000, (size_t)1 << 40, NULL);
    const int n = launches;
    if (s != PE_OK || n == 0) { printf("%s: status %d, %d launches\n", q->name, s, n); ++bad; continue; }
    for (int k = 1; k <= n; ++k) {
      launches = last_error = 0;
      fail_at = k;
      s = batched(q->count, mats, &o, (void*)0x100000000, (size_t)1 << 40, NULL);
      if (s != PE_EHIP || launches - k > 2) {
        printf("%s: launch %d of %d fails: status %d, %d launches behind it\n", q->name, k, n, s, launches - k);
        ++bad;
      }
    }
  }
  printf("launch checks: %d failures\n", bad);
  return bad != 0;
}
