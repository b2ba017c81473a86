/* A plain C caller that some calls of the runtime fail: its own hipMalloc stands in front of the runtime's and refuses
 * allocations above a size while `limit` is set, its hipStreamSynchronize waits but reports an error while `broken` is, and its
 * hipLaunchKernel counts.  Searches a scenario of at least 2^21 partitions without memory for tables, after a search whose wait
 * was reported as failed, and undisturbed.  tests/test_scarce_memory.py builds and runs it. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "chm.h"

static size_t limit = 0;
static int refused = 0;

int hipMalloc(void **p, size_t bytes) {
  static int (*real)(void **, size_t) = NULL;
  if (!real) *(void **)&real = dlsym(RTLD_NEXT, "hipMalloc");
  if (limit && bytes > limit) { ++refused; return 2; }          /* out of memory */
  return real(p, bytes);
}

static int broken = 0, launched = 0;
typedef struct { unsigned x, y, z; } dim3_t;

int hipStreamSynchronize(void *stream) {
  static int (*real)(void *) = NULL;
  if (!real) *(void **)&real = dlsym(RTLD_NEXT, "hipStreamSynchronize");
  const int rc = real(stream);
  return broken ? 999 : rc;                                     /* unknown error */
}

int hipLaunchKernel(const void *f, dim3_t grid, dim3_t block, void **args, size_t lds, void *stream) {
  static int (*real)(const void *, dim3_t, dim3_t, void **, size_t, void *) = NULL;
  if (!real) *(void **)&real = dlsym(RTLD_NEXT, "hipLaunchKernel");
  ++launched;
  return real(f, grid, block, args, lds, stream);
}

static void print_best(const char *what, int rc, const chm_best *b) {
  printf("%s rc=%d index=%llu cost=%lld strategy=%d t_step=%lld t_trans=%lld\n", what, rc, (unsigned long long)b->index,
         (long long)b->cost, b->strategy, (long long)b->t_step_us, (long long)b->t_trans_us);
}

int main(int argc, char **argv) {
  enum { L = 32, PP = 8, DP = 2 };
  int32_t fwd[L], bwd[L], mem[L], failed[1] = {3};
  if (argc != 1 + 3 * L) return 2;
  for (int l = 0; l < L; ++l) { fwd[l] = atoi(argv[1 + l]); bwd[l] = atoi(argv[1 + L + l]); mem[l] = atoi(argv[1 + 2 * L + l]); }
  chm_scenario_desc d;
  memset(&d, 0, sizeof(d));
  d.L = L; d.PP = PP; d.DP = DP; d.M = 9; d.fwd_us = fwd; d.bwd_us = bwd; d.mem_mib = mem; d.n_failed = 1; d.failed_nodes = failed;
  d.comm_us = 150; d.mem_cap_mib = 8000; d.horizon_steps = 2048; d.xfer_us_per_mib = 100; d.reconf_us[1] = 8000000;
  chm_scenario *s = NULL;
  int rc = chm_load_scenario(&d, &s);
  if (rc != CHM_OK) { printf("load rc=%d\n", rc); return 1; }
  chm_best b;
  for (uint32_t mask = 1; mask <= 7; mask = mask == 4 ? 7 : 2 * mask) {
    limit = 1;
    rc = chm_search_best(s, mask, &b, NULL);
    limit = 0;
    print_best("scarce", rc, &b);
  }
  printf("refused %d\n", refused);
  for (int i = 0; i < 3; ++i) {                                 /* the first one's wait fails */
    broken = i == 0;
    launched = 0;
    rc = chm_search_best(s, 7u, &b, NULL);
    broken = 0;
    printf("launches %d rc=%d\n", launched, rc);
    if (i > 0) print_best("after", rc, &b);
  }
  for (uint32_t mask = 1; mask <= 7; mask = mask == 4 ? 7 : 2 * mask) {
    rc = chm_search_best(s, mask, &b, NULL);
    print_best("plenty", rc, &b);
  }
  chm_free_scenario(s);
  return 0;
}
