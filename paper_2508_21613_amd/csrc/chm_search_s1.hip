// The search kernels of strategy 1 (re-partition), one instance per number of stages.
#include "chm_halves_kernel.h"
#include "chm_search_kernel.h"

int chmk_fast_search_s1(int sp, const FastLaunch &a, uint32_t blocks, uint32_t tile_bytes, void *stream, SearchVariant variant) {
  return launch_by_stages<1>(sp, a, blocks, tile_bytes, (hipStream_t)stream, variant);
}
int chmk_halves_s1(int sp, const HalvesLaunch &a, bool build, void *stream) {
  return halves_by_stages<1>(sp, a, build, (hipStream_t)stream);
}
