// The search and list kernels of strategy 0 (redundant computation), one instance per number of stages.
#include "chm_search_kernel.h"

int chmk_fast_search_s0(int sp, const FastLaunch &a, uint32_t blocks, uint32_t tile_bytes, void *stream, bool queued) {
  return launch_by_stages<0>(sp, a, blocks, tile_bytes, (hipStream_t)stream, queued);
}
int chmk_list_filter_s0(int sp, const ListFilter &a, uint32_t blocks, void *stream) {
  return filter_by_stages<0>(sp, a, blocks, (hipStream_t)stream);
}
