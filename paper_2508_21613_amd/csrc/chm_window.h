// Costs of a window of rerouting plan indices: what the kernels that expand partitions to plan indices share, and the one that works
// the partitions out itself.
#ifndef CHM_WINDOW_H
#define CHM_WINDOW_H
#include <hip/hip_runtime.h>

#include "chm_fast.h"

namespace {

// The same with 32-bit index arithmetic, for reroute spaces below 2^31 vectors per partition and launches
// of at most 2^31 plan indices: the host passes the partition (relative to the pass) and the reroute rank of
// the launch's first plan index, so a lane divides first_rr + gid, which fits 32 bits.
// Division of a 32-bit number by a divisor fixed at launch: one multiply-high, two shifts, an add and a subtract
// (round-up method of Granlund and Montgomery), exact for every dividend; the compiler's generic 32-bit
// division costs about five times as much.
struct FastDiv {
  uint32_t d, m, sh1, sh2;
};
static inline FastDiv make_fast_div(uint32_t d) {
  FastDiv f;
  f.d = d;
  uint32_t l = 0;
  while ((1ull << l) < d) ++l;                               // ceil(log2 d)
  f.m = (uint32_t)(((1ull << 32) * ((1ull << l) - d)) / d) + 1u;
  f.sh1 = l < 1 ? l : 1;
  f.sh2 = l > 0 ? l - 1 : 0;
  return f;
}
__device__ __forceinline__ uint32_t fast_div(uint32_t n, const FastDiv &f) {
  const uint32_t t = __umulhi(f.m, n);
  return (t + ((n - t) >> f.sh1)) >> f.sh2;
}

struct ExpandArgs32 {
  const uint64_t *base;
  const uint32_t *weights;
  const uint32_t *rows[DEV_MAX_AFF];
  FastDiv R[DEV_MAX_AFF];
  int32_t stride[DEV_MAX_AFF], peers[DEV_MAX_AFF];
  int32_t n_aff;
  FastDiv R_joint;
  uint32_t first_part, first_rr, count;
  uint64_t K;
  int64_t *costs;
};

// Plan indices per workgroup: EXPAND_PER consecutive tiles of BLOCK.  A lane computes its EXPAND_PER costs
// first and stores them back to back at the end: memory operations of a wave complete in order, so a load
// issued after a store would wait for that store to be acknowledged (microseconds when HBM is saturated
// with writes), and with one 512-byte store in flight per wave the kernel stayed below 1.5 TB/s.
constexpr int EXPAND_PER = 8;

}  // namespace

// One stage lost nodes and its vector table is small (k_window_plans).
struct WindowArgs {
  FastLaunch search;            // the rerouting family; the kernel fills in which partitions
  const uint32_t *rows;         // rank-ordered vectors, `stride` (4 or 8) entries each
  uint64_t part_first;          // partition and reroute rank of the first plan index
  uint32_t first_rr, count, tile, stride;
  FastDiv R;                    // vectors
  uint32_t step_parts, step_rr; // 2 * BLOCK plan indices on: whole partitions, and vectors
  uint64_t K;
  int64_t *costs;
};
// Plan indices per workgroup, a multiple of BLOCK * EXPAND_PER.  Partitions that a tile begins or ends in are worked out twice, and
// their lanes are one per partition: four times the least where 64 vectors and more leave a wavefront and a half of partitions
// (153 vectors, 2^26 plans: 212 us with the least, 137 with twice, 111 with four times that, 116 with 16 times), the least where a launch would have fewer workgroups than compute units.
enum { WINDOW_LEAST_R = 16 };
static inline uint32_t window_tile(uint32_t R, uint32_t count) {
  const uint32_t least = BLOCK * EXPAND_PER;
  return R >= 64 && count >= 256u * 4 * least ? 4 * least : least;
}
static_assert((BLOCK * EXPAND_PER + WINDOW_LEAST_R - 1) / WINDOW_LEAST_R + 1 <= BLOCK && (4 * BLOCK * EXPAND_PER + 63) / 64 + 1 <= BLOCK,
              "a lane for every partition of a tile");
int chmk_window_plans(int sp, const WindowArgs &a, uint32_t row_bytes, void *stream);       // 1 = no instance for these stages
#endif
