// Costs of a window of rerouting plan indices: what the kernels that expand partitions to plan indices share, and the one that works
// the partitions out itself.
#ifndef CHM_WINDOW_H
#define CHM_WINDOW_H
#include <hip/hip_runtime.h>

#include <algorithm>

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
  uint32_t in_place;            // 1: the vectors take the room of what the partitions took
  FastDiv R;                    // vectors
  uint32_t step_parts, step_rr; // 2 * BLOCK plan indices on: whole partitions, and vectors
  uint64_t K;
  int64_t *costs;
};
// WINDOW_LEAST_R: fewer vectors have more partitions in the smallest tile than lanes.  WINDOW_BEHIND: larger tables, bytes, take the room of
// what the partitions took (and are staged after them): three or four workgroups fit a compute unit then instead of two, and at most
// 53 KB are asked for.
enum { WINDOW_LEAST_R = 16, WINDOW_BEHIND = 8 << 10 };
// Plan indices per workgroup, a multiple of 2 * BLOCK.  The partitions a tile touches are worked out ahead of its stores, one per lane,
// those it begins or ends in twice; the least, 2,048, only where a launch would have fewer workgroups than compute units otherwise.
// - Fewer than 64 vectors: as many plan indices as have a lane for every partition, up to four times the least (us with the least / so:
//   36 vectors, 16 M plans of 8 stages 73 / 49, of 24 stages 145 / 67; 16 vectors, of 28 stages 166 / 114).
// - From 64 on four times the least (153 vectors, 2^26 plans of 8 stages: 212 with the least, 137 with twice, 111 with four times that,
//   116 with 16 times), and where a launch has more than three workgroups a compute unit then, as many as fill one wavefront with
//   partitions: it works out 64 of them in the time of five (1,891 vectors, 16 M plans of 24 stages 98 / 57, of 8 stages 57 / 50).
static inline uint32_t window_tile(uint32_t R, uint32_t count) {
  const uint32_t least = BLOCK * EXPAND_PER;
  if (R < 64) {
    const uint32_t tile = std::min(4 * least, (BLOCK - 1) * R / (2 * BLOCK) * (2 * BLOCK));
    return count >= 256u * tile ? tile : least;
  }
  const uint32_t times = count >= 256u * 4 * least ? 4 : 1;
  return std::max(times, std::min(64u * R / least, (count + 768u * least - 1) / (768u * least))) * least;
}
static_assert((BLOCK * EXPAND_PER + WINDOW_LEAST_R - 1) / WINDOW_LEAST_R + 1 <= BLOCK && (4 * BLOCK * EXPAND_PER + 63) / 64 + 1 <= BLOCK,
              "a lane for every partition of a tile");
int chmk_window_plans(int sp, const WindowArgs &a, uint32_t row_bytes, void *stream);       // 1 = no instance for these stages
#endif
