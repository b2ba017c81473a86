// Costs of a window of rerouting plan indices in one kernel.
#include "chm_search_kernel.h"
#include "chm_window.h"

namespace {

// One workgroup per tile of plan indices.  The partitions the tile's indices belong to are worked out first, one per lane (cost
// without penalty and peer stage times, into LDS, beside the vector table), then every index adds the penalty of its vector.  The
// vector memory path carries the stores and little else, and other workgroups store while this one works out its partitions (2^26
// plans, 153 vectors: 108 us, 5.0 TB/s; 118 us with a pass of its own over the partitions ahead, a plain fill of the buffer 78).
// What is left above the fill: the first partitions of every workgroup (8 us until its first store, five workgroups to a compute
// unit) and 63 us of VALU issue beside the stores.  A lane computes its EXPAND_PER costs before it stores them, two neighbouring ones as
// 16 bytes, streamed past the caches.

// More stages than this: class_time.  A tile has a few partitions a lane at most, so that its further instructions count less than the
// wavefronts that store meanwhile (16 stages, 81 vectors, 14 M plans: 64 us with the 159 registers of pipeline_time, 54 with 69).
constexpr int WINDOW_FLOW = 8;

template <int SP>
__global__ void __launch_bounds__(BLOCK) CHM_WAVES(SP, 2) k_window_plans(WindowArgs a) {
  typedef SearchShared<SP, 4> Shared;
  static_assert(sizeof(Shared) % sizeof(uint4) == 0, "the rows behind it");
  __shared__ uint64_t base[BLOCK];
  __shared__ __align__(16) uint32_t weights[BLOCK * ROWS_MAX_P];
  extern __shared__ uint4 room[];                      // what the partitions take, and the rows, [R * stride / 4], behind it or in its place
  Shared &sh = *(Shared *)room;
  uint4 *const rows = room + (a.in_place ? 0 : sizeof(Shared) / sizeof(uint4));
  const uint32_t R = a.R.d;
  const uint32_t tile_first = blockIdx.x * a.tile;     // < count by the grid size
  const uint32_t tile_end = min(tile_first + a.tile, a.count);
  const uint32_t p_first = fast_div(a.first_rr + tile_first, a.R);
  const uint32_t n_parts = min(fast_div(a.first_rr + tile_end - 1, a.R) - p_first + 1, (uint32_t)BLOCK);
  const uint4 *rows4 = (const uint4 *)a.rows;
  auto stage_rows = [&]() {
    for (uint32_t i = threadIdx.x; i < R * (a.stride / 4u); i += BLOCK) rows[i] = rows4[i];
  };
  if (!a.in_place) stage_rows();
  FastLaunch f = a.search;
  f.s.part_first = a.part_first + p_first;
  f.s.part_count = n_parts;
  f.base_out = base;
  f.weights_out = weights;
  search_partitions<SP, 2, 4, (SP > WINDOW_FLOW)>(f, 0, sh, nullptr);
  __syncthreads();
  // a partition that does not fit costs INT64_MAX whatever the vector: no multiples to add
  if (threadIdx.x < n_parts && base[threadIdx.x] == ~0ull) {
    base[threadIdx.x] = (uint64_t)CHM_INF_COST;
    for (int i = 0; i < ROWS_MAX_P; ++i) weights[threadIdx.x * ROWS_MAX_P + i] = 0;
  }
  if (a.in_place) stage_rows();                        // (uniform; nobody reads `sh` any more)
  __syncthreads();
  const uint4 *weights4 = (const uint4 *)weights;
  const bool aligned = (((uintptr_t)a.costs) & 15u) == 0;            // uniform
  const bool short_k = a.K <= 0xffffffffull;                         // uniform
  // partition (of the tile) and reroute rank of the lane's next plan index: divided once, then 2 * BLOCK indices on at a time
  uint32_t lp = fast_div(a.first_rr + tile_first + 2 * threadIdx.x, a.R);
  uint32_t rr = a.first_rr + tile_first + 2 * threadIdx.x - lp * R;
  lp -= p_first;
  auto cost_of = [&](uint32_t p, uint32_t r) -> int64_t {
    p = p < n_parts ? p : n_parts - 1;                               // (lanes past the end)
    const uint4 w_lo = weights4[2 * p];
    uint32_t m;
    if (a.stride == 4) {                                             // uniform
      const uint4 row = rows[r];
      m = max(max(__umul24(row.x, w_lo.x), __umul24(row.y, w_lo.y)), max(__umul24(row.z, w_lo.z), __umul24(row.w, w_lo.w)));
    } else {
      const uint4 w_hi = weights4[2 * p + 1];
      const uint4 row = rows[2 * r], row2 = rows[2 * r + 1];
      m = max(max(__umul24(row.x, w_lo.x), __umul24(row.y, w_lo.y)), max(__umul24(row.z, w_lo.z), __umul24(row.w, w_lo.w)));
      m = max(m, max(max(__umul24(row2.x, w_hi.x), __umul24(row2.y, w_hi.y)), max(__umul24(row2.z, w_hi.z), __umul24(row2.w, w_hi.w))));
    }
    return (int64_t)(base[p] + (short_k ? (uint64_t)(uint32_t)a.K * m : a.K * m));
  };
  for (uint32_t part = tile_first; part < tile_end; part += BLOCK * EXPAND_PER) {
    const uint32_t first = part + 2 * threadIdx.x;
    int64_t cost[EXPAND_PER];
#pragma unroll
    for (int rep = 0; rep < EXPAND_PER; rep += 2) {
      const bool over = rr + 1 >= R;                                 // the pair's second index is in the next partition
      cost[rep] = cost_of(lp, rr);
      cost[rep + 1] = cost_of(lp + (over ? 1u : 0u), over ? 0u : rr + 1);
      lp += a.step_parts;
      rr += a.step_rr;
      const bool wrap = rr >= R;
      lp += wrap ? 1u : 0u;
      rr -= wrap ? R : 0u;
    }
#pragma unroll
    for (int rep = 0; rep < EXPAND_PER; rep += 2) {
      const uint32_t gid = first + (rep >> 1) * (2 * BLOCK);
      if (aligned && gid + 1 < tile_end) {
        typedef long long pair_t __attribute__((ext_vector_type(2)));
        pair_t v;
        v.x = cost[rep];
        v.y = cost[rep + 1];
        __builtin_nontemporal_store(v, (pair_t *)(a.costs + gid));
      } else {
        if (gid < tile_end) __builtin_nontemporal_store(cost[rep], &a.costs[gid]);
        if (gid + 1 < tile_end) __builtin_nontemporal_store(cost[rep + 1], &a.costs[gid + 1]);
      }
    }
  }
}

}  // namespace

int chmk_window_plans(int sp, const WindowArgs &a, uint32_t row_bytes, void *stream) {
  const uint32_t blocks = (a.count + a.tile - 1) / a.tile;
#define CHM_CASE(SP) case SP: { \
    const uint32_t own = sizeof(SearchShared<SP, 4>), room = a.in_place ? (own > row_bytes ? own : row_bytes) : own + row_bytes; \
    hipLaunchKernelGGL((k_window_plans<SP>), dim3(blocks), dim3(BLOCK), room, (hipStream_t)stream, a); return 0; }
  switch (sp) {
    CHM_CASE(2) CHM_CASE(3) CHM_CASE(4) CHM_CASE(5) CHM_CASE(6) CHM_CASE(7) CHM_CASE(8) CHM_CASE(9) CHM_CASE(10) CHM_CASE(11)
    CHM_CASE(12) CHM_CASE(13) CHM_CASE(14) CHM_CASE(15) CHM_CASE(16) CHM_CASE(17) CHM_CASE(18) CHM_CASE(19) CHM_CASE(20)
    CHM_CASE(21) CHM_CASE(22) CHM_CASE(23) CHM_CASE(24) CHM_CASE(25) CHM_CASE(26) CHM_CASE(27) CHM_CASE(28) CHM_CASE(29)
    CHM_CASE(30) CHM_CASE(31) CHM_CASE(32)
    default: return 1;
  }
#undef CHM_CASE
}
