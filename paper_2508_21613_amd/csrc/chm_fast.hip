// Host side of the shape-specialised search path (chm_search_kernel.h): which strategies it covers, its tables and
// scratch, its launches; and the kernels around it: enumeration of the candidates of a bounded search, the
// rank-ordered reroute vectors and the cost store of rerouting plan indices.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "chm_fast.h"
#include "chm_pool.h"
#include "chm_window.h"

// typed front ends of the caching allocator (chm_pool.h)
template <typename T>
static inline bool pool_take(T *&p, size_t bytes) { p = (T *)pool_device_alloc(bytes); return p != nullptr; }
template <typename T>
static inline bool pool_take_pinned(T *&p, size_t bytes) { p = (T *)pool_pinned_alloc(bytes); return p != nullptr; }

namespace {

// ---------------------------------------------------------------------------------------
// bounded search: enumeration of the candidates (see CandidateSet)
// ---------------------------------------------------------------------------------------
// row[x] = candidates (of the arrangement being refined) whose current stage starts at or before x.  Finds by
// bisection the start in [lo, hi] whose block holds index idx, counting blocks from lo on, and leaves in idx
// the offset inside that block (an index beyond the last block lands on hi).
__host__ __device__ inline int candidate_start(const uint64_t *row, int lo, int hi, uint64_t &idx) {
  const uint64_t target = idx + (lo > 0 ? row[lo - 1] : 0);
  int a = lo, b = hi;
  while (a < b) {
    const int m = (a + b) >> 1;
    if (row[m] > target) b = m;
    else a = m + 1;
  }
  idx = target - (a > 0 ? row[a - 1] : 0);
  return a;
}

struct CandidateEnum {
  const uint64_t *ways;         // [stages][end][start]
  const uint8_t *low_pair;      // [stages][L+1]
  int32_t stages, L;
  uint32_t total;               // candidates of this launch
  uint64_t first, stride;       // launch index i stands for candidate (first + i) * stride
  uint4 *cut_list;              // [candidate] cut positions packed into bytes
  uint32_t *cut_pos;            // [candidate] = its index
  uint32_t *cut_count;          // [workgroup] candidates in its region of BLOCK slots
};

// Candidate `index` of the set, in ascending partition rank: the start of the last stage is chosen first
// (the candidates that share it form a block of ways[last][a][L] indices), then the start of the stage below
// it among those the pair limit allows, and so on down.  Every scan is bounded by the stage above it, so the
// cuts stay a valid partition whatever the tables hold.
__global__ void __launch_bounds__(BLOCK) k_enumerate_candidates(CandidateEnum e) {
  const uint32_t gid = blockIdx.x * BLOCK + threadIdx.x;
  if (threadIdx.x == 0) {
    const uint32_t first = blockIdx.x * BLOCK;
    e.cut_count[blockIdx.x] = first >= e.total ? 0u : (e.total - first < BLOCK ? e.total - first : (uint32_t)BLOCK);
  }
  if (gid >= e.total) return;
  const int W = e.L + 1;
  uint64_t idx = (e.first + gid) * e.stride;
  uint32_t words[4] = {0, 0, 0, 0};
  int s = e.stages - 1;                   // the stage whose start is being chosen
  int end = e.L;                          // its end
  // at least one layer for every stage below
  int start = candidate_start(e.ways + ((size_t)s * W + end) * W, s, end - 1, idx);
  for (;;) {
    words[(s - 1) >> 2] |= (uint32_t)start << (8 * ((s - 1) & 3));
    if (s == 1) break;
    // the stage below: layers [below, start), its pair with stage s ends at `end`
    const int lo = (int)e.low_pair[(size_t)(s - 1) * W + end];
    const int first = lo > s - 1 ? lo : s - 1;
    const int below = first >= start - 1 ? start - 1 : candidate_start(e.ways + ((size_t)(s - 1) * W + start) * W, first, start - 1, idx);
    end = start;
    start = below;
    --s;
  }
  e.cut_list[gid] = make_uint4(words[0], words[1], words[2], words[3]);
  e.cut_pos[gid] = gid;
}

// ---------------------------------------------------------------------------------------
// reroute vector table and the cost store of rerouting plan indices
// ---------------------------------------------------------------------------------------
// Row r of affected stage a = the reroute vector of rank r, decoded from the count table
// (count[left][remaining] = vectors of `left` entries summing to `remaining`); rows beyond the
// valid ones put every orphaned micro-batch on every peer (never better than a valid row).
__global__ void __launch_bounds__(BLOCK) k_make_rows(const DevScenario *__restrict__ scn, const uint64_t *__restrict__ comp,
                                                     int a, uint32_t *__restrict__ rows, uint32_t n_rows_padded, int stride) {
  const uint32_t r = blockIdx.x * BLOCK + threadIdx.x;
  if (r >= n_rows_padded) return;
  const int p = scn->aff_peers[a];
  const int total = scn->aff_total[a];
  uint32_t *row = rows + (size_t)r * stride;
  if ((uint64_t)r >= scn->aff_R[a]) {
    for (int i = 0; i < stride; ++i) row[i] = i < p ? (uint32_t)total : 0u;
    return;
  }
  const uint64_t *tab = comp + scn->comp_off[a];
  const uint32_t cs = scn->comp_stride[a];
  uint64_t rank = r;
  int rem = total;
  for (int pos = 0; pos < stride; ++pos) {
    int v = 0;
    if (pos < p) {
      const int left = p - 1 - pos;
      for (;; ++v) {
        const uint64_t cnt = tab[(uint32_t)left * cs + (uint32_t)(rem - v)];
        if (rank < cnt) break;
        rank -= cnt;
      }
      rem -= v;
    }
    row[pos] = (uint32_t)v;
  }
}
struct ExpandArgs {
  const uint64_t *base;         // [partition of the pass] cost without penalties, ~0 = does not fit
  const uint32_t *weights;      // [partition of the pass][affected stage][8]
  const uint32_t *rows[DEV_MAX_AFF];
  uint64_t R[DEV_MAX_AFF];      // valid reroute vectors per affected stage
  int32_t stride[DEV_MAX_AFF], peers[DEV_MAX_AFF];
  int32_t n_aff;
  uint64_t R_joint, K;
  uint64_t local_first, count;  // plan indices local to the family
  uint64_t part_base;           // first partition of the pass
  int64_t *costs;
};

// one lane per plan index: split the index into (partition, per-stage reroute ranks), look the
// vectors up, add the penalties to the partition's base cost, store (coalesced)
__global__ void __launch_bounds__(BLOCK) k_expand(ExpandArgs a) {
  const uint64_t gid = (uint64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (gid >= a.count) return;
  const uint64_t local = a.local_first + gid;
  const uint64_t part = local / a.R_joint;
  uint64_t rr = local - part * a.R_joint;
  const uint64_t pl = part - a.part_base;
  const uint64_t base = a.base[pl];
  uint64_t pen = 0;
  for (int s = a.n_aff - 1; s >= 0; --s) {          // last affected stage is least significant
    const uint64_t q = rr / a.R[s];
    const uint64_t r = rr - q * a.R[s];
    rr = q;
    const uint32_t *row = a.rows[s] + r * (uint64_t)a.stride[s];
    const uint32_t *w = a.weights + pl * (a.n_aff * ROWS_MAX_P) + s * 8;
    uint32_t m = 0;
    for (int i = 0; i < a.peers[s]; ++i) {
      const uint32_t v = base != ~0ull ? __umul24(row[i], w[i]) : 0u;
      m = m > v ? m : v;
    }
    pen += m;
  }
  __builtin_nontemporal_store((int64_t)(base == ~0ull ? CHM_INF_COST : (int64_t)(base + a.K * pen)), &a.costs[gid]);
}

// The same with 32-bit index arithmetic (ExpandArgs32), for reroute spaces below 2^31 vectors per partition and launches of at
// most 2^31 plan indices.
__device__ __forceinline__ int64_t expand_one(const ExpandArgs32 &a, uint32_t gid) {
  const uint32_t idx = a.first_rr + gid;
  const uint32_t q = fast_div(idx, a.R_joint);
  uint32_t rr = idx - q * a.R_joint.d;
  const uint32_t pl = a.first_part + q;
  const uint64_t base = a.base[pl];
  uint64_t pen = 0;
  // unrolled over the (at most four) affected stages so that the per-stage launch arguments are read with
  // constant offsets; rows are padded to 4 or 8 entries with zeros, so whole rows are read
#pragma unroll
  for (int s = DEV_MAX_AFF - 1; s >= 0; --s) {      // last affected stage is least significant
    if (s < a.n_aff) {
      uint32_t r = rr;
      if (s > 0) {                                  // the first stage takes what is left: no division
        const uint32_t qq = fast_div(rr, a.R[s]);
        r = rr - qq * a.R[s].d;
        rr = qq;
      }
      const uint32_t *w = a.weights + (size_t)pl * (a.n_aff * ROWS_MAX_P) + s * 8;
      const uint32_t *row = a.rows[s] + (size_t)r * (uint32_t)a.stride[s];
      uint32_t m = 0;
      if (a.stride[s] == 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) m = max(m, __umul24(row[i], w[i]));
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) m = max(m, __umul24(row[i], w[i]));
      }
      pen += m;
    }
  }
  return base == ~0ull ? CHM_INF_COST : (int64_t)(base + a.K * pen);
}

__global__ void __launch_bounds__(BLOCK) k_expand32(ExpandArgs32 a) {
  // a lane owns two neighbouring plan indices per tile of 2 * BLOCK and stores them as one 16-byte word
  const uint32_t first = blockIdx.x * (EXPAND_PER * BLOCK) + 2 * threadIdx.x;
  int64_t cost[EXPAND_PER];
#pragma unroll
  for (int rep = 0; rep < EXPAND_PER; ++rep) {
    const uint32_t gid = first + (rep >> 1) * (2 * BLOCK) + (rep & 1);
    cost[rep] = expand_one(a, gid < a.count ? gid : a.count - 1);   // lanes past the end redo the last index
  }
  const bool aligned = (((uintptr_t)a.costs) & 15u) == 0;            // uniform
#pragma unroll
  for (int rep = 0; rep < EXPAND_PER; rep += 2) {
    const uint32_t gid = first + (rep >> 1) * (2 * BLOCK);
    // streamed out, never read back here
    if (aligned && gid + 1 < a.count) {
      typedef long long pair_t __attribute__((ext_vector_type(2)));
      pair_t v;
      v.x = cost[rep];
      v.y = cost[rep + 1];
      __builtin_nontemporal_store(v, (pair_t *)(a.costs + gid));
    } else {
      if (gid < a.count) __builtin_nontemporal_store(cost[rep], &a.costs[gid]);
      if (gid + 1 < a.count) __builtin_nontemporal_store(cost[rep + 1], &a.costs[gid + 1]);
    }
  }
}

int launch_by_strategy(int strategy, int sp, const FastLaunch &a, uint32_t blocks, uint32_t tile_bytes, hipStream_t st, SearchVariant variant = SEARCH_PLAIN) {
  return strategy == 0 ? chmk_fast_search_s0(sp, a, blocks, tile_bytes, st, variant)
         : strategy == 1 ? chmk_fast_search_s1(sp, a, blocks, tile_bytes, st, variant)
                         : chmk_fast_search_s2(sp, a, blocks, tile_bytes, st, variant);
}

// most stages the kernels are instantiated for: any search, and one that packs its cuts (bounded, cut lists)
constexpr int PACKED_MAX_STAGES = 16;
constexpr uint32_t LIST_TILES = 16;
// Rows of cuts without stored costs: from this many on, what cannot win is left out (k_list_best).  2^20 rows: 8 stages with every option,
// strategy 0 57 us one by one, 60 so, strategy 2 62 and 65, 16 stages 53 and 46; 1.5 * 2^20 rows: 66 and 63, 76 and 72, 61 and 51.
constexpr uint32_t LIST_BEST_FROM = 3 << 19;
bool stages_covered(int sp) { return sp >= 2 && sp <= DEV_MAX_S; }

// Share of uniformly drawn partitions into `sp` stages whose largest per-node peak memory stays within the cap
// (the filter of largest_peak, on the host).  Only steers the choice between two kernels with equal results.
constexpr int FIT_SAMPLES = 128;
constexpr float QUEUE_BELOW_SHARE = 0.80f;
float estimate_fit_share(const DevScenario &h, const FastFamily &ff, int strat, int sp) {
  const int L = h.L, k = sp - 1, n = L - 1;
  uint64_t state = 0x9e3779b97f4a7c15ull ^ ((uint64_t)L << 32) ^ ((uint64_t)sp << 8) ^ (uint64_t)strat;
  auto next = [&state]() {                   // splitmix64
    uint64_t z = (state += 0x9e3779b97f4a7c15ull);
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
  };
  int fit = 0;
  for (int smp = 0; smp < FIT_SAMPLES; ++smp) {
    // k distinct cut positions out of 1..n, each subset equally likely: for j = n-k+1..n draw t from 1..j and
    // take t, or j when t is already taken; the chosen positions are bits of a mask
    uint64_t chosen[2] = {0, 0};
    for (int j = n - k + 1; j <= n; ++j) {
      const int t = 1 + (int)(((next() >> 32) * (uint64_t)j) >> 32);
      const int pick = (chosen[t >> 6] >> (t & 63)) & 1 ? j : t;
      chosen[pick >> 6] |= 1ull << (pick & 63);
    }
    int c[DEV_MAX_S + 1];
    c[0] = 0;
    int filled = 1;
    for (int w = 0; w < 2; ++w)
      for (uint64_t m = chosen[w]; m; m &= m - 1) c[filled++] = w * 64 + __builtin_ctzll(m);
    c[sp] = L;
    int64_t st[DEV_MAX_S], ac[DEV_MAX_S];
    for (int s = 0; s < sp; ++s) { st[s] = h.pw[c[s + 1]] - h.pw[c[s]]; ac[s] = h.pa[c[s + 1]] - h.pa[c[s]]; }
    int64_t peak = 0;
    for (int s = 0; s < sp; ++s) {
      const int coef = ff.mem_coef[s];
      if (coef < 0) continue;
      const int64_t a = strat == 0 ? st[s] + st[(s + 1) % sp] : st[s];
      const int64_t b = strat == 0 ? ac[s] + ac[(s + 1) % sp] : ac[s];
      peak = std::max(peak, a + (ff.has_act ? b * coef : 0));
    }
    if (peak <= (int64_t)h.cap) ++fit;
  }
  return (float)fit / (float)FIT_SAMPLES;
}

// Partitions of all families of a call up to which they are searched in one launch.  us a search, one launch after the other /
// together: 9,455 partitions of 4 stages 39 / 31, 0.5 M of 6 stages 65 / 52, 3.6 M of 8 stages at uneven speeds 127 / 106 and, where a
// tenth of them fits (apart, a ring per wavefront collects those that do), 100 / 80; 9.7 M 285 / 241 and 182 / 153; 18.6 M 360 / 353;
// 34 M 572 / 592 and 430 / 410: by then each family fills the device by itself.
constexpr uint64_t FAMILIES_UP_TO = 1ull << 24;

// Search by halves (chm_halves_kernel.h): which families.
//
// Partitions from which a family goes by halves: below, its seeds, its table and the fixed cost of a wavefront weigh more than the
// partitions.  The two meet at 1.1 to 2.0 M partitions, whatever the depth; us a search, range kernel / by halves, strategies 0 and 2: 5 stages,
// 1.5 M 40 / 44 and 46 / 48, 2.1 M 47 / 44 and 51 / 49, 10.3 M 94 / 53 and 98 / 54; 6 stages, 1.1 M 40 / 40 and 43 / 46, 2.1 M 49 / 42 and
// 53 / 47; 8 stages, 1.2 M 45 / 51 and 46 / 47, 2.6 M 63 / 46 and 63 / 48; 12 stages, 0.7 M 44 / 51 and 45 / 51, 2.5 M 76 / 58 and 73 / 56; 16
// stages, 0.5 M 51 / 53 and 53 / 55, 3.3 M 118 / 72 and 111 / 68.
constexpr uint64_t HALVES_FROM = 1ull << 21;
// Units of work a wavefront is given at least where there is more than one round of them (8 stages, 48 layers, one round / two / three 82 / 84 / 88
// us a search, strategy 0; 5.2 G partitions of 11 stages 3,240 / 2,880 / 2,660 us with 2 / 4 / 8 rounds).
constexpr uint64_t HALVES_UNITS = 256;
constexpr uint64_t HALVES_TWO_CHOICES = 1ull << 24;      // (see halves_walked)

// Most units of work of a wavefront: its workgroup counts the partitions that fit, up to 2 x 64 a unit, in 32 bits.
constexpr uint64_t HALVES_MOST_UNITS = 1ull << 22;

// The work of the search and the wavefronts it is shared out among: as many as are resident at a time, or several times as many where
// each still has a few hundred units.  Small families, which leave wavefronts idle however they are shared out, in shares of 16 units: setting
// a block up again for its next share costs less than walking on does (6 stages, 52 layers, us a search bounded / strategy 0 exhaustive,
// shares of 128, 64, 40, 24, 16: 72, 64, 61, 58, 58 / 48, 43, 42, 41, 41).
void halves_share(const DevScenario &h, int sp, int k, HalvesShape *hs) {
  const int walked = halves_walked(sp), kept = sp - 1 - walked;
  for (int c = 0; c < 2; ++c) {
    hs->units[c] = 0;
    for (int v = kept; v <= h.L - 1 - walked; ++v) hs->units[c] += halves_units(&h, walked, v) * halves_blocks(&h, kept, c + 1, v);
    auto items = [&](bool pruned) -> uint32_t {
      const uint64_t resident = 1024u * (uint64_t)halves_waves(sp, k, c + 1, pruned);
      const uint64_t rounds = std::min<uint64_t>(8, hs->units[c] / (HALVES_UNITS * resident));
      return (uint32_t)(rounds ? rounds * resident : std::max<uint64_t>(1, std::min<uint64_t>(resident, hs->units[c] / 16)));
    };
    hs->n_items[c] = items(false);
    if (c == 0) hs->n_items_pruned = items(true);
  }
}

HalvesShape halves_shape(const FastTables *t, const DevScenario &h, int k) {
  const FastFamily &ff = t->fam[k];
  const int sp = h.fam[k].stages;
  const HalvesShape none;
  if (h.fam[k].n_part < HALVES_FROM || sp < 5 || sp > 16 || !ff.time24 || (k == 0 && ff.allreduce > 0)) return none;
  for (int ci = 0; ci < ff.n_cls; ++ci)
    if (!ff.cls[ci].unit || ff.cls[ci].M < sp) return none;
  if (k != 0 && ff.n_time > 1) return none;
  for (int s = 0; k == 2 && s < h.n_aff; ++s)
    if (t->even_share[s] == 0) return none;
  HalvesShape hs;
  const int walked = halves_walked(sp), kept = sp - 1 - walked;
  if (h.L - 1 - walked < kept) return none;
  for (int v = kept; v <= h.L - 1 - walked; ++v) {
    // (ranks of the lanes' cuts are 32 bits wide, of up to two blocks beyond the last one)
    if (h.binom[kept][v - 1] >= (1ull << 32) - 128 || h.binom[kept - 1][v - 1] >= (1ull << 32) - 128) return none;
    const uint64_t blocks = halves_blocks(&h, kept, 1, v);
    hs.blocks += blocks;
    hs.steps += blocks * h.binom[walked][h.L - 1 - v];
  }
  halves_share(h, sp, k, &hs);
  for (int c = 0; c < 2; ++c)
    if (hs.units[c] / (c == 0 ? std::min(hs.n_items[0], hs.n_items_pruned) : hs.n_items[c]) >= HALVES_MOST_UNITS) return none;
  hs.walked = walked;
  return hs;
}

}  // namespace

static void fast_quiesce(FastState *f) {
  if (f->quiesce) f->quiesce(f->owner);
}

// rows of the rank-ordered vector table, decoded on the device (queued on the stream that reads them)
static bool build_vector_rows(FastState *f, const DevScenario &h, hipStream_t st) {
  const FastTables *t = &f->h_tables;
  if (!f->d_vecs && !pool_take(f->d_vecs, f->vec_words * sizeof(uint32_t))) return false;
  for (int a = 0; a < h.n_aff; ++a) {
    const int stride = h.aff_peers[a] <= 4 ? 4 : 8;
    hipLaunchKernelGGL(k_make_rows, dim3((t->vec_rows[a] + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, st, f->d_scn, f->d_comp, a,
                       f->d_vecs + t->vec_off[a], t->vec_rows[a], stride);
  }
  return hipGetLastError() == hipSuccess;
}

void fast_select(FastState *f, const DevScenario &h, bool int32_ok) {
  for (bool &u : f->usable) u = false;
  for (HalvesShape &hs : f->halves) hs = HalvesShape();
  f->large_reroute = f->rows_ok = false;
  f->mul24_reroute = false;
  f->vec_words = 16;
  memset(&f->h_tables, 0, sizeof(f->h_tables));
  if (!int32_ok) return;
  // memory side of the int32 kernels: doubled static sums plus the largest activation term stay below
  // 2^31, and the (doubled) activation sums fit the 24-bit multiply
  if (2 * h.pw[h.L] + 2 * h.pa[h.L] * (int64_t)DEV_MAX_S >= (1ll << 31) || 2 * h.pa[h.L] >= (1ll << 24)) return;
  // 24-bit multiplies in least_penalty need peer stage times below 2^24
  uint32_t q_aff = 65536;
  for (int a = 0; a < h.n_aff; ++a)
    for (int i = 0; i < h.aff_peers[a]; ++i) q_aff = std::max(q_aff, h.aff_q[a][i]);
  const bool w24 = (((h.pf[h.L] + h.pb[h.L]) * (int64_t)q_aff) >> 16) + 2 < (1ll << 24);
  f->mul24_reroute = w24;
  FastTables *t = &f->h_tables;
  size_t vec_words = 16;
  for (int k = 0; k < 3; ++k) {
    const DevFamily &fam = h.fam[k];
    if (!fam.n_part || !stages_covered(fam.stages)) continue;
    if (k == 1 && fam.fixed_step == CHM_INF_COST) continue;
    bool ok = true;
    FastFamily &ff = t->fam[k];
    ff.n_cls = fam.n_cls;
    ff.fixed_step = (int32_t)fam.fixed_step;
    ff.w_total = (int32_t)h.pw[h.L];
    for (int j = 0; j < DEV_MAX_S; ++j) ff.mem_coef[j] = fam.mem_coef[j];
    ff.has_act = h.pa[h.L] > 0 ? 1 : 0;
    ff.assign = h.assign;
    ff.allreduce = (int32_t)h.allreduce;
    ff.fixed_layers = (k == 1 && h.n_fixed > 0) ? h.p0_max_layers : 0;
    ff.node_exists = h.node_exists;
    // 24-bit multiplies in the sharper lower bound: micro-batches x (doubled) stage time, plus the prefix, below 2^31
    ff.lb_prefix = (2 * (h.pf[h.L] + h.pb[h.L]) < (1ll << 24)) && ((int64_t)(h.D * h.M + h.S) * 2 * (h.pf[h.L] + h.pb[h.L]) < (1ll << 31)) ? 1 : 0;
    if (k == 0 && h.allreduce > 0 && h.L > 64) continue;     // colour masks of the specialised kernel hold 64 colours
    for (int j = 0; j <= h.S; ++j) ff.w0[j] = (int32_t)h.pw[h.p0[j]];
    // Re-partition at nominal speed: the chains are alike and differ in their micro-batches alone, more of which never take
    // less time (every term of pipeline_time grows with M): the class with the most goes first and is the only one timed.
    std::vector<int> order;
    for (int ci = 0; ci < fam.n_cls; ++ci) order.push_back(ci);
    ff.n_time = fam.n_cls;
    // The class with the most work (micro-batches x factors of its nodes) goes first: a search by halves and a list of strategy 0
    // time the others only where that one does not decide already.
    auto work = [&fam](int c) {
      uint64_t w = 0;
      for (int j = 0; j < fam.cls[c].n; ++j) w += fam.cls[c].q[j];
      return w * (uint64_t)fam.cls[c].M;
    };
    std::stable_sort(order.begin(), order.end(), [&work](int a, int b) { return work(a) > work(b); });
    if (k == 1 && fam.n_cls > 0) {
      bool nominal = true;
      for (int ci = 0; ci < fam.n_cls; ++ci)
        for (int j = 0; j < fam.cls[ci].n; ++j) nominal = nominal && fam.cls[ci].q[j] == 65536u;
      if (nominal) {
        std::stable_sort(order.begin(), order.end(), [&fam](int a, int b) { return fam.cls[a].M > fam.cls[b].M; });
        ff.n_time = 1;
      }
    }
    uint32_t q_all = 65536;
    for (int ci = 0; ci < fam.n_cls && ok; ++ci) {
      const DevClass &c = fam.cls[order[ci]];
      FastClass &fc = ff.cls[ci];
      fc.n = c.n; fc.M = c.M; fc.comm_total = (int32_t)((c.n - 1) * h.comm);
      fc.dead = 0;
      fc.unit = 1;
      fc.q_min = c.n > 0 ? c.q[0] : 65536u;
      for (int j = 0; j < c.n; ++j) {
        fc.q_min = std::min(fc.q_min, c.q[j]);
        if (c.q[j] != 65536u) fc.unit = 0;
        fc.wlo[j] = (int32_t)h.pw[h.p0[c.host[j]]];
        fc.whi[j] = (int32_t)h.pw[h.p0[c.host[j] + 1]];
      }
      // every one of the (M + stages) scaled stage times in the bound may round down by up to two
      fc.lb_slack = fc.unit ? 0 : 2 * (c.M + fam.stages);
      if (c.n < 1 || (k != 0 && c.n != fam.stages)) ok = false;
      // per partition stage: its node's factor and position in the chain (strategy 0: some stages have none)
      for (int s = 0, j = 0; s < fam.stages; ++s) {
        const bool there = k != 0 || (j < c.n && c.src[j] == s);
        fc.q_stage[s] = there ? c.q[j] : 65536u;
        fc.steady[s] = there ? c.M - c.n + j : -1;
        if (there) ++j;
        else fc.dead |= 1u << s;
        fc.after[s] = c.n - j;
      }
      for (int j = 0; j < c.n; ++j) q_all = std::max(q_all, c.q[j]);
    }
    // stage times of the kernels are scaled (and, strategy 0, doubled) sums; prefix sums of them stay below the total
    ff.time24 = ((((h.pf[h.L] + h.pb[h.L]) * (k == 0 ? 2 : 1) * (int64_t)q_all) >> 16) + 2 * DEV_MAX_S) < (1ll << 24) ? 1 : 0;
    if (k == 2 && ok) {
      ok = w24;
      f->rows_ok = ok;
      uint64_t r_sum = 0;
      for (int a = 0; a < h.n_aff; ++a) {
        const int p = h.aff_peers[a];
        t->lb_mult[a] = (uint32_t)((h.aff_total[a] + p - 1) / p);
        t->lb_q[a] = h.aff_q[a][0];
        bool even = true;
        for (int i = 1; i < p; ++i) {
          t->lb_q[a] = std::min(t->lb_q[a], h.aff_q[a][i]);
          even = even && h.aff_q[a][i] == h.aff_q[a][0];
        }
        t->even_share[a] = even ? t->lb_mult[a] : 0u;
        if (p > ROWS_MAX_P || h.aff_R[a] > ROWS_MAX_R) { f->rows_ok = false; continue; }
        const int stride = p <= 4 ? 4 : 8;
        const uint32_t padded = (uint32_t)((h.aff_R[a] + 3) / 4 * 4);
        // stages with the same peer count, orphan count and cap share one table
        int same = -1;
        for (int b = 0; b < a; ++b)
          if (h.aff_peers[b] == p && h.aff_total[b] == h.aff_total[a]) same = b;
        t->vec_rows[a] = padded;
        if (same >= 0) t->vec_off[a] = t->vec_off[same];
        else { t->vec_off[a] = (uint32_t)vec_words; vec_words += ((size_t)padded * stride + 15) / 16 * 16; }
        r_sum += h.aff_R[a];
      }
      f->large_reroute = ok && f->rows_ok && r_sum > FAST_FUSED_R;
    }
    f->usable[k] = ok;
    if (ok) f->halves[k] = halves_shape(t, h, k);
    f->fit_share[k] = (ok && k != 2) ? -1.0f : 1.0f;      // sampled on first need
  }
  f->vec_words = vec_words;
}
int fast_prepare(FastState *f, const DevScenario &h, bool int32_ok, const DevScenario *d_scn, const uint64_t *d_comp) {
  fast_select(f, h, int32_ok);
  if (!f->usable[0] && !f->usable[1] && !f->usable[2]) return 0;
  f->d_scn = d_scn;
  f->d_comp = d_comp;
  f->vecs_ready = false;
  hipStream_t ls = (hipStream_t)f->load_stream;
  bool up = pool_take(f->d_tables, sizeof(FastTables));
  up = up && pool_staged_upload(&f->stage, f->d_tables, &f->h_tables, sizeof(FastTables), ls);
  up = (hipStreamSynchronize(ls) == hipSuccess) && up;
  f->stage.used = 0;
  return up ? 0 : 1;
}

namespace {

// scratch of plan-index scoring: per partition of a pass the cost without penalties and the peer stage times
bool ensure_scratch(FastState *f, uint64_t parts) {
  const uint32_t need = (uint32_t)std::min<uint64_t>(FAST_SUB, std::max<uint64_t>(parts, 1 << 12));
  if (f->d_base && f->d_weights && f->d_unread && f->scratch_parts >= need) return true;
  fast_quiesce(f);                                           // what is replaced may still be read by an asynchronous call
  if (f->d_unread) pool_release(f->d_unread);
  if (f->d_weights) pool_release(f->d_weights);
  if (f->d_base) pool_release(f->d_base);
  f->d_unread = nullptr; f->d_weights = nullptr; f->d_base = nullptr; f->scratch_parts = 0;
  bool ok = pool_take(f->d_base, (size_t)need * sizeof(uint64_t));
  ok = ok && pool_take(f->d_weights, (size_t)need * DEV_MAX_AFF * ROWS_MAX_P * sizeof(uint32_t));
  ok = ok && pool_take(f->d_unread, 16 * sizeof(uint64_t));
  if (ok) f->scratch_parts = need;
  return ok;
}

// Whether the lower bound of a list's rows leaves anything out: it knows the step time alone, which over the horizon has to outweigh what
// fetching the weights may cost (8 stages, 2^23 rows, a horizon of one step and dear weights: 115 us one by one, 130 with the bound; a horizon of
// 2,048 steps 99 and 68).  24-bit multiplies have to do, too.
bool times_decide(const DevScenario &h, const FastFamily &ff, int sp) {
  if (ff.lb_prefix == 0 || ff.n_cls == 0) return false;
  const double step = (double)ff.cls[0].M * (double)(h.pf[h.L] + h.pb[h.L]) / sp;
  return (double)h.K * step >= (double)h.xfer * (double)h.pw[h.L];
}

// Explicit list of partition ranks or cut positions.
int launch_list(FastState *f, const DevScenario &h, const SearchLaunch &a, hipStream_t st) {
  const int sp = h.fam[a.strategy].stages;
  // a bounded search prunes against the best cost evaluated so far: a short first launch makes one known early
  const bool bounded = a.incumbent != nullptr && a.costs_out == nullptr;
  for (uint32_t done = 0; done < a.part_count;) {
    const uint32_t n = bounded && done == 0 ? std::min<uint32_t>(LIST_FIRST, a.part_count) : a.part_count - done;
    FastLaunch fl;
    fl.s = a;
    fl.s.part_first = 0;
    fl.s.part_count = n;
    fl.s.ranks = a.ranks ? a.ranks + done : nullptr;
    fl.s.cuts = a.cuts ? a.cuts + (size_t)done * (size_t)(sp - 1) : nullptr;
    if (!bounded) fl.s.incumbent = nullptr;
    fl.pos_base = done;
    fl.tab = f->d_tables;
    // rounds of 64 entries per wavefront: as many as leave eight workgroups to every compute unit, up to LIST_TILES (the ring
    // is drained once per wavefront, by a wave that is filled in part)
    fl.per_lane = std::max<uint32_t>(1, std::min<uint32_t>(LIST_TILES, n / (BLOCK * 256 * 8)));
    fl.base_out = nullptr;
    fl.weights_out = nullptr;
    fl.cut_list = nullptr;
    fl.cut_pos = nullptr;
    fl.cut_count = nullptr;
    const uint32_t blocks = (n + BLOCK * fl.per_lane - 1) / (BLOCK * fl.per_lane);
    const bool best_only = !bounded && a.evaluated != nullptr;
    const int rc = best_only ? chmk_list_best(a.strategy, sp, fl, st) : launch_by_strategy(a.strategy, sp, fl, blocks, 0, st, SEARCH_LIST);
    if (rc) return rc;
    if (hipGetLastError() != hipSuccess) return -1;
    done += n;
  }
  return 0;
}

// Run length per lane.  Runs of at most 32 partitions (longer ones leave too few workgroups to even out the
// tail: 62.9 M partitions then make about 30 workgroups per compute unit, six rounds of the five that are
// resident); spaces below 2^25 partitions get at least 16 workgroups per compute unit and correspondingly shorter
// runs (measured on 10 to 15 M partitions: unranking once per 10 to 15 partitions costs less than the idle tail
// of fewer, longer workgroups; runs of 5 to 7 were 1 to 8 % slower).  Small spaces: runs of 4, or as short
// as lets every lane of five workgroups per CU have one: a second round of workgroups costs more than a second partition per
// lane.  (Five are resident up to 5 stages, with strategy 2 up to 8; deeper kernels hold four, three or two, and then
// run further rounds.)
uint64_t run_length(uint64_t partitions) {
  const uint64_t lanes_balanced = 256ull * 16 * BLOCK, lanes_resident = 256ull * 5 * BLOCK;
  uint64_t per = partitions / lanes_balanced;
  if (per < 4) per = std::min<uint64_t>(4, (partitions + lanes_resident - 1) / lanes_resident);
  return std::max<uint64_t>(1, std::min<uint64_t>(per, 32));
}

int launch_search(FastState *f, const DevScenario &h, const SearchLaunch &a, uint64_t *base_out, uint32_t *weights_out,
                  hipStream_t st) {
  FastLaunch fl;
  fl.s = a;
  fl.cut_list = nullptr;
  fl.cut_pos = nullptr;
  fl.cut_count = nullptr;
  fl.tab = f->d_tables;
  fl.base_out = base_out;
  fl.weights_out = weights_out;
  uint64_t per = run_length(a.part_count);
  if (a.jump_at != 0xffffffffu) per = 1;               // a run must not straddle two windows
  else if (a.costs_out != nullptr) per = std::min<uint64_t>(per, 8);   // bounds the LDS tile of the cost store
  fl.per_lane = (uint32_t)per;
  const uint32_t tile_bytes = (a.costs_out != nullptr && per > 1) ? (uint32_t)(BLOCK * per * sizeof(int64_t)) : 0u;
  const uint64_t lanes = (a.part_count + per - 1) / per;
  const uint32_t blocks = (uint32_t)((lanes + BLOCK - 1) / BLOCK);
  const int sp = h.fam[a.strategy].stages;
  // pure range search of a family in which a good share of the partitions fails the memory filter
  // (a bounded search needs the ring: only there a wave decides what to evaluate before it evaluates)
  const bool pure_range = a.costs_out == nullptr && base_out == nullptr;
  const bool queued = pure_range && sp <= PACKED_MAX_STAGES && (a.incumbent != nullptr ||
                                     (a.strategy != 2 && f->queue_mode != 0 &&
                                      (f->queue_mode > 0 || fast_fit_share(f, h, a.strategy) < QUEUE_BELOW_SHARE)));
  if (!queued) { fl.s.incumbent = nullptr; fl.s.evaluated = nullptr; }
  const int rc = launch_by_strategy(a.strategy, sp, fl, blocks, tile_bytes, st, queued ? SEARCH_QUEUED : SEARCH_PLAIN);
  if (rc) return rc;
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace

namespace {
int64_t scale_floor_host(int64_t x, uint32_t q) {
  return q == 65536u ? x : std::max<int64_t>(0, ((x * (int64_t)q) >> 16) - 1);
}
}  // namespace

bool fast_candidates_build(const FastState *f, const DevScenario &h, int k, uint64_t incumbent, CandidateSet *out) {
  out->total = 0;
  if (k < 0 || k > 2 || !f->usable[k] || incumbent == ~0ull) return false;
  const FastTables &t = f->h_tables;
  const FastFamily &ff = t.fam[k];
  const int sp = h.fam[k].stages, L = h.L;
  if (sp < 2 || sp > PACKED_MAX_STAGES || L > 255) return false;
  const size_t W = (size_t)L + 1;
  out->stages = sp;
  out->L = L;
  out->ways.assign((size_t)sp * W * W, 0);
  out->low_pair.assign((size_t)sp * W, 0);
  if (incumbent < (uint64_t)h.reconf[k]) return true;                     // nothing can reach it
  const int64_t limit = (int64_t)((incumbent - (uint64_t)h.reconf[k]) / (uint64_t)h.K);   // largest step time that may still win
  if ((int64_t)ff.fixed_step > limit) return true;
  auto pc = [&](int x) { return h.pf[x] + h.pb[x]; };
  // stage s = layers [b, e) taken alone (strategies 1 and 2): lower bound of the step time it implies, and its memory
  auto single_ok = [&](int s, int b, int e) {
    if (k == 0) return true;
    const int coef = ff.mem_coef[s];
    if (coef >= 0 && (h.pw[e] - h.pw[b]) + (ff.has_act ? (h.pa[e] - h.pa[b]) * coef : 0) > h.cap) return false;
    const int64_t c = pc(e) - pc(b);
    int64_t lb = 0;
    for (int ci = 0; ci < ff.n_cls; ++ci) {
      const FastClass &cl = ff.cls[ci];
      int64_t v = (int64_t)cl.M * c + pc(b);
      // At nominal speed also the wait before the stage's first backward counts: that one cannot start before
      // micro-batch 0 has gone forward through every stage and backward through the stages behind this one,
      // by which time the stage has at most run its warm-up forwards and one more (stages - 1 - s + 1 of them)
      if (cl.unit && cl.M >= sp - s) v += std::max<int64_t>(0, (pc(L) - pc(e)) - (int64_t)(sp - 1 - s) * (h.pf[e] - h.pf[b]));
      lb = std::max(lb, std::max<int64_t>(0, scale_floor_host(v, cl.q_min) - cl.lb_slack) + cl.comm_total);
    }
    if (ff.allreduce > 0) lb += (int64_t)ff.allreduce * (e - b);
    if (k == 2)
      for (int a = 0; a < h.n_aff; ++a)
        if (h.aff_stage[a] == s) lb += (int64_t)t.lb_mult[a] * scale_floor_host(c, t.lb_q[a]);
    return lb <= limit;
  };
  // node s of the ring under redundant computation runs stages s and s+1 = layers [a, e)
  auto pair_ok = [&](int s, int a, int e) {
    const int coef = ff.mem_coef[s];
    if (coef >= 0 && (h.pw[e] - h.pw[a]) + (ff.has_act ? (h.pa[e] - h.pa[a]) * coef : 0) > h.cap) return false;
    const int64_t c = pc(e) - pc(a);
    for (int ci = 0; ci < ff.n_cls; ++ci) {
      const FastClass &cl = ff.cls[ci];
      if ((cl.dead >> s) & 1u) continue;
      if (std::max<int64_t>(0, scale_floor_host((int64_t)cl.M * c, cl.q_min) - cl.lb_slack) + cl.comm_total > limit) return false;
    }
    return true;
  };
  if (k == 0) {
    // both terms fall as the pair starts later: the allowed starts are those from the first one on from which all pass
    for (int s = 0; s + 1 < sp; ++s)
      for (int e = s + 2; e <= L; ++e) {
        int a = e - 2;
        while (a >= 0 && pair_ok(s, a, e)) --a;
        out->low_pair[(size_t)s * W + e] = (uint8_t)(a + 1);              // e - 1: no start passes
      }
  }
  auto ways = [&](int s, int a, int b) -> uint64_t & { return out->ways[((size_t)s * W + b) * W + a]; };
  for (int b = 1; b <= L - (sp - 1); ++b)
    if (single_ok(0, 0, b)) ways(0, 0, b) = 1;
  std::vector<uint64_t> from(W + 1);
  for (int s = 1; s < sp; ++s) {
    for (int a = s; a <= L - (sp - s); ++a) {
      // from[x] = ways to arrange stages 0..s-1 with stage s-1 = [x', a), x' >= x
      from[a] = 0;
      for (int x = a - 1; x >= 0; --x) from[x] = from[x + 1] + ways(s - 1, x, a);
      const int b_lo = a + 1, b_hi = s == sp - 1 ? L : L - (sp - 1 - s);
      for (int b = (s == sp - 1 ? L : b_lo); b <= b_hi; ++b) {
        if (!single_ok(s, a, b)) continue;
        const int lo = std::min<int>(std::max<int>(out->low_pair[(size_t)(s - 1) * W + b], s - 1), a);
        ways(s, a, b) = from[lo];
      }
    }
  }
  uint64_t total = 0;
  for (int a = sp - 1; a < L; ++a) total += ways(sp - 1, a, L);
  out->total = total;
  // what the enumeration reads: per (stage, end) the counts accumulated over the starts
  for (int s2 = 0; s2 < sp; ++s2)
    for (int b = 0; b <= L; ++b) {
      uint64_t *row = out->ways.data() + ((size_t)s2 * W + b) * W;
      for (int a = 1; a <= L; ++a) row[a] += row[a - 1];
    }
  static uint64_t next_serial = 0;
  out->serial = __atomic_add_fetch(&next_serial, 1, __ATOMIC_RELAXED);
  return true;
}

void fast_candidate_cuts(const CandidateSet &cs, uint64_t idx, uint8_t *cuts) {
  const size_t W = (size_t)cs.L + 1;
  int s = cs.stages - 1, end = cs.L;
  int start = candidate_start(cs.ways.data() + ((size_t)s * W + end) * W, s, end - 1, idx);
  for (;;) {
    cuts[s - 1] = (uint8_t)start;
    if (s == 1) break;
    const int first = std::max<int>(cs.low_pair[(size_t)(s - 1) * W + end], s - 1);
    const int below = first >= start - 1 ? start - 1 : candidate_start(cs.ways.data() + ((size_t)(s - 1) * W + start) * W, first, start - 1, idx);
    end = start;
    start = below;
    --s;
  }
}

int fast_candidates_search(FastState *f, const DevScenario &h, const SearchLaunch &a, const CandidateSet &cs, uint64_t stride,
                           void *stream) {
  if (cs.total == 0 || a.part_count == 0) return 0;
  if (a.part_count > CAND_PASS || a.idx_bits < 23 || stride < 1 || (a.part_first + a.part_count - 1) * stride >= cs.total) return 1;
  hipStream_t st = (hipStream_t)stream;
  const uint32_t total = a.part_count;
  const uint32_t blocks = (total + BLOCK - 1) / BLOCK;
  if (f->cand_capacity < total) {
    fast_quiesce(f);
    if (f->d_cand_list) pool_release(f->d_cand_list);
    if (f->d_cand_pos) pool_release(f->d_cand_pos);
    if (f->d_cand_count) pool_release(f->d_cand_count);
    f->d_cand_list = nullptr; f->d_cand_pos = nullptr; f->d_cand_count = nullptr; f->cand_capacity = 0;
    const uint64_t cap = std::max<uint64_t>(1 << 16, (uint64_t)blocks * BLOCK);
    bool ok = pool_take(f->d_cand_list, cap * sizeof(uint4));
    ok = ok && pool_take(f->d_cand_pos, cap * sizeof(uint32_t));
    ok = ok && pool_take(f->d_cand_count, cap / BLOCK * sizeof(uint32_t));
    if (!ok) return -1;
    f->cand_capacity = cap;
  }
  if (f->cand_ways_capacity < cs.ways.size()) {
    fast_quiesce(f);
    if (f->d_cand_ways) pool_release(f->d_cand_ways);
    if (f->d_cand_low) pool_release(f->d_cand_low);
    f->d_cand_ways = nullptr; f->d_cand_low = nullptr; f->cand_ways_capacity = 0; f->cand_serial = 0;
    bool ok = pool_take(f->d_cand_ways, cs.ways.size() * sizeof(uint64_t));
    ok = ok && pool_take(f->d_cand_low, cs.ways.size());      // more than stages x (L+1)
    if (!ok) return -1;
    f->cand_ways_capacity = cs.ways.size();
  }
  if (f->cand_serial != cs.serial) {
    // The tables go through a pinned staging buffer: a copy from pageable memory keeps the host busy until the data
    // has left (tens of microseconds for the 150 KB of the 32-card shape, during which nothing is launched), a copy
    // from pinned memory is queued and done.  An event tells when the buffer may be written again.
    f->cand_serial = 0;
    const size_t ways_bytes = cs.ways.size() * sizeof(uint64_t), low_bytes = cs.low_pair.size();
    if (f->cand_stage_capacity < ways_bytes + low_bytes) {
      if (f->cand_copied && hipEventSynchronize((hipEvent_t)f->cand_copied) != hipSuccess) return -1;
      if (f->h_cand_stage) pool_release(f->h_cand_stage);
      f->h_cand_stage = nullptr; f->cand_stage_capacity = 0;
      if (!pool_take_pinned(f->h_cand_stage, ways_bytes + low_bytes)) return -1;
      f->cand_stage_capacity = ways_bytes + low_bytes;
    }
    if (!f->cand_copied) {
      hipEvent_t ev = nullptr;
      if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) return -1;
      f->cand_copied = ev;
    } else if (hipEventSynchronize((hipEvent_t)f->cand_copied) != hipSuccess) {
      return -1;
    }
    memcpy(f->h_cand_stage, cs.ways.data(), ways_bytes);
    memcpy(f->h_cand_stage + ways_bytes, cs.low_pair.data(), low_bytes);
    if (hipMemcpyAsync(f->d_cand_ways, f->h_cand_stage, ways_bytes, hipMemcpyHostToDevice, st) != hipSuccess) return -1;
    if (hipMemcpyAsync(f->d_cand_low, f->h_cand_stage + ways_bytes, low_bytes, hipMemcpyHostToDevice, st) != hipSuccess) return -1;
    if (hipEventRecord((hipEvent_t)f->cand_copied, st) != hipSuccess) return -1;
    f->cand_serial = cs.serial;
  }
  CandidateEnum e;
  e.ways = f->d_cand_ways; e.low_pair = f->d_cand_low; e.stages = cs.stages; e.L = cs.L; e.total = total; e.first = a.part_first; e.stride = stride;
  e.cut_list = (uint4 *)f->d_cand_list; e.cut_pos = f->d_cand_pos; e.cut_count = f->d_cand_count;
  hipLaunchKernelGGL(k_enumerate_candidates, dim3(blocks), dim3(BLOCK), 0, st, e);
  FastLaunch fl;
  fl.s = a;
  fl.s.ranks = nullptr;
  fl.s.cuts = nullptr;
  fl.s.costs_out = nullptr;
  fl.s.part_first = 0;
  fl.s.part_count = total;
  fl.s.evaluated = nullptr;
  fl.tab = f->d_tables;
  fl.per_lane = 1;                        // one round per region of BLOCK candidates
  fl.base_out = nullptr;
  fl.weights_out = nullptr;
  fl.cut_list = (const uint4 *)f->d_cand_list;
  fl.cut_pos = f->d_cand_pos;
  fl.cut_count = f->d_cand_count;
  const int sp = h.fam[a.strategy].stages;
  const int rc = launch_by_strategy(a.strategy, sp, fl, blocks, 0, st);
  if (rc) return rc;
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

float fast_fit_share(FastState *f, const DevScenario &h, int k) {
  if (k < 0 || k > 2) return 1.0f;
  if (f->fit_share[k] < 0.0f) f->fit_share[k] = estimate_fit_share(h, f->h_tables.fam[k], k, h.fam[k].stages);
  return f->fit_share[k];
}

bool fast_can_bound(const FastState *f, const DevScenario &h, const SearchLaunch &a) {
  if (a.strategy < 0 || a.strategy > 2 || !f->usable[a.strategy]) return false;
  return a.costs_out == nullptr && h.fam[a.strategy].stages <= PACKED_MAX_STAGES;
}

bool fast_list_leaves_out(const FastState *f, const DevScenario &h, const SearchLaunch &a, uint64_t n) {
  if (!fast_can_bound(f, h, a) || a.cuts == nullptr || a.incumbent != nullptr || n < LIST_BEST_FROM) return false;
  return times_decide(h, f->h_tables.fam[a.strategy], h.fam[a.strategy].stages);
}

bool fast_halves_covers(const FastState *f, const DevScenario &h, int k, uint64_t partitions) {
  return k >= 0 && k <= 2 && f->halves[k].walked != 0 && partitions == h.fam[k].n_part;
}

uint64_t fast_halves_blocks(const FastState *f, int k) { return f->halves[k].blocks; }

int fast_halves_choices(const FastState *f, const DevScenario &h, int k, bool bounded) {
  if (bounded || h.fam[k].stages < HALVES_TWO_CHOICES_FROM) return 1;
  if (f->halves_choices_set != 0) return f->halves_choices_set;
  return f->halves[k].units[0] >= HALVES_TWO_CHOICES ? 2 : 1;
}

int fast_halves_search(FastState *f, const DevScenario &h, const SearchLaunch &a, uint64_t partitions, uint32_t chunk_words,
                       bool may_allocate, bool bounded, void *stream) {
  const int k = a.strategy;
  if (!fast_halves_covers(f, h, k, partitions)) return 1;
  const HalvesShape &hs = f->halves[k];
  const int sp = h.fam[k].stages;
  if (!f->d_pairs[k]) {
    // (no memory for the table: the range kernel needs none)
    if (!may_allocate || !pool_take(f->d_pairs[k], halves_table_bytes(h.L))) return 1;
  }
  HalvesLaunch hl;
  hl.s = a;
  hl.tab = f->d_tables;
  hl.chunk_words = chunk_words;
  hl.bounded = bounded ? 1 : 0;
  hl.choices = (uint32_t)fast_halves_choices(f, h, k, bounded);
  hl.n_units = hs.units[hl.choices - 1];
  hl.n_items = f->halves_items_set != 0 ? (uint32_t)std::max<uint64_t>(f->halves_items_set, hl.n_units / HALVES_MOST_UNITS + 1) : bounded ? hs.n_items_pruned : hs.n_items[hl.choices - 1];
  hl.per_item = (hl.n_units + hl.n_items - 1) / hl.n_items;
  hl.n_rows = (uint32_t)(h.L + 1);
  hl.pairs = f->d_pairs[k];
  hl.items = (HalvesItems *)(f->d_pairs[k] + (size_t)((h.L + 1) * (h.L + 1)) * PAIR_RECORD_WORDS);     // (records are whole 32 bytes)
  const bool build = !f->pairs_ready[k];
  const int rc = k == 0 ? chmk_halves_s0(sp, hl, build, stream)
                 : k == 1 ? chmk_halves_s1(sp, hl, build, stream) : chmk_halves_s2(sp, hl, build, stream);
  if (rc) return rc;
  if (hipGetLastError() != hipSuccess) return -1;
  f->pairs_queued[k] = true;
  return 0;
}

void fast_halves_settled(FastState *f) {
  for (int k = 0; k < 3; ++k) {
    f->pairs_ready[k] = f->pairs_ready[k] || f->pairs_queued[k];
    f->pairs_queued[k] = false;
  }
}

int fast_search(FastState *f, const DevScenario &h, const SearchLaunch &a, void *stream) {
  if (a.strategy < 0 || a.strategy > 2 || !f->usable[a.strategy]) return 1;
  if (a.part_count == 0) return 0;
  hipStream_t st = (hipStream_t)stream;
  const bool list = a.ranks != nullptr || a.cuts != nullptr;
  if (list && h.fam[a.strategy].stages > PACKED_MAX_STAGES) return 1;
  return list ? launch_list(f, h, a, st) : launch_search(f, h, a, nullptr, nullptr, st);
}

int fast_search_families(FastState *f, const DevScenario &h, const SearchLaunch *a, int n, void *stream) {
  FamiliesLaunch fl;
  memset((void *)&fl, 0, sizeof(fl));
  uint64_t total = 0;
  int deep = 0, s1 = 0;
  for (int i = 0; i < n; ++i) {
    const int k = a[i].strategy;
    if (k < 0 || k > 2 || !f->usable[k] || a[i].ranks || a[i].cuts || a[i].costs_out || fl.family[k].tab) return 1;
    fl.family[k].s = a[i];
    fl.family[k].tab = f->d_tables;
    total += a[i].part_count;
    (k == 1 ? s1 : deep) = h.fam[k].stages;            // (strategies 0 and 2 have the stages of the grid)
  }
  if (deep == 0 || total > FAMILIES_UP_TO) return 1;
  if (s1 == 0) s1 = deep - 1;
  const uint64_t per = run_length(total);
  uint32_t blocks = 0;
  for (int k = 0; k < 3; ++k) {
    if (!fl.family[k].tab) continue;
    fl.family[k].per_lane = fl.family[k].s.jump_at != 0xffffffffu ? 1 : (uint32_t)per;       // (a run must not straddle two windows)
    fl.blocks[k] = (uint32_t)((fl.family[k].s.part_count + BLOCK * fl.family[k].per_lane - 1) / (BLOCK * fl.family[k].per_lane));
    blocks += fl.blocks[k];
  }
  if (blocks == 0) return 0;
  const int rc = deep <= 8 ? chmk_families_8(deep, s1, fl, blocks, stream) : deep <= 12 ? chmk_families_12(deep, s1, fl, blocks, stream)
                 : deep <= 16 ? chmk_families_16(deep, s1, fl, blocks, stream) : chmk_families_24(deep, s1, fl, blocks, stream);
  if (rc) return rc;
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int fast_score_reroute(FastState *f, const DevScenario &h, const DevScenario *d_scn, uint64_t local_first,
                       uint64_t count, int64_t *d_costs, void *stream) {
  if (!f->usable[2] || !f->rows_ok || h.n_aff == 0) return 1;
  if (count == 0) return 0;
  hipStream_t st = (hipStream_t)stream;
  if (!f->vecs_ready) {
    // in stream order ahead of what reads them (a call captured into a graph runs later: it brings its own)
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (!build_vector_rows(f, h, st) || hipStreamIsCapturing(st, &capture) != hipSuccess) return -1;
    f->vecs_ready = capture == hipStreamCaptureStatusNone;
  }
  const FastTables &t = f->h_tables;
  const uint64_t R = h.fam[2].n_reroute;
  // one stage lost nodes, a table of at most 32 KB: costs straight from the partitions, a tile of plan indices at a time
  const uint64_t row_bytes = R * (h.aff_peers[0] <= 4 ? 16u : 32u);
  if (h.n_aff == 1 && R >= WINDOW_LEAST_R && row_bytes <= (32u << 10)) {
    for (uint64_t done = 0; done < count;) {
      const uint64_t first = local_first + done;
      WindowArgs w;
      memset((void *)&w, 0, sizeof(w));
      w.search.s = SearchLaunch();
      w.search.s.scn = d_scn;
      w.search.s.strategy = 2;
      w.search.s.idx_bits = 1;
      w.search.tab = f->d_tables;
      w.search.per_lane = 1;
      w.part_first = first / R;
      w.first_rr = (uint32_t)(first % R);
      w.R = make_fast_div((uint32_t)R);
      w.step_parts = 2 * BLOCK / (uint32_t)R;
      w.step_rr = 2 * BLOCK % (uint32_t)R;
      w.rows = f->d_vecs + t.vec_off[0];
      w.stride = h.aff_peers[0] <= 4 ? 4 : 8;
      w.K = (uint64_t)h.K;
      w.count = (uint32_t)std::min<uint64_t>(count - done, (1ull << 31) - (1ull << 20));
      w.costs = d_costs + done;
      w.tile = window_tile((uint32_t)R, w.count);
      w.in_place = row_bytes > WINDOW_BEHIND ? 1 : 0;
      const int rc = chmk_window_plans(h.fam[2].stages, w, (uint32_t)row_bytes, stream);
      if (rc) return rc;
      if (hipGetLastError() != hipSuccess) return -1;
      done += w.count;
    }
    return 0;
  }
  if (!ensure_scratch(f, (local_first + count - 1) / R - local_first / R + 1)) return -1;
  ExpandArgs e;
  memset(&e, 0, sizeof(e));
  e.base = f->d_base;
  e.weights = f->d_weights;
  e.n_aff = h.n_aff;
  for (int s = 0; s < h.n_aff; ++s) {
    e.rows[s] = f->d_vecs + t.vec_off[s];
    e.R[s] = h.aff_R[s];
    e.stride[s] = h.aff_peers[s] <= 4 ? 4 : 8;
    e.peers[s] = h.aff_peers[s];
  }
  e.R_joint = R;
  e.K = (uint64_t)h.K;
  const uint64_t last = local_first + count - 1;
  const uint64_t part_lo = local_first / R, part_hi = last / R;
  for (uint64_t p = part_lo; p <= part_hi; p += FAST_SUB) {
    const uint64_t np = std::min<uint64_t>(FAST_SUB, part_hi - p + 1);
    SearchLaunch sub = SearchLaunch();
    sub.scn = d_scn;
    sub.strategy = 2;
    sub.part_first = p;
    sub.part_count = (uint32_t)np;
    sub.idx_bits = 1;
    sub.result = f->d_unread;            // not written in this mode
    sub.feasible = f->d_unread + 1;      // scratch counter, not read
    int rc = launch_search(f, h, sub, f->d_base, f->d_weights, st);
    if (rc) return rc;
    // the plan indices of this pass: those of partitions [p, p+np) clipped to the request
    const uint64_t lo = std::max<uint64_t>(local_first, p * R);
    const uint64_t hi = std::min<uint64_t>(last, (p + np) * R - 1);
    e.local_first = lo;
    e.count = hi - lo + 1;
    e.part_base = p;
    e.costs = d_costs + (lo - local_first);
    if (R < (1ull << 31)) {
      // 32-bit index arithmetic: launches of at most 2^31 - 2^20 plan indices
      for (uint64_t done = 0; done < e.count;) {
        const uint64_t first = e.local_first + done;
        ExpandArgs32 x;
        memset(&x, 0, sizeof(x));
        x.base = e.base; x.weights = e.weights; x.n_aff = e.n_aff; x.K = e.K;
        for (int s = 0; s < h.n_aff; ++s) { x.rows[s] = e.rows[s]; x.R[s] = make_fast_div((uint32_t)e.R[s]); x.stride[s] = e.stride[s]; x.peers[s] = e.peers[s]; }
        x.R_joint = make_fast_div((uint32_t)R);
        x.first_part = (uint32_t)(first / R - p);
        x.first_rr = (uint32_t)(first % R);
        x.count = (uint32_t)std::min<uint64_t>(e.count - done, (1ull << 31) - (1ull << 20));
        x.costs = e.costs + done;
        hipLaunchKernelGGL(k_expand32, dim3((x.count + BLOCK * EXPAND_PER - 1) / (BLOCK * EXPAND_PER)), dim3(BLOCK), 0, st, x);
        done += x.count;
      }
      if (hipGetLastError() != hipSuccess) return -1;
      continue;
    }
    for (uint64_t done = 0; done < e.count;) {       // keep each grid below 2^31 blocks
      ExpandArgs part = e;
      part.local_first = e.local_first + done;
      part.count = std::min<uint64_t>(e.count - done, 1ull << 36);
      part.costs = e.costs + done;
      const uint32_t blocks = (uint32_t)((part.count + BLOCK - 1) / BLOCK);
      hipLaunchKernelGGL(k_expand, dim3(blocks), dim3(BLOCK), 0, st, part);
      done += part.count;
    }
    if (hipGetLastError() != hipSuccess) return -1;
  }
  return 0;
}

void fast_release(FastState *f) {
  if (f->cand_copied) (void)hipEventDestroy((hipEvent_t)f->cand_copied);
  f->cand_copied = nullptr;
  if (f->h_cand_stage) pool_release(f->h_cand_stage);
  f->h_cand_stage = nullptr; f->cand_stage_capacity = 0;
  if (f->d_cand_low) pool_release(f->d_cand_low);
  if (f->d_cand_ways) pool_release(f->d_cand_ways);
  if (f->d_cand_count) pool_release(f->d_cand_count);
  if (f->d_cand_pos) pool_release(f->d_cand_pos);
  if (f->d_cand_list) pool_release(f->d_cand_list);
  f->d_cand_low = nullptr; f->d_cand_ways = nullptr; f->d_cand_count = nullptr; f->d_cand_pos = nullptr; f->d_cand_list = nullptr;
  f->cand_capacity = 0; f->cand_ways_capacity = 0;
  if (f->d_unread) pool_release(f->d_unread);
  if (f->d_weights) pool_release(f->d_weights);
  if (f->d_base) pool_release(f->d_base);
  if (f->d_vecs) pool_release(f->d_vecs);
  for (uint32_t *&p : f->d_pairs) { if (p) pool_release(p); p = nullptr; }
  if (f->d_tables) pool_release(f->d_tables);
  f->d_unread = nullptr; f->d_weights = nullptr; f->d_base = nullptr;
  f->d_vecs = nullptr;
  f->d_tables = nullptr;
}
