// Shape-specialised search kernels (chm_fast.hip): interface to the host part.
#ifndef CHM_FAST_H
#define CHM_FAST_H
#include <hip/hip_runtime.h>

#include "chm_dev.h"
#include "chm_pool.h"
#include <vector>

enum {
  BLOCK = 256,               // workgroup of the search kernels
  FAST_MAX_P = 15,           // peers a stage that lost nodes can have (DEV_MAX_D - 1)
  ROWS_MAX_P = 8,            // peers and
  ROWS_MAX_R = 1 << 23,      // reroute vectors per stage up to which the vectors are tabulated for the cost store of plan indices
  FAST_FUSED_R = 4096,       // more vectors than this (all stages): a large reroute space (see FastState::large_reroute)
  FAST_SUB = 1 << 20,        // partitions per pass of the cost store of plan indices (bounds its scratch memory: 136 MB;
                             // the scratch is sized for the passes actually asked for and grows when needed)
  LIST_FIRST = 1 << 16       // entries of the first launch of a bounded list search
};

// One pipeline class in the form the specialised kernels read (all int32).
struct FastClass {
  int32_t n, M;
  uint32_t dead;                  // bit s: partition stage s has no node in this chain (strategy 0)
  int32_t unit;                   // 1: every node of the chain runs at nominal speed (no scaling)
  uint32_t q_min;                 // smallest speed factor along the chain (lower bound of the step time)
  int32_t lb_slack;               // what rounding can take from that bound when q_min scales it (0 at nominal speed)
  int32_t comm_total;             // (n-1) * comm
  // per partition stage: speed factor of its node, nodes of the chain behind it, and micro-batches - nodes + position
  // (see pipeline_time; a stage without a node: factor 65536 and -1)
  uint32_t q_stage[DEV_MAX_S];
  int32_t after[DEV_MAX_S], steady[DEV_MAX_S];
  int32_t wlo[DEV_MAX_S], whi[DEV_MAX_S];   // memory prefix at the bounds of the fault-free stage of node j
};

struct FastFamily {
  int32_t n_cls;
  int32_t n_time;                 // classes that can be the slowest: the first n_time (see fast_select)
  int32_t fixed_step;             // strategy 1: step time of the untouched pipelines
  int32_t w0[DEV_MAX_S + 1];      // memory prefix at the fault-free stage bounds
  int32_t w_total;                // memory of the whole model
  int32_t mem_coef[DEV_MAX_S];    // see DevFamily::mem_coef
  int32_t has_act;                // 0: no activation table, the peak is the static sum
  int32_t assign;                 // strategy 1: 1 = least-total-transfer assignment of survivors to new stages
  int32_t allreduce;              // time of one round of gradient communication (0: not modelled)
  int32_t fixed_layers;           // strategy 1: layers of the largest stage on a node of an untouched pipeline, else 0
  uint32_t node_exists;           // strategy 0: bit s = some pipeline still has its node of stage s
  int32_t time24;                 // 1: (doubled, scaled) stage times and their sums stay below 2^24
  int32_t lb_prefix;              // 1: the sharper lower bound (24-bit multiplies are safe for these times)
  FastClass cls[DEV_MAX_CLS];
};

struct FastTables {
  FastFamily fam[3];
  // rerouting: per affected stage, all valid reroute vectors in rank order; a row has a stride of
  // 4 (up to 4 peers) or 8 dwords, and the row count is padded to a multiple of 4
  uint32_t vec_off[DEV_MAX_AFF];  // offset (in uint32) of stage a's rows in vecs[]
  uint32_t vec_rows[DEV_MAX_AFF]; // rows including the padding
  // peers of stage a all of one speed: the extra micro-batches of the fullest peer when they share evenly; else 0
  uint32_t even_share[DEV_MAX_AFF];
  // lower bound of stage a's reroute penalty: some peer takes at least lb_mult[a] = ceil(orphans / peers)
  // micro-batches whatever the cap, each at a stage time scaled by at least lb_q[a]
  uint32_t lb_mult[DEV_MAX_AFF], lb_q[DEV_MAX_AFF];
};

// What a wavefront of the search walks (chm_halves_kernel.h): the upper half's cuts and, of the lower half's, the last ones that leave its
// lanes enough choices of the cuts below.  One more walked cut leaves an eighth of the lanes' set-ups (300 instructions) to a family of 8
// stages, but more lanes idle (8 stages, 48 layers, two / three / four walked: strategy 0 91 / 82 / 114 us a search, strategy 2 85 / 85 / 113;
// 7 stages 46 / 48; 12 stages, 31 layers, three / four 134 / 115).  A lane may keep two choices of the cuts below: half the scalar instructions and
// record loads a partition, for four wavefronts per SIMD instead of five or six.  That pays where the search takes milliseconds and is
// exhaustive (HALVES_TWO_CHOICES units of work; 5.2 G partitions of 11 stages 2,960 / 2,650 us; 8 stages 47 / 48, strategy 0 52 / 58; 29 M of
// 15 stages, strategy 0 149 / 161).
constexpr int halves_walked(int stages) { return stages <= 7 ? 2 : stages <= 10 ? 3 : 4; }
enum { HALVES_TWO_CHOICES_FROM = 10 };
// Wavefronts per SIMD: 5 from 8 stages on and 4 from 11 on, so that the set-up and the outer loops keep their vector registers (with six and
// five up to 61 of them were spilled, which small families and strategy 1 paid for: us a search of all strategies, 14 stages, 25 layers
// 114 / 90, 16 stages, 26 layers 149 / 119, 29 layers 510 / 446).  Strategy 0 of up to 13 stages, exhaustive, is better off with 5 (11 stages, 30
// layers 71, 82 with 4; 37 layers 268 and 278); bounded searches of 8 and 9 stages, most of which is set-ups, with 6 (strategy 2 of 8 stages, 48
// layers 27, 30 with 5).
constexpr int halves_waves(int stages, int strategy, int choices, bool pruned) {
  if (choices == 2) return 4;
  if (stages <= 7) return strategy == 0 ? 6 : 7;
  if (pruned && strategy != 0 && stages <= 9) return 6;
  return stages <= 10 || (strategy == 0 && stages <= 13 && !pruned) ? 5 : 4;
}
// How a family is searched by halves (chm_halves_kernel.h); walked = 0: it is not.
struct HalvesShape {
  int walked = 0;               // upper cuts a wavefront walks
  uint64_t blocks = 0;          // of 64 choices of the cuts below, to be set up
  uint64_t steps = 0;           // blocks x choices of the walked cuts
  // with one choice of the lower cuts a lane, with two:
  uint32_t n_items[2] = {0, 0}; // wavefronts of the search
  uint32_t n_items_pruned = 0;  // of a bounded one (one choice)
  uint64_t units[2] = {0, 0};   // work to share out among them
};

struct FastState {
  bool usable[3] = {false, false, false};   // per strategy: a specialised kernel covers this scenario
  // rerouting: at most 8 peers and 2^23 vectors per stage, and more than FAST_FUSED_R vectors over all stages.
  // (chm_search_best_static refuses such a family, see chm.h; no search needs it any more.)
  bool large_reroute = false;
  bool rows_ok = false;                     // the vectors of every stage can be tabulated (cost store of plan indices)
  bool mul24_reroute = false;               // peer stage times stay below 2^24: what least_penalty needs
  // Range search of strategies 0 and 1: share of the partitions that pass the memory filter, estimated at load
  // from FIT_SAMPLES seeded random partitions; below QUEUE_BELOW_SHARE the search compacts the partitions that
  // fit through a ring per wave (k_fast_search, QUEUED).  queue_mode: -1 = by that estimate, 0 = never, 1 = always.
  float fit_share[3] = {1.0f, 1.0f, 1.0f};   // negative: not sampled yet (sampled when a search first asks)
  int queue_mode = -1;
  // Set by the owner of the state before fast_prepare: the stream the library's own uploads and table kernels
  // run on (only that stream is waited for), and a call that waits until no work launched through this handle is
  // in flight any more (made before a buffer that such work may touch is replaced).
  void *load_stream = nullptr;
  PoolStage stage;                          // pinned staging of the uploads at load (the owner's; may be empty)
  void (*quiesce)(void *) = nullptr;
  void *owner = nullptr;
  FastTables h_tables;
  FastTables *d_tables = nullptr;
  uint32_t *d_vecs = nullptr;
  // scratch of the cost store of plan indices, FAST_SUB partitions at a time; allocated when first needed
  uint64_t *d_base = nullptr;               // cost without penalties, ~0 for a partition that does not fit
  uint32_t *d_weights = nullptr;            // [partition][affected stage][8] peer stage times
  uint64_t *d_unread = nullptr;             // 16 words the base pass reports to, not read
  uint32_t scratch_parts = 0;               // partitions d_base and d_weights have room for
  // The rank-ordered vector table only serves the cost store of plan indices (up to 76 MB where the vectors are many)
  // and is decoded when one first asks for it.
  bool vecs_ready = false;                  // the rank-ordered vector table (d_vecs) has been decoded
  size_t vec_words = 0;                     // size of the vector table
  const DevScenario *d_scn = nullptr;       // the handle's device tables (for that later build)
  const uint64_t *d_comp = nullptr;
  // search by halves, per strategy: records of pairs of cuts and shares of work (halves_table_bytes), laid out by the first search
  uint32_t *d_pairs[3] = {nullptr, nullptr, nullptr};
  bool pairs_ready[3] = {false, false, false};      // the table is there: a search that filled it has been waited for
  bool pairs_queued[3] = {false, false, false};     // a launch of the current search fills it, or found it ready
  HalvesShape halves[3];
  int halves_choices_set = 0;               // chm_set_halves_shares: 0 = by the rules
  uint32_t halves_items_set = 0;
  // scratch of the candidate path of the bounded search; grown to what a search needs
  void *d_cand_list = nullptr;              // [candidate] cut positions, 16 bytes each
  uint32_t *d_cand_pos = nullptr;           // [candidate] its index
  uint32_t *d_cand_count = nullptr;         // [workgroup] candidates in its region of BLOCK slots
  uint64_t cand_capacity = 0;
  uint64_t *d_cand_ways = nullptr;          // CandidateSet::ways on the device
  uint8_t *d_cand_low = nullptr;            // CandidateSet::low_pair on the device
  size_t cand_ways_capacity = 0;
  uint64_t cand_serial = 0;                 // CandidateSet::serial of the tables the device holds
  uint8_t *h_cand_stage = nullptr;          // pinned staging of the two tables on their way to the device
  size_t cand_stage_capacity = 0;
  void *cand_copied = nullptr;              // hipEvent_t: the last copy out of the staging buffer is done
};

enum SearchVariant { SEARCH_PLAIN, SEARCH_QUEUED, SEARCH_LIST };
struct FastLaunch {
  SearchLaunch s;
  const FastTables *tab;
  uint32_t per_lane;            // consecutive partition ranks per lane
  // cost store of rerouting plan indices: the kernel leaves the penalties out and stores, per partition, the cost
  // without them and the peer stage times (null: otherwise)
  uint64_t *base_out;
  uint32_t *weights_out;
  uint32_t pos_base = 0;        // list mode: list position (chunk-local) of entry 0 of this launch
  // candidate mode (bounded search): workgroup b owns slots [b * per_lane * BLOCK, ...) of cut_list / cut_pos, of which the
  // first cut_count[b] are filled.  In round `it` lane t evaluates slot it * BLOCK + t: the partition whose cut positions
  // are the bytes of cut_list[slot], reported as number cut_pos[slot] (null: other modes)
  const uint4 *cut_list;
  const uint32_t *cut_pos;
  const uint32_t *cut_count;
};

// The families of one call in one launch (k_search_families); family[k] with blocks[k] workgroups, 0 = not among them.
struct FamiliesLaunch {
  FastLaunch family[3];
  uint32_t blocks[3];
};

// Exhaustive search of a whole family by halves (chm_halves_kernel.h).
enum { PAIR_RECORD_WORDS = 8 };
struct HalvesItems {
  int4 prefix[DEV_MAX_L + 1];   // prefix sums: forward, forward + backward, static memory, activation memory
  uint64_t first[2][DEV_MAX_L]; // per last cut of the lanes, its first unit of work (lanes of one choice, of two)
  uint32_t share[DEV_MAX_S];    // strategy 2: reroute penalty of a stage as a multiple of its time
  uint32_t units[4 * DEV_MAX_L];            // row i - 1: units of i walked cuts whose leading digit is below x
  uint32_t binom[DEV_MAX_S * DEV_MAX_L];    // row i - 1: C(x, i), 0 < i <= lower cuts
};
// Work of a block of 64 choices of the lanes' cuts (`kept` of them, the last one v): what a step of the innermost loop takes is a unit;
// its set-up and a turn of the loop around (a row) take as long as this many.
enum { HALVES_SETUP = 60, HALVES_ROW = 5 };
template <typename Scenario>
__host__ __device__ inline uint64_t halves_blocks(const Scenario &h, int kept, int choices, int v) {
  return (h->binom[kept - 1][v - 1] + 64 * choices - 1) / (64 * choices);
}
template <typename Scenario>
__host__ __device__ inline uint64_t halves_units(const Scenario &h, int walked, int v) {
  return HALVES_SETUP + h->binom[walked][h->L - 1 - v] + HALVES_ROW * h->binom[walked - 1][h->L - 2 - v];
}
// Bytes of device memory for all that (128 layers: 0.56 MB).
constexpr size_t halves_table_bytes(int L) { return (size_t)((L + 1) * (L + 1)) * PAIR_RECORD_WORDS * sizeof(uint32_t) + sizeof(HalvesItems); }
static_assert(halves_table_bytes(DEV_MAX_L) < 700000, "what chm_search_best promises");
struct HalvesLaunch {
  SearchLaunch s;               // result = words of the family's first chunk
  const FastTables *tab;
  uint32_t *pairs;              // records of pairs of cuts, (L + 1)^2 of PAIR_RECORD_WORDS words
  HalvesItems *items;
  uint32_t n_rows, n_items;     // layers + 1; wavefronts
  uint64_t n_units, per_item;   // units of work, of all and of a wavefront
  uint32_t choices;             // of the lower cuts, a lane
  uint32_t bounded;             // 1: what the cuts placed so far make too slow is left out
  uint32_t chunk_words;         // words from one chunk's argmin words to the next chunk's
};

// Bounded search, candidate path.  Every term of the lower bound of a plan's cost belongs to one stage
// (micro-batches x its time + the time of the layers ahead of it, its memory) or, under redundant computation,
// to one node's pair of adjacent stages, and each is monotone in where the stage (or pair) starts: with its end
// fixed, a later start only lowers it.  The partitions whose bound does not exceed the incumbent are therefore
// exactly those whose every stage s starts at or after low_single[s][end] and whose every pair starts at or
// after low_pair[s][end of the pair]: a set that can be counted and enumerated without touching the others.
// ways[s][a][b] = number of ways to place the cuts below a so that stages 0..s obey all of that, stage s being
// layers [a, b).  Candidates are numbered in ascending partition rank (highest cut most significant).
struct CandidateSet {
  int stages = 0, L = 0;
  std::vector<uint64_t> ways;               // [stages][end b][start a], (L+1) x (L+1) per stage; once built, accumulated over
                                            // the starts (entry a = ways with a start <= a), so that a block is found by bisection
  std::vector<uint8_t> low_pair;            // [stages][L+1]: lowest start of the pair (stages s, s+1) that ends at e; 0 = no such limit
  uint64_t total = 0;                       // candidates; 0 also when the bound excludes the whole family
  uint64_t serial = 0;                      // distinguishes the sets a process builds (the device keeps the last one uploaded)
};
enum {
  CAND_DIRECT = 1 << 17,      // up to this many candidates are always enumerated (cheaper than any range search)
  CAND_HALVES = 1 << 20,      // up to this many when the family is too large for a range search, but not for one by halves,
  CAND_MAX = 1 << 26,         // and up to this many when it is too large for either,
  CAND_PASS = 1 << 22,        // enumerated and evaluated this many at a time
  CAND_SAMPLE = 1 << 17       // candidates evaluated per round of tightening the incumbent (see run_search)
};

// Counts the candidates of a strategy against an incumbent cost (host).  Returns false when the strategy has no
// specialised kernel or the tables are out of the candidate path's limits.
bool fast_candidates_build(const FastState *f, const DevScenario &h, int strategy, uint64_t incumbent, CandidateSet *out);
// Enumerates the candidates on the device and runs the search kernel over them; the key written to a.result
// carries the candidate's index.  Same return convention as fast_search.
// Launch index i stands for candidate (a.part_first + i) * stride, a.part_count of them (at most CAND_PASS).
int fast_candidates_search(FastState *f, const DevScenario &h, const SearchLaunch &a, const CandidateSet &cs, uint64_t stride,
                           void *stream);
// Cut positions of candidate `index` (host).
void fast_candidate_cuts(const CandidateSet &cs, uint64_t index, uint8_t *cuts);

// Decides per strategy whether a specialised kernel applies and fills the host copy of its tables (host only;
// a re-partition family whose untouched pipelines do not fit is still reported as covered: its fixed step time
// is only known once the device has computed it).
void fast_select(FastState *f, const DevScenario &h, bool int32_ok);
// fast_select, then uploads the tables.  Returns 0, or non-zero on a failed HIP call.
int fast_prepare(FastState *f, const DevScenario &h, bool int32_ok, const DevScenario *d_scn, const uint64_t *d_comp);
// Launches the specialised search kernel for one chunk.  Returns 0 on success, a positive
// value when the strategy is not covered (the caller then uses the generic kernel), or a
// negative value on a HIP error.
int fast_search(FastState *f, const DevScenario &h, const SearchLaunch &a, void *stream);
// Whether fast_search would run this launch as a bounded search if a.incumbent were set (a search of a covered
// strategy of at most 16 stages without cost store).
bool fast_can_bound(const FastState *f, const DevScenario &h, const SearchLaunch &a);
// Whether fast_search would take a list of n entries, of which this launch is a part, to the kernel that leaves out rows that cannot win
// (k_list_best).  It does where a.evaluated is set, the counters of the rows whose times are worked out.
bool fast_list_leaves_out(const FastState *f, const DevScenario &h, const SearchLaunch &a, uint64_t n);
// The range searches of up to three families (one launch argument each, at most one per strategy) in one launch, exhaustive; an
// incumbent word set in them is lowered by what they find.  Same return convention; positive: some family is not covered, their
// stages have no common instance, or they are large enough to fill the device one after the other.
int fast_search_families(FastState *f, const DevScenario &h, const SearchLaunch *a, int n, void *stream);
// its kernels by stages (chm_families_*.hip): 1 = no instance
int chmk_families_8(int sp, int s1, const FamiliesLaunch &a, uint32_t blocks, void *stream);      // up to 8 stages
int chmk_families_12(int sp, int s1, const FamiliesLaunch &a, uint32_t blocks, void *stream);     // up to 12
int chmk_families_16(int sp, int s1, const FamiliesLaunch &a, uint32_t blocks, void *stream);
int chmk_families_24(int sp, int s1, const FamiliesLaunch &a, uint32_t blocks, void *stream);
// Kernel launchers by strategy (chm_search_s0/1/2.hip): 1 = no instance for this number of stages, else 0.
int chmk_list_best(int strategy, int sp, const FastLaunch &a, void *stream);       // 1 = no instance for these stages
int chmk_fast_search_s0(int sp, const FastLaunch &a, uint32_t blocks, uint32_t tile_bytes, void *stream, SearchVariant variant);
int chmk_fast_search_s1(int sp, const FastLaunch &a, uint32_t blocks, uint32_t tile_bytes, void *stream, SearchVariant variant);
int chmk_fast_search_s2(int sp, const FastLaunch &a, uint32_t blocks, uint32_t tile_bytes, void *stream, SearchVariant variant);
int chmk_halves_s0(int sp, const HalvesLaunch &a, bool build, void *stream);
int chmk_halves_s1(int sp, const HalvesLaunch &a, bool build, void *stream);
int chmk_halves_s2(int sp, const HalvesLaunch &a, bool build, void *stream);
// Choices of the lower cuts a lane keeps when a family is searched by halves.
int fast_halves_choices(const FastState *f, const DevScenario &h, int k, bool bounded);
// Exhaustive search of a whole family (a.part_first = 0, `partitions` of them, which may be more than one chunk) by
// halves.  a.result = words of its first chunk, those of the next chunk chunk_words further on; a.incumbent: as in a bounded
// search, only for what chm_halves_kernel.h says.  may_allocate = false, or no memory to be had: only with tables that are already there.  Same
// return convention as fast_search (positive: not covered, or smaller than what the range search does as fast).
// fast_halves_covers: whether it takes the family at all.
bool fast_halves_covers(const FastState *f, const DevScenario &h, int strategy, uint64_t partitions);
// Blocks of 64 choices of the lower cuts that its wavefronts set up, with one choice a lane.
uint64_t fast_halves_blocks(const FastState *f, int strategy);
int fast_halves_search(FastState *f, const DevScenario &h, const SearchLaunch &a, uint64_t partitions, uint32_t chunk_words,
                       bool may_allocate, bool bounded, void *stream);
// The stream of the last search has been waited for: the tables its launches filled are there.
void fast_halves_settled(FastState *f);
// Sampled share of partitions of a strategy that pass the memory filter (1.0 where no sample applies).
float fast_fit_share(FastState *f, const DevScenario &h, int strategy);
// Scores plan indices [local_first, local_first+count) of the rerouting family (indices local to
// the family) into d_costs: one pass of the search kernel stores each partition's cost without
// penalties and its peer stage times, then one lane per plan index adds the penalty of its
// reroute vectors (looked up in the rank-ordered table) and stores the cost.  Same return
// convention as fast_search.
int fast_score_reroute(FastState *f, const DevScenario &h, const DevScenario *d_scn, uint64_t local_first,
                       uint64_t count, int64_t *d_costs, void *stream);
// the caller has waited for everything launched through the handle: the buffers can be reused at once
void fast_release(FastState *f);
#endif
