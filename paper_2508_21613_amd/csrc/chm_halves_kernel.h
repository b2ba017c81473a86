// Exhaustive search of a whole family by halves: the kernels for large spaces.  Included by one translation unit per
// strategy, behind chm_search_kernel.h.
//
// A wavefront's lanes keep the first G cuts of a partition, a choice or two of them each, all with the same last one v; the W cuts
// above are walked as nested loops, one cut each.  What a step time is made of (pipeline_time in chm_search_kernel.h, read the way
// class_time does) is a state of six numbers that takes up one stage after the other: maxima of forward and backward times, and of the
// terms that have met neither end's turn, one of them or both.  So a loop over a cut adds the stage that the cut ends to the lane's state
// (Terms::add, 12 instructions), whose times are the same for all lanes, and the innermost one, over the last cut y, is left with the two
// last stages: 13 instructions (under redundant computation 22).  What is the same for all lanes of the last two levels is a function of two
// cuts and comes from a table of (L + 1)^2 records (k_cut_records, 32 bytes each, laid out once per handle and strategy).
//
// Times are floats.  A float addition or multiply-add issues beside a maximum of another wavefront (2.6 to 3 cycles an instruction for
// such streams, 4.2 for integers).  Up to 2^24 they are the whole numbers they stand for; above, sums are rounded, and the limit they are
// compared with is raised by more than that (TIME_SLACK).  They only decide which partitions may have a cost not above the lowest met; the cost
// of these is worked out anew, in integers (consider).  Times of pipeline classes but the one with the most work take part there, too.
//
// Bound by the issue of vector instructions (0.6 to 0.7 of the rate above while all wavefronts run) and, for searches of tens of
// microseconds, by the 6 us until the first lanes are set up and the end, when few wavefronts are left on a SIMD.  With one choice a lane
// no vector registers are spilled up to 7 stages, and 4 to 23 in the set-up and the outer loops of bounded searches of 8 and 9 stages, of strategy 0
// of 11 to 13 and of strategy 1 from 9 on, where one more wavefront per SIMD is worth more; with two choices, 3 to 71 from 10 stages on (11 stages,
// strategy 1: 1.0 GB of scratch written in 2.6 ms; with three wavefronts per SIMD, which need next to none, a re-plan takes 4.44 ms instead of
// 4.30).  62.9 M partitions of
// 8 stages: 44 us (integers, a lane for every lower half: 54; one by one 434), under redundant computation 54 (66; 516), 10.7 M of 7
// stages 13 to 18 (27), 5.2 G of 11 stages 2.65 ms (3.93; 51).
#ifndef CHM_HALVES_KERNEL_H
#define CHM_HALVES_KERNEL_H
#include <type_traits>

#include "chm_search_kernel.h"

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
typedef u32x16 record_pair __attribute__((aligned(32)));       // two neighbouring records: 32 bytes each, a scalar load of 64
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));

// least reroute penalty of a stage all of whose peers have one speed (stage_penalty; nothing else comes here)
__device__ __forceinline__ uint32_t even_penalty(ScnPtr scn, TabPtr tab, int st, int f, int b) {
  return tab->even_share[st] * peer_time(f, b, scn->aff_q[st][0]);
}
constexpr float NEVER = -1e30f, HUGE_TIME = 1e30f;     // terms that do not exist, times of what does not fit
// What a stage's node lacks of the weights it is to hold ([lo, hi) of the memory prefix, stage s); where the nodes' assignment is open, what
// the node lacks that holds most of them (N = 0: it is not).
template <int N, int STRAT>
__device__ __forceinline__ int lacking(FamPtr ff, int lo, int hi, int s) {
  auto held = [&](int a, int b) { return imax32(0, imin32(hi, b) - imax32(lo, a)); };
  if (STRAT != 1) return hi - lo - held(ff->w0[s], ff->w0[s + 1]);
  const ClsPtr cl = &ff->cls[0];
  if (N == 0 || !ff->assign) return hi - lo - held(cl->wlo[s], cl->whi[s]);
  int most = 0;
  for (int j = 0; j < N; ++j) most = imax32(most, held(cl->wlo[j], cl->whi[j]));
  return hi - lo - most;
}
// time of a step that fetching so much costs: a whole number not above it (four roundings of 2^-24: the size, the price, less 2^-21, their product)
__device__ __forceinline__ float fetch_time(ScnPtr scn, int mib) {
  return floorf((float)mib * ((float)((double)scn->xfer / (double)scn->K) * (1.0f - 1.0f / 2097152)));
}
constexpr int HALVES_UNFIT = 1 << 30;                  // in place of a share of a node's memory
// A time is a chain of at most two additions a level and four more, of numbers up to six times as large, rounded to 24 bits: 6 x (2 x 16 + 4) =
// 216 units of 2^-24 of it, and the limit is raised by 256 units of the longest time there may be (or of itself, if that is less).  What the limit
// is lowered by (communication, penalties, fetch times, which may be many times as long) adds 20 roundings, the limit itself, its
// difference from that, the record's share and the comparison's other side one each: 24 units of the limit, raised by 32.
constexpr double TIME_SLACK = 1.0 / 65536, LIMIT_SLACK = 1.0 / 524288;
constexpr uint32_t CLUSTER = 4;
// What a time less its limit, with that limit lowered later on, is rounded by at most, as a part of the limit before: six roundings of
// 2^-24 (the limit less what all its partitions have, that less the record's share, the time less it, what the limit falls by less this, their sum).
constexpr float LIMIT_ROUNDING = 1.0f / 2097152;
// Below this a time is exact: what it is the sum of, the whole model's time added twice at most, stays below 2^24.
constexpr float EXACT_TIME = 4194304.0f;

__device__ __forceinline__ float fmax2(float a, float b) { return __builtin_fmaxf(a, b); }
__device__ __forceinline__ float fmax3(float a, float b, float c) { return __builtin_fmaxf(__builtin_fmaxf(a, b), c); }

// The state of the stages (nodes) taken up so far: largest forward and backward time, and the largest sums of class_time.
struct Terms {
  float mf, mb, none, ou, ov, both;
  // takes up a stage: forward and backward time, its own term less the prefix, `after` stages behind it, the prefix at its end
  __device__ __forceinline__ void add(float f, float b, float own, float after, float end) {
    mf = fmax2(mf, f);
    mb = fmax2(mb, b);
    const float u = __builtin_fmaf(mb, after, end), w = __builtin_fmaf(mf, after, end);
    none = fmax2(none, own);
    ou = fmax2(ou, none + u);
    ov = fmax2(ov, none + w);
    both = fmax3(both, ou + w, ov + u);
  }
  // the same with times counted from the end of the last node taken up, c = f + b further on now
  __device__ __forceinline__ void add_from_end(float f, float b, float c, float own, float after) {
    both -= c;
    none += c;
    add(f, b, own, after, 0.0f);
  }
};

// Records of two cuts, 8 words each, in one table of (L + 1)^2: those of the innermost loop, x <= y, in row x and column y; those of the
// loop ahead of it, x < m < L, in what these leave free, row L - x and columns 0 on (step_index).
__device__ __forceinline__ uint32_t step_index(int L, int x, int m) { return (uint32_t)((L - x) * (L + 1) + (m - x - 1)); }
// The innermost loop's, x < y.  Strategies 1 and 2: x, y = the last two cuts; stage N-2 = [x, y) and stage N-1 = [y, L), times less
// the whole model's.  Strategy 0 (node s runs stages s and s+1): x = the last cut but two, y = the last one; node N-3 = [x, y), times
// from the end of node N-4.
enum { PAIR_LAST = 0,       // 1, 2: time of stage N-1; 0: its share of node N-1 (which also runs stage 0)
       PAIR_U, PAIR_V,      // 1, 2: what stage N-2's backward, forward exceeds that by, at least 0; 0: node N-2's terms from N-3's
       PAIR_OWN,            // own term of stage N-2 (0: node N-3) without the prefix
       PAIR_TERM,           // 1, 2: the last stage's whole term, HUGE_TIME where one of the two does not fit; 0: end of node N-3
       PAIR_COST,           // 1, 2: reroute penalties of the two stages, and the time to fetch what they lack; 0: U of node N-3
       PAIR_V3,             // 0: V of node N-3
       PAIR_FIT,            // 0: node N-1's share of memory, HALVES_UNFIT if N-3 does not fit; 1, 2, in the record (x, L): y that fit behind x (whole numbers)
       PAIR_WORDS };
// The loop's over the last cut but one, x < m.  Strategies 1 and 2: stage N-3 = [x, m).  Strategy 0: node N-4 = [x, m) and, whatever x,
// node N-2 = [m, L).
enum { STEP_F = 0, STEP_B,  // forward and backward time
       STEP_OWN,            // own term
       STEP_END,            // 1, 2: prefix at m less the whole model's; 0: time of node N-2
       STEP_COST,           // 1, 2: reroute penalty of the stage, and the time to fetch what it lacks; 0: forward time of node N-2
       STEP_LAYERS,         // 1, 2: layers of the stage; 0: backward time of node N-2
       STEP_FETCH,          // 0: time to fetch what the two last stages lack at least, wherever the last cut is; 1: what [x, m) lacks (whole number)
       STEP_FIT,            // whether what the record holds fits (whole number)
       STEP_WORDS };
static_assert((int)PAIR_WORDS == (int)PAIR_RECORD_WORDS && (int)STEP_WORDS == (int)PAIR_RECORD_WORDS, "a record of either kind");

// One wavefront per cut x, its lanes take the cuts above; the first workgroup also lays out what every workgroup of the search stages in
// LDS.
template <int N, int STRAT>
__global__ void __launch_bounds__(BLOCK) k_cut_records(HalvesLaunch a) {
  constexpr int K = N - 1, W = halves_walked(N), G = K - W, ROWS = G > W ? G : W;
  const ScnPtr scn = as_const(a.s.scn);
  const TabPtr tab = as_const(a.tab);
  const FamPtr ff = &tab->fam[STRAT];
  const ClsPtr cl = &ff->cls[0];
  const int L = scn->L;
  if (blockIdx.x == 0) {
    // (one choice a lane, two choices a lane)
    __shared__ uint64_t units[2 * DEV_MAX_L];
    static_assert(BLOCK == 2 * DEV_MAX_L, "a thread for each");
    const int v = (int)threadIdx.x % DEV_MAX_L, choices = (int)threadIdx.x / DEV_MAX_L + 1;
    units[threadIdx.x] = v >= G && v <= L - 1 - W ? halves_units(scn, W, v) * halves_blocks(scn, G, choices, v) : 0;
    __syncthreads();
    uint64_t first = 0;
    for (int i = 0; i < v; ++i) first += units[(choices - 1) * DEV_MAX_L + i];
    a.items->first[choices - 1][v] = first;
    for (int i = threadIdx.x; i < W * DEV_MAX_L; i += BLOCK) {
      const int n = i / DEV_MAX_L + 1, x = i % DEV_MAX_L;
      const uint64_t u = scn->binom[n][x] + (x > 0 ? HALVES_ROW * scn->binom[n - 1][x - 1] : 0);
      a.items->units[i] = u > 0xffffffffull ? 0xffffffffu : (uint32_t)u;
    }
    for (int i = threadIdx.x; i <= L; i += BLOCK)
      a.items->prefix[i] = make_int4((int)scn->pf[i], (int)(scn->pf[i] + scn->pb[i]), (int)scn->pw[i], (int)scn->pa[i]);
    // (peers of one speed, nominal: what the loss of a stage costs is so many times its time)
    if (STRAT == 2 && threadIdx.x < DEV_MAX_S) {
      uint32_t share = 0;
      for (int st = 0; st < scn->n_aff; ++st)
        if (scn->aff_stage[st] == (int)threadIdx.x) share = tab->even_share[st];
      a.items->share[threadIdx.x] = share;
    }
    // (binomials up to 2^32 - 1: ranks of lower halves are below that)
    for (int i = threadIdx.x; i < ROWS * DEV_MAX_L; i += BLOCK) {
      const uint64_t b = scn->binom[1 + i / DEV_MAX_L][i % DEV_MAX_L];
      a.items->binom[i] = b > 0xffffffffull ? 0xffffffffu : (uint32_t)b;
    }
  }
  const int lane = threadIdx.x & 63;
  const int x = __builtin_amdgcn_readfirstlane(blockIdx.x * (BLOCK / 64) + (threadIdx.x >> 6));
  if (x > L) return;
  auto fwd = [&](int lo, int hi) { return (int)(scn->pf[hi] - scn->pf[lo]); };
  auto both = [&](int lo, int hi) { return (int)(scn->pf[hi] - scn->pf[lo] + scn->pb[hi] - scn->pb[lo]); };
  const int cap = (int)scn->cap, M = cl->M;
  auto memory = [&](int lo, int hi, int s) {           // (0: nobody's)
    const int coef = ff->mem_coef[s];
    return coef < 0 ? 0 : (int)(scn->pw[hi] - scn->pw[lo]) + (ff->has_act ? (int)__umul24((uint32_t)(scn->pa[hi] - scn->pa[lo]), (uint32_t)coef) : 0);
  };
  auto penalty = [&](int lo, int hi, int s) {
    uint32_t pen = 0;
    for (int st = 0; STRAT == 2 && st < scn->n_aff; ++st)
      if (scn->aff_stage[st] == s) pen += even_penalty(scn, tab, st, fwd(lo, hi), both(lo, hi) - fwd(lo, hi));
    return (float)pen;
  };
  auto store = [&](uint32_t index, const float (&rec)[7], uint32_t last_word) {
    uint4 *dst = (uint4 *)(a.pairs + (size_t)index * PAIR_RECORD_WORDS);
    dst[0] = make_uint4(__float_as_uint(rec[0]), __float_as_uint(rec[1]), __float_as_uint(rec[2]), __float_as_uint(rec[3]));
    dst[1] = make_uint4(__float_as_uint(rec[4]), __float_as_uint(rec[5]), __float_as_uint(rec[6]), last_word);
  };
  auto lacks = [&](int lo, int hi, int s) { return lacking<N, STRAT>(ff, (int)scn->pw[lo], (int)scn->pw[hi], s); };
  uint32_t n_fit = 0;
  for (int y0 = 0; y0 <= L; y0 += 64) {
    const int y = y0 + lane;
    const bool there = x < y && y < L;
    const int lo = there ? x : 0, hi = there ? y : 0;
    const int f = fwd(lo, hi), c = both(lo, hi), last = both(hi, L), total = both(0, L);
    float pair[7] = {}, step[7] = {};
    uint32_t pair_word, step_word;
    if (STRAT == 0) {
      {
        constexpr int S = N - 3;
        const bool dead = (cl->dead >> S) & 1u, gone = (cl->dead >> (N - 1)) & 1u;
        const float b = dead ? 0.0f : (float)(c - f), ff3 = dead ? 0.0f : (float)f, cc = dead ? 0.0f : (float)c;
        pair[PAIR_LAST] = gone ? 0.0f : (float)last;
        pair[PAIR_U] = b * (float)cl->after[N - 2];
        pair[PAIR_V] = ff3 * (float)cl->after[N - 2];
        pair[PAIR_OWN] = dead ? NEVER : (float)cl->steady[S] * cc;
        pair[PAIR_TERM] = cc;
        pair[PAIR_COST] = b * (float)cl->after[S];
        pair[PAIR_V3] = ff3 * (float)cl->after[S];
        pair_word = (uint32_t)(there && memory(lo, hi, S) <= cap ? memory(hi, L, N - 1) : HALVES_UNFIT);
      }
      constexpr int S = N - 4;
      const bool dead = (cl->dead >> S) & 1u, gone = (cl->dead >> (N - 2)) & 1u;
      const float c2 = gone ? 0.0f : (float)last, f2 = gone ? 0.0f : (float)fwd(hi, L);
      step[STEP_F] = dead ? 0.0f : (float)f;
      step[STEP_B] = dead ? 0.0f : (float)(c - f);
      step[STEP_OWN] = dead ? NEVER : (float)cl->steady[S] * (float)c;
      step[STEP_END] = c2;
      step[STEP_COST] = f2;
      step[STEP_LAYERS] = c2 - f2;
      step[STEP_FETCH] = fetch_time(scn, imax32(0, ff->w0[N - 2] - (int)scn->pw[hi]));
      // (two cuts walked: node N-4 starts with the lanes' last cut but one, its memory is not looked at here)
      step_word = there && (W == 2 || memory(lo, hi, S) <= cap) && memory(hi, L, N - 2) <= cap ? 1u : 0u;
    } else {
      const bool fit = there && x >= 1 && memory(lo, hi, N - 2) <= cap && memory(hi, L, N - 1) <= cap;
      pair[PAIR_LAST] = (float)last;
      pair[PAIR_U] = (float)imax32(0, c - f - last);
      pair[PAIR_V] = (float)imax32(0, f - last);
      pair[PAIR_OWN] = (float)((M - 2) * c + last) + (float)total;
      pair[PAIR_TERM] = fit ? (float)((M - 1) * last) + (float)total : HUGE_TIME;
      pair[PAIR_COST] = penalty(lo, hi, N - 2) + penalty(hi, L, N - 1) + fetch_time(scn, lacks(lo, hi, N - 2) + lacks(hi, L, N - 1));
      n_fit += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(fit));
      pair_word = y == L ? n_fit : 0;
      step[STEP_F] = (float)f;
      step[STEP_B] = (float)(c - f);
      step[STEP_OWN] = (float)((M - 3) * c + last) + (float)total;
      step[STEP_END] = (float)-last;
      const int lack = lacks(lo, hi, N - 3);
      step[STEP_COST] = penalty(lo, hi, N - 3) + fetch_time(scn, lack);
      step[STEP_FETCH] = __int_as_float(lack);         // (read where the assignment is open: of any stage)
      step[STEP_LAYERS] = (float)(hi - lo);
      step_word = there && memory(lo, hi, N - 3) <= cap ? 1u : 0u;
    }
    if (y >= x && y <= L) store((uint32_t)(x * (L + 1) + y), pair, pair_word);
    if (there) store(step_index(L, x, y), step, step_word);
  }
}

// Digits x_K > ... > x_1 of `rem` = sum of C(x_i, i), as cuts c[i] = x_i + 1, all below `end`.  table[(i-1) * DEV_MAX_L + x] = C(x, i),
// which grows with x: a digit is built bit by bit, three instructions and a probe each, 6 of them up to 64 positions.  (The
// four-way search of unrank_digits waits for half as many probes, but takes five times the instructions, which count here.)
template <int K>
__device__ __forceinline__ void unrank_by_bits(uint32_t rem, int end, const uint32_t *table, int *c) {
#pragma unroll
  for (int i = K; i >= 2; --i) {
    const uint32_t *row = table + (i - 1) * DEV_MAX_L;
    int x = 0;
    uint32_t at = 0;                                   // C(x, i)
    auto bit = [&](int b) {
      const uint32_t t = row[x + b];
      const bool up = t <= rem;
      x = up ? x + b : x;
      at = up ? t : at;
    };
    if (end > 64) bit(64);                             // uniform
#pragma unroll
    for (int b = 32; b >= 1; b >>= 1) bit(b);
    rem -= at;
    c[i] = x + 1;
  }
  c[1] = (int)rem + 1;                                 // C(x, 1) = x
}

// A wavefront takes one stretch of units of work after the other, each of one v and 64 choices of the lanes' cuts that end with v; see
// the head of the file.  The upper cuts that go with v are numbered by falling digits x (position = sum of C(x_i, i) over W of them), cut =
// L-1-x; a stretch begins and ends with a row, a choice of all of them but the last.
// PRUNE: a bounded search (compiled apart: its tests in the loops over the outer cuts cost the exhaustive search 5 % as a flag).
template <int N, int STRAT, int R, bool PRUNE>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(halves_waves(N, STRAT, R, PRUNE)))) k_search_halves(HalvesLaunch a) {
  constexpr int K = N - 1, W = halves_walked(N), G = K - W, ROWS = G > W ? G : W;
  constexpr int LOW = STRAT == 0 ? G - 1 : G;         // nodes the lanes' cuts alone decide
  __shared__ int4 T[DEV_MAX_L + 1];
  __shared__ uint32_t BN[ROWS * DEV_MAX_L], UN[W * DEV_MAX_L];
  __shared__ uint64_t first_unit[DEV_MAX_L], RK[W * DEV_MAX_L];       // RK: row i - 1 = C(x, G + i), ranks of the walked cuts
  __shared__ uint64_t wave_cost[BLOCK / 64], wave_rank[BLOCK / 64];
  __shared__ uint32_t wave_fit[BLOCK / 64];
  const ScnPtr scn = as_const(a.s.scn);
  const TabPtr tab = as_const(a.tab);
  const FamPtr ff = &tab->fam[STRAT];
  const ClsPtr cl = &ff->cls[0];
  const CHM_CONST i32x4 *pre = (const CHM_CONST i32x4 *)(uintptr_t)a.items->prefix;      // {forward, both, memory, activations}
  const int L = scn->L;
  for (int i = threadIdx.x; i <= L; i += BLOCK) T[i] = a.items->prefix[i];
  for (int i = threadIdx.x; i < ROWS * DEV_MAX_L; i += BLOCK) BN[i] = a.items->binom[i];
  for (int i = threadIdx.x; i < W * DEV_MAX_L; i += BLOCK) UN[i] = a.items->units[i];
  if (threadIdx.x < DEV_MAX_L) first_unit[threadIdx.x] = a.items->first[R - 1][threadIdx.x];
  if ((int)threadIdx.x % DEV_MAX_L < L)
    for (int i = threadIdx.x; i < W * DEV_MAX_L; i += BLOCK) RK[i] = scn->binom[G + 1 + i / DEV_MAX_L][i % DEV_MAX_L];
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t item = __builtin_amdgcn_readfirstlane(blockIdx.x * (BLOCK / 64) + wave);
  uint64_t best_cost = ~0ull, best_rank = ~0ull;
  uint32_t n_fit = 0, considered = 0;
  uint64_t low_cost = umin64(a.s.incumbent0, __hip_atomic_load(a.s.incumbent, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));     // lowest known
  // The item's part of all units of work: blocks of 64 choices of the lanes' cuts, v by v, each its set-up and its upper cuts in turn.
  uint64_t unit = (uint64_t)item * a.per_item;
  const uint64_t unit_end = umin64(unit + a.per_item, a.n_units);
  while (unit < unit_end) {
    const uint64_t first_lo = first_unit[lane], first_hi = first_unit[lane + 64];
    // (units are numbered v by v: first grows with v, and is the same where v has none)
    const int v = (int)__popcll(__builtin_amdgcn_ballot_w64(first_lo <= unit)) + (int)__popcll(__builtin_amdgcn_ballot_w64(first_hi <= unit)) - 1;
    const uint64_t behind = unit - uniform64(first_unit[v]);
    auto choose = [&](int x, int i) -> uint32_t { return (uint32_t)__builtin_amdgcn_readfirstlane((int)BN[(i - 1) * DEV_MAX_L + x]); };      // C(x, i)
    const uint32_t n_up = choose(L - 1 - v, W);                // upper cuts that go with v
    const uint32_t n_low = choose(v - 1, G - 1);               // choices of the lanes' cuts that end with v
    const uint32_t units = HALVES_SETUP + n_up + HALVES_ROW * choose(L - 2 - v, W - 1);      // (halves_units)
    const uint32_t low_block = (behind >> 32) == 0 ? (uint32_t)behind / units : (uint32_t)(behind / units);
    const uint32_t from = (uint32_t)(behind - (uint64_t)low_block * units);
    const uint32_t to = unit_end - unit < units - from ? from + (uint32_t)(unit_end - unit) : units;
    unit += units - from;
    // Digits x[i], i = W .. 2, of the row (all but the last cut) that a unit of upper cuts belongs to; the rows' position is returned.
    // (C(x, i) positions have a leading digit below x, in C(x-1, i-1) rows.)
    auto row_of = [&](uint32_t rem, uint32_t (&x)[5]) -> uint32_t {
      uint32_t position = 0;
#pragma unroll
      for (int i = W; i >= 2; --i) {
        // largest x with that many units or fewer
        const uint32_t lo = UN[(i - 1) * DEV_MAX_L + lane], hi = UN[(i - 1) * DEV_MAX_L + lane + 64];
        x[i] = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(lo <= rem)) + (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(hi <= rem)) - 1u;
        rem -= (uint32_t)(x[i] < 64 ? __builtin_amdgcn_readlane((int)lo, (int)x[i]) : __builtin_amdgcn_readlane((int)hi, (int)x[i] - 64));
        position += (uint32_t)__builtin_amdgcn_readfirstlane((int)BN[(i - 1) * DEV_MAX_L + x[i]]);
      }
      return position;
    };
    uint32_t x[5] = {}, x_end[5];
    const uint32_t up_end = to == units ? n_up : row_of(to < HALVES_SETUP ? 0 : to - HALVES_SETUP, x_end);
    uint32_t left = up_end - row_of(from < HALVES_SETUP ? 0 : from - HALVES_SETUP, x);       // upper cuts still to walk
    if (left == 0) continue;
    uint32_t fit_up = 0;                               // strategies 1, 2: upper cuts that fit

    // ---- this lane's cuts, R choices of them
    const int cap = (int)scn->cap;
    const int total = pre[L].y;
    const float shift = (float)total;
    const bool open_nodes = STRAT == 1 && ff->assign != 0;
    const CHM_CONST uint32_t *share = as_const(a.items)->share;       // 2: share of a stage's time that its loss costs
    struct Choice {
      uint32_t cuts[(G + 3) / 4];                      // a byte each
      Terms low;
      float off, layers;                               // what the limit is lowered by (0: the comm term and the end of the last node)
      int mem_b, f_b, c_b;                             // 0: prefixes at cut G-1 (memory as node G-1 counts it)
      float zl;                                        // 0: stage 0's time on node N-1, and what it leaves of its memory
      int room_z;
      bool ok;
    };
    Choice mine[R];
    uint32_t low_fit = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      Choice &o = mine[r];
      const uint32_t q = low_block * (64u * R) + 64u * r + (uint32_t)lane;
      o.ok = q < n_low;
      o.low = {0, 0, NEVER, NEVER, NEVER, NEVER};
      if (STRAT == 1) o.low.both = (float)(ff->fixed_step - cl->comm_total);    // (untouched pipelines: whatever the cuts)
      o.off = (float)cl->comm_total;
      int c[G + 1];
      unrank_by_bits<G - 1>(o.ok ? q : 0u, v, BN, c);  // cuts 1..v-1
      c[0] = 0;
      c[G] = v;
#pragma unroll
      for (int i = 0; i < (G + 3) / 4; ++i) o.cuts[i] = 0;
#pragma unroll
      for (int i = 1; i <= G; ++i) o.cuts[(i - 1) >> 2] |= (uint32_t)c[i] << (8 * ((i - 1) & 3));
      int4 t[G + 1];
      t[0] = make_int4(0, 0, 0, 0);
#pragma unroll
      for (int i = 1; i <= G; ++i) t[i] = T[c[i]];
      o.layers = 0;
      if (STRAT != 0 && ff->allreduce > 0) {
        int layers = ff->fixed_layers;
#pragma unroll
        for (int s = 0; s < G; ++s) layers = imax32(layers, c[s + 1] - c[s]);
        o.layers = (float)layers;
      }
#pragma unroll
      for (int s = 0; s < LOW; ++s) {
        const int e = STRAT == 0 ? s + 2 : s + 1;
        int f = t[e].x - t[s].x, cc = t[e].y - t[s].y;
        const int coef = ff->mem_coef[s];
        const int m = t[e].z - t[s].z + (ff->has_act ? (int)__umul24((uint32_t)(t[e].w - t[s].w), (uint32_t)(coef < 0 ? 0 : coef)) : 0);
        o.ok = o.ok && (coef < 0 || m <= cap);
        if (STRAT == 2) o.off += (float)(int)((uint32_t)cc * share[s]);
        if (STRAT == 0) {
          const bool dead = (cl->dead >> s) & 1u;      // uniform
          if (dead) f = cc = 0;
          o.low.add_from_end((float)f, (float)(cc - f), (float)cc, dead ? NEVER : (float)cl->steady[s] * (float)cc, (float)cl->after[s]);
          o.off += (float)cc;
        } else {
          // (the whole model's time is left out of both prefixes a term holds: the records' are less by as much)
          o.low.add((float)f, (float)(cc - f), (float)((int)__umul24((uint32_t)(cl->M - N + s), (uint32_t)cc) - t[e].y + total) + shift, (float)(N - 1 - s),
                    (float)(t[e].y - total));
        }
      }
      int lacks = 0;
      if (open_nodes) {
#pragma unroll
        for (int s = 0; s < G; ++s) lacks += (int)a.pairs[step_index(L, c[s], c[s + 1]) * STEP_WORDS + STEP_FETCH];
      } else {
#pragma unroll
        for (int s = 0; s < G; ++s) lacks += lacking<0, STRAT>(ff, t[s].z, t[s + 1].z, s);
      }
      o.off += fetch_time(scn, lacks);
      if (STRAT == 0) {
        const int coef_g = ff->mem_coef[G - 1], coef_z = ff->mem_coef[N - 1];
        o.f_b = t[G - 1].x;
        o.c_b = t[G - 1].y;
        o.mem_b = coef_g < 0 ? 0 : t[G - 1].z + (ff->has_act ? (int)__umul24((uint32_t)t[G - 1].w, (uint32_t)coef_g) : 0);
        o.zl = ((cl->dead >> (N - 1)) & 1u) ? 0.0f : (float)t[1].y;
        o.room_z = coef_z < 0 ? HALVES_UNFIT - 1 : cap - t[1].z - (ff->has_act ? (int)__umul24((uint32_t)t[1].w, (uint32_t)coef_z) : 0);
      }
      low_fit += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(o.ok));
    }
    if (low_fit == 0) left = 0;                        // uniform: none of these lower cuts fits
    const i32x4 tv = pre[v];

    // ---- the upper cuts
    const int rounds = STRAT != 0 ? ff->allreduce : 0;
    const double per_step = 1.0 / (double)scn->K;
    // (the closed form's two ends and its own term, of sums up to twice the model's time)
    const double longest = (double)(cl->M + N + 4) * (double)total * 2.0;
    auto limit_of = [&](uint64_t cost) -> float {      // no step time above this can reach `cost`
      const uint64_t reconf = (uint64_t)scn->reconf[STRAT];
      if (cost == ~0ull) return HUGE_TIME / 2;
      if (cost < reconf) return NEVER;
      const double most = (double)(cost - reconf) * per_step + 1.0;
      return (float)(most + __builtin_fmin(most, longest) * TIME_SLACK + most * LIMIT_SLACK);
    };
    float limit = limit_of(low_cost);
    // memory of a node above the lanes' cuts, the same for all lanes
    auto peak = [&](i32x4 lo, i32x4 hi, int s) {
      const int coef = ff->mem_coef[s];
      return coef < 0 ? 0 : hi.z - lo.z + (hi.w - lo.w) * coef;
    };
    auto gone = [&](int s) { return STRAT == 0 && ((cl->dead >> s) & 1u) != 0; };
    const int M = cl->M;
    const RowPtr pairs = as_const((const uint32_t *)a.pairs);
    const float after_g = STRAT == 0 ? (float)cl->after[N - 4] : 0.0f;
    const float after_y = STRAT == 0 ? (float)cl->after[N - 3] : 0.0f, after_m = STRAT == 0 ? (float)cl->after[N - 2] : 0.0f;
    const float last_m = STRAT == 0 ? (float)(cl->steady[N - 2] + 1) : 0.0f;      // (0, a node that is gone: as good as no own term)
    const float last_own = STRAT == 0 ? (float)(cl->steady[N - 1] + 1) : 0.0f;

    i32x4 at[W + 1];                                   // prefixes at the cuts walked: at[0] = v, at[i] = cut G+i
    int cut[W + 1];
    at[0] = tv;
    cut[0] = v;
    // of the levels above the innermost loop: everything below stage N-2 (0: node N-3), the limit, and, strategy 0, what of the last nodes is
    // the same for a row
    struct Row {
      Terms now;
      float lim, off;
      float um, vm, xb, xf;
      int room;
    };
    Row row[R];
    float own_m = 0, c_m = 0;

    auto lower_to = [&](uint64_t cost) {
      low_cost = cost;
      limit = limit_of(cost);
#pragma unroll
      for (int r = 0; r < R; ++r) row[r].lim = __builtin_fminf(row[r].lim, limit - row[r].off);
    };
    // the few that may win: time of every class, weights to fetch, cost, ties by rank, all in integers
    // (`here`: the lane has one; y, half and its time t, as far as that is a whole number, are its own)
    auto consider = [&](bool here, int y, int half, float t) {
      // (the compiler is not to know that cuts and tables are the same each time: kept across the loops, what follows from them takes the
      // registers)
      uint64_t tables = (uint64_t)(uintptr_t)scn, family = (uint64_t)(uintptr_t)ff;
      asm volatile("" : "+s"(tables), "+s"(family));
      const ScnPtr scn = (ScnPtr)(uintptr_t)tables;
      const FamPtr ff = (FamPtr)(uintptr_t)family;
      // what others have found by now counts, too
      auto lowest_of_all = [&]() { return __hip_atomic_load(a.s.incumbent, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
      uint64_t known = ~0ull;
      const bool asks = STRAT != 2 && (R == 2 || considered >= CLUSTER);       // (two choices a lane: the count would be one more register to spill)
      if (R == 1) ++considered;
      if (asks) known = lowest_of_all();
      int c[N + 1];
      c[0] = 0;
      c[N] = L;
      uint32_t words[(G + 3) / 4];
#pragma unroll
      for (int i = 0; i < (G + 3) / 4; ++i) {
        words[i] = mine[0].cuts[i];
        if (R == 2) words[i] = half != 0 ? mine[R - 1].cuts[i] : words[i];
        asm volatile("" : "+v"(words[i]));
      }
      asm volatile("" : "+s"(c[N]));
#pragma unroll
      for (int i = 1; i <= G; ++i) c[i] = (int)((words[(i - 1) >> 2] >> (8 * ((i - 1) & 3))) & 0xffu);
#pragma unroll
      for (int i = 1; i < W; ++i) {
        c[G + i] = cut[i];
        asm volatile("" : "+s"(c[G + i]));
      }
      c[K] = y;
      int step = STRAT == 1 ? ff->fixed_step : 0;
      auto prefix_at = [&](int i) { return i == 0 ? make_int2(0, 0) : make_int2(T[c[i]].x, T[c[i]].y); };
      if (STRAT != 0) {                                // (one class is timed)
        if (__builtin_amdgcn_ballot_w64(here && t >= EXACT_TIME) == 0) step = imax32(step, (int)t + ff->cls[0].comm_total);
        else step = imax32(step, class_time<N, STRAT, true, true>(&ff->cls[0], prefix_at));
      } else {
        for (int ci = 0; ci < ff->n_time; ++ci) {
#pragma unroll
          for (int i = 1; i <= G; ++i) asm volatile("" : "+v"(c[i]));
          step = imax32(step, class_time<N, STRAT, true, true>(&ff->cls[ci], prefix_at));
          if (__builtin_amdgcn_ballot_w64(here && (float)step <= limit) == 0) return;
        }
      }
      if (STRAT == 2) {
        for (int st = 0; st < scn->n_aff; ++st) {
#pragma unroll
          for (int s = 0; s < N; ++s)
            if (scn->aff_stage[st] == s) {             // uniform
              const int4 lo = T[c[s]], hi = T[c[s + 1]];
              step += (int)even_penalty(scn, tab, st, hi.x - lo.x, hi.y - lo.y - (hi.x - lo.x));
            }
        }
      }
      if (rounds > 0) {
        int layers = ff->fixed_layers;
#pragma unroll
        for (int s = 0; s < N; ++s) layers = imax32(layers, c[s + 1] - c[s]);
        step += ff->allreduce * layers;
      }
      if (__builtin_amdgcn_ballot_w64(here && (float)step <= limit) == 0) return;
      // (One wavefront may have to work out a whole cluster of partitions, one after the other, most of which others have beaten by then: it
      // asks from the CLUSTER-th on, while it works out the times, which under strategy 2 takes less time than to ask.)
      if (asks) {
        known = uniform64(known);
        if (known < low_cost) lower_to(known);
      }
      const bool near_best = here && (float)step <= limit;
      if (__builtin_amdgcn_ballot_w64(near_best) == 0) return;
      int wp[N + 1];
      wp[0] = 0;
#pragma unroll
      for (int i = 1; i <= N; ++i) wp[i] = T[c[i]].z;
      const uint64_t cost = (uint64_t)scn->K * (uint32_t)step + (uint64_t)scn->reconf[STRAT] +
                            (uint64_t)scn->xfer * (uint32_t)missing_weights<N, STRAT>(ff, wp);
      const bool lowest = near_best && cost <= low_cost;
      if (__builtin_amdgcn_ballot_w64(lowest) == 0) return;
      if (!asks) known = lowest_of_all();
      uint64_t rank = (uint64_t)(low_block * (64u * R) + 64u * (uint32_t)half + (uint32_t)lane) + BN[(G - 1) * DEV_MAX_L + v - 1] + RK[(W - 1) * DEV_MAX_L + y - 1];
#pragma unroll
      for (int i = 1; i < W; ++i) rank += RK[(i - 1) * DEV_MAX_L + cut[i] - 1];
      if (lowest && (cost < best_cost || (cost == best_cost && rank < best_rank))) { best_cost = cost; best_rank = rank; }
      const uint64_t least = uniform64(wave_min(lowest ? cost : ~0ull));
      known = uniform64(known);
      if (least < umin64(known, low_cost) && lane == 0) atomicMin((unsigned long long *)a.s.incumbent, (unsigned long long)least);
      if (umin64(least, known) < low_cost) lower_to(umin64(least, known));
    };

    // Innermost loop: last cuts m+n, m+n-1, ... m+1, the others being fixed; src = records of the first two.  Four records a round.
    // (Strategies 1 and 2: a record behind the last one, y = m, is HUGE_TIME; what lies ahead of that, in the row or before it, is read along
    // and not looked at.  m > 2: something does.)
    auto walk = [&](RowPtr src, int m, uint32_t n) {
      for (;;) {
        const u32x16 first = *(const CHM_CONST record_pair *)src, second = *(const CHM_CONST record_pair *)(src - 2 * PAIR_WORDS);
        src -= 4 * PAIR_WORDS;
        constexpr int A = PAIR_WORDS, B = 0;           // words of y's record and of y - 1's
        // a partition's time and what it may be at most (strategy 0: from the end of node N-3)
        auto time_of = [&](const Row &w, float zl, const u32x16 &r, int o, float *most) -> float {
          auto word = [&](int i) { return __uint_as_float(r[i]); };
          if (STRAT == 0) {
            const float end = word(o + PAIR_TERM), cz = word(o + PAIR_LAST) + zl;
            const float su2 = fmax3(cz, w.um, word(o + PAIR_U)), sv2 = fmax3(cz, w.vm, word(o + PAIR_V));
            const float su = fmax3(su2 + c_m, w.xb, word(o + PAIR_COST)), sv = fmax3(sv2 + c_m, w.xf, word(o + PAIR_V3));
            const float t = fmax3(__builtin_fmaf(cz, last_own, c_m), su2 + sv2 + own_m, su + sv + fmax2(w.now.none + end, word(o + PAIR_OWN)));
            *most = w.lim - end;
            return fmax3(t, w.now.ou + sv, w.now.ov + su);
          }
          const float last = word(o + PAIR_LAST);
          const float su = fmax2(w.now.mb - last, word(o + PAIR_U)), sv = fmax2(w.now.mf - last, word(o + PAIR_V));
          const float t = fmax3(fmax2(w.now.none, word(o + PAIR_OWN)) + su + sv, w.now.ou + sv, w.now.ov + su);
          *most = w.lim - word(o + PAIR_COST);
          return fmax3(t, w.now.both, word(o + PAIR_TERM));
        };
        auto may_win = [&](int i, const u32x16 &r, int o, bool there) -> uint64_t {
          float most;
          const float t = time_of(row[i], mine[i].zl, r, o, &most);
          uint64_t near = __builtin_amdgcn_ballot_w64(t <= most);
          if (STRAT == 0) {
            uint64_t fit = __builtin_amdgcn_ballot_w64((int)r[o + PAIR_FIT] <= row[i].room);
            fit = there ? fit : 0;
            n_fit += (uint32_t)__popcll(fit);
            near &= fit;
          }
          return near;
        };
        uint64_t any = 0;
#pragma unroll
        for (int i = 0; i < R; ++i) any |= may_win(i, first, A, true) | may_win(i, first, B, n >= 2);
        if (n > 2) {
#pragma unroll
          for (int i = 0; i < R; ++i) any |= may_win(i, second, A, true) | may_win(i, second, B, n >= 4);
        }
        if (__builtin_expect(any != 0, 0)) {
          // the lanes' best ones together, then the next best, until none is left within the limit
          float over[4 * R], time[4 * R];
#pragma unroll
          for (int e = 0; e < 4 * R; ++e) {
            const int o = (e & 1) ? B : A;
            const u32x16 &r = (e & 2) ? second : first;
            float most;
            time[e] = time_of(row[e >> 2], mine[e >> 2].zl, r, o, &most);
            over[e] = time[e] - most;
            const bool fit = (uint32_t)(e & 3) < n && (STRAT != 0 || (int)r[o + PAIR_FIT] <= row[e >> 2].room);
            over[e] = fit ? over[e] : HUGE_TIME;
          }
#pragma unroll 1
          for (;;) {
            float least = over[0], t = time[0];
            int which = 0;
#pragma unroll
            for (int e = 1; e < 4 * R; ++e) {
              const bool less = over[e] < least;
              least = less ? over[e] : least;
              t = less ? time[e] : t;
              which = less ? e : which;
            }
            const bool here = least <= 0.0f;
            if (__builtin_amdgcn_ballot_w64(here) == 0) break;
            const float before = limit;
            consider(here, m + (int)n - (which & 3), which >> 2, t);
            // (the new limit may be thousandths of the one before: a plan that fetches nothing behind one that fetches gigabytes)
            const float lowered = before - limit - before * LIMIT_ROUNDING;
#pragma unroll
            for (int e = 0; e < 4 * R; ++e) over[e] = here && which == e ? HUGE_TIME : over[e] + lowered;
          }
        }
        if (n <= 4) break;
        n -= 4;
      }
    };

    // A loop's cut i (1 .. W-2) is placed: whether the stage it ends (0: the node it ends) fits (in any lane),
    float off_i[R][W], layers_i[R][W];
    Terms state[R][W];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      state[r][0] = mine[r].low;
      off_i[r][0] = mine[r].ok ? mine[r].off : HUGE_TIME;        // (so that nothing above can win)
      layers_i[r][0] = mine[r].layers;
    }
    auto fits = [&](auto level) -> bool {
      constexpr int I = decltype(level)::value;
      cut[I] = L - 1 - (int)x[W + 1 - I];
      at[I] = pre[cut[I]];
      if constexpr (STRAT == 0 && I == 1) {            // node G-1 = [cut G-1, cut G+1)
        const int coef = ff->mem_coef[G - 1], need = coef < 0 ? 0 : at[1].z + at[1].w * coef;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const bool fit = mine[r].ok && need - mine[r].mem_b <= cap;
          row[r].room = fit ? mine[r].room_z : (int)0x80000000;
          off_i[r][1] = fit ? mine[r].off : HUGE_TIME;
        }
        return true;
      } else if constexpr (STRAT == 0) {               // node s = [cut s, cut s+2)
        return peak(at[I - 2], at[I], G + I - 2) <= cap;
      } else {                                         // stage s = [cut s, cut s+1)
        return peak(at[I - 1], at[I], G + I - 1) <= cap;
      }
    };
    // it joins the state,
    auto take_up = [&](auto level) {
      constexpr int I = decltype(level)::value;
      int lack;
      if (open_nodes) lack = (int)pairs[step_index(L, cut[I - 1], cut[I]) * STEP_WORDS + STEP_FETCH];
      else lack = lacking<0, STRAT>(ff, at[I - 1].z, at[I].z, G + I - 1);
      const float fetch = fetch_time(scn, lack);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        Terms t = state[r][I - 1];
        if constexpr (STRAT == 0) {
          constexpr int s = G + I - 2;
          const int f_0 = I == 1 ? mine[r].f_b : at[I == 1 ? 0 : I - 2].x, c_0 = I == 1 ? mine[r].c_b : at[I == 1 ? 0 : I - 2].y;
          const float f = gone(s) ? 0.0f : (float)(at[I].x - f_0), c = gone(s) ? 0.0f : (float)(at[I].y - c_0);
          t.add_from_end(f, c - f, c, gone(s) ? NEVER : (float)cl->steady[s] * c, (float)cl->after[s]);
          off_i[r][I] = off_i[r][I == 1 ? 1 : I - 1] + (c + fetch);
        } else {
          constexpr int s = G + I - 1;
          const int f = at[I].x - at[I - 1].x, c = at[I].y - at[I - 1].y, end = at[I].y - total;
          t.add((float)f, (float)(c - f), (float)((M - N + s) * c - end) + shift, (float)(N - 1 - s), (float)end);
          off_i[r][I] = off_i[r][I - 1] + fetch;
          if (STRAT == 2) off_i[r][I] += (float)(int)(share[G + I - 1] * (uint32_t)c);
          if (rounds > 0) layers_i[r][I] = fmax2(layers_i[r][I - 1], (float)(cut[I] - cut[I - 1]));
        }
        state[r][I] = t;
      }
    };
    // and whether, in a bounded search, some lane may still win whatever the cuts above are (times of strategies 1 and 2 are less by the
    // whole model's, which every term still gets).
    auto may_win_yet = [&](auto level) -> bool {
      constexpr int I = decltype(level)::value;
      if (!PRUNE) return true;
      uint64_t any = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const Terms &t = state[r][I];
        any |= __builtin_amdgcn_ballot_w64(fmax2(fmax3(t.none, t.ou, t.ov), t.both) <= limit - off_i[r][I]);
      }
      return any != 0;
    };
    auto left_out = [&](uint32_t all) { left = left > all ? left - all : 0; };       // (the part may end sooner)
    if (PRUNE && STRAT != 0) {
      uint64_t any = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) any |= __builtin_amdgcn_ballot_w64(mine[r].low.both <= limit - off_i[r][0]);
      if (any == 0) left = 0;
    }
    // cut K-1, and the innermost loop: the stage it ends comes from a record
    auto over_m = [&] {
      constexpr int P = W - 2;
      const uint32_t width = (uint32_t)(L + 1) * PAIR_RECORD_WORDS;
      int m = L - 1 - (int)x[2];
      RowPtr step = pairs + step_index(L, STRAT != 0 ? cut[P] : W == 2 ? 0 : cut[W == 2 ? 0 : P - 1], m) * STEP_WORDS;
      RowPtr pair = pairs + (uint32_t)(STRAT != 0 ? m : cut[P]) * width + (uint32_t)(L - 2) * PAIR_WORDS;
      u32x8 next = *(const CHM_CONST u32x8 *)step;
      do {
        const u32x8 rec = next;
        step -= STEP_WORDS;
        next = *(const CHM_CONST u32x8 *)step;         // (ahead of the first one lies the end of another row)
        auto word = [&](int i) { return __uint_as_float(rec[i]); };
        const uint32_t n = x[2];
        cut[W - 1] = m;
        bool open = rec[STEP_FIT] != 0;
        if (open) {
          uint64_t any = 0;
          if constexpr (STRAT == 0) {
            c_m = word(STEP_END);
            own_m = c_m * last_m;
          }
          i32x4 tm = {};
          if constexpr (STRAT == 0 && W == 2) tm = pre[m];
#pragma unroll
          for (int r = 0; r < R; ++r) {
            Row &w = row[r];
            w.now = state[r][P];
            if constexpr (STRAT == 0) {
              float f = word(STEP_F), b = word(STEP_B), own = word(STEP_OWN);
              if constexpr (W == 2) {                  // node N-4 = [cut G-1, m)
                const int coef = ff->mem_coef[G - 1];
                const bool fit = mine[r].ok && (coef < 0 ? 0 : tm.z + tm.w * coef) - mine[r].mem_b <= cap;
                w.room = fit ? mine[r].room_z : (int)0x80000000;
                f = gone(G - 1) ? 0.0f : (float)(tm.x - mine[r].f_b);
                b = gone(G - 1) ? 0.0f : (float)(tm.y - mine[r].c_b) - f;
                own = gone(G - 1) ? NEVER : (float)cl->steady[G - 1] * (f + b);
              }
              w.now.add_from_end(f, b, f + b, own, after_g);
              w.off = off_i[r][P] + (f + b) + word(STEP_FETCH);
              w.um = fmax2(w.now.mb, word(STEP_LAYERS)) * after_m;
              w.vm = fmax2(w.now.mf, word(STEP_COST)) * after_m;
              w.xb = w.now.mb * after_y;
              w.xf = w.now.mf * after_y;
              // (a path that turns at both ends within the nodes so far does not get longer)
              w.lim = limit - w.off;
              w.lim = w.now.both <= w.lim ? w.lim : NEVER;
            } else {
              w.now.add(word(STEP_F), word(STEP_B), word(STEP_OWN), 2.0f, word(STEP_END));
              w.off = off_i[r][P] + word(STEP_COST);
              // (rounds of communication: at least the layers of the largest stage so far)
              int some = rounds;
              asm volatile("" : "+s"(some));           // (kept a branch)
              if (some > 0) w.off += (float)some * fmax2(layers_i[r][P], word(STEP_LAYERS));
              w.lim = limit - w.off;
            }
            // (strategy 0: with the least that the last two nodes' turns add, and the own term of node N-2, whole by now)
            const float none = STRAT == 0 ? w.now.none + (w.xb + w.xf) : w.now.none, ou = STRAT == 0 ? w.now.ou + w.xf : w.now.ou;
            const float ov = STRAT == 0 ? w.now.ov + w.xb : w.now.ov, least = STRAT == 0 ? fmax2(w.now.both, w.um + w.vm + own_m) : w.now.both;
            if (PRUNE) any |= __builtin_amdgcn_ballot_w64(fmax2(fmax3(none, ou, ov), least) <= w.lim);
          }
          if (PRUNE) open = any != 0;
        }
        if (open) {
          if (STRAT != 0) fit_up += pair[2 * PAIR_WORDS + PAIR_FIT];
          walk(pair, m, n);
        }
        if (STRAT != 0) pair -= width;
        --m;
        left -= n;
        ++x[2];
      } while (left != 0 && W >= 3 && x[2] < x[3]);
    };
    // the cuts before, if they are walked; one that is left out takes with it what is left of its choices of the cuts above
    auto over_g = [&] {
      if constexpr (W < 3) {
        over_m();
      } else {
        constexpr std::integral_constant<int, W - 2> level;
        auto leave_out = [&] { left_out(x[3] * (x[3] - 1) / 2 - x[2] * (x[2] - 1) / 2); };
        do {
          if (fits(level)) {
            take_up(level);
            if (may_win_yet(level)) over_m();
            else leave_out();
          } else {
            leave_out();
          }
          ++x[3];
          x[2] = 1;
        } while (left != 0 && W >= 4 && x[3] < x[4]);
      }
    };
    while (left != 0) {
      if constexpr (W < 4) {
        over_g();
      } else {
        constexpr std::integral_constant<int, W - 3> level;
        auto leave_out = [&] {
          left_out(x[4] * (x[4] - 1) * (x[4] - 2) / 6 - x[3] * (x[3] - 1) * (x[3] - 2) / 6 - x[2] * (x[2] - 1) / 2);
        };
        if (fits(level)) {
          take_up(level);
          if (may_win_yet(level)) over_g();
          else leave_out();
        } else {
          leave_out();
        }
        ++x[4];
        x[3] = 2;
        x[2] = 1;
      }
    }
    if (STRAT != 0) n_fit += fit_up * low_fit;
  }
  // ---- lowest cost of the workgroup, then lowest rank
  {
    const uint64_t low = wave_min(best_cost);
    const uint64_t low_rank = wave_min(best_cost == low ? best_rank : ~0ull);
    if (lane == 0) { wave_cost[wave] = low; wave_rank[wave] = low_rank; wave_fit[wave] = n_fit; }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t cost = wave_cost[0], rank = wave_rank[0];
    uint32_t fit = wave_fit[0];
#pragma unroll
    for (int i = 1; i < BLOCK / 64; ++i) {
      if (wave_cost[i] < cost || (wave_cost[i] == cost && wave_rank[i] < rank)) { cost = wave_cost[i]; rank = wave_rank[i]; }
      fit += wave_fit[i];
    }
    const uint32_t slot = (blockIdx.x & a.s.slot_mask) * a.s.slot_stride;
    if (fit) atomicAdd((unsigned long long *)a.s.feasible + slot, (unsigned long long)fit);
    if (cost != ~0ull) {
      // the chunk of 2^idx_bits ranks the plan lies in has words of its own
      const uint64_t chunk = rank >> a.s.idx_bits, local = rank & ((1ull << a.s.idx_bits) - 1ull);
      atomicMin((unsigned long long *)a.s.result + chunk * a.chunk_words + slot, (unsigned long long)((cost << a.s.idx_bits) | local));
    }
  }
}

template <int STRAT, int N>
int launch_halves(const HalvesLaunch &a, bool build, hipStream_t st) {
  if (build) hipLaunchKernelGGL((k_cut_records<N, STRAT>), dim3((a.n_rows + BLOCK / 64 - 1) / (BLOCK / 64)), dim3(BLOCK), 0, st, a);
  const uint32_t blocks = (a.n_items + BLOCK / 64 - 1) / (BLOCK / 64);
  if (a.bounded) hipLaunchKernelGGL((k_search_halves<N, STRAT, 1, true>), dim3(blocks), dim3(BLOCK), 0, st, a);
  else if (a.choices == 1) hipLaunchKernelGGL((k_search_halves<N, STRAT, 1, false>), dim3(blocks), dim3(BLOCK), 0, st, a);
  else if constexpr (N >= HALVES_TWO_CHOICES_FROM) hipLaunchKernelGGL((k_search_halves<N, STRAT, 2, false>), dim3(blocks), dim3(BLOCK), 0, st, a);
  else return 1;
  return 0;
}

// build: the tables are filled first.  1 = no instance for this number of stages.
template <int STRAT>
int halves_by_stages(int sp, const HalvesLaunch &a, bool build, hipStream_t st) {
#define CHM_CASE(SPV) case SPV: return launch_halves<STRAT, SPV>(a, build, st);
  switch (sp) {
#ifdef CHM_TUNING_SUBSET
    CHM_CASE(7) CHM_CASE(8) CHM_CASE(10) CHM_CASE(11)
#else
    CHM_CASE(5) CHM_CASE(6) CHM_CASE(7) CHM_CASE(8) CHM_CASE(9) CHM_CASE(10)
    CHM_CASE(11) CHM_CASE(12) CHM_CASE(13) CHM_CASE(14) CHM_CASE(15) CHM_CASE(16)
#endif
    default: return 1;
  }
#undef CHM_CASE
}

}  // namespace
#endif
