// Exhaustive search of a whole family by halves: the kernels for large spaces.  Included by one translation unit per
// strategy, behind chm_search_kernel.h.
//
// A partition is a lower half (its first H cuts) and an upper half (its last UP cuts).  Everything a plan's step time is
// made of (pipeline_time in chm_search_kernel.h) splits at the cut between them: maxima and sums over the stages of one
// half alone, and a few terms of the stages that cross.  A lane keeps one lower half in registers and its wavefront walks the
// upper halves as nested loops, one cut each.  All lanes of a wavefront have the same last lower cut v, so the stage between
// the halves, and every stage above it, is the same for all of them: its times and memory are scalars, and what a cut decides
// is worked out where its loop stands.  Only what depends on the last cut is left to the innermost loop, and of that
// the scalar share (a function of two cuts) is read from a table of (L + 1)^2 records (k_pair_records, 32 bytes each,
// laid out once per handle and strategy).
// Bound by VALU issue: 14 to 17 instructions a partition in the innermost loop (26 under redundant computation), 20 to 28 in all;
// working every lane's upper stages out on their own took 51 to 54 (104 with two classes of pipelines), one partition at a time
// 200 and more.  62.9 M partitions of 8 stages: 54 us (120; one by one 434), under redundant computation 66 (209; 516), 5.2 G of
// 11 stages 4.0 ms (6.4; 51).  As many waves per SIMD as the registers leave hide the scalar loads: 7 up to 8 stages, 6 up to 11, 5
// beyond, under redundant computation 5 up to 10 and 4 beyond (strategy 1 of 11, 15 and 16 stages spills two to nine registers).
//
// Every partition's memory peak and the time of its longest pipeline class are worked out.  The time of other classes (strategy
// 0: pipelines without the failed nodes) and the weights to fetch (the transition time) only where horizon x that time does not
// already exceed the lowest cost met so far in the search: elsewhere they cannot change the argmin, ties included.
#ifndef CHM_HALVES_KERNEL_H
#define CHM_HALVES_KERNEL_H
#include "chm_search_kernel.h"

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
typedef u32x16 record_pair __attribute__((aligned(32)));       // two neighbouring records: 32 bytes each, a scalar load of 64

// least reroute penalty of a stage all of whose peers have one speed (stage_penalty; nothing else comes here)
__device__ __forceinline__ uint32_t even_penalty(ScnPtr scn, TabPtr tab, int st, int f, int b) {
  return tab->even_share[st] * peer_time(f, b, scn->aff_q[st][0]);
}
constexpr int HALVES_NEVER = TERM_NEVER;
constexpr int HALVES_UNFIT = 1 << 30;      // in place of a memory peak or a time: these partitions do not fit

// A record of two cuts x < y.  Strategies 1 and 2: x, y = the last two cuts; stage N-2 = [x, y) and stage N-1 = [y, L), times as
// prefixes from the front.  Strategy 0 (node s runs stages s and s+1): x = the last cut but two, y = the last one; node N-3 =
// [x, y), times relative to the end of node N-4 less the prefix at x.
enum { PAIR_END = 0,        // end of stage N-2 (strategy 0: of node N-3)
       PAIR_U, PAIR_V,      // U and V of pipeline_time of that stage alone, under 1 and 2 not below those of the last stage
       PAIR_OWN,            // its (M - n + s) C - P
       PAIR_LAST,           // 1, 2: the last stage's whole term; 0: its share of node N-1 (which also runs stage 0): time
       PAIR_PENALTY,        // 2: reroute penalties of the two stages; 0: node N-1's share of memory, HALVES_UNFIT if N-3 does not fit
       PAIR_ROUNDS,         // 1, 2: communication rounds of the larger of the two stages; 0: U of node N-2 from N-3's backward
       PAIR_FIT,            // 1, 2: 1 = both fit; 0: V of node N-2 from N-3's forward
       PAIR_WORDS };

// One lane per pair of cuts; the first workgroup also lays out what every workgroup of the search stages in LDS.
template <int N, int STRAT, int UP>
__global__ void __launch_bounds__(BLOCK) k_pair_records(HalvesLaunch a) {
  constexpr int K = N - 1, H = K - UP;
  const ScnPtr scn = as_const(a.s.scn);
  const TabPtr tab = as_const(a.tab);
  const FamPtr ff = &tab->fam[STRAT];
  const ClsPtr cl = &ff->cls[0];
  const int L = scn->L, W = L + 1;
  if (blockIdx.x == 0) {
    __shared__ uint32_t items[DEV_MAX_L];
    const int v = (int)threadIdx.x;
    if (v < DEV_MAX_L) {
      // wavefront items per last lower cut v, and where v's first one is
      uint32_t n = 0;
      if (v >= H && v <= L - 1 - UP) {
        const uint32_t low = (uint32_t)scn->binom[H - 1][v - 1], up = (uint32_t)scn->binom[UP][L - 1 - v];
        n = ((low + 63u) / 64u) * ((up + a.chunk - 1) / a.chunk);
      }
      items[v] = n;
    }
    __syncthreads();
    if (v < DEV_MAX_L) {
      uint32_t first = 0;
      for (int i = 0; i < v; ++i) first += items[i];
      a.items->first[v] = first;
    }
    for (int i = threadIdx.x; i <= L; i += BLOCK)
      a.items->prefix[i] = make_int4((int)scn->pf[i], (int)(scn->pf[i] + scn->pb[i]), (int)scn->pw[i], (int)scn->pa[i]);
    // (binomials up to 2^32 - 1: ranks of lower halves are below that)
    for (int i = threadIdx.x; i < H * DEV_MAX_L; i += BLOCK) {
      const uint64_t b = scn->binom[1 + i / DEV_MAX_L][i % DEV_MAX_L];
      a.items->binom[i] = b > 0xffffffffull ? 0xffffffffu : (uint32_t)b;
    }
  }
  const uint32_t p = blockIdx.x * BLOCK + threadIdx.x;
  if (p >= (uint32_t)(W * W)) return;
  const int x = (int)p / W, y = (int)p % W;
  uint32_t rec[PAIR_WORDS];
#pragma unroll
  for (int i = 0; i < PAIR_WORDS; ++i) rec[i] = 0;
  if (x >= 1 && x < y && y < L) {
    auto fwd = [&](int lo, int hi) { return (int)(scn->pf[hi] - scn->pf[lo]); };
    auto both = [&](int lo, int hi) { return (int)(scn->pf[hi] - scn->pf[lo] + scn->pb[hi] - scn->pb[lo]); };
    auto peak = [&](int lo, int hi, int s) {           // (0: nobody's)
      const int coef = ff->mem_coef[s];
      return coef < 0 ? 0 : (int)(scn->pw[hi] - scn->pw[lo]) + (ff->has_act ? (int)__umul24((uint32_t)(scn->pa[hi] - scn->pa[lo]), (uint32_t)coef) : 0);
    };
    const int cap = (int)scn->cap;
    const int end = both(0, y);
    if (STRAT == 0) {
      constexpr int S = N - 3;
      const bool dead = (cl->dead >> S) & 1u, gone = (cl->dead >> (N - 1)) & 1u;
      const int f = dead ? 0 : fwd(x, y), c = dead ? 0 : both(x, y), e = dead ? both(0, x) : end;
      rec[PAIR_END] = (uint32_t)e;
      rec[PAIR_U] = (uint32_t)(e + cl->after[S] * (c - f));
      rec[PAIR_V] = (uint32_t)(e + cl->after[S] * f);
      rec[PAIR_OWN] = (uint32_t)(cl->steady[S] < 0 ? HALVES_NEVER : cl->steady[S] * c - e);
      rec[PAIR_LAST] = (uint32_t)(gone ? 0 : both(y, L));
      const int coef = ff->mem_coef[N - 1];
      const int share = coef < 0 ? 0 : (int)(scn->pw[L] - scn->pw[y]) + (ff->has_act ? (int)__umul24((uint32_t)(scn->pa[L] - scn->pa[y]), (uint32_t)coef) : 0);
      rec[PAIR_PENALTY] = (uint32_t)(peak(x, y, S) <= cap ? share : HALVES_UNFIT);
      rec[PAIR_ROUNDS] = (uint32_t)(e + cl->after[N - 2] * (c - f));
      rec[PAIR_FIT] = (uint32_t)(e + cl->after[N - 2] * f);
    } else {
      const int f = fwd(x, y), c = both(x, y), total = both(0, L);
      rec[PAIR_END] = (uint32_t)end;
      rec[PAIR_U] = (uint32_t)imax32(total, end + (c - f));
      rec[PAIR_V] = (uint32_t)imax32(total, end + f);
      rec[PAIR_OWN] = (uint32_t)(cl->steady[N - 2] * c - end);
      rec[PAIR_LAST] = (uint32_t)(cl->steady[N - 1] * both(y, L) + total);
      if (STRAT == 2) {
        uint32_t pen = 0;
        for (int st = 0; st < scn->n_aff; ++st) {
          const int sa = scn->aff_stage[st];
          if (sa == N - 2) pen += even_penalty(scn, tab, st, f, c - f);
          if (sa == N - 1) pen += even_penalty(scn, tab, st, fwd(y, L), both(y, L) - fwd(y, L));
        }
        rec[PAIR_PENALTY] = pen;
      }
      rec[PAIR_ROUNDS] = (uint32_t)(ff->allreduce * imax32(y - x, L - y));
      rec[PAIR_FIT] = peak(x, y, N - 2) <= cap && peak(y, L, N - 1) <= cap ? 1u : 0u;
    }
  }
  uint4 *dst = (uint4 *)(a.pairs + (size_t)p * PAIR_WORDS);
  dst[0] = make_uint4(rec[0], rec[1], rec[2], rec[3]);
  dst[1] = make_uint4(rec[4], rec[5], rec[6], rec[7]);
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

// One wavefront per (v, 64 lower halves that end with cut v, `chunk` upper halves); see the head of the file.  The upper halves
// that go with v are numbered by falling digits x (position = sum of C(x_i, i) over UP of them), cut = L-1-x.
// PRUNE: a bounded search (compiled apart: its tests in the loops over the outer cuts cost the exhaustive search 5 % as a flag).
template <int N, int STRAT, int UP, bool PRUNE>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(STRAT == 0 ? (N <= 10 ? 5 : 4) : N <= 8 ? 7 : N <= 11 ? 6 : 5))) k_search_halves(HalvesLaunch a) {
  constexpr int K = N - 1, H = K - UP;
  constexpr int LOW = STRAT == 0 ? H - 1 : H;         // nodes of the lower half alone
  __shared__ int4 T[DEV_MAX_L + 1];
  __shared__ uint32_t BN[H * DEV_MAX_L];
  __shared__ uint64_t wave_cost[BLOCK / 64], wave_rank[BLOCK / 64];
  __shared__ uint32_t wave_fit[BLOCK / 64];
  const ScnPtr scn = as_const(a.s.scn);
  const TabPtr tab = as_const(a.tab);
  const FamPtr ff = &tab->fam[STRAT];
  const ClsPtr cl = &ff->cls[0];
  const CHM_CONST i32x4 *pre = (const CHM_CONST i32x4 *)(uintptr_t)a.items->prefix;      // {forward, both, memory, activations}
  const int L = scn->L;
  for (int i = threadIdx.x; i <= L; i += BLOCK) T[i] = a.items->prefix[i];
  for (int i = threadIdx.x; i < H * DEV_MAX_L; i += BLOCK) BN[i] = a.items->binom[i];
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t item = __builtin_amdgcn_readfirstlane(blockIdx.x * (BLOCK / 64) + wave);
  uint64_t best_cost = ~0ull, best_rank = ~0ull;
  uint32_t n_fit = 0;
  const uint64_t inc0 = umin64(a.s.incumbent0, __hip_atomic_load(a.s.incumbent, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  if (item < a.n_items) {
    // the item's v: items are numbered v by v
    const uint64_t below_lo = __builtin_amdgcn_ballot_w64(a.items->first[lane] <= item);
    const uint64_t below_hi = __builtin_amdgcn_ballot_w64(a.items->first[lane + 64] <= item);
    const int v = (int)__popcll(below_lo) + (int)__popcll(below_hi) - 1;     // first_item grows with v (equal where v has none)
    const uint32_t local = item - as_const(a.items->first)[v];
    const uint32_t n_up = (uint32_t)scn->binom[UP][L - 1 - v];               // upper halves that go with v
    const uint32_t n_low = (uint32_t)scn->binom[H - 1][v - 1];               // lower halves that end with v
    const uint32_t low_blocks = (n_low + 63u) / 64u;
    const uint32_t part = local / low_blocks, low_block = local - part * low_blocks;
    const uint32_t up_first = part * a.chunk;
    uint32_t left = n_up - up_first < a.chunk ? n_up - up_first : a.chunk;   // upper halves still to walk
    // digits of the first one: x[i], i = UP .. 1
    int x[UP + 1];
    {
      uint32_t rem = up_first;
#pragma unroll
      for (int i = UP; i >= 1; --i) {
        // largest x with C(x, i) <= rem (binomials of up to three cuts grow strictly from i - 1 on)
        const uint64_t lo = __builtin_amdgcn_ballot_w64(BN[(i - 1) * DEV_MAX_L + lane] <= rem);
        const uint64_t hi = __builtin_amdgcn_ballot_w64(BN[(i - 1) * DEV_MAX_L + lane + 64] <= rem);
        x[i] = (int)__popcll(lo) + (int)__popcll(hi) - 1;
        rem -= as_const(a.items->binom)[(i - 1) * DEV_MAX_L + x[i]];
      }
    }

    // ---- this lane's lower half
    const uint32_t q = low_block * 64u + (uint32_t)lane;
    const bool active = q < n_low;
    uint32_t low_cuts[(H + 3) / 4];                    // its cuts, a byte each
    int c_first, c_before;                             // cut 1; cut H-1 (strategy 0)
    int layers_low = 0;
    int none = HALVES_NEVER, only_u = HALVES_NEVER, only_v = HALVES_NEVER, both = HALVES_NEVER;     // see class_time
    int sum_low = 0, mf = 0, mb = 0;
    int pen_low = 0;
    bool ok = active;
    const int cap = (int)scn->cap;
    {
      int c[H + 1];
      unrank_by_bits<H - 1>(active ? q : 0u, v, BN, c);          // cuts 1..v-1
      c[0] = 0;
      c[H] = v;
#pragma unroll
      for (int i = 0; i < (H + 3) / 4; ++i) low_cuts[i] = 0;
#pragma unroll
      for (int i = 1; i <= H; ++i) low_cuts[(i - 1) >> 2] |= (uint32_t)c[i] << (8 * ((i - 1) & 3));
      c_first = c[1];
      c_before = c[H - 1];
      int4 t[H + 1];
      t[0] = make_int4(0, 0, 0, 0);
#pragma unroll
      for (int i = 1; i <= H; ++i) t[i] = T[c[i]];
#pragma unroll
      for (int s = 0; s < H; ++s) layers_low = imax32(layers_low, c[s + 1] - c[s]);
      if (STRAT != 0) layers_low = imax32(layers_low, ff->fixed_layers);
#pragma unroll
      for (int s = 0; s < LOW; ++s) {
        const int e = STRAT == 0 ? s + 2 : s + 1;
        int f = t[e].x - t[s].x, cc = t[e].y - t[s].y;
        const int coef = ff->mem_coef[s];
        const int m = t[e].z - t[s].z + (ff->has_act ? (int)__umul24((uint32_t)(t[e].w - t[s].w), (uint32_t)(coef < 0 ? 0 : coef)) : 0);
        ok = ok && (coef < 0 || m <= cap);
        if (STRAT == 2)
          for (int st = 0; st < scn->n_aff; ++st)
            if (scn->aff_stage[st] == s) pen_low += (int)even_penalty(scn, tab, st, f, cc - f);      // uniform
        if (STRAT == 0 && ((cl->dead >> s) & 1u)) f = cc = 0;
        sum_low += cc;
        mf = imax32(mf, f);
        mb = imax32(mb, cc - f);
        const int u = (int)__umul24((uint32_t)mb, (uint32_t)cl->after[s]) + sum_low, w = (int)__umul24((uint32_t)mf, (uint32_t)cl->after[s]) + sum_low;
        none = imax32(none, cl->steady[s] < 0 ? HALVES_NEVER : (int)__umul24((uint32_t)cc, (uint32_t)cl->steady[s]) - sum_low);
        only_u = imax32(only_u, none + u);
        only_v = imax32(only_v, none + w);
        both = imax32(both, imax32(only_u + w, only_v + u));
      }
    }
    const i32x4 tv = pre[v], tl = pre[L];
    // strategy 0: the lane's shares of nodes H-1 = [cut H-1, g) and N-1 (stage 0 of it)
    int4 tb = make_int4(0, 0, 0, 0);
    int zl = 0, room_z = 0;                            // stage 0's time, and what it leaves of node N-1's memory
    if (STRAT == 0) {
      tb = T[c_before];
      const int coef_g = ff->mem_coef[H - 1], coef_z = ff->mem_coef[N - 1];
      const int4 t1 = T[c_first];
      zl = ((cl->dead >> (N - 1)) & 1u) ? 0 : t1.y;
      room_z = coef_z < 0 ? HALVES_UNFIT - 1 : cap - t1.z - (ff->has_act ? (int)__umul24((uint32_t)t1.w, (uint32_t)coef_z) : 0);
      // (from here on the memory of the lower share of node H-1 in tb.z: one subtraction per g)
      tb.z = coef_g < 0 ? 0 : tb.z + (ff->has_act ? (int)__umul24((uint32_t)tb.w, (uint32_t)coef_g) : 0);
    }
    const uint64_t low_mask = __builtin_amdgcn_ballot_w64(ok);
    const uint32_t low_fit = (uint32_t)__popcll(low_mask);
    if (low_mask == 0) left = 0;                       // uniform: none of these lower halves fits

    // ---- the upper halves
    const int rounds = STRAT != 0 ? ff->allreduce : 0;
    const int fixed_step = ff->fixed_step, comm = cl->comm_total;
    const double per_step = 1.0 / (double)scn->K;
    auto limit_of = [&](uint64_t cost) -> int {       // no step time above this can reach `cost` (rounded up)
      const uint64_t reconf = (uint64_t)scn->reconf[STRAT];
      if (cost == ~0ull) return 0x7fffffff;
      if (cost < reconf) return -1;
      const double y = (double)(cost - reconf) * per_step + 1.0;
      return y >= 2147483647.0 ? 0x7fffffff : (int)y;
    };
    int limit = __builtin_amdgcn_readfirstlane(limit_of(inc0));
    // a node above the lower half, the same for all lanes: times (0 when nobody runs it), and whether it fits
    auto scalar_peak = [&](i32x4 lo, i32x4 hi, int s) {
      const int coef = ff->mem_coef[s];
      return coef < 0 ? 0 : hi.z - lo.z + (hi.w - lo.w) * coef;
    };
    auto gone = [&](int s) { return STRAT == 0 && ((cl->dead >> s) & 1u) != 0; };
    const int M = cl->M;
    auto scalar_own = [&](int s, int c, int p) {       // (strategies 1, 2: every stage has its node)
      const int k = STRAT == 0 ? cl->steady[s] : M - N + s;
      return STRAT == 0 && k < 0 ? HALVES_NEVER : k * c - p;
    };
    uint32_t share_h = 0, share_m = 0;                 // strategy 2: share of a stage's time that its loss costs, stages H and N-3
    if (STRAT == 2) {
      for (int st = 0; st < scn->n_aff; ++st) {
        if (scn->aff_stage[st] == H) share_h = tab->even_share[st];
        if (UP == 3 && scn->aff_stage[st] == N - 3) share_m = tab->even_share[st];
      }
    }
    const RowPtr pairs = as_const((const uint32_t *)a.pairs);

    int g = 0;                                         // cut H+1
    i32x4 tg = tv;
    // of the levels above the innermost loop, per lane (see the kernel's use of them)
    int xf = 0, xb = 0, u_h = 0, v_h = 0, gmax = 0, both_lim = 0, lim = 0, off = 0;
    int xf2 = 0, xb2 = 0, u_m = 0, v_m = 0, own_m = 0;
    int u_g = 0, v_g = 0, own_h = 0, room = 0, layers_up = 0, rounds_low = 0, pen_up = 0;
    int bf = 0, bb = 0, c0 = 0;
    bool ok_g = ok;
    if (STRAT != 0) {
      both_lim = both;
      off = comm;
      lim = ok ? __builtin_elementwise_sub_sat(limit, off) : (int)0x80000000;
    }

    auto upper_rank = [&](int m, int y) -> uint64_t {
      uint64_t r = 0;
      if (UP == 3) r = scn->binom[H + 1][g - 1];
      return r + scn->binom[K - 1][m - 1] + scn->binom[K][y - 1];
    };
    // the few that may win: other classes, weights to fetch, cost, ties by rank
    auto consider = [&](uint64_t mask, int r, int m, int y, int pen, int pair_rounds) {
      int c[N + 1];
      c[0] = 0;
      c[N] = L;
#pragma unroll
      for (int i = 1; i <= H; ++i) c[i] = (int)((low_cuts[(i - 1) >> 2] >> (8 * ((i - 1) & 3))) & 0xffu);
      if (UP == 3) c[H + 1] = g;
      c[K - 1] = m;
      c[K] = y;
      int step = r + off;                              // (off: what the limits of this level have been lowered by)
      if (STRAT != 0) {
        const int pens = pen_low + pen_up;
        step = imax32(step - pens, fixed_step) + pens + pen;
        if (rounds > 0) step += imax32(rounds_low, pair_rounds);
      } else {
        for (int ci = 1; ci < ff->n_time; ++ci)
          step = imax32(step, class_time<N, STRAT, true, true>(&ff->cls[ci], [&](int i) { const int4 t = T[c[i]]; return make_int2(t.x, t.y); }));
      }
      const bool near_best = ((mask >> lane) & 1u) && step <= limit;
      if (__builtin_amdgcn_ballot_w64(near_best) == 0) return;
      int wp[N + 1];
      wp[0] = 0;
#pragma unroll
      for (int i = 1; i <= N; ++i) wp[i] = T[c[i]].z;
      const uint64_t cost = (uint64_t)scn->K * (uint32_t)step + (uint64_t)scn->reconf[STRAT] +
                            (uint64_t)scn->xfer * (uint32_t)missing_weights<N, STRAT>(ff, wp);
      const uint64_t rank = (uint64_t)q + BN[(H - 1) * DEV_MAX_L + v - 1] + upper_rank(m, y);
      if (near_best && (cost < best_cost || (cost == best_cost && rank < best_rank))) { best_cost = cost; best_rank = rank; }
      const int seen = __builtin_amdgcn_readfirstlane(limit_of(wave_min(near_best ? cost : ~0ull)));
      if (seen < limit) {
        limit = seen;
        lim = ok_g ? __builtin_elementwise_sub_sat(limit, off) : (int)0x80000000;
      }
    };

    // Innermost loop: upper halves whose last cut is y, y-1, ... (n of them), the others being fixed.  Two records a round, the
    // next two on their way.
    auto walk = [&](int row, int m, int y, uint32_t n, int c2, int own_z) {
      // (y > m > 2: there are records ahead of (row, y))
      RowPtr at = pairs + (size_t)(uint32_t)(row * (L + 1) + y - 1) * PAIR_WORDS;
      u32x16 next = *(const CHM_CONST record_pair *)at;
      for (;;) {
        const u32x16 r = next;
        constexpr int A = PAIR_WORDS, B = 0;           // words of y's record and of y - 1's
        at -= 2 * PAIR_WORDS;
        next = *(const CHM_CONST record_pair *)at;
        const bool two = n >= 2;
        // the longest class's time less what is common to the level (off)
        auto time_of = [&](int o) -> int {
          int su, sv, t;
          if (STRAT == 0) {
            const int end = (int)r[o + PAIR_END], cz = (int)r[o + PAIR_LAST] + zl;
            const int last = end + (cz + c2);
            t = (int)__umul24((uint32_t)cz, (uint32_t)own_z) + last;
            su = imax32(imax32(last, (int)r[o + PAIR_ROUNDS] + c2), end + u_m);
            sv = imax32(imax32(last, (int)r[o + PAIR_FIT] + c2), end + v_m);
            t = imax32(t, su + sv + (own_m - end));
            su = imax32(imax32(su, (int)r[o + PAIR_U]), end + xb2);
            sv = imax32(imax32(sv, (int)r[o + PAIR_V]), end + xf2);
            t = imax32(t, su + sv + (int)r[o + PAIR_OWN]);
            if (UP == 3) {
              su = imax32(su, u_h);
              sv = imax32(sv, v_h);
              t = imax32(t, su + sv + own_h);
            }
            su = imax32(su, u_g);
            sv = imax32(sv, v_g);
          } else {
            su = imax32((int)r[o + PAIR_U], (int)r[o + PAIR_END] + xb2);
            sv = imax32((int)r[o + PAIR_V], (int)r[o + PAIR_END] + xf2);
            t = imax32((int)r[o + PAIR_LAST], su + sv + (int)r[o + PAIR_OWN]);
            if (UP == 3) {
              su = imax32(su, u_m);
              sv = imax32(sv, v_m);
              t = imax32(t, su + sv + own_m);
            }
            su = imax32(su, u_h);
            sv = imax32(sv, v_h);
          }
          t = imax32(t, su + sv + gmax);
          t = imax32(imax32(t, only_u + sv), only_v + su);
          return imax32(t, both_lim);
        };
        uint64_t near_a, near_b;
        int ta, tb2;
        if (STRAT == 0) {
          const uint64_t fit_a = __builtin_amdgcn_ballot_w64((int)r[A + PAIR_PENALTY] <= room);
          uint64_t fit_b = __builtin_amdgcn_ballot_w64((int)r[B + PAIR_PENALTY] <= room);
          fit_b = two ? fit_b : 0;
          near_a = near_b = 0;
          // (nothing to time where no lane fits: a cap that next to nothing fits)
          if ((fit_a | fit_b) != 0) {
            n_fit += (uint32_t)__popcll(fit_a) + (uint32_t)__popcll(fit_b);
            ta = time_of(A);
            near_a = __builtin_amdgcn_ballot_w64(ta <= lim) & fit_a;
            if (two) {
              tb2 = time_of(B);
              near_b = __builtin_amdgcn_ballot_w64(tb2 <= lim) & fit_b;
            }
          }
        } else {
          auto test = [&](int o, int &t) -> uint64_t {
            n_fit += r[o + PAIR_FIT];
            t = time_of(o);
            int w = t;
            if (STRAT == 2) w += (int)r[o + PAIR_PENALTY];
            if (rounds > 0) {                          // uniform
              asm volatile("");                        // (kept a branch)
              w += imax32(rounds_low, (int)r[o + PAIR_ROUNDS]);
            }
            return __builtin_amdgcn_ballot_w64(w <= lim);
          };
          near_a = test(A, ta);
          near_b = 0;
          if (two) near_b = test(B, tb2);
        }
        if ((near_a | near_b) != 0) {
#pragma unroll 1
          for (int e = 0; e < 2; ++e) {
            const bool b = e != 0;
            const uint64_t mask = b ? near_b : near_a;
            if (mask == 0 || (STRAT != 0 && (b ? r[B + PAIR_FIT] : r[A + PAIR_FIT]) == 0)) continue;
            consider(mask, b ? tb2 : ta, m, b ? y - 1 : y, STRAT == 2 ? (int)(b ? r[B + PAIR_PENALTY] : r[A + PAIR_PENALTY]) : 0,
                     (int)(b ? r[B + PAIR_ROUNDS] : r[A + PAIR_ROUNDS]));
          }
        }
        if (n <= 2) break;
        n -= 2;
        y -= 2;
      }
    };
    // A bounded search: whether some lane may still win, given what the cuts placed so far are worth at least.  su, sv: lower bounds of
    // the suffix maxima that reach the terms of node H (strategy 0: of node H-1) and below.
    auto hopeless = [&](int su, int sv, int least) -> bool {
      const int t = imax32(imax32(least, su + sv + gmax), imax32(imax32(only_u + sv, only_v + su), both_lim));
      return __builtin_amdgcn_ballot_w64(t <= lim) == 0;
    };
    if (PRUNE && STRAT != 0 && __builtin_amdgcn_ballot_w64(both <= __builtin_elementwise_sub_sat(lim, pen_low)) == 0) left = 0;
    while (left != 0) {
      bool fits = true;
      int pen_g = 0, c_h = 0, f_h = 0;
      if (UP == 3) {
        g = L - 1 - x[UP];
        tg = pre[g];
        if (STRAT != 0) {
          // stage H = [v, g)
          f_h = tg.x - tv.x;
          c_h = tg.y - tv.y;
          fits = scalar_peak(tv, tg, H) <= cap;
          xf = imax32(mf, f_h);
          xb = imax32(mb, c_h - f_h);
          u_h = tg.y + (N - 1 - H) * xb;
          v_h = tg.y + (N - 1 - H) * xf;
          gmax = imax32(none, scalar_own(H, c_h, tg.y));
          if (STRAT == 2) pen_g = (int)share_h * c_h;
          layers_up = imax32(layers_low, g - v);
          if (PRUNE) {
            if (STRAT == 2) lim = ok ? __builtin_elementwise_sub_sat(limit, comm + pen_low + pen_g) : (int)0x80000000;
            fits = fits && !hopeless(imax32(u_h, tl.y), imax32(v_h, tl.y), 0);
          }
        }
      }
      do {
        const int m = L - 1 - x[2];
        const i32x4 tm = pre[m];
        uint32_t n = (uint32_t)(x[2] - x[1]);
        n = n < left ? n : left;
        left -= n;
        const int y = L - 1 - x[1];
        x[1] = 0;
        ++x[2];
        if (STRAT != 0) {
          if (UP == 3) {
            // stage N-3 = [g, m)
            const int f = tm.x - tg.x, c = tm.y - tg.y;
            if (!fits || scalar_peak(tg, tm, N - 3) > cap || n == 0) continue;
            xf2 = imax32(xf, f);
            xb2 = imax32(xb, c - f);
            u_m = tm.y + 2 * xb2;
            v_m = tm.y + 2 * xf2;
            own_m = scalar_own(N - 3, c, tm.y);
            pen_up = STRAT == 2 ? pen_g + (int)share_m * c : 0;
            if (rounds > 0) rounds_low = rounds * imax32(layers_up, m - g);
          } else {
            // stage H = N-3 = [v, m)
            const int f = tm.x - tv.x, c = tm.y - tv.y;
            if (scalar_peak(tv, tm, H) > cap || n == 0) continue;
            xf2 = imax32(mf, f);
            xb2 = imax32(mb, c - f);
            u_h = tm.y + 2 * xb2;
            v_h = tm.y + 2 * xf2;
            gmax = imax32(none, scalar_own(H, c, tm.y));
            pen_up = STRAT == 2 ? (int)share_h * c : 0;
            if (rounds > 0) rounds_low = rounds * imax32(layers_low, m - v);
          }
          if (STRAT == 2) {
            off = comm + pen_low + pen_up;
            lim = ok ? __builtin_elementwise_sub_sat(limit, off) : (int)0x80000000;
          }
          if (PRUNE) {
            int su = tl.y, sv = tl.y, least = 0;
            if (UP == 3) {
              su = imax32(su, u_m);
              sv = imax32(sv, v_m);
              least = su + sv + own_m;
            }
            if (hopeless(imax32(su, u_h), imax32(sv, v_h), least)) continue;
          }
          walk(m, m, y, n, 0, 0);
        } else {
          // node H-1 = [cut H-1, cut H+1); UP = 3: node H = [v, m); node N-2 = [m, L)
          const i32x4 tu = UP == 3 ? tg : tm;
          if (scalar_peak(tm, tl, N - 2) > cap || (UP == 3 && scalar_peak(tv, tm, H) > cap) || n == 0) continue;
          const int coef_g = ff->mem_coef[H - 1];
          const int need_g = coef_g < 0 ? 0 : tu.z + tu.w * coef_g;
          ok_g = ok && need_g - tb.z <= cap;
          const bool gone_g = gone(H - 1);
          const int f0 = gone_g ? 0 : tu.x - tb.x;
          c0 = gone_g ? 0 : tu.y - tb.y;
          bf = imax32(mf, f0);
          bb = imax32(mb, c0 - f0);
          if (UP == 3 && !gone(H)) { f_h = tm.x - tv.x; c_h = tm.y - tv.y; } else { f_h = c_h = 0; }
          const int base = UP == 3 ? tg.y : tv.y;      // end of node N-4 in the records' times
          const int x1f = imax32(bf, f_h), x1b = imax32(bb, c_h - f_h);
          const int p_g = base - c_h;
          const int shift = sum_low + c0 - p_g;
          u_g = p_g + (int)__umul24((uint32_t)bb, (uint32_t)cl->after[H - 1]);
          v_g = p_g + (int)__umul24((uint32_t)bf, (uint32_t)cl->after[H - 1]);
          const int k_g = cl->steady[H - 1];
          gmax = imax32(none + shift, k_g < 0 ? HALVES_NEVER : (int)__umul24((uint32_t)c0, (uint32_t)k_g) - p_g);
          if (UP == 3) {
            u_h = base + (int)__umul24((uint32_t)x1b, (uint32_t)cl->after[H]);
            v_h = base + (int)__umul24((uint32_t)x1f, (uint32_t)cl->after[H]);
            own_h = scalar_own(H, c_h, base);
          }
          xb2 = (int)__umul24((uint32_t)x1b, (uint32_t)cl->after[N - 3]);
          xf2 = (int)__umul24((uint32_t)x1f, (uint32_t)cl->after[N - 3]);
          const int f2 = gone(N - 2) ? 0 : tl.x - tm.x, c2 = gone(N - 2) ? 0 : tl.y - tm.y;
          u_m = c2 + (int)__umul24((uint32_t)imax32(x1b, c2 - f2), (uint32_t)cl->after[N - 2]);
          v_m = c2 + (int)__umul24((uint32_t)imax32(x1f, f2), (uint32_t)cl->after[N - 2]);
          own_m = scalar_own(N - 2, c2, c2);
          both_lim = both - shift;
          off = shift + comm;
          lim = ok_g ? __builtin_elementwise_sub_sat(limit, off) : (int)0x80000000;
          room = ok_g ? room_z : (int)0x80000000;
          const int k_z = cl->steady[N - 1];
          if (PRUNE) {
            // (the ends of the records' nodes lie behind `base`)
            int su = base + imax32(u_m, xb2), sv = base + imax32(v_m, xf2), least = 0;
            if (UP == 3) {
              su = imax32(su, u_h);
              sv = imax32(sv, v_h);
              least = su + sv + own_h;
            }
            if (hopeless(imax32(su, u_g), imax32(sv, v_g), least)) continue;
          }
          walk(UP == 3 ? g : v, m, y, n, c2, k_z < 0 ? 0 : k_z);
        }
      } while (left != 0 && UP == 3 && x[2] < x[UP]);
      if (UP == 3) { ++x[UP]; x[2] = 1; }
    }
    if (STRAT != 0) n_fit *= low_fit;

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
      if (cost < inc0) atomicMin((unsigned long long *)a.s.incumbent, (unsigned long long)cost);
      atomicMin((unsigned long long *)a.s.result + chunk * a.chunk_words + slot, (unsigned long long)((cost << a.s.idx_bits) | local));
    }
  }
}

template <int STRAT, int N, int UP>
void launch_halves(const HalvesLaunch &a, bool build, hipStream_t st) {
  if (build) hipLaunchKernelGGL((k_pair_records<N, STRAT, UP>), dim3((a.n_pairs + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, st, a);
  const uint32_t blocks = (a.n_items + BLOCK / 64 - 1) / (BLOCK / 64);
  if (a.bounded) hipLaunchKernelGGL((k_search_halves<N, STRAT, UP, true>), dim3(blocks), dim3(BLOCK), 0, st, a);
  else hipLaunchKernelGGL((k_search_halves<N, STRAT, UP, false>), dim3(blocks), dim3(BLOCK), 0, st, a);
}

// build: the table of pairs is filled first.  1 = no instance for this shape.
template <int STRAT>
int halves_by_stages(int sp, int up, const HalvesLaunch &a, bool build, hipStream_t st) {
#define CHM_CASE(SPV)                                                                                                        \
  case SPV:                                                                                                                  \
    if constexpr (SPV <= HALVES_TWO_UP_TO) { if (up == 2) { launch_halves<STRAT, SPV, 2>(a, build, st); return 0; } }        \
    if constexpr (SPV >= HALVES_THREE_FROM) { if (up == 3) { launch_halves<STRAT, SPV, 3>(a, build, st); return 0; } }       \
    return 1;
  switch (sp) {
#ifdef CHM_TUNING_SUBSET
    CHM_CASE(7) CHM_CASE(8)
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
