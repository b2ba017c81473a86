// Exhaustive search of a whole family by halves: the kernels for large spaces.  Included by one translation unit per
// strategy, behind chm_search_kernel.h.
//
// A partition is a lower half (its first H cuts) and an upper half (its last UP cuts).  Everything a plan's step time is
// made of (pipeline_time in chm_search_kernel.h) splits at the cut between them: maxima and sums over the stages of one
// half alone, and a few terms of the stage that crosses.  So a lane keeps one lower half in registers, a wavefront walks
// a list of upper halves whose share was worked out once for all lower halves (k_upper_halves) and arrives through
// scalar loads.  Bound by VALU issue: a partition costs 51 to 54 lane instructions at 7 and 8 stages (104 with the two pipeline
// classes of strategy 0), lanes without a lower half and the wavefronts' own lower halves included, where working it out on
// its own costs over 200 at 8 stages and 300 at 11; a step of the loop costs the same at any depth, idle lanes weigh where
// lower halves are few (fast_select decides for which families it pays and how many cuts an upper half takes).  62.9 M partitions
// of 8 stages: 0.12 ms (0.44 ms one by one in the range kernel), 5.2 G of 11 stages: 6.4 ms (51).  64 VGPRs or fewer at one
// class: 8 waves per SIMD, which hide the scalar loads.  All lanes of a wavefront have the same last lower cut v, and the list is ordered by its
// first cut, descending: the upper halves that go with v are the first C(L-1-v, UP) of the list, for every v.
//
// Every partition's memory peak and step time are worked out.  The weights to fetch (the transition time) only where
// horizon x step time alone does not already exceed the lowest cost met so far in the search: elsewhere they cannot
// change the argmin, ties included.
#ifndef CHM_HALVES_KERNEL_H
#define CHM_HALVES_KERNEL_H
#include "chm_search_kernel.h"

namespace {

// a uniform value held in a vector register
__device__ __forceinline__ int in_vector(int x) {
  asm volatile("v_mov_b32 %0, %1" : "=v"(x) : "s"(x));
  return x;
}
// least reroute penalty of a stage all of whose peers have one speed (stage_penalty; nothing else comes here)
__device__ __forceinline__ uint32_t even_penalty(ScnPtr scn, TabPtr tab, int st, int f, int b) {
  return tab->even_share[st] * peer_time(f, b, scn->aff_q[st][0]);
}
constexpr int HALVES_NEVER = -(1 << 30);   // a term of a maximum that does not exist
// memory peak of a lane without a lower half: above every cap (the peaks of plans stay below it by the bound that selects
// these kernels, so a cap of 2^31 - 1, "no limit", can be taken as one less)
constexpr int IDLE_PEAK = 0x7fffffff;

// Words of an upper half's record.  UP cuts c[H+1..K]; the stages behind the crossing one, s = H+1..N-1, have UP nodes
// of which the last has no waiting behind it.  (Strategy 0: node s runs stages s and s+1, the last node also stage 0.)
// The words every partition needs come first: they are what the loop loads, one record ahead.
template <int STRAT, int UP, int NC>
struct Upper {
  enum {
    PC1 = 0, PF1, PW1,                    // prefixes at c[H+1]: forward + backward, forward, memory
    PEAK,                                 // largest memory peak of the upper stages alone
    PENALTY,                              // reroute penalties of upper stages (strategy 2; strategy 0: see below)
    PC2 = 4, PF2, PW2,                    // strategy 0: prefixes at c[H+2] (at L when UP is 1)
    WRAP_C, WRAP_W,                       // strategy 0: the last stage's times and memory (its node also runs stage 0)
    CLASS0 = STRAT == 0 ? WRAP_W + 1 : PENALTY + 1,
    // per class, relative to the end of the crossing node H: for the nodes s = N-2 .. H+1, their R (time from H up to and
    // with s), the suffix maxima of U and V over the upper nodes alone, and (M-n+s) C - R; then R of the node N-2 (strategy
    // 0) or N-1, and (other strategies) the last node's own term
    MID = 4, LAST = MID * (UP - 1), PER_CLASS = LAST + (STRAT == 0 ? 1 : 2),
    HOT = CLASS0 + NC * PER_CLASS,
    CUTS = HOT,                           // all UP cuts, a byte each
    RANK_LO, RANK_HI,                     // their share of the partition rank
    LAYERS,                               // layers of the largest upper stage
    PA1, PA2, WRAP_A,                     // activation memory, like PW1, PW2, WRAP_W
    WORDS = (WRAP_A + 1 + 3) / 4 * 4
  };
};

// One lane per upper half, in the order of the list: position p = sum of C(x_i, i) over UP falling digits x, and the cuts
// are L-1-x, ascending.
template <int N, int STRAT, int UP, int NC>
__global__ void __launch_bounds__(BLOCK) k_upper_halves(HalvesLaunch a) {
  constexpr int K = N - 1, H = K - UP;
  typedef Upper<STRAT, UP, NC> R;
  constexpr int W = R::WORDS;
  __shared__ int4 T[DEV_MAX_L + 1];
  __shared__ uint64_t BN[K * DEV_MAX_L];
  const ScnPtr scn = as_const(a.s.scn);
  const TabPtr tab = as_const(a.tab);
  const FamPtr ff = &tab->fam[STRAT];
  const int L = scn->L;
  for (int i = threadIdx.x; i <= L; i += BLOCK) T[i] = make_int4((int)scn->pf[i], (int)(scn->pf[i] + scn->pb[i]), (int)scn->pw[i], (int)scn->pa[i]);
  for (int i = threadIdx.x; i < K * DEV_MAX_L; i += BLOCK) BN[i] = scn->binom[1 + i / DEV_MAX_L][i % DEV_MAX_L];
  __shared__ uint32_t items[DEV_MAX_L];
  if (blockIdx.x == 0 && threadIdx.x < DEV_MAX_L) {
    // wavefront items per last lower cut v, and where v's first one is
    const int v = (int)threadIdx.x;
    uint32_t n = 0;
    if (v >= H && v <= L - 1 - UP) {
      const uint32_t low = (uint32_t)scn->binom[H - 1][v - 1], up = (uint32_t)scn->binom[UP][L - 1 - v];
      n = ((low + 63u) / 64u) * ((up + a.chunk - 1) / a.chunk);
    }
    items[v] = n;
  }
  __syncthreads();
  if (blockIdx.x == 0 && threadIdx.x < DEV_MAX_L) {
    uint32_t first = 0;
    for (int v = 0; v < (int)threadIdx.x; ++v) first += items[v];
    a.items->first[threadIdx.x] = first;
  }
  if (blockIdx.x == 0) {
    // what every workgroup of the search stages in LDS, in the form it wants it (binomials up to 2^32 - 1: ranks of lower
    // halves are below that)
    for (int i = threadIdx.x; i <= L; i += BLOCK) a.items->prefix[i] = T[i];
    for (int i = threadIdx.x; i < H * DEV_MAX_L; i += BLOCK) a.items->binom[i] = BN[i] > 0xffffffffull ? 0xffffffffu : (uint32_t)BN[i];
  }
  const uint32_t p = blockIdx.x * BLOCK + threadIdx.x;
  if (p >= a.n_upper) return;
  int x[UP + 2];
  unrank_digits<UP, uint64_t>(p, L, (L - 1) <= 64 ? 3 : 4, BN, x);              // x[i] = digit + 1, i = 1..UP
  int c[UP + 2];                                                       // c[1..UP] = c[H+1..K]; c[UP+1] = L
#pragma unroll
  for (int i = 1; i <= UP; ++i) c[i] = L - x[UP + 1 - i];
  c[UP + 1] = L;
  int4 t[UP + 2];
  uint64_t rank = 0;
  uint32_t packed = 0;
#pragma unroll
  for (int i = 1; i <= UP + 1; ++i) {
    t[i] = T[c[i]];
    if (i <= UP) {
      rank += BN[(H + i - 1) * DEV_MAX_L + c[i] - 1];
      packed |= (uint32_t)c[i] << (8 * (i - 1));
    }
  }
  uint32_t rec[W];
#pragma unroll
  for (int i = 0; i < W; ++i) rec[i] = 0;
  rec[R::PC1] = (uint32_t)t[1].y; rec[R::PF1] = (uint32_t)t[1].x; rec[R::PW1] = (uint32_t)t[1].z; rec[R::PA1] = (uint32_t)t[1].w;
  rec[R::CUTS] = packed;
  rec[R::RANK_LO] = (uint32_t)rank; rec[R::RANK_HI] = (uint32_t)(rank >> 32);
  // times of the upper nodes H+i, i = 1..UP: stage H+i = [c[i], c[i+1]) (strategy 0: two stages, [c[i], c[i+2]); the last
  // node's second one is stage 0, added by the lower half)
  int F[UP + 1], C[UP + 1];
  int peak = 0, layers = 0;
#pragma unroll
  for (int i = 1; i <= UP; ++i) {
    const int e = STRAT == 0 && i < UP ? i + 2 : i + 1;
    F[i] = t[e].x - t[i].x;
    C[i] = t[e].y - t[i].y;
    const int coef = ff->mem_coef[H + i];
    const int m = t[e].z - t[i].z + (ff->has_act ? (int)__umul24((uint32_t)(t[e].w - t[i].w), (uint32_t)(coef < 0 ? 0 : coef)) : 0);
    if (!(STRAT == 0 && i == UP)) peak = imax32(peak, coef < 0 ? 0 : m);
    layers = imax32(layers, c[i + 1] - c[i]);
  }
  rec[R::PEAK] = (uint32_t)peak;
  rec[R::LAYERS] = (uint32_t)layers;
  if (STRAT == 0) {
    const int second = UP >= 2 ? 2 : UP + 1;
    rec[R::PC2] = (uint32_t)t[second].y; rec[R::PF2] = (uint32_t)t[second].x; rec[R::PW2] = (uint32_t)t[second].z; rec[R::PA2] = (uint32_t)t[second].w;
    rec[R::WRAP_C] = (uint32_t)C[UP];
    rec[R::WRAP_W] = (uint32_t)(t[UP + 1].z - t[UP].z);
    rec[R::WRAP_A] = (uint32_t)(t[UP + 1].w - t[UP].w);
  }
  if (STRAT == 2) {
    uint32_t pen = 0;
    for (int st = 0; st < scn->n_aff; ++st) {
      const int sa = scn->aff_stage[st] - H;                           // uniform
      if (sa < 1) continue;
      int f = F[1], cc = C[1];
#pragma unroll
      for (int i = 2; i <= UP; ++i) { f = sa == i ? F[i] : f; cc = sa == i ? C[i] : cc; }
      pen += even_penalty(scn, tab, st, f, cc - f);
    }
    rec[R::PENALTY] = pen;
  }
#pragma unroll
  for (int ci = 0; ci < NC; ++ci) {
    const ClsPtr cl = &ff->cls[ci];
    int r[UP + 1], u[UP + 1], v[UP + 1], own[UP + 1];
    int sum = 0, mf = 0, mb = 0;
#pragma unroll
    for (int i = 1; i <= UP; ++i) {
      const bool dead = STRAT == 0 && ((cl->dead >> (H + i)) & 1u);
      const int f = dead ? 0 : F[i], cc = dead ? 0 : C[i];
      sum += cc;
      mf = imax32(mf, f);
      mb = imax32(mb, cc - f);
      r[i] = sum;
      u[i] = sum + cl->after[H + i] * mb;
      v[i] = sum + cl->after[H + i] * mf;
      own[i] = cl->steady[H + i] < 0 ? HALVES_NEVER : cl->steady[H + i] * cc - sum;
    }
    uint32_t *out = rec + R::CLASS0 + ci * R::PER_CLASS;
    int su = STRAT == 0 ? 0 : r[UP], sv = su;        // (strategy 0: the last node's time is not known here)
#pragma unroll
    for (int i = UP - 1; i >= 1; --i) {
      su = imax32(su, u[i]);
      sv = imax32(sv, v[i]);
      uint32_t *mid = out + R::MID * (UP - 1 - i);
      mid[0] = (uint32_t)r[i]; mid[1] = (uint32_t)su; mid[2] = (uint32_t)sv; mid[3] = (uint32_t)own[i];
    }
    out[R::LAST] = (uint32_t)(STRAT == 0 ? (UP >= 2 ? r[UP - 1] : 0) : r[UP]);
    if (STRAT != 0) out[R::LAST + 1] = (uint32_t)(r[UP] + r[UP] + own[UP]);
  }
  uint4 *dst = (uint4 *)(a.upper + (size_t)p * W);
#pragma unroll
  for (int i = 0; i < W / 4; ++i) dst[i] = make_uint4(rec[4 * i], rec[4 * i + 1], rec[4 * i + 2], rec[4 * i + 3]);
}

// One wavefront per (v, 64 lower halves that end with cut v, `chunk` upper halves); see the head of the file.
template <int N, int STRAT, int UP, int NC>
__global__ void __launch_bounds__(BLOCK) k_search_halves(HalvesLaunch a) {
  constexpr int K = N - 1, H = K - UP;
  constexpr int LOW = STRAT == 0 ? H - 1 : H;         // nodes of the lower half alone; the next one (strategy 0: two) cross
  typedef Upper<STRAT, UP, NC> R;
  constexpr int W = R::WORDS;
  __shared__ int4 T[DEV_MAX_L + 1];
  __shared__ uint32_t BN[H * DEV_MAX_L];
  __shared__ uint64_t wave_cost[BLOCK / 64], wave_rank[BLOCK / 64];
  __shared__ uint32_t wave_fit[BLOCK / 64];
  const ScnPtr scn = as_const(a.s.scn);
  const TabPtr tab = as_const(a.tab);
  const FamPtr ff = &tab->fam[STRAT];
  const int L = scn->L;
  for (int i = threadIdx.x; i <= L; i += BLOCK) T[i] = a.items->prefix[i];
  for (int i = threadIdx.x; i < H * DEV_MAX_L; i += BLOCK) BN[i] = a.items->binom[i];
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t item = __builtin_amdgcn_readfirstlane(blockIdx.x * (BLOCK / 64) + wave);
  uint64_t best_cost = ~0ull, best_rank = ~0ull;
  uint32_t n_fit = 0;
  const uint64_t inc0 = __hip_atomic_load(a.s.incumbent, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (item < a.n_items) {
    // the item's v: items are numbered v by v
    const uint64_t below_lo = __builtin_amdgcn_ballot_w64(a.items->first[lane] <= item);
    const uint64_t below_hi = __builtin_amdgcn_ballot_w64(a.items->first[lane + 64] <= item);
    const int v = (int)__popcll(below_lo) + (int)__popcll(below_hi) - 1;     // first_item grows with v (equal where v has none)
    const uint32_t local = item - (uint32_t)__builtin_amdgcn_readfirstlane(a.items->first[v]);
    const uint32_t n_up = (uint32_t)scn->binom[UP][L - 1 - v];               // upper halves that go with v
    const uint32_t n_low = (uint32_t)scn->binom[H - 1][v - 1];               // lower halves that end with v
    const uint32_t low_blocks = (n_low + 63u) / 64u;
    const uint32_t part = local / low_blocks, low_block = local - part * low_blocks;
    uint32_t up = part * a.chunk;
    const uint32_t up_end = up + a.chunk < n_up ? up + a.chunk : n_up;

    // ---- this lane's lower half
    const uint32_t q = low_block * 64u + (uint32_t)lane;
    const bool active = q < n_low;
    int c[H + 1];
    unrank_digits<H - 1, uint32_t>(active ? q : 0u, v, (v - 1) <= 64 ? 3 : 4, BN, c);   // digits 0..v-2: cuts 1..v-1
    c[0] = 0;
    c[H] = v;
    const uint64_t low_rank = (uint64_t)q + BN[(H - 1) * DEV_MAX_L + v - 1];
    int4 t[H + 1];
    t[0] = make_int4(0, 0, 0, 0);
#pragma unroll
    for (int i = 1; i <= H; ++i) t[i] = T[c[i]];
    int peak_low = active ? 0 : IDLE_PEAK, layers_low = ff->fixed_layers;
    int F[LOW > 0 ? LOW : 1], C[LOW > 0 ? LOW : 1];
#pragma unroll
    for (int s = 0; s < LOW; ++s) {
      const int e = STRAT == 0 ? s + 2 : s + 1;
      F[s] = t[e].x - t[s].x;
      C[s] = t[e].y - t[s].y;
      const int coef = ff->mem_coef[s];
      const int m = t[e].z - t[s].z + (ff->has_act ? (int)__umul24((uint32_t)(t[e].w - t[s].w), (uint32_t)(coef < 0 ? 0 : coef)) : 0);
      peak_low = imax32(peak_low, coef < 0 ? 0 : m);
    }
#pragma unroll
    for (int s = 0; s < H; ++s) layers_low = imax32(layers_low, c[s + 1] - c[s]);
    uint32_t pen_low = 0, share_h = 0;
    if (STRAT == 2) {
      for (int st = 0; st < scn->n_aff; ++st) {
        const int sa = scn->aff_stage[st];                                   // uniform
        if (sa < H) {
          int f = F[0], cc = C[0];
#pragma unroll
          for (int s = 1; s < LOW; ++s) { f = sa == s ? F[s] : f; cc = sa == s ? C[s] : cc; }
          pen_low += even_penalty(scn, tab, st, f, cc - f);
        } else if (sa == H) {
          share_h = tab->even_share[st];
        }
      }
    }
    // per class: what the lower nodes contribute (see pipeline_time): maxima of forward and backward, time of the lower
    // nodes, and the maxima over the lower j of the terms own_j + {both, one, none} of the lower suffix maxima
    int mf[NC], mb[NC], sum_low[NC], both[NC], only_u[NC], only_v[NC], none[NC];
    // what the loop multiplies per class, in vector registers (an instruction takes one scalar operand, and that is the
    // record's): nodes behind and micro-batches - nodes + position (no node: 0) of the crossing nodes H, H-1 and N-1
    struct Crossing { int after, steady; };
    Crossing at_h[NC], at_g[NC], at_z[NC];
    int after_mid[NC][UP], comm[NC];
#pragma unroll
    for (int ci = 0; ci < NC; ++ci) {
      const ClsPtr cl = &ff->cls[ci];
      int u[LOW > 0 ? LOW : 1], w[LOW > 0 ? LOW : 1], own[LOW > 0 ? LOW : 1];
      int sum = 0;
      mf[ci] = mb[ci] = 0;
#pragma unroll
      for (int s = 0; s < LOW; ++s) {
        const bool dead = STRAT == 0 && ((cl->dead >> s) & 1u);
        const int f = dead ? 0 : F[s], cc = dead ? 0 : C[s];
        sum += cc;
        mf[ci] = imax32(mf[ci], f);
        mb[ci] = imax32(mb[ci], cc - f);
        u[s] = (int)__umul24((uint32_t)mb[ci], (uint32_t)cl->after[s]) + sum;
        w[s] = (int)__umul24((uint32_t)mf[ci], (uint32_t)cl->after[s]) + sum;
        own[s] = cl->steady[s] < 0 ? HALVES_NEVER : (int)__umul24((uint32_t)cc, (uint32_t)cl->steady[s]) - sum;
      }
      sum_low[ci] = sum;
      both[ci] = only_u[ci] = only_v[ci] = none[ci] = HALVES_NEVER;
      int su = 0, sv = 0;
#pragma unroll
      for (int s = LOW - 1; s >= 0; --s) {
        su = imax32(su, u[s]);
        sv = imax32(sv, w[s]);
        both[ci] = imax32(both[ci], su + sv + own[s]);
        only_u[ci] = imax32(only_u[ci], su + own[s]);
        only_v[ci] = imax32(only_v[ci], sv + own[s]);
        none[ci] = imax32(none[ci], own[s]);
      }
#pragma unroll
      for (int i = 1; i < UP; ++i) after_mid[ci][i] = in_vector(cl->after[H + i]);
      auto crossing = [cl](int s) {
        const int k = cl->steady[s];
        return Crossing{in_vector(cl->after[s]), in_vector(k < 0 ? 0 : k)};
      };
      at_h[ci] = crossing(H);
      at_g[ci] = STRAT == 0 ? crossing(H - 1) : Crossing{0, 0};
      at_z[ci] = STRAT == 0 ? crossing(N - 1) : Crossing{0, 0};
      comm[ci] = in_vector(cl->comm_total);
      both[ci] += comm[ci];
    }
    const int4 tv = t[H], tw = t[STRAT == 0 ? H - 1 : H], t1 = t[1];

    // ---- the upper halves
    int cap = imin32((int)scn->cap, IDLE_PEAK - 1);
    asm("" : "+s"(cap));     // (a compiler that sees this bound tests for idle lanes apart in every step: 1.3 % of the re-plan's time)
    const int fixed_step = in_vector(ff->fixed_step);
    const double per_step = 1.0 / (double)scn->K;
    auto limit_of = [&](uint64_t cost) -> int {       // no step time above this can reach `cost` (rounded up)
      const uint64_t reconf = (uint64_t)scn->reconf[STRAT];
      if (cost == ~0ull) return 0x7fffffff;
      if (cost < reconf) return -1;
      const double x = (double)(cost - reconf) * per_step + 1.0;
      return x >= 2147483647.0 ? 0x7fffffff : (int)x;
    };
    int limit = __builtin_amdgcn_readfirstlane(limit_of(inc0));
    const RowPtr list = as_const((const uint32_t *)a.upper);
    // exceptions to the plain memory check and step time, all uniform
    enum { ACTIVATIONS = 1, FREE_G = 2, FREE_H = 4, FREE_Z = 8, ROUNDS = 16, PEAKS = ACTIVATIONS | FREE_G | FREE_H | FREE_Z, GONE = 32 };
    uint32_t odd = (ff->has_act ? ACTIVATIONS : 0) | (ff->mem_coef[H] < 0 ? FREE_H : 0);
    if (STRAT == 0) odd |= (ff->mem_coef[H - 1] < 0 ? FREE_G : 0) | (ff->mem_coef[N - 1] < 0 ? FREE_Z : 0);
    else odd |= ff->allreduce > 0 ? ROUNDS : 0;
    uint32_t gone[NC];                                // per class: crossing nodes it does without (bits of their stages)
#pragma unroll
    for (int ci = 0; ci < NC; ++ci) {
      gone[ci] = STRAT == 0 ? ff->cls[ci].dead & ((1u << H) | (1u << (H - 1)) | (1u << (N - 1))) : 0u;
      odd |= gone[ci] ? GONE << ci : 0;
    }
    uint32_t nx[R::HOT];
#pragma unroll
    for (int i = 0; i < R::HOT; ++i) nx[i] = list[(size_t)up * W + i];
    for (; up < up_end; ++up) {
      uint32_t rec[R::HOT];
#pragma unroll
      for (int i = 0; i < R::HOT; ++i) rec[i] = nx[i];
      const RowPtr cold = list + (size_t)up * W;
      const RowPtr next = up + 1 < up_end ? cold + W : cold;
#pragma unroll
      for (int i = 0; i < R::HOT; ++i) nx[i] = next[i];
      if ((int)rec[R::PEAK] > cap) continue;           // uniform: none of these partitions fits
      // memory and times of the crossing nodes: H = [c[H], c[H+1]); strategy 0: H-1 = [c[H-1], c[H+1]), H = [c[H],
      // c[H+2]) and the last node, which also runs stage 0
      int fh, ch, fg = 0, cg = 0, cz = 0, mh, mg = 0, mz = 0;
      if (STRAT == 0) {
        fg = (int)rec[R::PF1] - tw.x;
        cg = (int)rec[R::PC1] - tw.y;
        mg = (int)rec[R::PW1] - tw.z;
        fh = (int)rec[R::PF2] - tv.x;
        ch = (int)rec[R::PC2] - tv.y;
        mh = (int)rec[R::PW2] - tv.z;
        cz = (int)rec[R::WRAP_C] + t1.y;
        mz = (int)rec[R::WRAP_W] + t1.z;
      } else {
        fh = (int)rec[R::PF1] - tv.x;
        ch = (int)rec[R::PC1] - tv.y;
        mh = (int)rec[R::PW1] - tv.z;
      }
      if (odd & PEAKS) {
        if (odd & ACTIVATIONS) {
          auto act = [&](int mib, int s) { const int coef = ff->mem_coef[s]; return (int)__umul24((uint32_t)mib, (uint32_t)(coef < 0 ? 0 : coef)); };
          mh += act((int)cold[STRAT == 0 ? R::PA2 : R::PA1] - tv.w, H);
          if (STRAT == 0) { mg += act((int)cold[R::PA1] - tw.w, H - 1); mz += act((int)cold[R::WRAP_A] + t1.w, N - 1); }
        }
        if (odd & FREE_H) mh = 0;
        if (odd & FREE_G) mg = 0;
        if (odd & FREE_Z) mz = 0;
      }
      const int bh = ch - fh, bg = cg - fg;
      const int peak = STRAT == 0 ? imax32(imax32(peak_low, mh), imax32(mg, mz)) : imax32(peak_low, mh);
      const uint64_t fit_mask = __builtin_amdgcn_ballot_w64(peak <= cap);
      // Nothing to time where no lane fits (uniform).  Strategy 0's nodes hold two stages and its time is the longest: under a
      // cap that next to nothing fits, 15.4 M partitions 64 instead of 85 us.  (The shorter times of the other strategies gain 2 us
      // there and lose as much everywhere else to the branch.)
      if (STRAT == 0 && fit_mask == 0) continue;
      n_fit += (uint32_t)__popcll(fit_mask);
      // ---- step time: the sum of pipeline_time from the last node down, relative to the end of node H
      int step = fixed_step;
#pragma unroll
      for (int ci = 0; ci < NC; ++ci) {
        const uint32_t *up_c = rec + R::CLASS0 + ci * R::PER_CLASS;
        int f1 = fh, b1 = bh, c1 = ch, f0 = fg, b0 = bg, c0 = cg, cl_z = cz;
        if (STRAT == 0 && (odd & (GONE << ci))) {      // uniform, seldom
          asm volatile("");                            // (kept a branch: as selects it would cost every class)
          if ((gone[ci] >> H) & 1u) f1 = b1 = c1 = 0;
          if ((gone[ci] >> (H - 1)) & 1u) f0 = b0 = c0 = 0;
          if ((gone[ci] >> (N - 1)) & 1u) cl_z = 0;
        }
        // largest forward and backward up to node H (strategy 0: and up to H-1)
        const int bf = STRAT == 0 ? imax32(mf[ci], f0) : mf[ci], bb = STRAT == 0 ? imax32(mb[ci], b0) : mb[ci];
        const uint32_t xf = (uint32_t)imax32(bf, f1), xb = (uint32_t)imax32(bb, b1);
        int su, sv, r;
        if (STRAT == 0) {
          su = sv = (int)up_c[R::LAST] + cl_z;
          r = (int)__umul24((uint32_t)cl_z, (uint32_t)at_z[ci].steady) + su;        // (no such node: 0 x 0 + su, covered by others)
        } else {
          su = sv = (int)up_c[R::LAST];
          r = (int)up_c[R::LAST + 1];
        }
#pragma unroll
        for (int i = UP - 1; i >= 1; --i) {
          const uint32_t *mid = up_c + R::MID * (UP - 1 - i);
          const uint32_t k = STRAT == 0 ? (uint32_t)after_mid[ci][i] : (uint32_t)(UP - i);
          // (the record's suffix maxima hold the last node's too, except under strategy 0)
          const int ub = (int)__umul24(xb, k) + (int)mid[0], uf = (int)__umul24(xf, k) + (int)mid[0];
          if (STRAT != 0 && i == UP - 1) {
            su = imax32((int)mid[1], ub);
            sv = imax32((int)mid[2], uf);
          } else {
            su = imax32(imax32(su, (int)mid[1]), ub);
            sv = imax32(imax32(sv, (int)mid[2]), uf);
          }
          r = imax32(r, su + sv + (int)mid[3]);
        }
        su = imax32(su, (int)__umul24(xb, STRAT == 0 ? (uint32_t)at_h[ci].after : (uint32_t)UP));
        sv = imax32(sv, (int)__umul24(xf, STRAT == 0 ? (uint32_t)at_h[ci].after : (uint32_t)UP));
        int ss = su + sv;
        r = imax32(r, (int)__umul24((uint32_t)c1, (uint32_t)at_h[ci].steady) + ss);
        int end_h = sum_low[ci] + c1;                  // time of the nodes up to H
        if (STRAT == 0) {
          su = imax32(su, (int)__umul24((uint32_t)bb, (uint32_t)at_g[ci].after) - c1);
          sv = imax32(sv, (int)__umul24((uint32_t)bf, (uint32_t)at_g[ci].after) - c1);
          ss = su + sv;
          r = imax32(r, (int)__umul24((uint32_t)c0, (uint32_t)at_g[ci].steady) + ss + c1);
          end_h += c0;
        }
        // the lower nodes' terms
        r = imax32(imax32(r, only_u[ci] + sv), only_v[ci] + su);
        r = imax32(r, ss + none[ci] + end_h);
        step = imax32(step, imax32(r + end_h + comm[ci], both[ci]));
      }
      if (STRAT == 2) step += (int)(pen_low + rec[R::PENALTY] + __umul24(share_h, (uint32_t)ch));
      if (STRAT != 0 && (odd & ROUNDS)) {
        const int stage_h = (int)(cold[R::CUTS] & 0xffu) - v;
        step += ff->allreduce * imax32(imax32(layers_low, stage_h), (int)cold[R::LAYERS]);
      }
      const bool near_best = peak <= cap && step <= limit;
      if (__builtin_amdgcn_ballot_w64(near_best) == 0) continue;
      // ---- the few that may win: weights to fetch, cost, ties by rank
      int wp[N + 1];
      wp[0] = 0;
      wp[N] = T[L].z;
      const uint32_t cuts = cold[R::CUTS];
#pragma unroll
      for (int i = 1; i <= K; ++i) wp[i] = i <= H ? t[i <= H ? i : 0].z : T[(cuts >> (8 * (i <= H ? 0 : i - H - 1))) & 0xffu].z;
      const uint64_t cost = (uint64_t)scn->K * (uint32_t)step + (uint64_t)scn->reconf[STRAT] +
                            (uint64_t)scn->xfer * (uint32_t)missing_weights<N, STRAT>(ff, wp);
      const uint64_t rank = low_rank + ((uint64_t)cold[R::RANK_LO] | ((uint64_t)cold[R::RANK_HI] << 32));
      if (near_best && (cost < best_cost || (cost == best_cost && rank < best_rank))) { best_cost = cost; best_rank = rank; }
      const int seen = __builtin_amdgcn_readfirstlane(limit_of(wave_min(near_best ? cost : ~0ull)));
      limit = limit < seen ? limit : seen;
    }
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

template <int STRAT, int N, int UP, int NC>
void launch_halves(const HalvesLaunch &a, bool build, hipStream_t st) {
  if (build) hipLaunchKernelGGL((k_upper_halves<N, STRAT, UP, NC>), dim3((a.n_upper + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, st, a);
  const uint32_t blocks = (a.n_items + BLOCK / 64 - 1) / (BLOCK / 64);
  hipLaunchKernelGGL((k_search_halves<N, STRAT, UP, NC>), dim3(blocks), dim3(BLOCK), 0, st, a);
}

template <int STRAT, int N>
int halves_by_shape(int up, int n_cls, const HalvesLaunch &a, bool build, hipStream_t st) {
#define CHM_SHAPE(UPV, NCV) if (up == UPV && n_cls == NCV) { launch_halves<STRAT, N, UPV, NCV>(a, build, st); return 0; }
  CHM_SHAPE(2, 1)
  if constexpr (STRAT == 0) { CHM_SHAPE(2, 2) CHM_SHAPE(2, 3) }
  if constexpr (N >= 7) { CHM_SHAPE(3, 1) }          // (fewer stages: lower halves of one or two cuts, too few for 64 lanes)
  if constexpr (N >= 7 && STRAT == 0) { CHM_SHAPE(3, 2) CHM_SHAPE(3, 3) }
#undef CHM_SHAPE
  return 1;
}

// build: the table of upper halves is filled first.  1 = no instance for this shape.
template <int STRAT>
int halves_by_stages(int sp, int up, int n_cls, const HalvesLaunch &a, bool build, hipStream_t st) {
  switch (sp) {
#define CHM_CASE(SPV) case SPV: return halves_by_shape<STRAT, SPV>(up, n_cls, a, build, st);
#ifdef CHM_TUNING_SUBSET
    CHM_CASE(7) CHM_CASE(8)
#else
    CHM_CASE(5) CHM_CASE(6) CHM_CASE(7) CHM_CASE(8) CHM_CASE(9) CHM_CASE(10)
    CHM_CASE(11) CHM_CASE(12) CHM_CASE(13) CHM_CASE(14) CHM_CASE(15) CHM_CASE(16)
#endif
#undef CHM_CASE
    default: return 1;
  }
}

// words of an upper half's record
template <int STRAT>
int halves_words(int up, int n_cls) {
  if (up == 3) return n_cls == 1 ? (int)Upper<STRAT, 3, 1>::WORDS : n_cls == 2 ? (int)Upper<STRAT, 3, 2>::WORDS : (int)Upper<STRAT, 3, 3>::WORDS;
  return n_cls == 1 ? (int)Upper<STRAT, 2, 1>::WORDS : n_cls == 2 ? (int)Upper<STRAT, 2, 2>::WORDS : (int)Upper<STRAT, 2, 3>::WORDS;
}

}  // namespace
#endif
