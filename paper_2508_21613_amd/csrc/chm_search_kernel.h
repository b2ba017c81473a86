// Shape-specialised search kernels of libchm for gfx950 (wave64, plain VALU integer work: the path is a max-plus
// longest path, not a dense contraction, so no MFMA).  Included by one translation unit per strategy, which
// instantiates the kernels for every number of stages.
//
// One lane owns a run of consecutive partition ranks.  It unranks the first one
// (combinatorial number system), then walks to each next partition with a branch-free
// successor step, so unranking is amortised over the run.  Everything a plan needs lives
// in registers: the cut positions, the per-stage sums (read from one LDS table of prefix
// sums staged once per workgroup), and the few sums and maxima the pipeline time is made of (pipeline_time).
// All values are int32: the host only selects these kernels when its load-time bound shows
// that no intermediate can reach 2^31, in which case the results equal the int64 ones.
//
// Data rerouting: after the base step time of a partition, the least penalty over all valid reroute vectors of
// every stage that lost nodes is added (least_penalty).
//
// Argmin: per lane a running (cost, run position) with strict less-than, so the lowest
// index wins inside a lane; then a DPP/shuffle wave reduction of the packed 64-bit key
// (cost << idx_bits | chunk-local partition index), one LDS step per workgroup and one
// 64-bit atomicMin per workgroup.
#ifndef CHM_SEARCH_KERNEL_H
#define CHM_SEARCH_KERNEL_H
#include <hip/hip_runtime.h>

#include "chm_fast.h"

namespace {

// The scenario tables are never written while a search kernel runs.  Reading them through the
// constant address space tells the compiler so: uniform reads become scalar loads (wide
// s_load_dwordx16 for the reroute rows) even though the kernel also stores costs to global memory.
#define CHM_CONST __attribute__((address_space(4)))
typedef const CHM_CONST DevScenario *ScnPtr;
typedef const CHM_CONST FastTables *TabPtr;
typedef const CHM_CONST FastFamily *FamPtr;
typedef const CHM_CONST FastClass *ClsPtr;
typedef const CHM_CONST uint32_t *RowPtr;
template <typename T>
__device__ __forceinline__ const CHM_CONST T *as_const(const T *p) {
  return (const CHM_CONST T *)(uintptr_t)p;
}

__device__ __forceinline__ int imax32(int a, int b) { return a > b ? a : b; }
__device__ __forceinline__ int imin32(int a, int b) { return a < b ? a : b; }
// a - b, 0 when that is negative (both below 2^31 and not negative): one saturating subtract
__device__ __forceinline__ uint32_t sub_floor(int a, int b) { return __builtin_elementwise_sub_sat((uint32_t)a, (uint32_t)b); }

// (x*q + 32768) >> 16 for 0 <= x < 2^31, q <= 2^20, result < 2^31
__device__ __forceinline__ int scale32(int x, uint32_t q) {
  return (int)(((uint64_t)(uint32_t)x * q + 32768u) >> 16);
}

// lower bound of scale32(f, q') + scale32(b, q') for any q' >= q, given x = f + b: each rounding loses less
// than one, so the sum is at least floor(x * q / 65536) - 1
__device__ __forceinline__ int scale_floor(int x, uint32_t q) {
  return q == 65536u ? x : imax32(0, (int)(((uint64_t)(uint32_t)x * q) >> 16) - 1);
}

// forward + backward time of a stage on a peer with factor q (uniform): nominal peers need no scaling
__device__ __forceinline__ uint32_t peer_time(int f, int b, uint32_t q) {
  return q == 65536u ? (uint32_t)(f + b) : (uint32_t)(scale32(f, q) + scale32(b, q));
}

// product of two numbers below 2^24 (low 32 bits), or of any two where the times do not fit 24 bits
template <bool M24>
__device__ __forceinline__ uint32_t times(uint32_t x, uint32_t y) { return M24 ? __umul24(x, y) : x * y; }

// 1F1B time of N stages, M micro-batches; F = forward, C = forward + backward per stage.  The estimator's dependency
// recurrence (eq. (transition); 2 N M cells) is the longest path of a graph so regular that its optimum is known in
// closed form, for every N, M >= 1:
//     T = max over j with M - N + j >= 0 of   SU[j] + SV[j] - P[j] + (M - N + j) C[j],
//     P[s] = C[0] + ... + C[s],  SU[j] = max over s >= j of P[s] + (N-1-s) max(B[0..s]),  SV[j] likewise with F.
// Why.  Run the rounds "forward t on every stage, then backward t-(N-1-s) on stage s" backwards in time from the end
// of the last backward of stage 0.  A path stands on a stage and every round it crosses adds one term:
//  - the N-1 rounds of backwards only: a round on stage k adds B[k] and the path stays or moves on to k+1; reaching
//    stage s takes B[0..s-1] once each, the N-1-s rounds left over are best spent on the largest B[0..s] met;
//  - the round of the last forward adds C[s] (with the forwards F[0..s-1] that lead to it: P[s] in all);
//  - the steady rounds: a round that adds C[k] leads to stage k+1, from where any stage up to k+1 can be next, so a
//    path climbs one stage per round, falls freely, and may stay on one stage j for as long as it likes; rounds not
//    needed for climbing belong to the largest C met;
//  - the warm-up mirrors the end with F in the place of B: from round N-1-s on stage s has forwards only, so a path
//    that leaves j climbs along that edge to some s (C[j+1..s] once each) and spends the N-1-s rounds left on the
//    largest F[0..s].
// Both ends use N-1-s and s-j rounds whatever s they turn at, which leaves exactly M-N+j rounds for C[j], and none
// of the choices depends on the others: hence the sum.  N maxima of N terms instead of 2 N M cells: at 8 stages and 16
// micro-batches about 80 instead of 280 instructions, at 16 and 64 about 160 instead of 2,000.
// A node that is left out of the pipeline (UNI: redundant computation, coefficients from the class) has F = C = 0,
// after = nodes behind it and steady = -1; its own term is never the largest (its neighbours' cover it).
template <int N, bool UNI, bool M24>
__device__ __forceinline__ int pipeline_time_m(const int (&F)[N], const int (&C)[N], ClsPtr cl) {
  const int M = cl->M;
  uint32_t U[N], V[N];
  uint32_t p = 0, max_f = 0, max_b = 0;              // p = P[s] on the way up, P[j] on the way down
#pragma unroll
  for (int s = 0; s < N; ++s) {
    const uint32_t f = (uint32_t)F[s], b = (uint32_t)(C[s] - F[s]);
    p += (uint32_t)C[s];
    max_f = max_f > f ? max_f : f;
    max_b = max_b > b ? max_b : b;
    const uint32_t after = UNI ? (uint32_t)cl->after[s] : (uint32_t)(N - 1 - s);
    U[s] = times<M24>(max_b, after) + p;
    V[s] = times<M24>(max_f, after) + p;
  }
  uint32_t su = 0, sv = 0, r = 0;
  if (M >= N) {                                      // uniform
#pragma unroll
    for (int j = N - 1; j >= 0; --j) {
      su = su > U[j] ? su : U[j];
      sv = sv > V[j] ? sv : V[j];
      const uint32_t k = UNI ? (uint32_t)cl->steady[j] : (uint32_t)(M - N + j);
      const uint32_t t = times<M24>((uint32_t)C[j], k) + su + (sv - p);
      r = r > t ? r : t;
      p -= (uint32_t)C[j];
    }
  } else {
#pragma unroll
    for (int j = N - 1; j >= 0; --j) {
      su = su > U[j] ? su : U[j];
      sv = sv > V[j] ? sv : V[j];
      const int k = UNI ? cl->steady[j] : M - N + j;
      if (k >= 0) {                                  // uniform
        const uint32_t t = times<M24>((uint32_t)C[j], (uint32_t)k) + su + (sv - p);
        r = r > t ? r : t;
      }
      p -= (uint32_t)C[j];
    }
  }
  return (int)r + cl->comm_total;
}

template <int N, bool UNI>
__device__ __forceinline__ int pipeline_time(const int (&F)[N], const int (&C)[N], ClsPtr cl, int time24) {
  return time24 ? pipeline_time_m<N, UNI, true>(F, C, cl) : pipeline_time_m<N, UNI, false>(F, C, cl);
}

constexpr int TERM_NEVER = -(1 << 30);   // a term of a maximum that does not exist

// Time of one pipeline class of a partition, stage after stage (at(i): prefixes of forward and forward + backward time at cut
// i).  The maximum of pipeline_time, read the other way round: a pair of stages (s, s') at which the two ends turn goes with
// the best own term of a stage not above either.  Four running maxima take the place of the arrays (16 instructions a stage
// instead of 13, but no registers that grow with the stages).
// EVEN: all nodes of the class have speed 1.
template <int N, int STRAT, bool M24, bool EVEN, typename At>
__device__ __forceinline__ int class_time(ClsPtr cl, At at) {
  const int M = cl->M;
  int none = TERM_NEVER, only_u = TERM_NEVER, only_v = TERM_NEVER, both = TERM_NEVER;
  int p = 0, mf = 0, mb = 0;
#pragma unroll
  for (int s = 0; s < N; ++s) {
    const int2 lo = at(s), hi = at(STRAT == 0 ? (s + 2 <= N ? s + 2 : N) : s + 1);
    int f = hi.x - lo.x, c = hi.y - lo.y;              // (strategy 0: a node runs two stages)
    if (STRAT == 0) {
      if (s == N - 1) { f += at(1).x; c += at(1).y; }
      const int keep = ((cl->dead >> s) & 1u) ? 0 : -1;          // uniform
      f &= keep;
      c &= keep;
    }
    if (!EVEN && !cl->unit) {                          // uniform
      const uint32_t q = cl->q_stage[s];
      const int b = scale32(c - f, q);
      f = scale32(f, q);
      c = f + b;
    }
    p += c;
    mf = imax32(mf, f);
    mb = imax32(mb, c - f);
    const int k = STRAT == 0 ? cl->steady[s] : M - N + s;
    if (k < 0) continue;                               // uniform: no own term, and no turn counts ahead of the first one
    const uint32_t after = STRAT == 0 ? (uint32_t)cl->after[s] : (uint32_t)(N - 1 - s);
    const int u = (int)(times<M24>((uint32_t)mb, after) + (uint32_t)p), v = (int)(times<M24>((uint32_t)mf, after) + (uint32_t)p);
    none = imax32(none, (int)times<M24>((uint32_t)c, (uint32_t)k) - p);
    only_u = imax32(only_u, none + u);
    only_v = imax32(only_v, none + v);
    both = imax32(imax32(both, only_u + v), only_v + u);
  }
  return both + cl->comm_total;
}

// The least of max_i r_i * w_i over all valid reroute vectors (0 <= r_i <= cap, sum = orphans), w_i = the stage's
// forward + backward time on peer i, all below 2^24.  Of the multiples w_i, 2 w_i, ..., cap w_i of all peers taken
// together a vector whose maximum is v uses only ones up to v, at least `orphans` of them; so the minimum is the
// orphans-th smallest multiple (equal ones counted one by one).  A peer whose time is 0 (a small factor rounds it down)
// has cap multiples of 0: they are taken first, and the peer takes no more.  Of the others' multiples those below
// (orphans left) / sum(1 / w_i) are fewer than the orphans left (floats, rounded well to the safe side), the few left are
// merged one at a time: about as many steps as there are peers, each a minimum over the peers, whatever the number of
// vectors (2,380,833 for 32 micro-batches over seven peers, which a sweep that shares their common entries took 318 us
// for; 153 for 16 over three).
// w[i] = NO_MULTIPLES for a peer without any left to take; taken = multiples of 0 taken already; most = multiples a peer has
// (cap, or all orphans); P = the most peers this instance takes.  Up to 4 (the usual case) everything is worked out for all
// four, which costs less than a branch per peer: two stages of 2 peers and 9 vectors each, 1.6 M partitions of 8 stages: 87 us
// a search, 97 with the instance for 15 peers (sweeping the 9 vectors 87).
constexpr uint32_t NO_MULTIPLES = 0xffffffffu;
template <int P>
__device__ __forceinline__ uint32_t least_penalty(const uint32_t (&w)[P], int peers, uint32_t taken, uint32_t orphans, uint32_t most) {
  constexpr bool ALL = P <= 4;
  float inv_sum = 0.0f;                              // (peers without multiples add next to nothing, to the safe side)
#pragma unroll
  for (int i = 0; i < P; ++i) {
    if (ALL || i < peers) inv_sum += __builtin_amdgcn_rcpf((float)w[i]);      // uniform
  }
  const float v0 = taken < orphans ? (float)(orphans - taken) * __builtin_amdgcn_rcpf(inv_sum) * 0.99999f : 0.0f;
  uint32_t next[P];                                  // peer i's smallest multiple not taken yet
#pragma unroll
  for (int i = 0; i < P; ++i) {
    next[i] = NO_MULTIPLES;
    if (ALL || i < peers) {
      uint32_t r = (uint32_t)(v0 * __builtin_amdgcn_rcpf((float)w[i]));      // (v0 < 2^31: 0 for a peer without multiples)
      r = r < most ? r : most;
      taken += r;
      next[i] = r < most && w[i] != NO_MULTIPLES ? __umul24(r + 1, w[i]) : NO_MULTIPLES;
    }
  }
  uint32_t least = 0;
  for (uint32_t guard = 0; taken < orphans && guard < 1100u; ++guard) {   // (at most 4 x 256 orphans: one step takes at least one)
    least = NO_MULTIPLES;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      if (ALL || i < peers) least = least < next[i] ? least : next[i];
    }
#pragma unroll
    for (int i = 0; i < P; ++i) {
      if (ALL || i < peers) {
        const bool hit = next[i] == least;
        taken += hit ? 1u : 0u;
        uint32_t after = next[i] + w[i];
        if (most < orphans && after > __umul24(most, w[i])) after = NO_MULTIPLES;
        next[i] = hit ? after : next[i];
      }
    }
  }
  return least;
}

// least reroute penalty of affected stage `st` whose forward and backward times are f and b.  Peers of equal speed
// share the orphans evenly: the fullest takes ceil(orphans / peers), which a cap that admits any vector admits too.
// (More than 10 stages have the instance for 15 peers alone: a second one costs their kernels, which are the longest and short
// of registers, 1 % where nothing needs it.)
template <int SP>
__device__ __forceinline__ uint32_t stage_penalty(ScnPtr scn, TabPtr tab, int st, int f, int b) {
  const int p = scn->aff_peers[st];
  if (tab->even_share[st] != 0) return tab->even_share[st] * peer_time(f, b, scn->aff_q[st][0]);    // uniform
  const uint32_t orphans = (uint32_t)scn->aff_total[st];
  const uint32_t most = scn->rcap > 0 && (uint32_t)scn->rcap < orphans ? (uint32_t)scn->rcap : orphans;
  uint32_t taken = 0;
  auto time_of = [&](int i) -> uint32_t {
    if (i >= p) return NO_MULTIPLES;                 // uniform
    const uint32_t w = peer_time(f, b, scn->aff_q[st][i]);
    taken += w ? 0u : most;
    return w ? w : NO_MULTIPLES;
  };
  if (SP <= 10 && p <= 4) {                          // uniform
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = time_of(i);
    return least_penalty<4>(w, p, taken, orphans, most);
  }
  uint32_t w[FAST_MAX_P];
#pragma unroll
  for (int i = 0; i < FAST_MAX_P; ++i) w[i] = time_of(i);
  return least_penalty<FAST_MAX_P>(w, p, taken, orphans, most);
}

__device__ __forceinline__ uint64_t umin64(uint64_t a, uint64_t b) { return a < b ? a : b; }

// 1-based position of the n-th set bit of x (1 <= n <= popcount(x)): which half holds it is decided
// by a population count, six times
__device__ __forceinline__ int nth_set_bit(uint64_t x, int n) {
  const uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32);
  int c = __popc(lo);
  bool up = n > c;
  uint32_t w = up ? hi : lo;
  int r = up ? n - c : n;
  int pos = up ? 32 : 0;
#pragma unroll
  for (int sh = 16; sh >= 1; sh >>= 1) {
    const uint32_t part = w & ((1u << sh) - 1u);
    c = __popc(part);
    up = r > c;
    w = up ? (w >> sh) : part;
    r = up ? r - c : r;
    pos += up ? sh : 0;
  }
  return pos + 1;
}

// Rounds of gradient communication under redundant computation (see comm_rounds in chm_kernels.hip):
// the colour set of stage s = the n_s lowest colours not used by stage s-1 (if its node exists) nor,
// for the last stage, by stage 0 (if the last node exists); sets are 64-bit masks, L <= 64.
template <int SP>
__device__ __forceinline__ int ring_rounds(const int (&c)[SP + 1], uint32_t node_exists) {
  uint64_t prev = 0, first = 0;
  int rounds = 0;
#pragma unroll
  for (int s = 0; s < SP; ++s) {
    const int n = c[s + 1] - c[s];
    uint64_t f = 0;
    if (s >= 1) f |= ((node_exists >> (s - 1)) & 1u) ? prev : 0ull;
    if (s >= 1 && s == SP - 1) f |= ((node_exists >> s) & 1u) ? first : 0ull;
    const int p = nth_set_bit(~f, n);
    const uint64_t low = p >= 64 ? ~0ull : ((1ull << p) - 1ull);
    const uint64_t cur = ~f & low;
    rounds = imax32(rounds, p);
    if (s == 0) first = cur;
    prev = cur;
  }
  return rounds;
}

template <int CTRL>
__device__ __forceinline__ uint64_t dpp_min(uint64_t v) {
  const int lo = __builtin_amdgcn_update_dpp((int)(uint32_t)v, (int)(uint32_t)v, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(uint32_t)(v >> 32), (int)(uint32_t)(v >> 32), CTRL, 0xF, 0xF, false);
  return umin64(v, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

__device__ __forceinline__ uint64_t wave_min(uint64_t v) {
  v = dpp_min<0xB1>(v);     // quad_perm [1,0,3,2]
  v = dpp_min<0x4E>(v);     // quad_perm [2,3,0,1]
  v = dpp_min<0x141>(v);    // row_half_mirror
  v = dpp_min<0x140>(v);    // row_mirror
  v = umin64(v, __shfl_xor(v, 16, 64));
  v = umin64(v, __shfl_xor(v, 32, 64));
  return v;
}

// a value all lanes agree on, as a scalar
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
}

// Combinadic digits of `rem` (a partition rank): for i = K..1 the largest x with C(x, i) <= rem.
// C(., i) grows with x, so each digit is found by a four-way search over [i-1, previous digit - 1]:
// three independent table probes per step, the range shrinks to a quarter; all lanes take the same number of steps (no
// divergence): unrank_steps of the L - K candidates a digit has at most (the digits above and below it narrow its range).
__device__ __forceinline__ int unrank_steps(int candidates) { return candidates <= 4 ? 1 : candidates <= 16 ? 2 : candidates <= 64 ? 3 : 4; }

template <int K, typename Rank>
__device__ __forceinline__ void unrank_digits(Rank rem, int L, int steps, const Rank *table, int (&c)[K + 2]) {
  // table[(i-1) * DEV_MAX_L + x] = C(x, i)
  auto column = [table](int i, int x) { return table[(i - 1) * DEV_MAX_L + x]; };
  int hi = L - 2;
#pragma unroll
  for (int i = K; i >= 1; --i) {
    int lo = i - 1;                                  // C(i-1, i) = 0 <= rem always
    for (int s = 0; s < steps; ++s) {
      const int q = (hi - lo + 4) >> 2;              // ceil((range size) / 4), 0 only when hi < lo
      const int m1 = lo + q, m2 = m1 + q, m3 = m2 + q;
      // (all three in flight before any is looked at: written with &&, each became a branch of its own behind the one before)
      const Rank t1 = column(i, imin32(m1, hi)), t2 = column(i, imin32(m2, hi)), t3 = column(i, imin32(m3, hi));
      const bool a1 = (m1 <= hi) & (t1 <= rem), a2 = (m2 <= hi) & (t2 <= rem), a3 = (m3 <= hi) & (t3 <= rem);
      // the answer lies in [lo, m1-1], [m1, m2-1], [m2, m3-1] or [m3, hi]
      const int nlo = a3 ? m3 : (a2 ? m2 : (a1 ? m1 : lo));
      const int nhi = a3 ? hi : (a2 ? m3 - 1 : (a1 ? m2 - 1 : m1 - 1));
      lo = nlo;
      hi = nhi < hi ? nhi : hi;
    }
    c[i] = lo + 1;
    rem -= column(i, lo);
    hi = lo - 1;
  }
}

// largest peak memory over the nodes of a plan: static + (pipeline length - position) * activations of the
// most demanding node of every stage (strategy 0: a node holds its stage and its ring successor's)
// (at[] = memory prefix at the cuts)
template <int SP, int STRAT>
__device__ __forceinline__ int peak_from(FamPtr ff, const int (&c)[SP + 1], const int (&at)[SP + 1], const int *pa) {
  int mmax = 0;
  // strategy 0: [c[j], c[j+2]) is two stages; the last node's second one is stage 0
  if (ff->has_act) {
    int ac[SP + 1];
    ac[0] = 0;
#pragma unroll
    for (int j = 1; j <= SP; ++j) ac[j] = pa[c[j]];
#pragma unroll
    for (int j = 0; j < SP; ++j) {
      const int coef = ff->mem_coef[j];
      const int e = STRAT == 0 ? (j + 2 <= SP ? j + 2 : SP) : j + 1;
      const int w = at[e] - at[j] + (STRAT == 0 && j == SP - 1 ? at[1] : 0), a = ac[e] - ac[j] + (STRAT == 0 && j == SP - 1 ? ac[1] : 0);
      const int m = w + (int)__umul24((uint32_t)a, (uint32_t)(coef < 0 ? 0 : coef));
      mmax = imax32(mmax, coef < 0 ? 0 : m);
    }
  } else {
#pragma unroll
    for (int j = 0; j < SP; ++j) {
      const int e = STRAT == 0 ? (j + 2 <= SP ? j + 2 : SP) : j + 1;
      const int m = at[e] - at[j] + (STRAT == 0 && j == SP - 1 ? at[1] : 0);
      mmax = imax32(mmax, ff->mem_coef[j] < 0 ? 0 : m);
    }
  }
  return mmax;
}

template <int SP, int STRAT>
__device__ __forceinline__ int largest_peak(FamPtr ff, const int (&c)[SP + 1], const int *pw, const int *pa) {
  int at[SP + 1];
  at[0] = 0;
#pragma unroll
  for (int j = 1; j <= SP; ++j) at[j] = pw[c[j]];
  return peak_from<SP, STRAT>(ff, c, at, pa);
}

// Weights a plan's nodes must fetch (MiB), from the memory prefix at its cuts: stage sizes minus what their nodes already
// hold (prefix sums are monotone, so the prefix at the larger of two positions is the larger of the two prefixes).
// Strategy 1: the largest total over the pipelines that lost nodes, per survivor in stage order or by the
// least-transfer assignment.
// (The assignment's outer loop is unrolled for few stages only: 1,024 cells in a row keep the compiler busy for hours.)
template <int SP, int STRAT>
__device__ __forceinline__ int missing_weights(FamPtr ff, const int (&wp)[SP + 1]) {
  if (STRAT != 1) {
    uint32_t have = 0;
#pragma unroll
    for (int j = 0; j < SP; ++j) have += sub_floor(imin32(wp[j + 1], ff->w0[j + 1]), imax32(wp[j], ff->w0[j]));
    return ff->w_total - (int)have;
  }
  int missing = 0;
  for (int ci = 0; ci < ff->n_cls; ++ci) {
    const ClsPtr cl = &ff->cls[ci];
    int have = 0;
    if (ff->assign) {
      // least-transfer assignment = largest total overlap of a non-crossing matching of survivors
      // and new stages (both are in layer order, see best_overlap in chm_kernels.hip); one row of
      // the two-index recurrence lives in registers.  A negative raw overlap needs no clamp:
      // diag + (negative) < diag <= G[j], which is already among the operands of the max.
      constexpr int OUTER = SP > 8 ? 1 : SP;
      int G[SP + 1];
#pragma unroll
      for (int j = 0; j <= SP; ++j) G[j] = 0;
#pragma unroll OUTER
      for (int i = 0; i < SP; ++i) {
        const int wlo_i = cl->wlo[i], whi_i = cl->whi[i];
        int diag = 0;
#pragma unroll
        for (int j = 0; j < SP; ++j) {
          const int above = G[j + 1];
          const int cand = diag + (imin32(wp[j + 1], whi_i) - imax32(wp[j], wlo_i));
          G[j + 1] = imax32(imax32(above, G[j]), cand);
          diag = above;
        }
      }
      have = G[SP];
    } else {
#pragma unroll
      for (int j = 0; j < SP; ++j)
        have += (int)sub_floor(imin32(wp[j + 1], cl->whi[j]), imax32(wp[j], cl->wlo[j]));
    }
    missing = imax32(missing, ff->w_total - have);
  }
  return missing;
}

// Lower bound of a plan's cost from its cuts c[0..SP] and the forward + backward time cs[] of its stages.
template <int SP, int STRAT>
__device__ __forceinline__ uint64_t cost_lower_bound(ScnPtr scn, TabPtr tab, FamPtr ff, const int (&cs)[SP], const int (&c)[SP + 1]) {
    // Lower bound of the plan's cost.  Every stage of a pipeline runs its M forwards and M backwards one
    // after the other, so the pipeline takes at least M x the largest (forward + backward) of its chain;
    // rounds of gradient communication: at least the layers of the largest stage; a stage that lost
    // nodes leaves some peer with at least ceil(orphans / peers) extra micro-batches; the weight transfer
    // is at least zero.  Above the incumbent the partition can neither win nor tie.
    // (Sharper where the times allow 24-bit multiplies: stage s cannot start before the forwards of the
    // stages ahead of it and is followed by their backwards: M x its own time + the times of stages 0..s-1.)
    int lb = ff->fixed_step;
    if (STRAT == 0) {
      int cd[SP];
#pragma unroll
      for (int j = 0; j < SP; ++j) cd[j] = cs[j] + cs[(j + 1) % SP];
      for (int ci = 0; ci < ff->n_cls; ++ci) {
        const ClsPtr cl = &ff->cls[ci];
        int v = 0;
        if (ff->lb_prefix) {
          int pre = 0;
#pragma unroll
          for (int j = 0; j < SP; ++j) {
            const int cj = ((cl->dead >> j) & 1u) ? 0 : cd[j];
            v = imax32(v, (int)__umul24((uint32_t)cl->M, (uint32_t)cj) + pre);
            pre += cj;
          }
        } else {
#pragma unroll
          for (int j = 0; j < SP; ++j) v = imax32(v, ((cl->dead >> j) & 1u) ? 0 : cd[j]);
          v *= cl->M;
        }
        lb = imax32(lb, imax32(0, scale_floor(v, cl->q_min) - cl->lb_slack) + cl->comm_total);
      }
    } else {
      for (int ci = 0; ci < ff->n_cls; ++ci) {
        const ClsPtr cl = &ff->cls[ci];
        int v = 0;
        if (ff->lb_prefix) {
          int pre = 0;
#pragma unroll
          for (int j = 0; j < SP; ++j) {
            v = imax32(v, (int)__umul24((uint32_t)cl->M, (uint32_t)cs[j]) + pre);
            pre += cs[j];
          }
        } else {
#pragma unroll
          for (int j = 0; j < SP; ++j) v = imax32(v, cs[j]);
          v *= cl->M;
        }
        lb = imax32(lb, imax32(0, scale_floor(v, cl->q_min) - cl->lb_slack) + cl->comm_total);
      }
    }
    if (ff->allreduce > 0) {
      int layers = STRAT == 0 ? 0 : ff->fixed_layers;
#pragma unroll
      for (int j = 0; j < SP; ++j) layers = imax32(layers, c[j + 1] - c[j]);
      lb += ff->allreduce * layers;
    }
    if (STRAT == 2) {
      for (int st = 0; st < scn->n_aff; ++st) {
        const int sa = scn->aff_stage[st];
        int c_st = cs[0];
#pragma unroll
        for (int j = 1; j < SP; ++j) c_st = sa == j ? cs[j] : c_st;
        lb += (int)tab->lb_mult[st] * scale_floor(c_st, tab->lb_q[st]);
      }
    }
    return (uint64_t)scn->K * (uint32_t)lb + (uint64_t)scn->reconf[STRAT];
}

// forward and forward + backward time of stage `sa` (uniform)
template <int SP>
__device__ __forceinline__ int2 stage_times(const int2 *tc, const int (&c)[SP + 1], int sa) {
  int lo = c[0], hi = c[1];
#pragma unroll
  for (int j = 1; j < SP; ++j) {
    lo = sa == j ? c[j] : lo;
    hi = sa == j ? c[j + 1] : hi;
  }
  const int2 a = tc[lo], b = tc[hi];
  return make_int2(b.x - a.x, b.y - a.y);
}

// Entries of a wave's queue of partitions that fit (QUEUED kernels): a ring of twice the wave width,
// since a round appends at most 64 entries to fewer than 64 waiting ones.
constexpr int QCAP = 128;

// More stages than this: class_time (20 stages: 112 vector registers instead of 180, four waves per SIMD instead of two, a search
// 89 instead of 107 us); fewer: pipeline_time, whose instructions are fewer (lists of 16 stages 658 us, 734 with class_time;
// searches of 11 stages 125 and 131, of 6 174 and 185).
constexpr int FLOW_FROM = 16;

// Waves per SIMD the register allocator is asked to keep possible: 5 up to 5 stages (at most 96 vector registers), 4 up to
// 10 (128), 3 up to 16 (168), 4 up to 24 and 3 beyond, without spills (class_time).  Strategy 2, whose loops over the peers
// need the most: 5 up to 8 stages, which fit 96 without spills when asked to (97 unasked: a range of 3 M partitions of 8
// stages 69 instead of 73 us, 2.6 M of uneven speeds 201 instead of 224).
//
// QUEUED (range search of strategies 0 and 1 without cost store): lanes whose partition fails the memory
// filter would idle through the recurrence of their wave, and consecutive ranks share their upper cuts, so
// whole runs of a lane fail together.  Each wave therefore first only filters: every lane takes the next
// partition of its run, and those that fit are appended (cut positions packed into bytes, position) to a
// ring in LDS that belongs to the wave.  Whenever 64 entries wait, the wave evaluates them, one per lane,
// with every lane busy; what is left after the last round is evaluated by a partly filled wave.  A ring is
// written and read by one wave only, whose LDS operations complete in order: no barrier is needed.
// MODE 0: every lane evaluates its own partitions; 1: QUEUED; 2: QUEUED with the bounds of a bounded search (a
// variant of its own: the bounds cost the plain queued kernel registers it does not have, 36 instead of 16
// spilled bytes per lane at 8 stages and 4 % of its time); 3: QUEUED, fed from a list; 4: the partitions of a window of plan indices, for
// the workgroup that calls it (k_window_plans), without an argmin.
// Lists of more stages than this have their next entry on its way while one is worked on: a tile waits for memory otherwise,
// which three or four wavefronts per SIMD do not hide (2^22 rows of 16 stages, strategy 2: 105 us without, 102 with it; strategy 0
// 87 and 85).  With fewer stages more of them are resident, and the load, which waits for the cost stores ahead of it, costs more than
// it saves (with a cost store: 7 stages, strategy 1, 65 us without, 69 with it; 5 stages, strategy 0, 67 and 69).
constexpr int LIST_AHEAD_FROM = 10;
// Lists of redundant computation, which has a class of pipelines for every node that is short, and deep ones of strategy 1, whose
// weights to fetch are many: the rows come in no order, so that after a few rounds next to none of 64 can win.  The class with the most
// work decides first, and the others and the weights to fetch are worked out only where it leaves a cost not above the wavefront's
// lowest (strategy 0, 2^22 rows: 8 stages 72 us without, 67 with it, 12 stages 79 and 73, 16 stages 90 and 84; strategy 1, 15 stages,
// 2^24 rows 199 and 191, but 2^20 rows 43.7 and 44.4 of 13).  From this many rounds of a workgroup on: with fewer there is nothing to
// compare with yet.  Nowhere else: neighbouring ranks have neighbouring costs, so that some of 64 may nearly always win, and what is left
// out with one class of pipelines costs less than the comparison (10 M ranks of 7 stages, strategy 1, 104 us with it, 90 without; of 8
// stages, strategy 2, 134 and 120; lists of 2^22 rows of 4 stages 54 and 51, of 14 stages, strategy 2, 96 and 92).
constexpr uint32_t NARROW_ROUNDS = 8;

template <int SP, int MODE>
struct SearchShared {
  static constexpr bool QUEUED = MODE >= 1 && MODE <= 3;
  uint4 q_cuts[QUEUED ? (BLOCK / 64) * QCAP : 1];
  uint64_t BN[(SP > 1 ? SP - 1 : 1) * DEV_MAX_L];       // BN[(i-1)*128 + x] = C(x, i), i = 1..K
  // prefix sums: forward and forward + backward; static memory; activation memory
  int2 TC[DEV_MAX_L + 1];
  uint64_t wave_keys[BLOCK / 64];
  uint32_t q_pos[QUEUED ? (BLOCK / 64) * QCAP : 1];
  int PW[DEV_MAX_L + 1], PA[DEV_MAX_L + 1];
  uint32_t wave_fit[BLOCK / 64], wave_eval[BLOCK / 64];
};

// One workgroup (`block` of the family's) of a search.  cost_tile: BLOCK * per_lane costs when a cost store with per_lane > 1 is
// asked for.
// FLOW: times by class_time.
template <int SP, int STRAT, int MODE, bool FLOW = (SP > FLOW_FROM)>
__device__ __forceinline__ void search_partitions(const FastLaunch &a, uint32_t block, SearchShared<SP, MODE> &sh, int64_t *cost_tile) {
  constexpr bool QUEUED = MODE >= 1 && MODE <= 3, LIST = MODE == 3, WINDOW = MODE == 4;
  constexpr int K = SP - 1;
  constexpr bool AHEAD = LIST && SP > LIST_AHEAD_FROM, NARROWS = LIST && (STRAT == 0 || (STRAT == 1 && SP > LIST_AHEAD_FROM));
  constexpr bool FETCH_LATE = NARROWS || AHEAD || FLOW;   // weights to fetch after the times, which need the registers first
  // cost store of plan indices: costs without penalties and the peers' stage times, for the kernel that expands them
  const bool expands = WINDOW || (!QUEUED && STRAT == 2 && a.base_out != nullptr);
  uint4 *const q_cuts = sh.q_cuts;
  uint32_t *const q_pos = sh.q_pos;
  int2 *const TC = sh.TC;
  int *const PW = sh.PW, *const PA = sh.PA;
  uint64_t *const BN = sh.BN, *const wave_keys = sh.wave_keys;
  uint32_t *const wave_fit = sh.wave_fit, *const wave_eval = sh.wave_eval;
  const ScnPtr scn = as_const(a.s.scn);
  const TabPtr tab = as_const(a.tab);
  const FamPtr ff = &tab->fam[STRAT];
  const int L = scn->L;
  const bool compact = !QUEUED && !WINDOW && a.cut_list != nullptr;
  const uint32_t n_slots = compact ? a.cut_count[block] : 0u;       // filled slots of this workgroup's region
  if (compact && n_slots == 0) return;
  for (int i = threadIdx.x; i <= L; i += BLOCK) {
    TC[i] = make_int2((int)scn->pf[i], (int)(scn->pf[i] + scn->pb[i]));
    PW[i] = (int)scn->pw[i];
    PA[i] = (int)scn->pa[i];
  }
  if (!compact && !(LIST && a.s.cuts != nullptr))               // positions given as cuts need no unranking
    for (int i = threadIdx.x; i < K * DEV_MAX_L; i += BLOCK) BN[i] = scn->binom[1 + i / DEV_MAX_L][i % DEV_MAX_L];
  __syncthreads();

  const uint32_t lane_id = block * BLOCK + threadIdx.x;
  const uint32_t run_first = lane_id * a.per_lane;                       // chunk-local (a chunk holds at most 2^30 partitions)
  const uint32_t run_len = (LIST || compact || run_first >= a.s.part_count) ? 0u
                           : (uint32_t)(a.s.part_count - run_first < a.per_lane ? a.s.part_count - run_first : a.per_lane);
  const uint32_t region = block * a.per_lane * BLOCK;               // compact mode: first slot of this workgroup

  // cut positions c[1..K]; c[0] = 0 and c[SP] = L are constants
  int c[SP + 1];
  c[0] = 0;
  c[SP] = L;
  // (a wavefront without partitions has nothing to unrank: most of a window's tile)
  const bool idle = WINDOW && __builtin_amdgcn_ballot_w64(run_len != 0) == 0;
  if (!compact && !LIST && !idle) {
    uint64_t rem = run_len ? a.s.part_first + run_first + (run_first >= a.s.jump_at ? a.s.jump_by : 0) : 0;   // idle lanes walk from rank 0: always valid cuts
    // combinadic digits from the LDS copy of the binomial table
    unrank_digits<K, uint64_t>(rem, L, unrank_steps(L - K), BN, c);
  }

  const int cap = (int)scn->cap;
  uint64_t best_cost = ~0ull;
  uint64_t wave_low = ~0ull;    // lowest cost the wave has met (uniform)
  uint32_t best_pos = 0;        // output position (chunk-local partition index or list position) of the lane's best
  uint32_t n_fit = 0;           // wave-uniform count of partitions that pass the memory filter

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t q_head = 0, q_tail = 0;        // wave-uniform: entries [q_head, q_tail) of the wave's ring wait
  // bounded search: the lowest cost evaluated so far, by this wave or (as of its last look) by any other
  const bool bounded = MODE >= 2 && a.s.incumbent != nullptr;
  uint64_t incumbent = ~0ull;
  uint32_t n_eval = 0;                    // wave-uniform count of partitions whose recurrences were run
  if (bounded) incumbent = umin64(a.s.incumbent0, __hip_atomic_load(a.s.incumbent, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  // Bounded search, a whole run at once.  Consecutive ranks differ in their lowest cuts.  When the run of a lane
  // stays inside the block of ranks that share the cuts above the h lowest ones (its offset among the
  // arrangements of those h cuts, plus its length, does not exceed their number C(c[h+1]-1, h)), the stages
  // from h+1 on are the same for every partition of the run, and so is their part of the lower bound: stage s
  // contributes M x its time + the time of all layers ahead of it, whatever the lower cuts are.  If that
  // alone lies above the incumbent for every lane, the wave has nothing to look at.
  bool wave_dead = false;
  if (MODE == 2 && bounded && K >= 2) {
    uint64_t offset = 0;
    int first_fixed = SP;                   // stages first_fixed.. are the same throughout the run
#pragma unroll
    for (int h = 1; h < K; ++h) {
      offset += BN[(h - 1) * DEV_MAX_L + (c[h] - 1)];
      const bool stays = offset + run_len <= BN[(h - 1) * DEV_MAX_L + (c[h + 1] - 1)];
      first_fixed = (first_fixed == SP && stays) ? h + 1 : first_fixed;
    }
    int pc[SP + 1];                         // forward + backward time of the layers ahead of stage s
#pragma unroll
    for (int s2 = 1; s2 <= SP; ++s2) pc[s2] = TC[c[s2]].y;
    int lb = ff->fixed_step;
    for (int ci = 0; ci < ff->n_cls; ++ci) {
      const ClsPtr cl = &ff->cls[ci];
      int v = 0;
#pragma unroll
      for (int s2 = 1; s2 < SP; ++s2) {
        int vs;
        if (STRAT == 0) {
          // a node's own stage and its successor's; the pair that wraps around to stage 0 is left out
          const int pair = s2 + 2 <= SP ? pc[s2 + 2 <= SP ? s2 + 2 : SP] - pc[s2] : 0;
          vs = ((cl->dead >> s2) & 1u) ? 0 : cl->M * pair;
        } else {
          const int own = pc[s2 + 1] - pc[s2];
          vs = ff->lb_prefix ? (int)__umul24((uint32_t)cl->M, (uint32_t)own) + pc[s2] : cl->M * own;
        }
        v = imax32(v, s2 >= first_fixed ? vs : 0);
      }
      lb = imax32(lb, imax32(0, scale_floor(v, cl->q_min) - cl->lb_slack) + cl->comm_total);
    }
    const uint64_t lb_cost = (uint64_t)scn->K * (uint32_t)lb + (uint64_t)scn->reconf[STRAT];
    const bool look = run_len != 0 && !(first_fixed < SP && lb_cost > incumbent);
    wave_dead = __builtin_amdgcn_ballot_w64(look) == 0;
  }
  // evaluation cuts: the lane's own cuts, or (QUEUED) those of the entry it takes from the ring
  int ce[SP + 1];
  ce[0] = 0;
  ce[SP] = L;

  auto row_of_list = [&](uint32_t entry, uint32_t (&w)[4]) {
    const uint64_t at = (uint64_t)entry * K;
    if (at + 16 <= (uint64_t)a.s.part_count * K) {
      __builtin_memcpy(w, a.s.cuts + at, 16);                  // (unaligned; bytes behind the row are not looked at)
    } else {
      for (int i = 0; i < K; ++i) {
        const uint32_t b = (uint32_t)a.s.cuts[at + i] << (8 * (i & 3));
        w[0] |= i < 4 ? b : 0; w[1] |= (i >> 2) == 1 ? b : 0; w[2] |= (i >> 2) == 2 ? b : 0; w[3] |= (i >> 2) == 3 ? b : 0;
      }
    }
  };
  uint32_t ahead[4] = {0, 0, 0, 0};                // AHEAD: the next entry, its cuts or its rank
  auto look_ahead = [&](uint32_t it) {
    const uint32_t entry = (block * a.per_lane + it) * BLOCK + threadIdx.x;
    const bool there = entry < a.s.part_count;
    ahead[0] = ahead[1] = ahead[2] = ahead[3] = 0;
    if (a.s.cuts != nullptr) {
      row_of_list(there ? entry : 0, ahead);
    } else {
      const uint64_t r = there ? a.s.ranks[entry] : 0;
      ahead[0] = (uint32_t)r; ahead[1] = (uint32_t)(r >> 32);
    }
  };
  if (AHEAD) look_ahead(0);

  for (uint32_t it = 0; it < (wave_dead || idle ? 0u : a.per_lane + (QUEUED ? 1u : 0u)); ++it) {
    bool live = it < run_len;             // this lane has a partition in this round
    uint32_t pos = run_first + it;        // where its result is reported
    if (QUEUED) {
      if (it < a.per_lane) {              // uniform; the extra round only drains the ring
        // ---- filter the lane's next partition and append it to the ring if it fits
        uint32_t words[4] = {0, 0, 0, 0};     // its cut positions, a byte each
        bool valid = true;
        if (LIST) {
          // tile `it` of this workgroup's part of the list: neighbouring lanes read neighbouring entries
          const uint32_t entry = (block * a.per_lane + it) * BLOCK + threadIdx.x;
          live = entry < a.s.part_count;
          pos = a.pos_base + entry;
          const uint64_t ahead_rank = (uint64_t)ahead[0] | ((uint64_t)ahead[1] << 32);
          if (AHEAD) {
            for (int w = 0; w < 4; ++w) words[w] = ahead[w];
            if (it + 1 < a.per_lane) look_ahead(it + 1);
          }
          if (a.s.cuts != nullptr) {
            if (!AHEAD) row_of_list(live ? entry : 0, words);
            // a row that does not increase strictly within 1..L-1 does not fit; 1..K stands in for it
            int prev = 0;
#pragma unroll
            for (int i = 1; i <= K; ++i) {
              const int ci = (int)((words[(i - 1) >> 2] >> (8 * ((i - 1) & 3))) & 0xffu);
              valid = valid && ci > prev;
              prev = ci;
            }
            valid = valid && prev <= L - 1;
            const uint32_t first[4] = {0x04030201u, 0x08070605u, 0x0c0b0a09u, 0x000f0e0du};
#pragma unroll
            for (int w = 0; w < 4; ++w) words[w] = valid ? words[w] : first[w];
#pragma unroll
            for (int i = 1; i <= K; ++i) c[i] = (int)((words[(i - 1) >> 2] >> (8 * ((i - 1) & 3))) & 0xffu);
          } else {
            for (int w = 0; w < 4 && AHEAD; ++w) words[w] = 0;
            uint64_t rem = live ? (AHEAD ? ahead_rank : a.s.ranks[entry]) : 0;
            valid = rem < scn->fam[STRAT].n_part;
            if (!valid) rem = 0;
            unrank_digits<K, uint64_t>(rem, L, unrank_steps(L - K), BN, c);
          }
        }
        bool fits = live && valid && largest_peak<SP, STRAT>(ff, c, PW, PA) <= cap;
        const uint64_t in_memory = __builtin_amdgcn_ballot_w64(fits);
        if (!LIST) n_fit += (uint32_t)__popcll(in_memory);
        if (bounded && in_memory != 0) {      // uniform; nothing to bound where nothing fits
          int cs[SP];                           // forward + backward time per stage
          int before = 0;
#pragma unroll
          for (int j = 0; j < SP; ++j) {
            const int behind = TC[c[j + 1]].y;
            cs[j] = behind - before;
            before = behind;
          }
          const uint64_t lb_cost = cost_lower_bound<SP, STRAT>(scn, tab, ff, cs, c);
          fits = fits && lb_cost <= incumbent;
        }
        const uint64_t fit_mask = __builtin_amdgcn_ballot_w64(fits);
        if (LIST) {
          n_fit += (uint32_t)__popcll(fit_mask);      // (of a bounded search: those that pass the bound too)
          if (a.s.costs_out != nullptr && live && !fits) a.s.costs_out[pos] = CHM_INF_COST;
        }
        if (fits) {
          const uint32_t slot = (uint32_t)wave * QCAP + ((q_tail + (uint32_t)__popcll(fit_mask & ((1ull << lane) - 1ull))) & (QCAP - 1));
          if (!LIST || a.s.cuts == nullptr) {
#pragma unroll
            for (int i = 1; i <= K; ++i) words[(i - 1) >> 2] |= (uint32_t)c[i] << (8 * ((i - 1) & 3));
          }
          q_cuts[slot] = make_uint4(words[0], words[1], words[2], words[3]);
          q_pos[slot] = (uint32_t)pos;
        }
        q_tail += (uint32_t)__popcll(fit_mask);
        // next partition of the run
        bool done = LIST;
#pragma unroll
        for (int i = 1; i <= K && !LIST; ++i) {
          const bool can = c[i] + 1 < c[i + 1];
          c[i] = done ? c[i] : (can ? c[i] + 1 : i);
          done = done || can;
        }
      }
      const uint32_t waiting = q_tail - q_head;
      if (waiting < 64 && !(it == a.per_lane && waiting > 0)) continue;     // uniform
      // ---- evaluate up to 64 waiting entries, one per lane
      const uint32_t take = waiting < 64 ? waiting : 64u;
      live = (uint32_t)lane < take;
      const uint32_t slot = (uint32_t)wave * QCAP + ((q_head + (uint32_t)lane) & (QCAP - 1));
      // lanes past the end take the first partition (cuts 1..K): always valid
      const uint4 packed = live ? q_cuts[slot] : make_uint4(0x04030201u, 0x08070605u, 0x0c0b0a09u, 0x000f0e0du);
      const uint32_t words[4] = {packed.x, packed.y, packed.z, packed.w};
#pragma unroll
      for (int i = 1; i <= K; ++i) ce[i] = (int)((words[(i - 1) >> 2] >> (8 * ((i - 1) & 3))) & 0xffu);
      pos = live ? q_pos[slot] : 0;
      q_head += take;
    }
    if (compact) {
      if (it * BLOCK >= n_slots) break;   // uniform: the region is used up
      const uint32_t slot = it * BLOCK + threadIdx.x;
      live = slot < n_slots;
      // lanes past the end take the first partition (cuts 1..K): always valid
      const uint4 packed = live ? a.cut_list[region + slot] : make_uint4(0x04030201u, 0x08070605u, 0x0c0b0a09u, 0x000f0e0du);
      const uint32_t words[4] = {packed.x, packed.y, packed.z, packed.w};
#pragma unroll
      for (int i = 1; i <= K; ++i) c[i] = (int)((words[(i - 1) >> 2] >> (8 * ((i - 1) & 3))) & 0xffu);
      pos = live ? a.cut_pos[region + slot] : 0;
    }
    if (!QUEUED) {
#pragma unroll
      for (int i = 1; i <= K; ++i) ce[i] = c[i];
    }
    // ---- memory filter
    // (QUEUED: every entry of the ring has passed it already)
    const bool ok = QUEUED ? live : (largest_peak<SP, STRAT>(ff, ce, PW, PA) <= cap && live);
    uint64_t cost = (uint64_t)CHM_INF_COST;
    const uint64_t ok_mask = __builtin_amdgcn_ballot_w64(ok);
    if (!QUEUED) n_fit += (uint32_t)__popcll(ok_mask);
    if (ok_mask != 0) {
      int t_step = ff->fixed_step;
      auto weights_to_fetch = [&]() -> int {
        int wp[SP + 1];                     // memory prefix at the cuts
        wp[0] = 0;
#pragma unroll
        for (int j = 1; j <= SP; ++j) wp[j] = PW[ce[j]];
        return missing_weights<SP, STRAT>(ff, wp);
      };
      int missing = 0;
      if (!FETCH_LATE) missing = weights_to_fetch();
      // (NARROWS) whether some partition of the wavefront may still win: what is not worked out yet only adds to its cost
      const bool every = a.s.costs_out != nullptr || a.per_lane < NARROW_ROUNDS;
      auto may_win = [&]() -> bool {
        const uint64_t least = (uint64_t)scn->K * (uint32_t)t_step + (uint64_t)scn->reconf[STRAT];
        return every || __builtin_amdgcn_ballot_w64(ok && least <= wave_low) != 0;
      };
      bool open = true;
      // Times per pipeline class.  The stage sums are read from the LDS table again for every class: at 16 stages keeping them
      // for the next class costs a wave per SIMD (two pipelines of 16 stages alike or not, 168 registers and spills).
      for (int ci = 0; ci < ff->n_time && (!NARROWS || open); ++ci) {
        const ClsPtr cl = &ff->cls[ci];
        // (the compiler is not to know that these reads are the same for every class)
#pragma unroll
        for (int j = 1; j <= K; ++j) asm volatile("" : "+v"(ce[j]));
        int time;
        if constexpr (FLOW) {
          auto at = [&](int i) -> int2 { return i == 0 ? make_int2(0, 0) : TC[ce[i]]; };
          time = ff->time24 ? class_time<SP, STRAT, true, false>(cl, at) : class_time<SP, STRAT, false, false>(cl, at);
        } else {
          int F[SP], C[SP];
          int2 t[SP + 1];
          t[0] = make_int2(0, 0);
#pragma unroll
          for (int j = 1; j <= SP; ++j) t[j] = TC[ce[j]];
          const uint32_t dead = STRAT == 0 ? cl->dead : 0u;
#pragma unroll
          for (int j = 0; j < SP; ++j) {
            const int e = STRAT == 0 ? (j + 2 <= SP ? j + 2 : SP) : j + 1;      // (strategy 0: a node runs two stages)
            F[j] = t[e].x - t[j].x;
            C[j] = t[e].y - t[j].y;
            if (STRAT == 0) {
              if (j == SP - 1) { F[j] += t[1].x; C[j] += t[1].y; }
              const int keep = ((dead >> j) & 1u) ? 0 : -1;            // uniform
              F[j] &= keep;
              C[j] &= keep;
            }
          }
          if (!cl->unit) {
#pragma unroll
            for (int j = 0; j < SP; ++j) {
              const uint32_t q = cl->q_stage[j];
              const int b = scale32(C[j] - F[j], q);
              F[j] = scale32(F[j], q);
              C[j] = F[j] + b;
            }
          }
          time = pipeline_time<SP, STRAT == 0>(F, C, cl, ff->time24);
        }
        t_step = imax32(t_step, time);
        if (NARROWS) open = may_win();
      }
      if (!NARROWS || open) {
        if (ff->allreduce > 0) {
          // rounds of gradient communication: largest stage on any device, or the ring colouring when nodes hold two stages
          int rounds;
          if (STRAT == 0) {
            rounds = ring_rounds<SP>(ce, ff->node_exists);
          } else {
            rounds = ff->fixed_layers;
#pragma unroll
            for (int j = 0; j < SP; ++j) rounds = imax32(rounds, ce[j + 1] - ce[j]);
          }
          t_step += ff->allreduce * rounds;
        }
        if (STRAT == 2 && !expands) {
          // least penalty over the reroute vectors of every stage that lost nodes
          for (int st = 0; st < scn->n_aff; ++st) {
            const int2 t = stage_times<SP>(TC, ce, scn->aff_stage[st]);
            t_step += (int)stage_penalty<SP>(scn, tab, st, t.x, t.y - t.x);
          }
        }
        if (expands) {
          if (ok) {
            uint4 *wout = (uint4 *)(a.weights_out + (size_t)(run_first + it) * (scn->n_aff * ROWS_MAX_P));
            for (int st = 0; st < scn->n_aff; ++st) {
              const int2 t = stage_times<SP>(TC, ce, scn->aff_stage[st]);
              const int p = scn->aff_peers[st];
              uint32_t w[ROWS_MAX_P];
#pragma unroll
              for (int i = 0; i < ROWS_MAX_P; ++i) w[i] = i < p ? peer_time(t.x, t.y - t.x, scn->aff_q[st][i]) : 0u;
              wout[2 * st] = make_uint4(w[0], w[1], w[2], w[3]);
              wout[2 * st + 1] = make_uint4(w[4], w[5], w[6], w[7]);
            }
          }
        }
        if (FETCH_LATE) missing = weights_to_fetch();
        cost = (uint64_t)scn->K * (uint32_t)t_step + (uint64_t)scn->reconf[STRAT] + (uint64_t)scn->xfer * (uint32_t)missing;
        // a lane meets the entries of a compacted list or of a ring in no particular order of position:
        // there the lower position wins among equal costs; a run is walked in ascending order
        const bool lower = (QUEUED || compact) ? (cost < best_cost || (cost == best_cost && pos < best_pos)) : cost < best_cost;
        if (ok && lower) { best_cost = cost; best_pos = pos; }
        if (NARROWS && !every && __builtin_amdgcn_ballot_w64(ok && cost < wave_low) != 0) wave_low = uniform64(wave_min(ok ? cost : ~0ull));
      }
      if (bounded) {
        // the round's lowest cost becomes known to every wave; what the others found is picked up in turn
        n_eval += (uint32_t)__popcll(ok_mask);
        const uint64_t round_best = wave_min(ok ? cost : ~0ull);
        if (round_best < incumbent) {
          incumbent = round_best;
          if (lane == 0) atomicMin((unsigned long long *)a.s.incumbent, (unsigned long long)round_best);
        }
        incumbent = umin64(incumbent, __hip_atomic_load(a.s.incumbent, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        if (NARROWS) wave_low = umin64(wave_low, uniform64(incumbent));
      }
      if (expands && ok) a.base_out[run_first + it] = cost;
    }
    if (expands && !ok && it < run_len) a.base_out[run_first + it] = ~0ull;
    if (LIST && a.s.costs_out != nullptr && live) a.s.costs_out[pos] = (int64_t)cost;
    if (!QUEUED && !WINDOW && a.s.costs_out != nullptr) {
      // per_lane == 1: the store is coalesced as it is; longer runs go through an LDS tile
      // (laid out in output order) and are written out together after the loop
      const int64_t v = ok ? (int64_t)cost : CHM_INF_COST;
      if (a.per_lane == 1 || compact) { if (live) a.s.costs_out[pos] = v; }
      else cost_tile[threadIdx.x * a.per_lane + it] = v;
    }
    // ---- next partition in rank order: bump the lowest cut that has room, reset those below
    if (!compact && !QUEUED) {
      bool done = false;
#pragma unroll
      for (int i = 1; i <= K; ++i) {
        const bool can = c[i] + 1 < c[i + 1];
        c[i] = done ? c[i] : (can ? c[i] + 1 : i);
        done = done || can;
      }
    }
  }

  if (!QUEUED && !WINDOW && a.s.costs_out != nullptr && a.per_lane > 1 && !compact) {
    __syncthreads();
    const uint64_t block_first = (uint64_t)block * BLOCK * a.per_lane;
    const uint32_t n_tile = BLOCK * a.per_lane;
    for (uint32_t i = threadIdx.x; i < n_tile; i += BLOCK)
      if (block_first + i < a.s.part_count) a.s.costs_out[block_first + i] = cost_tile[i];
  }
  if (WINDOW) return;
  uint64_t key = best_cost == ~0ull ? CHM_KEY_NONE
                                    : ((best_cost << a.s.idx_bits) | (uint64_t)best_pos);
  if (expands) key = CHM_KEY_NONE;   // the combine kernel takes the argmin
  key = wave_min(key);
  if (lane == 0) { wave_keys[wave] = key; wave_fit[wave] = n_fit; wave_eval[wave] = n_eval; }
  __syncthreads();
  if (threadIdx.x == 0) {
    // one atomic of each kind per workgroup, spread over several words (see SearchLaunch)
    const uint32_t slot = (block & a.s.slot_mask) * a.s.slot_stride;
    uint64_t k = wave_keys[0];
    uint32_t fit = wave_fit[0], evaluated = wave_eval[0];
#pragma unroll
    for (int i = 1; i < BLOCK / 64; ++i) { k = umin64(k, wave_keys[i]); fit += wave_fit[i]; evaluated += wave_eval[i]; }
    if (fit) atomicAdd((unsigned long long *)a.s.feasible + slot, (unsigned long long)fit);
    if (MODE == 2 && bounded && evaluated) atomicAdd((unsigned long long *)a.s.evaluated + slot, (unsigned long long)evaluated);
    // a search over a list of candidates of a bounded search makes its best cost known to what follows
    if (!QUEUED && a.s.incumbent != nullptr && k != CHM_KEY_NONE)
      atomicMin((unsigned long long *)a.s.incumbent, (unsigned long long)(k >> a.s.idx_bits));
    if (k != CHM_KEY_NONE) atomicMin((unsigned long long *)a.s.result + slot, (unsigned long long)k);
  }
}

// Lists ask for four wavefronts per SIMD as deep as that needs no spills (2^22 rows of 15 stages, strategy 1: 80 us with 133 registers and
// three, 75 with 128; of 14 stages, strategy 0: 85 and 77).
constexpr int list_four_waves(int strategy) { return strategy == 0 ? 14 : 15; }
#define CHM_WAVES(SP, STRAT) __attribute__((amdgpu_waves_per_eu((SP) <= (STRAT == 2 ? 8 : 5) ? 5 : (SP) <= 10 ? 4 : (SP) <= 16 ? 3 : (SP) <= 24 ? 4 : 3)))
template <int SP, int STRAT, int MODE = 0>
__global__ void __launch_bounds__(BLOCK) CHM_WAVES((MODE == 3 && SP > 10 && SP <= list_four_waves(STRAT) ? 10 : SP), STRAT) k_fast_search(FastLaunch a) {
  __shared__ SearchShared<SP, MODE> sh;
  extern __shared__ int64_t cost_tile[];
  search_partitions<SP, STRAT, MODE>(a, blockIdx.x, sh, cost_tile);
}

// The families of a call in one launch: strategies 2 and 0 of SP stages, 1 of S1.  Small families take microseconds, as long as
// it takes to launch the next: side by side they take as long as the
// longest (9,455 partitions of 4 stages: kernels of 5, 5.5 and 7 us, a search 39 us one after the other, 31 together).
template <int SP, int S1>
__global__ void __launch_bounds__(BLOCK) CHM_WAVES(SP, 2) k_search_families(FamiliesLaunch a) {
  typedef SearchShared<SP, 0> Shared;                  // (S1 < SP: room for both)
  static_assert(S1 < SP && sizeof(SearchShared<S1, 0>) <= sizeof(Shared), "one shared block for all families");
  __shared__ Shared sh;
  const uint32_t b = blockIdx.x;
  if (b < a.blocks[2]) search_partitions<SP, 2, 0>(a.family[2], b, sh, nullptr);
  else if (b < a.blocks[2] + a.blocks[0]) search_partitions<SP, 0, 0>(a.family[0], b - a.blocks[2], sh, nullptr);
  else search_partitions<S1, 1, 0, (SP > FLOW_FROM)>(a.family[1], b - a.blocks[2] - a.blocks[0], *(SearchShared<S1, 0> *)&sh, nullptr);
}

// Which variant of the search kernel: every lane its own partitions; the partitions that fit (and, in a bounded search, may
// still win) compacted through a ring per wave; the same fed from an explicit list.
template <int STRAT>
int launch_by_stages(int sp, const FastLaunch &a, uint32_t blocks, uint32_t tile_bytes, hipStream_t st, SearchVariant variant) {
  // (the ring of strategy 2 exists with bounds only: without them nothing has shown a use for it)
  const bool bounds = STRAT == 2 || a.s.incumbent != nullptr;
#define CHM_CASE(SPV)                                                                         \
  case SPV:                                                                                   \
    if (variant == SEARCH_LIST)                                                               \
      hipLaunchKernelGGL((k_fast_search<SPV, STRAT, 3>), dim3(blocks), dim3(BLOCK), 0, st, a); \
    else if (variant == SEARCH_QUEUED && bounds)                                              \
      hipLaunchKernelGGL((k_fast_search<SPV, STRAT, 2>), dim3(blocks), dim3(BLOCK), 0, st, a); \
    else if (variant == SEARCH_QUEUED)                                                        \
      hipLaunchKernelGGL((k_fast_search<SPV, STRAT, (STRAT == 2 ? 2 : 1)>), dim3(blocks), dim3(BLOCK), 0, st, a); \
    else                                                                                      \
      hipLaunchKernelGGL((k_fast_search<SPV, STRAT>), dim3(blocks), dim3(BLOCK), tile_bytes, st, a); \
    return 0;
// (a ring or list entry holds up to 16 cuts: deeper pipelines have the plain range kernel only)
#define CHM_DEEP(SPV)                                                                         \
  case SPV:                                                                                   \
    if (variant != SEARCH_PLAIN || a.cut_list != nullptr) return 1;                           \
    hipLaunchKernelGGL((k_fast_search<SPV, STRAT>), dim3(blocks), dim3(BLOCK), tile_bytes, st, a); \
    return 0;
  switch (sp) {
#ifdef CHM_TUNING_SUBSET        // (-DCHM_TUNING_SUBSET: a few stage counts, for quick rebuilds while tuning)
    CHM_CASE(7) CHM_CASE(8) CHM_CASE(15) CHM_CASE(16)
#else
    CHM_CASE(2) CHM_CASE(3) CHM_CASE(4) CHM_CASE(5) CHM_CASE(6) CHM_CASE(7) CHM_CASE(8)
    CHM_CASE(9) CHM_CASE(10) CHM_CASE(11) CHM_CASE(12) CHM_CASE(13) CHM_CASE(14) CHM_CASE(15) CHM_CASE(16)
    CHM_DEEP(17) CHM_DEEP(18) CHM_DEEP(19) CHM_DEEP(20) CHM_DEEP(21) CHM_DEEP(22) CHM_DEEP(23) CHM_DEEP(24)
    CHM_DEEP(25) CHM_DEEP(26) CHM_DEEP(27) CHM_DEEP(28) CHM_DEEP(29) CHM_DEEP(30) CHM_DEEP(31) CHM_DEEP(32)
#endif
    default: return 1;
  }
#undef CHM_DEEP
#undef CHM_CASE
}

}  // namespace

#endif
