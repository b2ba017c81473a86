// The best of a long list of partitions, given as rows of cut positions, whose costs are not stored.
#include "chm_search_kernel.h"

namespace {

// Whether the first K bytes of a row of cuts rise strictly, the first one above 0, all below 128 (four at a time: a byte of 128 +
// cut less (the one before it + 1) keeps its top bit where the cut is larger, and borrows nothing).
template <int K>
__device__ __forceinline__ bool strictly_rising(const uint32_t (&w)[4]) {
  uint32_t wrong = 0;
#pragma unroll
  for (int i = 0; i < (K + 3) / 4; ++i) {
    const uint32_t before = (w[i] << 8) | (i > 0 ? w[i > 0 ? i - 1 : 0] >> 24 : 0u);
    const uint32_t rises = (w[i] | 0x80808080u) - (before + 0x01010101u);
    const uint32_t counted = K - 4 * i >= 4 ? 0x80808080u : 0x80808080u >> (8 * (4 - (K - 4 * i > 0 ? K - 4 * i : 1)));
    wrong |= (w[i] | ~rises) & counted;
  }
  return wrong == 0;
}

// With no more rows of 64 that fit than this, working them out costs less than the bound of all 64.
constexpr int FEW_ROWS = 16;
// Where more than so many eighths of the rows that fit pass the bound (a list of neighbours of one plan, or uneven speeds, which weaken the
// bound), it is not looked at for half as many rounds as there have been.
constexpr int USELESS_SHARE = 5;
constexpr uint32_t FIRST_LOOKS = 4;       // (the first rounds lower the cost: random rows pass them, too)

// cuts c[0..SP] from words of a byte each
template <int SP>
__device__ __forceinline__ void unpack_cuts(const uint32_t (&words)[4], int L, int (&c)[SP + 1]) {
  c[0] = 0;
  c[SP] = L;
#pragma unroll
  for (int i = 1; i < SP; ++i) c[i] = (int)((words[(i - 1) >> 2] >> (8 * ((i - 1) & 3))) & 0xffu);
}

// What a row of a list must pass to be worked out: it fits, and a lower bound of its step time (cost_lower_bound's, of the class of
// pipelines with the most work and the first stage that lost nodes) does not exceed what the lowest cost met leaves.  All that is the same for
// all rows is read once, ahead of them: in the loop over the rows every scalar load is a wait that three wavefronts per SIMD do not hide.
template <int SP, int STRAT>
struct ListBound {
  int M, slack, add, lost, limit, rounds, fixed_layers;
  uint32_t q, dead, mult, lost_q;
  double per_step;
  uint64_t reconf;
  bool plain_memory;
  __device__ __forceinline__ void start(ScnPtr scn, TabPtr tab, FamPtr ff) {
    const ClsPtr cl = &ff->cls[0];
    M = cl->M;
    q = cl->q_min;
    slack = cl->lb_slack;
    dead = STRAT == 0 ? cl->dead : 0u;
    add = cl->comm_total;
    rounds = ff->allreduce;
    fixed_layers = ff->fixed_layers;
    lost = STRAT == 2 && scn->n_aff > 0 ? scn->aff_stage[0] : -1;
    mult = lost >= 0 ? (uint32_t)tab->lb_mult[0] : 0u;
    lost_q = lost >= 0 ? (uint32_t)tab->lb_q[0] : 65536u;
    per_step = 1.0 / (double)scn->K;
    reconf = (uint64_t)scn->reconf[STRAT];
    plain_memory = ff->has_act == 0;
#pragma unroll
    for (int j = 0; j < SP; ++j) plain_memory = plain_memory && ff->mem_coef[j] >= 0;
  }
  // no step time above `limit` can reach the cost (the division is rounded: one more than it says)
  __device__ __forceinline__ void lower_to(uint64_t cost) {
    const double most = cost < reconf ? -1.0 : (double)(cost - reconf) * per_step + 1.0;
    limit = __builtin_amdgcn_readfirstlane(most < 2147483647.0 ? (int)most : 2147483647);
  }
  // words = the cuts a byte each; cw = prefixes {forward + backward, memory}; in_memory: the lanes whose row fits; look: whether the bound is
  // looked at (few rows that fit cost less than the bound)
  __device__ __forceinline__ bool passes(FamPtr ff, const uint32_t (&words)[4], int L, const int2 *cw, const int *pa, int cap, bool valid,
                                         bool look, uint64_t *in_memory) const {
    int t[SP + 1], at[SP + 1];
    t[0] = at[0] = 0;
#pragma unroll
    for (int j = 1; j <= SP; ++j) {
      // (a byte times the size of an entry is one dot product of bytes)
      const uint32_t offset = __builtin_amdgcn_udot4(words[(j - 1) >> 2], (uint32_t)sizeof(int2) << (8 * ((j - 1) & 3)), 0u, false);
      const int2 both = j < SP ? *(const int2 *)((const char *)cw + offset) : cw[L];
      t[j] = both.x;
      at[j] = both.y;
    }
    int peak = 0;
    if (plain_memory) {
#pragma unroll
      for (int j = 0; j < SP; ++j) {
        const int e = STRAT == 0 ? (j + 2 <= SP ? j + 2 : SP) : j + 1;
        peak = imax32(peak, at[e] - at[j] + (STRAT == 0 && j == SP - 1 ? at[1] : 0));
      }
    } else {
      int c[SP + 1];
      unpack_cuts<SP>(words, L, c);
      peak = peak_from<SP, STRAT>(ff, c, at, pa);
    }
    const bool fits = valid && peak <= cap;
    *in_memory = __builtin_amdgcn_ballot_w64(fits);
    if (!look || limit == 2147483647 || __popcll(*in_memory) <= FEW_ROWS) return fits;         // uniform
    int v = 0;
    if (STRAT == 0) {
      int before = 0;
#pragma unroll
      for (int j = 0; j < SP; ++j) {
        int pair = t[j + 2 <= SP ? j + 2 : SP] - t[j] + (j == SP - 1 ? t[1] : 0);
        pair &= ((dead >> j) & 1u) ? 0 : -1;             // uniform
        v = imax32(v, (int)__umul24((uint32_t)M, (uint32_t)pair) + before);
        before += pair;
      }
    } else {
#pragma unroll
      for (int j = 0; j < SP; ++j) v = imax32(v, (int)__umul24((uint32_t)M, (uint32_t)(t[j + 1] - t[j])) + t[j]);
    }
    if (q != 65536u) v = imax32(0, scale_floor(v, q) - slack);
    v += add;
    if (rounds > 0) {
      int c[SP + 1];
      unpack_cuts<SP>(words, L, c);
      int layers = STRAT == 0 ? 0 : fixed_layers;
#pragma unroll
      for (int j = 0; j < SP; ++j) layers = imax32(layers, c[j + 1] - c[j]);
      v += rounds * layers;
    }
    if (STRAT == 2 && lost >= 0) {
      auto cut = [&](int i) -> int {                     // 0 < i < SP, uniform
        const int w = (i - 1) >> 2;
        const uint32_t low = w == 0 ? words[0] : words[1], high = w == 2 ? words[2] : words[3];
        return (int)(((w < 2 ? low : high) >> (8 * ((i - 1) & 3))) & 0xffu);
      };
      const int from = lost == 0 ? 0 : cw[cut(lost)].x, to = lost == SP - 1 ? t[SP] : cw[cut(lost + 1)].x;
      v += (int)mult * scale_floor(to - from, lost_q);
    }
    return fits && v <= limit;
  }
};

// Wavefronts per SIMD, and workgroups (of four) per compute unit: as many as the closed form's arrays leave without spilled vector registers
// (strategy 2 spills about 50 scalars at any depth).
constexpr int list_best_waves(int stages) { return stages <= 8 ? 5 : stages <= 12 ? 4 : 3; }

// One workgroup to a share of the rows; a wavefront filters 64 rows a round and works out those in its ring that may win, 64 at a time.
// Rows of a list come in no order, so that after the first 64 next to none can win: a row takes 160 to 215 instructions (16 stages) instead of
// 190 to 330.  Bound by VALU issue and the prefixes' LDS reads.  2^23 rows, us, one by one / so: 16 stages 119 / 84, 116 / 71 and 159 / 90
// (strategies 0, 1, 2), 8 stages 98 / 64, 87 / 54 and 109 / 72, at uneven speeds 148 / 112, 95 / 60 and 242 / 116.  Lists of which nearly all
// may win (neighbours of one plan, one row over and over) take what they take one by one, within 8 % (the shortest, of six rounds a wavefront,
// within 18 %): the bound is looked at ever more seldom and times come from the closed form as there.  (Stage after stage, class_time, leaves room for a fifth or sixth wavefront per SIMD, but such lists
// took 15 to 37 % longer and random ones no less.)
template <int SP, int STRAT>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(list_best_waves(SP)))) k_list_best(FastLaunch a) {
  constexpr int K = SP - 1;
  __shared__ uint4 q_cuts[(BLOCK / 64) * QCAP];
  __shared__ uint32_t q_pos[(BLOCK / 64) * QCAP];
  __shared__ int2 CW[DEV_MAX_L + 1], TC[DEV_MAX_L + 1];      // prefixes: {forward + backward, memory}, {forward, forward + backward}
  __shared__ int PA[DEV_MAX_L + 1];
  __shared__ uint64_t wave_keys[BLOCK / 64];
  __shared__ uint32_t wave_fit[BLOCK / 64], wave_worked[BLOCK / 64];
  const ScnPtr scn = as_const(a.s.scn);
  const TabPtr tab = as_const(a.tab);
  const FamPtr ff = &tab->fam[STRAT];
  const int L = scn->L, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int i = threadIdx.x; i <= L; i += BLOCK) {
    const int f = (int)scn->pf[i], both = (int)(scn->pf[i] + scn->pb[i]);
    TC[i] = make_int2(f, both);
    CW[i] = make_int2(both, (int)scn->pw[i]);
    PA[i] = (int)scn->pa[i];
  }
  uint64_t low_cost = ~0ull;               // lowest cost the wavefront has met
  ListBound<SP, STRAT> bound;
  bound.start(scn, tab, ff);
  bound.lower_to(low_cost);
  __syncthreads();

  const int cap = (int)scn->cap;
  uint64_t best_cost = ~0ull;
  uint32_t best_pos = 0, n_fit = 0, n_worked = 0, q_head = 0, q_tail = 0;
  // Row of round `it`: neighbouring lanes read neighbouring rows, a workgroup's rounds lie across the whole list, the last one comes first: in
  // a list in order of cost, rising or falling, the lowest costs are met within two rounds.
  auto entry_of = [&](uint32_t it) { return ((it == 0 ? a.per_lane - 1 : it - 1) * gridDim.x + blockIdx.x) * BLOCK + threadIdx.x; };
  auto row_of = [&](uint32_t it, uint32_t (&w)[4]) {
    const uint32_t entry = entry_of(it);
    const uint64_t at = (uint64_t)(entry < a.s.part_count ? entry : 0) * K;
    w[0] = w[1] = w[2] = w[3] = 0;
    if (at + 16 <= (uint64_t)a.s.part_count * K) {
      __builtin_memcpy(w, a.s.cuts + at, 16);                  // (unaligned; bytes behind the row are not looked at)
    } else {
      for (int i = 0; i < K; ++i) {
        const uint32_t b = (uint32_t)a.s.cuts[at + i] << (8 * (i & 3));
        w[0] |= i < 4 ? b : 0; w[1] |= (i >> 2) == 1 ? b : 0; w[2] |= (i >> 2) == 2 ? b : 0; w[3] |= (i >> 2) == 3 ? b : 0;
      }
    }
  };
  // up to 64 rows of the ring, one a lane: their costs
  auto work_out = [&](uint32_t take) {
    const bool live = (uint32_t)lane < take;
    n_worked += take;
    const uint32_t at_slot = (uint32_t)wave * QCAP + ((q_head + (uint32_t)lane) & (QCAP - 1));
    // (lanes past the end take the first partition, cuts 1..K: always valid)
    const uint4 packed = live ? q_cuts[at_slot] : make_uint4(0x04030201u, 0x08070605u, 0x0c0b0a09u, 0x000f0e0du);
    const uint32_t pos = live ? q_pos[at_slot] : 0;
    const uint32_t words[4] = {packed.x, packed.y, packed.z, packed.w};
    int c[SP + 1];
    unpack_cuts<SP>(words, L, c);
    int t_step = ff->fixed_step;
    // (what is not worked out yet only adds to the cost)
    auto may_win = [&]() { return __builtin_amdgcn_ballot_w64(live && t_step <= bound.limit) != 0; };
    for (int ci = 0; ci < ff->n_time; ++ci) {
      const ClsPtr cl = &ff->cls[ci];
#pragma unroll
      for (int j = 1; j <= K; ++j) asm volatile("" : "+v"(c[j]));
      int F[SP], C[SP];
      int2 t[SP + 1];
      t[0] = make_int2(0, 0);
#pragma unroll
      for (int j = 1; j <= SP; ++j) t[j] = TC[c[j]];
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
      t_step = imax32(t_step, pipeline_time<SP, STRAT == 0>(F, C, cl, ff->time24));
      if (!may_win()) return;
    }
    if (ff->allreduce > 0) {
      // rounds of gradient communication: largest stage on any device, or the ring colouring when nodes hold two stages
      int rounds;
      if (STRAT == 0) {
        rounds = ring_rounds<SP>(c, ff->node_exists);
      } else {
        rounds = ff->fixed_layers;
#pragma unroll
        for (int j = 0; j < SP; ++j) rounds = imax32(rounds, c[j + 1] - c[j]);
      }
      t_step += ff->allreduce * rounds;
    }
    if (STRAT == 2) {
      // least penalty over the reroute vectors of every stage that lost nodes
      for (int st = 0; st < scn->n_aff; ++st) {
        const int2 t = stage_times<SP>(TC, c, scn->aff_stage[st]);
        t_step += (int)stage_penalty<SP>(scn, tab, st, t.x, t.y - t.x);
      }
    }
    if (!may_win()) return;
    int wp[SP + 1];                         // memory prefix at the cuts
    wp[0] = 0;
#pragma unroll
    for (int j = 1; j <= SP; ++j) wp[j] = CW[c[j]].y;
    const uint64_t cost = (uint64_t)scn->K * (uint32_t)t_step + (uint64_t)scn->reconf[STRAT] + (uint64_t)scn->xfer * (uint32_t)missing_weights<SP, STRAT>(ff, wp);
    // (the lower position wins among equal costs)
    if (live && (cost < best_cost || (cost == best_cost && pos < best_pos))) { best_cost = cost; best_pos = pos; }
    if (__builtin_amdgcn_ballot_w64(live && cost < low_cost) != 0) {
      low_cost = uniform64(wave_min(live ? cost : ~0ull));
      bound.lower_to(low_cost);
    }
  };

  uint32_t next_look = 0;                  // round from which on the bound is looked at
  uint32_t words[4], next[4];
  row_of(0, next);
  for (uint32_t it = 0; it < a.per_lane; ++it) {
    const uint32_t entry = entry_of(it);
#pragma unroll
    for (int w = 0; w < 4; ++w) words[w] = next[w];
    if (it + 1 < a.per_lane) row_of(it + 1, next);
    // a row that does not increase strictly within 1..L-1 does not fit; 1..K stands in for it
    const bool valid = strictly_rising<K>(words) && (int)((words[(K - 1) >> 2] >> (8 * ((K - 1) & 3))) & 0xffu) <= L - 1;
    const uint32_t first[4] = {0x04030201u, 0x08070605u, 0x0c0b0a09u, 0x000f0e0du};
#pragma unroll
    for (int w = 0; w < 4; ++w) words[w] = valid ? words[w] : first[w];
    uint64_t in_memory;
    const bool stays = bound.passes(ff, words, L, CW, PA, cap, entry < a.s.part_count && valid, it >= next_look, &in_memory);
    n_fit += (uint32_t)__popcll(in_memory);
    const uint64_t stay_mask = __builtin_amdgcn_ballot_w64(stays);
    if (stay_mask == 0) continue;           // uniform
    if (stays) {
      const uint32_t at_slot = (uint32_t)wave * QCAP + ((q_tail + (uint32_t)__popcll(stay_mask & ((1ull << lane) - 1ull))) & (QCAP - 1));
      q_cuts[at_slot] = make_uint4(words[0], words[1], words[2], words[3]);
      q_pos[at_slot] = a.pos_base + entry;
    }
    q_tail += (uint32_t)__popcll(stay_mask);
    if (q_tail - q_head < 64) continue;
    // (told where the ring is full: elsewhere too little stays for it to matter, and a scalar instruction a round costs half a percent)
    if (it >= next_look && it >= FIRST_LOOKS && 8 * __popcll(stay_mask) > USELESS_SHARE * __popcll(in_memory)) next_look = it + it / 2 + 2;
    work_out(64u);
    q_head += 64;
  }
  if (q_tail != q_head) work_out(q_tail - q_head);

  uint64_t key = best_cost == ~0ull ? CHM_KEY_NONE : ((best_cost << a.s.idx_bits) | (uint64_t)best_pos);
  key = wave_min(key);
  if (lane == 0) { wave_keys[wave] = key; wave_fit[wave] = n_fit; wave_worked[wave] = n_worked; }
  __syncthreads();
  if (threadIdx.x == 0) {
    // one atomic of each kind per workgroup, spread over several words (see SearchLaunch)
    const uint32_t word = (blockIdx.x & a.s.slot_mask) * a.s.slot_stride;
    uint64_t k = wave_keys[0];
    uint32_t fit = wave_fit[0], worked = wave_worked[0];
#pragma unroll
    for (int i = 1; i < BLOCK / 64; ++i) { k = umin64(k, wave_keys[i]); fit += wave_fit[i]; worked += wave_worked[i]; }
    if (fit) atomicAdd((unsigned long long *)a.s.feasible + word, (unsigned long long)fit);
    if (worked) atomicAdd((unsigned long long *)a.s.evaluated + word, (unsigned long long)worked);
    if (k != CHM_KEY_NONE) atomicMin((unsigned long long *)a.s.result + word, (unsigned long long)k);
  }
}

template <int STRAT>
int launch_list_best(int sp, FastLaunch a, hipStream_t st) {
  // as many workgroups as are resident together
  const uint32_t resident = 256u * (uint32_t)list_best_waves(sp);
  a.per_lane = (a.s.part_count + BLOCK * resident - 1) / (BLOCK * resident);
  const uint32_t blocks = (a.s.part_count + BLOCK * a.per_lane - 1) / (BLOCK * a.per_lane);
#define CHM_CASE(SP) case SP: hipLaunchKernelGGL((k_list_best<SP, STRAT>), dim3(blocks), dim3(BLOCK), 0, st, a); return 0;
  switch (sp) {
    CHM_CASE(2) CHM_CASE(3) CHM_CASE(4) CHM_CASE(5) CHM_CASE(6) CHM_CASE(7) CHM_CASE(8) CHM_CASE(9) CHM_CASE(10) CHM_CASE(11)
    CHM_CASE(12) CHM_CASE(13) CHM_CASE(14) CHM_CASE(15) CHM_CASE(16)
    default: return 1;
  }
#undef CHM_CASE
}

}  // namespace

int chmk_list_best(int strategy, int sp, const FastLaunch &a, void *stream) {
  hipStream_t st = (hipStream_t)stream;
  return strategy == 0 ? launch_list_best<0>(sp, a, st) : strategy == 1 ? launch_list_best<1>(sp, a, st) : launch_list_best<2>(sp, a, st);
}
