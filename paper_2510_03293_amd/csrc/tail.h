// The tail of a routing call: the load-ordered chain over the flexible tokens and the
// finishing pass that writes the dispatch tables (Algorithm 1 of the paper, appendix
// "Pseudo Code"; Method: Final assignment).  Device code only, shared by the tail kernel
// and by the fused kernel that runs a whole single-tile call in one launch.
#pragma once

#include <type_traits>

#include "analyse.h"
#include "laser_internal.h"

namespace laser {

// ------------------------------------------------------------------ tail -----
//
// One kernel after the analysis: workgroup 0 is the chain, every other workgroup
// finishes 4 tiles (one wavefront each).  Calls whose tokens may nearly all be load-dependent have up to
// 64 more workgroups, which walk the chain in blocks beside workgroup 0 (see "the chain in blocks").
//
// Chain workgroup (4 wavefronts):
//   prefix  (all waves)  exclusive prefix over tiles of the fixed tokens' per-expert
//           counts -> tile_base; for every tile the number of flexible tokens before it,
//           and the list of those tokens.  Then flag 1 is published: everything is final if no tile holds a flexible token.
//   chain   decides the flexible tokens in token order.  The counters a flexible token
//           sees are loads_in + fixed prefix of its tile + fixed tokens before it
//           inside the tile (carried by its record) + flexible choices so far.
//           Candidate key = (load << 4) + rank: ascending load, ties by score rank; the
//           k smallest keys win.  Two evaluations, same result:
//           - a window of consecutive flexible tokens at once (lane = token), 64 of them in wave 0
//             ("window evaluation") or 256 in four waves ("window of 256 tokens"); used first when
//             there are enough tokens;
//           - sequential (wave 0): a candidate is chosen iff fewer than k candidate keys are
//             smaller than its own, see "sequential walk" and "walks of up to 8 candidates"
//             below.  Takes over where the window evaluation stops paying.
//           Waves that do not evaluate stage the records in LDS ahead of those that do.
//   totals  loads and offsets, then flag 2 (or 3: the blocks were first).
//   Output of the chain, per expert: one bit per flexible token of the call in token
//   order (chain_bits, 32 per word) and the running count of chosen bits at every
//   32-token boundary (chain_cum).
//
// Finishing wavefront (lane = token of its tile): loads what does not depend on the
// chain, waits for flag 1 (and for flag 2 if any tile holds flexible tokens), then
// gives flexible tokens their experts (in score order) and weights from the chain's
// bits and places every assignment slot t*k+j at
//   expert_offsets[e] + (assignments to e in earlier tiles) + (earlier tokens of
//   this tile assigned to e),
// which is the stable counting sort of the flat expert_ids array.  The middle term is
// the fixed tokens' prefix (tile_base) plus the flexible choices of earlier tiles
// (chain_cum at the last boundary + the bits since).
//
// The waits are bounded polls of flags that the analysis kernel of the same call
// cleared.  Workgroup 0 waits for nobody, neither for the blocks of its chain, which it does not need, nor for
// any other workgroup, and it is dispatched ahead of those that wait for it, so the polls
// end, whatever else is on the GPU.  A poll of a finishing wavefront that runs out sets
// ws.status[kStatusError] and the wave leaves without writing; the caller learns of it through
// laser_status().  A block whose wait runs out just leaves.

constexpr int kChainWaves = 4;
constexpr int kTailThreads = kChainWaves * 64;
// workgroups that finish the tiles of a call
__host__ __device__ inline int finish_groups(int ntiles) { return (ntiles + kChainWaves - 1) / kChainWaves; }
constexpr int kSelfPrefixTiles = 1024;  // up to here finishing workgroups sum the counts themselves
// (see "a handful of flexible tokens" below)
constexpr int kFastMaxTiles = 256;
constexpr int kFastTiles = 4;
constexpr int kFastTokens = 8;

// (not for wide calls: the shortcut reads the 16-candidate records)
__device__ __forceinline__ bool fast_path_applies(int ntiles, int nflex_tiles, int nflex_tok, int cw) {
  return cw == kMaxC && ntiles <= kFastMaxTiles && nflex_tiles > 0 && nflex_tiles <= kFastTiles &&
         nflex_tok <= kFastTokens;
}


constexpr int kChainLdsBytes = 57 * 1024;  // dynamic LDS of a chain workgroup, used by one phase after the other
constexpr int kChainStageTiles = kChainLdsBytes / 64;  // tiles of byte counts that fit the LDS

// Data published by the chain workgroup is read with agent-scope atomic loads: they
// see what the publisher wrote back before raising the flag, without the reader
// having to invalidate its whole L2 (the chain may run on another XCD).
__device__ __forceinline__ int load_published(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned load_published(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Flips this lane's bit of a 64-bit mask of lanes in LDS.  As a 32-bit operation on the
// word the bit is in: lanes 0..31 and 32..63 that flip bits of the same mask then work on
// different addresses, and an LDS atomic on one address is served lane after lane.
__device__ __forceinline__ void flip_lane_bit(unsigned long long* mask, int lane) {
  atomicXor(reinterpret_cast<unsigned*>(mask) + (lane >> 5), 1u << (lane & 31));
}

// Orders this wavefront's LDS traffic (another lane's write before this lane's read)
// without waiting for anything in flight to memory: a fence at workgroup scope would
// also wait for the chain's output stores.
__device__ __forceinline__ void lds_wave_fence() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// (every lane its own word)
__device__ __forceinline__ bool poll_word(const int* word, int want, long long limit) {
  for (long long it = 0; it < limit; ++it) {
    if (__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= want) return true;
    __builtin_amdgcn_s_sleep(4);
  }
  return false;
}
// What the flag holds once it is at least `want` (> 0); 0 where the polls run out.
__device__ __forceinline__ int poll_flag(const int* flag, int want, long long limit) {
  for (long long it = 0; it < limit; ++it) {
    const int seen = __builtin_amdgcn_readfirstlane(
        __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    if (seen >= want) return seen;
    __builtin_amdgcn_s_sleep(4);
  }
  return 0;
}

// A chain that is walked in one piece and in blocks at the same time (see "the chain in blocks"):
// whoever is through first claims the call, and a walk that is under way looks every few microseconds
// whether somebody has.  One wavefront asks memory for the claim and looks at the answer at its next
// turn; the others learn of it through LDS, and all of them leave behind the same barrier.
// ON false: nobody else walks the call (no code).
template <bool ON>
struct Race {
  const int* claim;  // NULL: nobody else walks this call
  int* stop;         // LDS, two words
  __device__ __forceinline__ bool on() const { return ON && claim != nullptr; }
  __device__ __forceinline__ int ask() const {
    return on() ? __hip_atomic_load(claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
  }
  // (before a barrier of LDS traffic)
  __device__ __forceinline__ void hand_out(int answer, int lane, int word = 0) const {
    if (on() && lane == 0) stop[word] = answer;
  }
  // (behind that barrier; between reading a word and writing it again there is another one)
  __device__ __forceinline__ bool over(int word = 0) const {
    return on() && __builtin_amdgcn_readfirstlane(stop[word]) != 0;
  }
};

// cnt += number of the 4 lanes named by the bytes of `w` whose key is smaller than this
// lane's key.  Written in assembly because the order of the instructions is the
// point: on gfx950 a vector instruction that reads an SGPR written by the vector
// instruction just before it (lane read -> compare -> add-with-carry) needs two wait
// states each time; grouped as 4 lane reads, 4 compares, 4 adds every producer is at
// least three instructions ahead of its consumer and nothing waits.
__device__ __forceinline__ void count_smaller4(unsigned key, unsigned w, int& cnt) {
  unsigned e0, e1, e2, e3;
  unsigned long long c0, c1, c2, c3, cy;
  asm volatile(
      "s_nop 1\n\t"
      "s_bfe_u32 %[e0], %[w], 0x80000\n\t"
      "s_bfe_u32 %[e1], %[w], 0x80008\n\t"
      "s_bfe_u32 %[e2], %[w], 0x80010\n\t"
      "s_lshr_b32 %[e3], %[w], 24\n\t"
      "v_readlane_b32 %[e0], %[key], %[e0]\n\t"
      "v_readlane_b32 %[e1], %[key], %[e1]\n\t"
      "v_readlane_b32 %[e2], %[key], %[e2]\n\t"
      "v_readlane_b32 %[e3], %[key], %[e3]\n\t"
      "v_cmp_lt_u32_e64 %[c0], %[e0], %[key]\n\t"
      "v_cmp_lt_u32_e64 %[c1], %[e1], %[key]\n\t"
      "v_cmp_lt_u32_e64 %[c2], %[e2], %[key]\n\t"
      "v_cmp_lt_u32_e64 %[c3], %[e3], %[key]\n\t"
      "v_addc_co_u32_e64 %[cnt], %[cy], %[cnt], 0, %[c0]\n\t"
      "v_addc_co_u32_e64 %[cnt], %[cy], %[cnt], 0, %[c1]\n\t"
      "v_addc_co_u32_e64 %[cnt], %[cy], %[cnt], 0, %[c2]\n\t"
      "v_addc_co_u32_e64 %[cnt], %[cy], %[cnt], 0, %[c3]\n\t"
      "s_nop 1\n\t"
      : [cnt] "+v"(cnt), [e0] "=&s"(e0), [e1] "=&s"(e1), [e2] "=&s"(e2), [e3] "=&s"(e3),
        [c0] "=&s"(c0), [c1] "=&s"(c1), [c2] "=&s"(c2), [c3] "=&s"(c3), [cy] "=&s"(cy)
      : [key] "v"(key), [w] "s"(w)
      : "scc");  // (the scalar bit-field extracts and the shift set SCC)
}

// One flexible token of up to 16 candidates (lanes named by the bytes of `ids`): returns
// whether this lane's expert is chosen.  Needs nothing in LDS; for the few tokens that a
// finishing workgroup resolves by itself.
__device__ __forceinline__ bool chain_step(unsigned key, bool cand, const uint4 ids, int k) {
  // (two counts: the second group's additions do not wait for the first group's)
  int smaller = 0, more = 0;
  count_smaller4(key, __builtin_amdgcn_readfirstlane(ids.x), smaller);
  count_smaller4(key, __builtin_amdgcn_readfirstlane(ids.y), more);
  count_smaller4(key, __builtin_amdgcn_readfirstlane(ids.z), smaller);
  count_smaller4(key, __builtin_amdgcn_readfirstlane(ids.w), more);
  return cand && smaller + more < k;
}

// Wave-wide minimum as a scalar: two exchanges inside the quads, the half-row and row
// mirrors (every lane of a 16-lane row then holds the row's minimum), one lane of each
// row read out.
__device__ __forceinline__ unsigned wave_min_u32(unsigned v) {
  constexpr int kRowMirror = 0x140;
  v = min(v, (unsigned)dpp_int<kQuadXor1>((int)v));
  v = min(v, (unsigned)dpp_int<kQuadXor2>((int)v));
  v = min(v, (unsigned)dpp_int<kRowHalfMirror>((int)v));
  v = min(v, (unsigned)dpp_int<kRowMirror>((int)v));
  const unsigned r0 = __builtin_amdgcn_readlane(v, 0), r1 = __builtin_amdgcn_readlane(v, 16);
  const unsigned r2 = __builtin_amdgcn_readlane(v, 32), r3 = __builtin_amdgcn_readlane(v, 48);
  return min(min(r0, r1), min(r2, r3));
}

// x summed over the four quarters of the wavefront: lane l gets the sum over lanes l % 16 + 16 q.
__device__ __forceinline__ unsigned add_quarters(unsigned x) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  u32x2 p = __builtin_amdgcn_permlane32_swap(x, x, false, false);  // (both halves of x, in both halves)
  x = p[0] + p[1];
  p = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return p[0] + p[1];
}

// One flexible token of a wide call (up to 64 candidates), in general: the k candidates with the
// smallest (load, rank).  The candidates are taken level by level of their counters, from the
// lowest one up, a whole level at a time as long as all of it is wanted; of the last level the
// lowest ranks.  Sets of experts are masks in scalar registers; the ranks of a level's experts are
// counted in the lanes of the ranks (`id`: the bit of the expert of rank = lane, 0 where there is
// no candidate) and taken back to the lanes of the experts (`rank`: the bit of the expert's rank).
// `level`: where the token before ended.  Returns 1 in the lanes of the chosen experts, else 0.
__device__ __forceinline__ unsigned chain_step_wide(unsigned load, unsigned long long rank, unsigned long long id, int k,
                                                    unsigned& level) {
  unsigned long long at = __builtin_amdgcn_ballot_w64(load == level);
  const unsigned long long below = __builtin_amdgcn_ballot_w64(load < level);
  // lane = rank: the `want` lowest ranks of the level `at`, then back to lane = expert
  auto lowest = [&](int want) {
    const unsigned long long ranks = __builtin_amdgcn_ballot_w64((at & id) != 0ull);
    const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(ranks >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)ranks, 0));
    const unsigned long long won = __builtin_amdgcn_ballot_w64(before < want) & ranks;
    return (won & rank) != 0ull ? 1u : 0u;
  };
  if (below == 0ull && __builtin_popcountll(at) >= k) return lowest(k);
  if (below != 0ull) {
    level = wave_min_u32(load);
    at = __builtin_amdgcn_ballot_w64(load == level);
  }
  unsigned long long taken = 0ull;
  int want = k;
  // (there are more than k candidates, so the levels of the others are not reached)
  for (int n = __builtin_popcountll(at); n < want; n = __builtin_popcountll(at)) {
    taken |= at;
    want -= n;
    at = __builtin_amdgcn_ballot_w64(load == level + 1);
    if (at != 0ull) {
      ++level;
    } else {
      level = wave_min_u32(load > level ? load : 0xFFFFFFFFu);
      at = __builtin_amdgcn_ballot_w64(load == level);
    }
  }
  return lowest(want) | ((unsigned)(taken >> (threadIdx.x & 63)) & 1u);
}

// What a walk derives from the lane number is computed when the walk begins: the compiler would
// otherwise do it ahead of the loop over a call's segments and keep all walks' masks and
// addresses in registers across everything (51 registers above what two workgroups per
// compute unit leave).
__device__ __forceinline__ void own_lane(int& lane) {
  asm volatile("" : "+v"(lane));
}

// ---- sequential walk ---------------------------------------------------------------------
//
// One dependent step per flexible token, by wave 0 (lane = expert, G = the flexible choices of
// the lane's expert so far); the other waves turn the records into what the step reads, a batch
// ahead, in LDS.  What bounds it is the dependent instructions of a step: a lone wavefront issues
// one every 4.2 to 5 cycles, an LDS lane exchange takes 57 (measured at 2.4 GHz), so the step is
// built to have few of both on the path from one token's choice to the next one's.
//
// Up to 8 candidates: chain_walk_pairs and chain_walk_lag, further down.
// Up to 16 candidates: the keys of the candidates are gathered from the lanes of their experts;
// lane 16 q + i compares the key of rank i with those of ranks 4 q .. 4 q + 3 and the four quarters
// are added across the wavefront (c = 16: 258 -> 132 ns per token).
constexpr int kSeqBatch = 48;  // flexible tokens per LDS batch
struct SeqTok {
  unsigned rec[64];   // per expert: (counter without flexible choices) << 4 | rank, or kSeqNoCand
  uint8_t addr[16];   // per rank: 4 * the candidate's lane (padded with a lane that holds none)
};
constexpr unsigned kSeqNoCand = 0x8000000Du;  // (compares above every key)
static_assert((2 * kSeqBatch + 1) * (int)sizeof(SeqTok) <= kChainLdsBytes, "two batches and a token of read-ahead");

// Wide calls (up to 64 candidates).
// The walk that load-balancing itself produces -- k of the candidates on the level where the last
// token left off, and nobody below it -- needs no search: chain_step_wide written out for that
// case, without a scalar instruction that reads a comparison's result (it would wait for 16
// cycles); that it was the case is looked at when the choice is there.  (8192 tokens, 64
// candidates, k = 6: 113 -> 99 ns per token, the call 952 -> 862 us)
constexpr int kSeqWideBatch = 21;
struct SeqTokWide {
  uint4 bits[64];     // x, y: of the expert of rank = lane; z, w: of the rank of the lane's expert
  unsigned base[64];  // per expert: its counter without flexible choices, or kSeqWideNoCand
};
constexpr unsigned kSeqWideNoCand = 0x40000000u;
static_assert((2 * kSeqWideBatch + 1) * (int)sizeof(SeqTokWide) <= kChainLdsBytes, "two batches and a token of read-ahead");

template <int CP>
struct SeqTraits {
  typedef SeqTok Tok;
  static constexpr int batch = kSeqBatch;
  static constexpr int half = 8;   // tokens whose records a producer wave has in flight together:
};                                 // half of its share of a batch
template <>
struct SeqTraits<0> {
  typedef SeqTokWide Tok;
  static constexpr int batch = kSeqWideBatch;
  static constexpr int half = 4;
};

// What a producer wave needs of some tokens, on its way from memory.
template <int N>
struct SeqLoads {
  unsigned rec[N], cids[N];
  int base[N];
};

// Producer wave pw (0, 1, 2) takes tokens pw, pw + 3, ... of every batch, in two halves.
// Lane i: where the record of its i-th token of batch `batch` is.
template <int CP>
__device__ __forceinline__ int seq_slots(int batch, int nflex_tok, const Workspace& ws, int pw, int lane) {
  constexpr int NB = SeqTraits<CP>::batch;
  const int f = batch * NB + pw + 3 * min(lane, (NB + 2) / 3);
  // (loads without conditions stay in flight: any token of the call stands in for none)
  return ws.flex_slot[min(f, nflex_tok - 1)];
}
template <int CP, int N>
__device__ __forceinline__ void seq_load(SeqLoads<N>& L, int slots, int i0, const RouteArgs& a, const Workspace& ws,
                                         int lane) {
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int slot = __builtin_amdgcn_readlane(slots, i0 + u);
    L.rec[u] = (ws.rec_lane + (size_t)slot * a.EP)[(unsigned)min(lane, a.EP - 1)];
    L.base[u] = ws.tile_base[(size_t)(slot >> 6) * 64 + lane];
    if constexpr (CP != 0) L.cids[u] = ws.rec_cids[(size_t)slot * 16 + (lane & 15)];
  }
}
template <int CP, int N>
__device__ __forceinline__ void seq_store(typename SeqTraits<CP>::Tok* dst, const SeqLoads<N>& L, int i0, int pw,
                                          int EP, int lane, int lin) {
#pragma unroll
  for (int u = 0; u < N; ++u) {
    if (pw + 3 * (i0 + u) >= SeqTraits<CP>::batch) break;
    auto* tok = dst + pw + 3 * (i0 + u);
    const bool cand = lane < EP && L.rec[u] != 0xFFFFu;
    const unsigned base = (unsigned)(lin + L.base[u]);
    if constexpr (CP != 0) {
      tok->rec[lane] = cand ? (base << 4) + L.rec[u] : kSeqNoCand;
      if (lane < 16) tok->addr[lane] = (uint8_t)(4 * L.cids[u]);
    } else {
      // (the ranks of the candidates, then the others: every lane sends its number to one of its own)
      const unsigned long long all = __builtin_amdgcn_ballot_w64(cand);
      const int ncand = __builtin_popcountll(all);
      const int other = lane - __builtin_amdgcn_mbcnt_hi((unsigned)(all >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)all, 0));
      const int rank = cand ? (int)(L.rec[u] & 63u) : ncand + other;
      const int id = __builtin_amdgcn_ds_permute(4 * rank, lane);
      const unsigned long long id_bit = lane < ncand ? 1ull << id : 0ull, rank_bit = cand ? 1ull << rank : 0ull;
      tok->bits[lane] = make_uint4((unsigned)id_bit, (unsigned)(id_bit >> 32), (unsigned)rank_bit, (unsigned)(rank_bit >> 32));
      tok->base[lane] = cand ? base + (L.rec[u] >> 6) : kSeqWideNoCand;
    }
  }
}

// Walks the flexible tokens from token `f0` of the call on.  `hist0`: the bits of output word
// f0 / 32 that are decided already.  The output (chain_bits, chain_cum) is indexed by the
// flexible token's number within the call.  CP: 16 candidates, 0: a wide call.  Returns whether the
// walk has come to its end (see Race).
template <int CP, bool RACE>
__device__ __forceinline__ bool chain_walk(uint8_t* lds, int f0, unsigned hist0, int nflex_tok, const RouteArgs& a,
                                           const Workspace& ws, int wave, int lane, int lin, int& gflex, Race<RACE> race) {
  own_lane(lane);
  typedef typename SeqTraits<CP>::Tok Tok;
  constexpr int NB = SeqTraits<CP>::batch;
  Tok* const buf = reinterpret_cast<Tok*>(lds);
  // wave-uniform values that arrive through LDS or memory: tell the compiler so, or the
  // loops below are compiled as divergent ones
  f0 = __builtin_amdgcn_readfirstlane(f0);
  nflex_tok = __builtin_amdgcn_readfirstlane(nflex_tok);
  const int b0 = f0 / NB, b1 = (nflex_tok + NB - 1) / NB;
  const unsigned k = (unsigned)a.k;
  int f = f0;
  unsigned G = (unsigned)gflex;
  // bits of the current output word, the last token's lowest
  unsigned hist = (f0 & 31) != 0 ? __builtin_bitreverse32(hist0) >> (32 - (f0 & 31)) : 0u;
  unsigned level = 0xFFFFFFFFu;  // (wide: no counter of a candidate is known to be below)
  unsigned chosen = 0u;          // (wide: of the last token, not in hist yet)
  // The producers are two batches ahead with the list of records, and half a batch ahead with
  // the records themselves: a batch is decided in a few microseconds, a record is two dependent
  // memory round trips away.  (The barriers leave loads in flight alone.)
  constexpr int NH = SeqTraits<CP>::half;
  const int pw = wave - 1;
  int slots = 0, slots_n = 0;  // of the batch being stored, of the next one
  SeqLoads<NH> first, second;
  if (wave != 0) {
    slots = seq_slots<CP>(b0, nflex_tok, ws, pw, lane);
    slots_n = seq_slots<CP>(b0 + 1, nflex_tok, ws, pw, lane);
    seq_load<CP, NH>(first, slots, 0, a, ws, lane);
    seq_load<CP, NH>(second, slots, NH, a, ws, lane);
    Tok* dst = buf + (b0 & 1) * NB;
    seq_store<CP, NH>(dst, first, 0, pw, a.EP, lane, lin);
    seq_load<CP, NH>(first, slots_n, 0, a, ws, lane);
    seq_store<CP, NH>(dst, second, NH, pw, a.EP, lane, lin);
  }
  // (looks at the claim are a few tokens apart: a token of a wide call can take a microsecond)
  constexpr int kPiece = !RACE ? 32 : CP != 0 ? 16 : 8;
  int answer = 0;
  if (RACE && wave == 0) {
    race.hand_out(0, lane, 0);
    race.hand_out(0, lane, 1);
    answer = race.ask();
  }
  lds_barrier();
  for (int b = b0; b < b1; ++b) {
    if (wave != 0) {
      if (b + 1 < b1) {
        slots = slots_n;
        slots_n = seq_slots<CP>(b + 2, nflex_tok, ws, pw, lane);
        seq_load<CP, NH>(second, slots, NH, a, ws, lane);
        Tok* dst = buf + ((b + 1) & 1) * NB;
        seq_store<CP, NH>(dst, first, 0, pw, a.EP, lane, lin);
        seq_load<CP, NH>(first, slots_n, 0, a, ws, lane);
        seq_store<CP, NH>(dst, second, NH, pw, a.EP, lane, lin);
      }
    } else {
      const Tok* cur = buf + (b & 1) * NB;
      const int n = min(NB, nflex_tok - b * NB);
      int r = f - b * NB;
      auto look = [&]() {
        if (!RACE || !race.on()) return false;
        const bool over = __builtin_amdgcn_readfirstlane(answer) != 0;
        answer = race.ask();
        if (over) race.hand_out(1, lane, b & 1);
        return over;
      };
      if constexpr (CP != 0) {
        constexpr int kPer = 4;  // keys a lane compares with
        unsigned rec = cur[r].rec[lane];
        unsigned ai = cur[r].addr[lane & 15], aj[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) aj[u] = cur[r].addr[4 * (lane >> 4) + u];
        // (the next token's record is read while this one is decided; behind the last one of a
        // batch it is read and not used)
        auto step = [&](const Tok& next) {
          const unsigned key = (G << 4) + rec;
          const unsigned ki = (unsigned)__builtin_amdgcn_ds_bpermute((int)ai, (int)key);
          unsigned kj[kPer];
#pragma unroll
          for (int u = 0; u < kPer; ++u) kj[u] = (unsigned)__builtin_amdgcn_ds_bpermute((int)aj[u], (int)key);
          __builtin_amdgcn_sched_barrier(0);
          const unsigned rec_n = next.rec[lane];
          const unsigned ai_n = next.addr[lane & 15];
          unsigned aj_n[kPer];
#pragma unroll
          for (int u = 0; u < kPer; ++u) aj_n[u] = next.addr[4 * (lane >> 4) + u];
          __builtin_amdgcn_sched_barrier(0);
          const unsigned shift = (rec & 15u) | ((rec >> 27) & 16u);  // (no candidate: a bit that is not set)
          unsigned cnt = 0;
#pragma unroll
          for (int u = 0; u < kPer; ++u) cnt += kj[u] < ki ? 1u : 0u;
          cnt = add_quarters(cnt);
          const unsigned won = (unsigned)__builtin_amdgcn_ballot_w64(cnt < k) & 0xFFFFu;
          const bool chosen = ((won >> shift) & 1u) != 0u;
          G += chosen ? 1u : 0u;
          hist = hist + hist + (chosen ? 1u : 0u);
          rec = rec_n;
          ai = ai_n;
#pragma unroll
          for (int u = 0; u < kPer; ++u) aj[u] = aj_n[u];
        };
        while (r < n) {
          // up to the end of the batch or of the 32-token output word (or half of it), whichever is first
          const int end = min(n, r + kPiece - (f & (kPiece - 1)));
          f += end - r;
          if (look()) break;
          for (; r + 4 <= end; r += 4) {
            step(cur[r + 1]);
            step(cur[r + 2]);
            step(cur[r + 3]);
            step(cur[r + 4]);
          }
          for (; r < end; ++r) step(cur[r + 1]);
          if ((f & 31) == 0) {
            ws.chain_bits[(size_t)((f >> 5) - 1) * 64 + lane] = __builtin_bitreverse32(hist);
            ws.chain_cum[(size_t)(f >> 5) * 64 + lane] = (int)G;
            hist = 0;
          }
        }
      } else {
        uint4 bits = cur[r].bits[lane];
        unsigned base = cur[r].base[lane];
        const unsigned none = 64u;
        auto step = [&](const Tok& next) {
          const unsigned load = base + G;
          const uint4 bits_n = next.bits[lane];
          const unsigned base_n = next.base[lane];
          // (what is read out of a comparison's scalar is at least two instructions behind it; the
          // named registers are the blocks' own, since k and k - 1 are read after they are written)
          unsigned x;
          unsigned long long kth;
          asm("v_cmp_eq_u32 s[88:89], %[load], %[level]\n\t"           // on the level
              "v_cmp_lt_u32 s[90:91], %[load], %[level]\n\t"
              "v_lshl_or_b32 %[hist], %[hist], 1, %[chosen]\n\t"       // (the token before)
              "v_and_b32 %[x], s88, %[id0]\n\t"
              "v_bitop3_b32 %[x], %[id1], %[x], s89 bitop3:0xec\n\t"   // x | (s89 & id1): by rank
              "v_cmp_ne_u32 s[92:93], 0, %[x]\n\t"
              "s_cmp_lg_u64 s[90:91], 0\n\t"                           // somebody is below the level
              "s_nop 0\n\t"
              "v_mbcnt_lo_u32_b32 %[x], s92, 0\n\t"                    // how many of lower rank are
              "v_mbcnt_hi_u32_b32 %[x], s93, %[x]\n\t"
              "v_cndmask_b32 %[x], %[none], %[x], s[92:93]\n\t"
              "v_cmp_gt_u32 s[94:95], %[k], %[x]\n\t"                  // chosen
              "v_cmp_eq_u32 s[92:93], %[km1], %[x]\n\t"                // the last one of the k
              "s_nop 0\n\t"
              "v_and_b32 %[x], s94, %[r0]\n\t"
              "v_bitop3_b32 %[x], %[r1], %[x], s95 bitop3:0xec\n\t"    // by expert
              "v_min_u32 %[x], 1, %[x]\n\t"
              "s_cselect_b64 %[kth], 0, s[92:93]\n\t"
              : [hist] "+v"(hist), [x] "=&v"(x), [kth] "=&s"(kth)
              : [load] "v"(load), [level] "v"(level), [chosen] "v"(chosen), [id0] "v"(bits.x), [id1] "v"(bits.y),
                [r0] "v"(bits.z), [r1] "v"(bits.w), [none] "v"(none), [k] "s"(k), [km1] "s"(k - 1)
              : "s88", "s89", "s90", "s91", "s92", "s93", "s94", "s95", "scc");
          chosen = x;
          if (__builtin_expect(kth == 0ull, 0)) {
            // fewer than k on the level (or somebody below it): all of those, and the lowest ranks
            // of the level above, in the same manner
            unsigned n0;
            unsigned long long below;
            asm("v_cmp_eq_u32 s[90:91], %[load], %[level]\n\t"
                "v_cmp_eq_u32 s[88:89], %[load], %[next]\n\t"
                "s_nop 0\n\t"
                "v_bcnt_u32_b32 %[n0], s90, 0\n\t"
                "v_bcnt_u32_b32 %[n0], s91, %[n0]\n\t"
                "v_and_b32 %[x], s88, %[id0]\n\t"
                "v_bitop3_b32 %[x], %[id1], %[x], s89 bitop3:0xec\n\t"
                "v_cmp_ne_u32 s[92:93], 0, %[x]\n\t"
                "v_cmp_lt_u32 s[88:89], %[load], %[level]\n\t"
                "s_nop 0\n\t"
                "v_mbcnt_lo_u32_b32 %[x], s92, %[n0]\n\t"
                "v_mbcnt_hi_u32_b32 %[x], s93, %[x]\n\t"
                "v_cndmask_b32 %[x], %[none], %[x], s[92:93]\n\t"
                "v_cmp_gt_u32 s[94:95], %[k], %[x]\n\t"
                "v_cmp_eq_u32 s[92:93], %[km1], %[x]\n\t"
                "s_nop 0\n\t"
                "v_and_b32 %[x], s94, %[r0]\n\t"
                "v_bitop3_b32 %[x], %[r1], %[x], s95 bitop3:0xec\n\t"
                "v_min_u32 %[x], 1, %[x]\n\t"
                "v_cndmask_b32 %[x], %[x], 1, s[90:91]\n\t"
                "s_mov_b64 %[below], s[88:89]\n\t"
                "s_mov_b64 %[kth], s[92:93]\n\t"
                : [x] "=&v"(x), [n0] "=&v"(n0), [below] "=&s"(below), [kth] "=&s"(kth)
                : [load] "v"(load), [level] "v"(level), [next] "v"(level + 1u), [id0] "v"(bits.x), [id1] "v"(bits.y),
                  [r0] "v"(bits.z), [r1] "v"(bits.w), [none] "v"(none), [k] "s"(k), [km1] "s"(k - 1)
                : "s88", "s89", "s90", "s91", "s92", "s93", "s94", "s95");
            chosen = x;
            if (kth != 0ull && below == 0ull)
              ++level;
            else
              chosen = chain_step_wide(load, ((unsigned long long)bits.w << 32) | bits.z,
                                       ((unsigned long long)bits.y << 32) | bits.x, (int)k, level);
          }
          G += chosen;
          bits = bits_n;
          base = base_n;
        };
        while (r < n) {
          const int end = min(n, r + kPiece - (f & (kPiece - 1)));
          f += end - r;
          if (look()) break;
          for (; r + 2 <= end; r += 2) {
            step(cur[r + 1]);
            step(cur[r + 2]);
          }
          for (; r < end; ++r) step(cur[r + 1]);
          if ((f & 31) == 0) {
            hist = (hist << 1) | chosen;
            ws.chain_bits[(size_t)((f >> 5) - 1) * 64 + lane] = __builtin_bitreverse32(hist);
            ws.chain_cum[(size_t)(f >> 5) * 64 + lane] = (int)G;
            hist = chosen = 0u;
          }
        }
      }
    }
    lds_barrier();
    if (RACE && race.over(b & 1)) return false;
  }
  if (wave == 0) {
    gflex = (int)G;
    if constexpr (CP == 0) hist = (hist << 1) | chosen;
    if ((f & 31) != 0)
      ws.chain_bits[(size_t)(f >> 5) * 64 + lane] = __builtin_bitreverse32(hist) >> (32 - (f & 31));
  }
  return true;
}

// ---- walks of up to 8 candidates --------------------------------------------------------
//
// All pairs of candidates at once.  Candidate j is before candidate i exactly if
//     G[j] - G[i] <= U,
// with G the flexible choices so far and U a number that the counters without them and the ranks
// give beforehand.  There are 28 pairs i < j, one per lane; the comparison leaves them as bits in a
// scalar register, and the number of candidates before any one of them is a bit count: of its
// pairs' bits, those flipped in which it is the second one.  It is chosen iff there are fewer
// than k.  A lone wavefront issues a vector instruction every 4.2 to 4.7 cycles, whether it needs
// the result of the one before or not (measured, 2.4 GHz); a lane exchange through LDS takes 56,
// and a vector instruction that reads the scalar of the comparison before it waits for two
// others in between.  So what counts is the number of instructions, that none waits for an
// exchange, and that other work stands behind the comparisons.

// The pair of this lane (lanes 28 and up: 0, 0).
__device__ __forceinline__ void lane_pair(int lane, int& i, int& j) {
  int rest = lane;
  i = 0;
  while (i < 7 && rest >= 7 - i) {
    rest -= 7 - i;
    ++i;
  }
  j = i + 1 + rest;
  if (lane >= 28) i = j = 0;
}
// How many are before number e: the bits of (pairs ^ flip) & mask.
struct PairCount {
  unsigned flip, mask;
};
__device__ __forceinline__ PairCount pair_count(int e, int i, int j, int lane) {
  PairCount c = {0u, 0u};
#pragma unroll
  for (int n = 0; n < 8; ++n) {
    const unsigned second = (unsigned)__builtin_amdgcn_ballot_w64(lane < 28 && j == n);
    const unsigned first = (unsigned)__builtin_amdgcn_ballot_w64(lane < 28 && i == n);
    c.flip = e == n ? second : c.flip;
    c.mask = e == n ? first | second : c.mask;
  }
  return c;
}
__device__ __forceinline__ int count_before(unsigned pairs, const PairCount& c, int start) {
  // (the instruction adds as well; the compiler would make an instruction of its own of it)
  int n;
  asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(n) : "v"((pairs ^ c.flip) & c.mask), "v"(start));
  return n;
}
// U of a pair with the keys ki, kj ((counter << 4) + rank, below 2^31; negative: no candidate):
// kj + 16 G[j] < ki + 16 G[i].  Who is no candidate is behind every candidate, of which there
// are more than k.
__device__ __forceinline__ int pair_bound(int ki, int kj) {
  constexpr int kBeyond = 1 << 30;  // (every difference of the choices)
  const int u = (ki + ~kj) >> 4;
  return kj < 0 ? -kBeyond : ki < 0 ? kBeyond : u;
}

// More than 8 experts.  A pair is one of ranks, and G lives in the lanes of the experts: the
// difference would have to be exchanged for every token on the path from one choice to the
// next.  Instead it is gathered a token early, before the choice of the token in between
// is known; that one enters as two bits of W, the mask of its chosen ranks: whether ci, and
// whether cj, was among them, at places that are known beforehand.
// All of that is prepared by waves 1 and 2, 16 tokens at a time in an LDS ring of three such
// batches (the consumer looks four tokens ahead, so the batch behind the current one is complete
// before the current one is begun).
// What bounds the step: 16 vector instructions, four LDS instructions -- a lane exchange keeps the
// wavefront from issuing for about 15 cycles --, waits; 105 cycles, and 9 of the batch's barrier.
// (A scalar move that reads the comparison's result costs 16 more.)
// 16384 tokens, 64 experts, k = 6, c = 8, all load-dependent: 69 -> 53 ns per token, the call 1156 ->
// 878 us, all but about 30 of it the walk.
constexpr int kLagBatch = 16;
struct LagTok {
  int4 v[32];  // per pair: U; 4 * lane of ci; 4 * lane of cj; their places in the W of the token
};             // before, a byte each
constexpr unsigned kLagNone = 15;  // (a bit of W that is never set)
// Per expert its place in the token's W: rows of 64 bytes, for each of the two producers of a batch
// that of the token before its eight and theirs.
constexpr int kLagPlaceRows = 9;
constexpr int kLagPlaceOffset = 3 * kLagBatch * (int)sizeof(LagTok);
static_assert(kLagPlaceOffset + 3 * 2 * kLagPlaceRows * 64 <= kChainLdsBytes, "ring of three batches");

// The loads of the producers have no conditions (any token of the call stands in for none): those
// stay in flight where one behind a branch would be waited for at its end.
__device__ __forceinline__ int lag_slot(int f, int nflex_tok, const Workspace& ws) {
  return ws.flex_slot[min(max(f, 0), nflex_tok - 1)];
}

// What a producer needs of its eight tokens, lane (s, r) = (lane / 8, lane % 8): candidate of
// rank r of token s.
struct LagCand {
  unsigned cid, pref;
  unsigned cid_before;  // candidate of rank r of the token before the eight
  int base;             // assignments in the tiles before the token's
};
// f: number of the first of the eight; at_i, at_j: see below.
__device__ __forceinline__ void lag_store(LagTok* dst, uint8_t* places, const LagCand& c, int f, int f0, int nflex_tok,
                                          int lane, int at_i, int at_j, int lin) {
  const int tok = f + (lane >> 3), r = lane & 7;
  const bool live = tok >= f0 && tok < nflex_tok;
  // ---- the places: rank of the expert, or none ----------------------------------------
  constexpr unsigned kNone4 = kLagNone * 0x01010101u;
  reinterpret_cast<uint2*>(places)[lane] = make_uint2(kNone4, kNone4);
  if (lane < 16) reinterpret_cast<unsigned*>(places)[128 + lane] = kNone4;
  asm volatile("" ::: "memory");  // (a wavefront's LDS traffic stays in order)
  // (ranks beyond the working set share a lane that holds no candidate; their bits of W are 0)
  if (live) places[(1 + (lane >> 3)) * 64 + c.cid] = (uint8_t)r;
  if (lane < 8 && f > f0 && f <= nflex_tok) places[c.cid_before] = (uint8_t)r;
  asm volatile("" ::: "memory");
  // ---- the pairs, lane (h, p) = (lane / 32, lane % 32): pair p of tokens 2 q + h ---------------
  const int before = c.base + __builtin_amdgcn_ds_bpermute(4 * (int)c.cid, lin) + (int)c.pref;
  const int key = (c.pref != 0xFFu && live) ? (before << 4) + r : -1;
  int ci[4], cj[4], ki[4], kj[4], wi[4], wj[4];  // (all exchanges in flight together)
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    ci[q] = __builtin_amdgcn_ds_bpermute(at_i + 64 * q, (int)c.cid);
    cj[q] = __builtin_amdgcn_ds_bpermute(at_j + 64 * q, (int)c.cid);
    ki[q] = __builtin_amdgcn_ds_bpermute(at_i + 64 * q, key);
    kj[q] = __builtin_amdgcn_ds_bpermute(at_j + 64 * q, key);
  }
  __builtin_amdgcn_sched_barrier(0);
  const int h = lane >> 5;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    wi[q] = places[(2 * q + h) * 64 + ci[q]];
    wj[q] = places[(2 * q + h) * 64 + cj[q]];
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < 4; ++q)
    dst[2 * q + h].v[lane & 31] = make_int4(pair_bound(ki[q], kj[q]), 4 * ci[q], 4 * cj[q], wi[q] | (wj[q] << 8));
}

// (f0, hist0 and what it returns: as chain_walk)
template <bool RACE>
__device__ __forceinline__ bool chain_walk_lag(uint8_t* lds, int f0, unsigned hist0, int nflex_tok, const RouteArgs& a,
                                               const Workspace& ws, int wave, int lane, int lin, int& gflex,
                                               Race<RACE> race) {
  own_lane(lane);
  LagTok* const ring = reinterpret_cast<LagTok*>(lds);
  uint8_t* const places = lds + kLagPlaceOffset;
  f0 = __builtin_amdgcn_readfirstlane(f0);
  nflex_tok = __builtin_amdgcn_readfirstlane(nflex_tok);
  const int b0 = f0 / kLagBatch, b1 = (nflex_tok + kLagBatch - 1) / kLagBatch;
  int pi, pj;
  lane_pair(lane & 31, pi, pj);
  // (a look at the claim every four batches, 3.4 us; in loops around those over the batches, and only where
  // it is RACE: a test in the consumer's loop over the batches cost the walk 5 %, loops around it 1.4 %)
  constexpr int kLook = 4;
  bool whole = true;
  auto stretches = [&](auto batches) {  // batches(b, be): from b on, before be
    if constexpr (RACE) {
      for (int b = b0, be; b < b1 && whole; b = be) {
        be = race.on() ? min(b1, b + kLook) : b1;
        batches(b, be);
        if (be < b1 && race.over()) whole = false;
      }
    } else {
      batches(b0, b1);
    }
  };
  if (wave == 1 || wave == 2) {
    // ---- producers: two batches ahead of the consumer in LDS, and two more with every load that
    // leads to another one -- where the records are, the records, the counters of the candidates
    // (the barriers leave loads in flight alone) ----
    const int pw = wave - 1, tok = 8 * pw + (lane >> 3);
    const int at_i = 32 * (lane >> 5) + 4 * pi, at_j = 32 * (lane >> 5) + 4 * pj;
    struct Slots {
      int own, before;
    };
    auto slot_of = [&](int n) {
      return Slots{lag_slot(n * kLagBatch + tok, nflex_tok, ws), lag_slot(n * kLagBatch + 8 * pw - 1, nflex_tok, ws)};
    };
    auto records = [&](LagCand& c, const Slots& s) {
      c.cid = ws.rec_cids[(size_t)s.own * 16 + (lane & 7)];
      c.pref = ws.rec_pref[(size_t)s.own * 16 + (lane & 7)];
      c.cid_before = ws.rec_cids[(size_t)s.before * 16 + (lane & 7)];
      c.base = s.own >> 6;  // (the tile, until the counter is loaded)
    };
    auto counter = [&](LagCand& c, const LagCand& r) {
      c.cid = r.cid;
      c.pref = r.pref;
      c.cid_before = r.cid_before;
      c.base = ws.tile_base[(size_t)r.base * 64 + r.cid];
    };
    Slots s0 = slot_of(b0), s1 = slot_of(b0 + 1);
    LagCand r0, r1, c0, c1;
    records(r0, s0);
    records(r1, s1);
    s0 = slot_of(b0 + 2);
    s1 = slot_of(b0 + 3);
    counter(c0, r0);
    counter(c1, r1);
    records(r0, s0);
    records(r1, s1);
    s0 = slot_of(b0 + 4);
    s1 = slot_of(b0 + 5);
    int buf = 0;  // of batch n
    auto fill = [&](int n, LagCand& c, LagCand& r, Slots& s) {
      lag_store(ring + buf * kLagBatch + 8 * pw, places + (2 * buf + pw) * kLagPlaceRows * 64, c, n * kLagBatch + 8 * pw, f0,
                nflex_tok, lane, at_i, at_j, lin);
      buf = buf == 2 ? 0 : buf + 1;
      counter(c, r);
      records(r, s);
      s = slot_of(n + 6);
    };
    fill(b0, c0, r0, s0);
    fill(b0 + 1, c1, r1, s1);
    lds_barrier();
    // (what is filled behind the last batch is not read)
    stretches([&](int b, int be) {
      for (; b < be; b += 2) {
        fill(b + 2, c0, r0, s0);
        lds_barrier();
        if (b + 1 >= be) break;
        fill(b + 3, c1, r1, s1);
        lds_barrier();
      }
    });
  } else if (wave != 0) {
    lds_barrier();
    stretches([&](int b, int be) {
      const int answer = race.ask();
      for (; b < be; ++b) {
        if (RACE && b + 1 == be && be < b1) race.hand_out(answer, lane);
        lds_barrier();
      }
    });
  } else {
    // ---- consumer ----------------------------------------------------------------------
    int G = gflex;
    unsigned hist = 0;  // the choices of the output word's tokens so far, the last one lowest
    const int k = a.k;
    // lane r < 8 counts for rank r; the others' bits of W stay 0
    const PairCount rank = pair_count(lane, pi, pj, lane);
    const int pair = lane & 31;
    const int start = lane < 8 ? 0 : 64;
    auto gather = [&](int from) { return __builtin_amdgcn_ds_bpermute(from, G); };
    lds_barrier();
    const LagTok* cur = ring;
    const uint8_t* cur_places = places + lane;  // row of the batch's token 0
    auto row = [](int u) { return ((u >> 3) * kLagPlaceRows + 1 + (u & 7)) * 64; };
    const LagTok* const ring_end = ring + 3 * kLagBatch;
    int4 d0 = cur[0].v[pair], d1 = cur[1].v[pair], d2 = cur[2].v[pair], d3 = cur[3].v[pair];
    unsigned place = cur_places[row(0)], place1 = cur_places[row(1)];
    // (no bytes from here on: carried as bytes they would be widened, hence waited for, at the head of
    // every batch)
    asm volatile("" : "+v"(place), "+v"(place1));
    int i1 = gather(d1.y), j1 = gather(d1.z);
    // (the choice before the first token is in G)
    int diff = gather(d0.z) - gather(d0.y);
    unsigned chosen = 0u;  // (lane = expert: of the token before)
    stretches([&](int b, int be) {
      for (; b < be; ++b) {
        const bool wrap = cur + kLagBatch == ring_end;
        const LagTok* const next = wrap ? ring : cur + kLagBatch;
        const uint8_t* const next_places = wrap ? places + lane : cur_places + 2 * kLagPlaceRows * 64;
  #pragma unroll
        for (int u = 0; u < kLagBatch; ++u) {
          // From the difference to W and the choice of the lane's expert, in assembly because the
          // order is the point: what is read out of a comparison's scalar must be two instructions
          // behind it, and these do something.
          unsigned next_j;
          unsigned long long won;
          asm("v_cmp_le_i32 vcc, %[diff], %[U]\n\t"
              "v_lshl_or_b32 %[hist], %[hist], 1, %[chosen]\n\t"  // (the token before)
              "v_lshrrev_b32 %[nj], 8, %[w1]\n\t"
              "v_bitop3_b32 %[diff], %[flip], %[mask], vcc_lo bitop3:0x48\n\t"  // (pairs ^ flip) & mask
              "v_bcnt_u32_b32 %[diff], %[diff], %[start]\n\t"
              "v_cmp_gt_i32 s[98:99], %[k], %[diff]\n\t"
              : [diff] "+v"(diff), [hist] "+v"(hist), [nj] "=&v"(next_j), [won] "={s[98:99]}"(won)
              : [chosen] "v"(chosen), [U] "v"(d0.x), [w1] "v"(d1.w), [flip] "v"(rank.flip), [mask] "v"(rank.mask),
                [start] "v"(start), [k] "s"(k)
              : "vcc");
          // (two blocks, so that the difference gathered for the next token is waited for here only)
          asm("v_sub_u32 %[diff], %[j1], %[i1]\n\t"
              "s_nop 0\n\t"
              "v_bfe_u32 %[chosen], s98, %[place], 1\n\t"
              "v_add_u32 %[G], %[G], %[chosen]\n\t"
              : [diff] "=&v"(diff), [chosen] "=&v"(chosen), [G] "+v"(G)
              : [i1] "v"(i1), [j1] "v"(j1), [place] "v"(place), [won] "{s[98:99]}"(won));
          // (a scalar instruction that read it would wait for 16 cycles)
          const unsigned W = (unsigned)won;
          const int i2 = gather(d2.y), j2 = gather(d2.z);
          __builtin_amdgcn_sched_barrier(0);
          const int next_chose_i = (int)__builtin_amdgcn_sbfe((int)W, (unsigned)d1.w, 1);
          const int next_chose_j = (int)__builtin_amdgcn_ubfe(W, next_j, 1);
          __builtin_amdgcn_sched_barrier(0);
          diff = diff + next_chose_i + next_chose_j;
          place = place1;
          place1 = u + 2 < kLagBatch ? cur_places[row(u + 2)] : next_places[row(u + 2 - kLagBatch)];
          i1 = i2;
          j1 = j2;
          d0 = d1;
          d1 = d2;
          d2 = d3;
          // (behind the last token of the call: read and not used)
          d3 = u + 4 < kLagBatch ? cur[u + 4].v[pair] : next[u + 4 - kLagBatch].v[pair];
          __builtin_amdgcn_sched_barrier(0);
        }
        const int w = b >> 1;
        if ((b & 1) != 0 || b + 1 == b1) {
          hist = (hist << 1) | chosen;
          if ((b & 1) == 0) hist <<= kLagBatch;
          const unsigned word = __builtin_bitreverse32(hist) | (w == (f0 >> 5) ? hist0 : 0u);
          ws.chain_bits[(size_t)w * 64 + lane] = word;
          if (32 * (w + 1) <= nflex_tok) ws.chain_cum[(size_t)(w + 1) * 64 + lane] = G;
          hist = chosen = 0u;
        }
        cur = next;
        cur_places = next_places;
        lds_barrier();
      }
    });
    gflex = G;
  }
  return whole;
}

// Up to 8 experts (all of a call's flexible tokens).  A pair is one of experts: the lane itself
// keeps the difference D of their choices, counts for both and adds (j chosen) - (i chosen);
// nothing is exchanged at all.  Eight instructions per token and none that only waits: the
// comparison is T <= U - D, with T what the token before adds and U - D made behind that token's
// comparison.  Lanes 28 to 35 count for one expert each, for the output: there D is shifted by
// one per token, and holds the experts' last 32 choices.
// What bounds a step: eight instructions at 4.7 cycles, and a sixteen-byte read per four tokens, issued
// for about 16 (two groups ahead, held there against the compiler, which would sink it to its use).
// Waves 1 and 2 prepare U, eight tokens per memory instruction, 96 tokens per batch; wave 3 writes
// out the choices (whose stores the producers' loads would wait for).
// 8 experts, k = 2, c = 4, every one of 16384 tokens load-dependent: 17.7 ns per token whatever the
// counters are, the call 318 us.  (Nine instructions and a wait, and 32 lane exchanges and 32 writes per
// 16 tokens in the producers: 21.6 ns, 379 us.  The window evaluation: 303 us where no tokens compete,
// 1906 us where they do.)  Four layers of 16384 tokens, a tenth of them load-dependent: 316 -> 290 us.
constexpr int kPairBatch = 96;  // tokens per LDS batch: 48 per producer wave
struct PairGroup {
  int4 v[32];  // per pair: U of four tokens
};
constexpr int kPairGroups = kPairBatch / 4, kPairWords = kPairBatch / 32;
// A ring of three batches (the consumer reads two groups ahead, so the batch behind the current one is
// complete before the current one is begun), and two batches' words of output.
constexpr int kPairOutOffset = 3 * kPairGroups * (int)sizeof(PairGroup);
static_assert(kPairOutOffset + 2 * kPairWords * 64 * 4 <= kChainLdsBytes, "ring and output");
constexpr int kPairLoads = kPairBatch / 2 / 8;  // of eight tokens each, per producer and batch

__device__ __forceinline__ void chain_walk_pairs(uint8_t* lds, int nflex_tok, const Workspace& ws, int k, int wave,
                                                 int lane, int lin, int& gflex) {
  own_lane(lane);
  PairGroup* const ring = reinterpret_cast<PairGroup*>(lds);
  unsigned (*const out)[64] = reinterpret_cast<unsigned (*)[64]>(lds + kPairOutOffset);
  nflex_tok = __builtin_amdgcn_readfirstlane(nflex_tok);
  const int nb = (nflex_tok + kPairBatch - 1) / kPairBatch;
  int pi, pj;
  if (wave == 1 || wave == 2) {
    // ---- producers: lane (s, e): token s of eight, expert e; then lane (h, p): pair p of tokens
    // 4 h .. 4 h + 3 -----------------------------------------------------------------------
    lane_pair(lane & 31, pi, pj);
    const int pw = wave - 1;
    const int lin_e = __builtin_amdgcn_ds_bpermute(4 * (lane & 7), lin);
    const int at_i = 128 * (lane >> 5) + 4 * pi, at_j = 128 * (lane >> 5) + 4 * pj;
    int slot[kPairLoads], base[kPairLoads];
    unsigned rec[kPairLoads];
    auto first = [&](int n, int r) { return n * kPairBatch + kPairBatch / 2 * pw + 8 * r; };
    auto load_slots = [&](int n) {
#pragma unroll
      for (int r = 0; r < kPairLoads; ++r) slot[r] = lag_slot(first(n, r) + (lane >> 3), nflex_tok, ws);
    };
    auto load_records = [&]() {
#pragma unroll
      for (int r = 0; r < kPairLoads; ++r) {
        rec[r] = ws.rec_lane[(size_t)slot[r] * 8 + (lane & 7)];
        base[r] = ws.tile_base[(size_t)(slot[r] >> 6) * 64 + (lane & 7)];
      }
    };
    int buf = 0;  // of batch n
    auto fill = [&](int n) {
      PairGroup* dst = ring + buf * kPairGroups + kPairGroups / 2 * pw + (lane >> 5);
      buf = buf == 2 ? 0 : buf + 1;
#pragma unroll
      for (int r = 0; r < kPairLoads; ++r) {
        // (counter << 3) + rank, below 2^30; who is no candidate is as far behind that as the choices
        // can differ.  (Tokens behind the last one: whatever comes out, their bits are not taken)
        const int key = rec[r] != 0xFFFFu ? ((lin_e + base[r] + (int)(rec[r] >> 4)) << 3) + (int)(rec[r] & 7u) : 0x7FFFFFF8;
        int u[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int ki = __builtin_amdgcn_ds_bpermute(at_i + 32 * q, key);
          const int kj = __builtin_amdgcn_ds_bpermute(at_j + 32 * q, key);
          u[q] = (ki + ~kj) >> 3;  // kj + 8 G[j] < ki + 8 G[i]
        }
        dst[2 * r].v[lane & 31] = make_int4(u[0], u[1], u[2], u[3]);
      }
    };
    load_slots(0);
    load_records();
    load_slots(1);
    fill(0);
    load_records();
    load_slots(2);
    fill(1);
    load_records();
    load_slots(3);
    lds_barrier();
    for (int n = 0; n < nb; ++n) {
      fill(n + 2);  // (behind the last batch: not used)
      load_records();
      load_slots(n + 4);
      lds_barrier();
    }
  } else if (wave == 3) {
    // ---- output: the words that the consumer has left of a batch (lane = expert; the first token's
    // bit is the highest, and set where the expert is not chosen) -----------------------------
    int before = 0;
    auto put_out = [&](int n) {
#pragma unroll
      for (int u = 0; u < kPairWords; ++u) {
        const int w = n * kPairWords + u, left = nflex_tok - 32 * w;
        if (left <= 0) break;
        const unsigned all = ~out[(n & 1) * kPairWords + u][(28 + lane) & 63];
        const unsigned word = lane < 8 ? __builtin_bitreverse32(all) & (left < 32 ? (1u << left) - 1u : ~0u) : 0u;
        before += __builtin_popcount(word);
        ws.chain_bits[(size_t)w * 64 + lane] = word;
        if (left >= 32) ws.chain_cum[(size_t)(w + 1) * 64 + lane] = before;
      }
    };
    lds_barrier();
    for (int n = 0; n < nb; ++n) {
      if (n > 0) put_out(n - 1);
      lds_barrier();
    }
    put_out(nb - 1);
  } else {
    // ---- consumer ----------------------------------------------------------------------
    lane_pair(lane, pi, pj);
    int D = 0, T = 0, G = 0;  // (G: of the output lane's expert)
    const bool output = lane >= 28 && lane < 36;
    const PairCount count_i = pair_count(output ? lane - 28 : pi, pi, pj, lane);
    PairCount count_j = pair_count(pj, pi, pj, lane);
    if (output) count_j = {0u, 0u};  // (fewer than k: T is 0 where the expert is chosen, else 1)
    const int shift = output ? 1 : 0;
    const int minus_k = -k;
    // (in assembly for the order, see chain_walk_lag; the counts are negative where the expert is
    // chosen: byte 3 is the sign)
#define LASER_PAIR_STEP(U_NEXT_)                                                               \
  "v_cmp_le_i32 vcc, %[T], %[V]\n\t"                                                          \
  "v_lshl_add_u32 %[D], %[D], %[shift], %[T]\n\t"                                             \
  "v_sub_u32 %[V], " U_NEXT_ ", %[D]\n\t"                                                     \
  "v_bitop3_b32 %[ci], %[fi], %[mi], vcc_lo bitop3:0x48\n\t" /* (pairs ^ flip) & mask */      \
  "v_bitop3_b32 %[cj], %[fj], %[mj], vcc_lo bitop3:0x48\n\t"                                  \
  "v_bcnt_u32_b32 %[ci], %[ci], %[mk]\n\t"                                                    \
  "v_bcnt_u32_b32 %[cj], %[cj], %[mk]\n\t"                                                    \
  "v_sub_u32_sdwa %[T], sext(%[ci]), sext(%[cj]) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:BYTE_3\n\t"
    int V;
    auto steps = [&](const int4& x, int next) {
      int ci, cj;
      asm(LASER_PAIR_STEP("%[x1]") LASER_PAIR_STEP("%[x2]") LASER_PAIR_STEP("%[x3]") LASER_PAIR_STEP("%[x4]")
          : [D] "+v"(D), [T] "+v"(T), [V] "+v"(V), [ci] "=&v"(ci), [cj] "=&v"(cj)
          : [x1] "v"(x.y), [x2] "v"(x.z), [x3] "v"(x.w), [x4] "v"(next), [fi] "v"(count_i.flip), [mi] "v"(count_i.mask),
            [fj] "v"(count_j.flip), [mj] "v"(count_j.mask), [mk] "s"(minus_k), [shift] "v"(shift)
          : "vcc");
    };
#undef LASER_PAIR_STEP
    lds_barrier();
    const PairGroup* cur = ring;
    int4 x = cur[0].v[lane & 31], x_1 = cur[1].v[lane & 31];
    V = x.x;
    unsigned all = 0;
    for (int n = 0; n < nb; ++n) {
      const int words = min(kPairWords, (nflex_tok - n * kPairBatch + 31) >> 5);
      for (int u = 0; u < words; ++u) {
        const PairGroup* const next = cur + 8 == ring + 3 * kPairGroups ? ring : cur + 8;
#pragma unroll
        for (int g = 0; g < 8; ++g) {
          // (behind the call's last token: read and not used)
          const int4 x_2 = g < 6 ? cur[g + 2].v[lane & 31] : next[g - 6].v[lane & 31];
          __builtin_amdgcn_sched_barrier(0);
          steps(x, x_1.x);
          __builtin_amdgcn_sched_barrier(0);
          x = x_1;
          x_1 = x_2;
        }
        cur = next;
        all = ((unsigned)D << 1) + (unsigned)T;  // (the last token's T is not in D yet)
        out[(n & 1) * kPairWords + u][lane] = all;
        G += 32 - __builtin_popcount(all);
      }
      lds_barrier();
    }
    // (the bits behind the call's last token do not count)
    G -= __builtin_popcount(~all & ((1u << (-nflex_tok & 31)) - 1u));
    gflex = __builtin_amdgcn_ds_bpermute(4 * (28 + (lane & 7)), G);
    gflex = lane < 8 ? gflex : 0;
  }
}

// ------------------------------------------------ window evaluation of the chain ----
//
// The sequential walk above costs one dependent step per flexible token.  Where
// consecutive flexible tokens rarely compete for the same experts at nearly equal
// loads, most of them can be decided side by side.  Wave 0 holds a window of 64
// consecutive flexible tokens, one per lane, each with a tentative choice.  A sweep
// re-decides every token of the window against
//     counters before the window  +  tentative choices of the window tokens before it,
// all lanes at once.  If q is the first token whose choice changed in a sweep, the new
// choices of tokens 0..q are final: each was computed from choices that did not change,
// hence from final ones (induction from the window head, whose inputs are all final).
// They leave the window, the next tokens enter with an empty tentative choice.  The
// result is the sequential one exactly, whatever the order of evaluation.  If too few
// tokens retire per sweep, the workgroup goes over to the sequential walk for the rest.
//
// Lane = token side: candidates by rank (ids), their counters without any flexible
// choice (b: loads_in + fixed prefix of the tile + fixed tokens before it inside the
// tile), tentative choice as a bit mask over ranks.  Lane = expert side, in LDS: the
// window lanes that tentatively chose the expert (64-bit mask) and the final
// flexible choices so far (G).  Lane l holds the token f of the window with
// f % 64 == l, so nothing moves when the window advances.
//
// Waves 1 to 3 prepare the per-token data two segments ahead in an LDS ring; the
// workgroup meets at a barrier once per segment of 192 tokens.

constexpr int kSpecSeg = 192;                 // tokens per segment (64 per producer wave)
constexpr int kSpecRing = 3 * kSpecSeg;       // tokens in the LDS ring
constexpr unsigned kSpecInvalid = 1u << 27;   // counter of a rank beyond the working set
constexpr int kSpecMinTokens = 256;           // fewer flexible tokens: sequential walk
constexpr int kSpecCheckSweeps = 8;           // progress is judged over this many sweeps
// Window of 64, up to 8 candidates.  Break-even with the walk: a sweep costs 0.56 / 0.9 us for 4 / 8
// candidates, a step of the walk 0.052, so 10.8 / 17.3 tokens per sweep.  It is given up when a run of
// sweeps is below that and the sweeps so far have cost more than walking their tokens -- if the run
// retired at least half of break-even, more by a walk over an eighth of the tokens that are left.
// The first sweeps, of tokens that all come in without a choice, mostly also at counters that are
// still equal, are not judged.  (16384 tokens, all load-dependent, 9 to 31 experts: 310..470 us in windows
// where no tokens compete, 850 walked; where they do, 860 with the attempt.)
constexpr int spec_break_even(int cp) { return cp <= 4 ? 88 : 140; }  // per kSpecCheckSweeps
constexpr int kSpecWarmUp = 4;
// Window of 64, up to 16 candidates: fewer than this many tokens in the last run of sweeps, and in all of
// them on the average.
constexpr int kSpecMinProgress = 56;  // per kSpecCheckSweeps

template <int CP>
struct SpecTok {
  uint4 ids;       // candidate experts by rank, one byte each
  unsigned b[CP];  // their counters without flexible choices
};
struct __align__(16) SpecExp {
  unsigned long long mask;  // window lanes that tentatively chose the expert
  int G;                    // final flexible choices of the expert so far
  int pad;
};
static_assert(kSpecRing * (int)sizeof(SpecTok<16>) <= kChainLdsBytes, "ring must fit the chain LDS");

template <int N>
__device__ __forceinline__ void sort_ascending_u32(unsigned (&K)[N]) {
  constexpr SortNet<N> net = make_sort_net<N>();
#pragma unroll
  for (int i = 0; i < net.n; ++i) {
    const unsigned lo = min(K[net.a[i]], K[net.b[i]]), hi = max(K[net.a[i]], K[net.b[i]]);
    K[net.a[i]] = lo;
    K[net.b[i]] = hi;
  }
}

// Bit mask over the CP key slots (slot = low 4 bits of a key) of the K smallest keys.
// With K known: a partial network that finds the min(K, CP - K) extreme keys by merging
// sorted pairs, quads, ... and keeping only that many per group; the keys are distinct.
template <int N, int M, bool LARGEST>
__device__ __forceinline__ void extreme_keys(const unsigned (&K)[N], unsigned (&out)[M]) {
  // groups of G keys, each reduced to its M' = min(G, M) extreme keys, sorted (most
  // extreme first); G doubles every round
  unsigned cur[N];
#pragma unroll
  for (int i = 0; i < N; ++i) cur[i] = K[i];
  auto better = [](unsigned x, unsigned y) { return LARGEST ? max(x, y) : min(x, y); };
  auto worse = [](unsigned x, unsigned y) { return LARGEST ? min(x, y) : max(x, y); };
  static_assert(M == 1 || M == 2, "at most two extreme keys");
  if (M == 1) {
#pragma unroll
    for (int g = 1; g < N; g *= 2)
#pragma unroll
      for (int i = 0; i + g < N; i += 2 * g) cur[i] = better(cur[i], cur[i + g]);
    out[0] = cur[0];
  } else {
    // pairs: (first, second)
#pragma unroll
    for (int i = 0; i < N; i += 2) {
      const unsigned a = better(cur[i], cur[i + 1]), b = worse(cur[i], cur[i + 1]);
      cur[i] = a;
      cur[i + 1] = b;
    }
#pragma unroll
    for (int g = 2; g < N; g *= 2)
#pragma unroll
      for (int i = 0; i + g < N; i += 2 * g) {
        const unsigned a0 = cur[i], b0 = cur[i + 1], a1 = cur[i + g], b1 = cur[i + g + 1];
        cur[i] = better(a0, a1);
        cur[i + 1] = better(worse(a0, a1), better(b0, b1));
      }
    out[0] = cur[0];
    out[1] = cur[1];
  }
}

template <int CP, int KK>
__device__ __forceinline__ unsigned smallest_k_slots(unsigned (&key)[CP], int k) {
  unsigned sel = 0;
  if (KK > 0 && KK <= 2 && KK < CP) {
    unsigned ext[KK > 0 && KK <= 2 ? KK : 1];
    extreme_keys<CP, (KK > 0 && KK <= 2 ? KK : 1), false>(key, ext);
#pragma unroll
    for (int i = 0; i < KK; ++i) sel |= 1u << (ext[i < 2 ? i : 0] & 15u);
  } else if (KK > 0 && CP - KK >= 1 && CP - KK <= 2) {
    constexpr int D = (KK > 0 && CP - KK >= 1 && CP - KK <= 2) ? CP - KK : 1;
    unsigned ext[D];
    extreme_keys<CP, D, true>(key, ext);
    sel = (1u << CP) - 1u;
#pragma unroll
    for (int i = 0; i < D; ++i) sel &= ~(1u << (ext[i] & 15u));
  } else {
    sort_ascending_u32<CP>(key);
#pragma unroll
    for (int i = 0; i < CP; ++i)
      if (i < k) sel |= 1u << (key[i] & 15u);
  }
  return sel;
}

__device__ __forceinline__ unsigned long long rotl64(unsigned long long x, int s) {  // s in [0, 63]
  return s ? (x << s) | (x >> (64 - s)) : x;
}
__device__ __forceinline__ unsigned long long rotr64(unsigned long long x, int s) {
  return s ? (x >> s) | (x << (64 - s)) : x;
}

// Producer: tokens seg*192 + half*64 + lane of the call -> ring (half = 0, 1, 2).
template <int CP, int KK>
__device__ __forceinline__ void spec_fill(SpecTok<CP>* ring, int seg, int half, int nflex_tok, const Workspace& ws,
                          const int* lin_tab, int lane) {
  const int f = seg * kSpecSeg + half * 64 + lane;
  if (f >= nflex_tok) return;
  const int slot = ws.flex_slot[f];
  const int tile = slot >> 6;
  const uint4 ids = reinterpret_cast<const uint4*>(ws.rec_cids)[slot];
  const uint4 pref = reinterpret_cast<const uint4*>(ws.rec_pref)[slot];
  const unsigned idw[4] = {ids.x, ids.y, ids.z, ids.w};
  const unsigned pfw[4] = {pref.x, pref.y, pref.z, pref.w};
  SpecTok<CP>* dst = &ring[f % kSpecRing];
  dst->ids = ids;
  int base[CP];
#pragma unroll
  for (int j = 0; j < CP; ++j) {
    const int e = (idw[j >> 2] >> (8 * (j & 3))) & 255;
    base[j] = ws.tile_base[(size_t)tile * 64 + e] + lin_tab[e];
  }
#pragma unroll
  for (int j = 0; j < CP; ++j) {
    const unsigned pf = (pfw[j >> 2] >> (8 * (j & 3))) & 255u;
    dst->b[j] = pf == 0xFFu ? kSpecInvalid : (unsigned)base[j] + pf;
  }
}

// Runs the window evaluation from flexible token 0.  All four waves call it.  Returns
// (to every wave) the number of flexible tokens decided, or -1 where somebody else has claimed the
// call (see Race); wave 0 leaves the flexible choices so far in `gflex` (lane = expert), the bits of the
// unfinished output word in `hist` and the number of sweeps in `nsweeps` (a status word where nobody
// else walks the call).  KK = k when known at compile time, else 0.
// LDS of the window evaluation beside the ring (one copy for all compiled variants).
struct SpecShared {
  SpecExp M[64];
  int lin_tab[64];
  int sh_done[2], sh_bail[2];  // by segment parity: written before, read after a barrier
};

template <int CP, int KK, bool RACE>
__device__ __forceinline__ int spec_walk(uint8_t* lds, SpecShared& sp, int nflex_tok, const RouteArgs& a,
                         const Workspace& ws, int wave, int lane, int lin, int& gflex, unsigned& hist, int& nsweeps,
                         Race<RACE> race) {
  own_lane(lane);
  nflex_tok = __builtin_amdgcn_readfirstlane(nflex_tok);
  SpecTok<CP>* ring = reinterpret_cast<SpecTok<CP>*>(lds);
  SpecExp* M = sp.M;
  int* lin_tab = sp.lin_tab;
  int* sh_done = sp.sh_done;
  int* sh_bail = sp.sh_bail;
  const int k = KK > 0 ? KK : a.k;
  if (wave == 0) {
    M[lane].mask = 0ull;
    M[lane].G = 0;
    lin_tab[lane] = lin;
  }
  __syncthreads();
  const bool producer = wave != 0;
  if (producer) {
    spec_fill<CP, KK>(ring, 0, wave - 1, nflex_tok, ws, lin_tab, lane);
    spec_fill<CP, KK>(ring, 1, wave - 1, nflex_tok, ws, lin_tab, lane);
  }
  __syncthreads();

  // consumer state (wave 0)
  int ex[CP];       // candidate experts by rank
  unsigned b[CP];   // their counters without flexible choices
#pragma unroll
  for (int j = 0; j < CP; ++j) {
    ex[j] = 0;
    b[j] = kSpecInvalid;
  }
  unsigned sel = 0;
  int cur_f = -1;                  // token whose data this lane holds
  int ridx = lane - 64;            // its place in the ring (advances by 64 per token)
  int done = 0;                    // tokens decided (uniform)
  int G = 0;                       // lane = expert: final flexible choices
  unsigned long long pend = 0ull;  // lane = expert: decided bits not yet written, from token 32*w
  int pn = 0, w = 0, gflushed = 0;
  int sweeps = 0, done_mark = 0, total_sweeps = 0;
  bool bail = false, stop = false;
  int decided = 0;
  const unsigned long long lb = lanes_below(lane);

  int answer = RACE && !producer ? race.ask() : 0;
  const int nep = (nflex_tok + kSpecSeg - 1) / kSpecSeg;
  for (int ep = 0; ep < nep; ++ep) {
    if (producer) {
      spec_fill<CP, KK>(ring, ep + 2, wave - 1, nflex_tok, ws, lin_tab, lane);
    } else {
      const int avail = min(nflex_tok, (ep + 2) * kSpecSeg);
      const int target = min(nflex_tok, (ep + 1) * kSpecSeg);
      while (done < target && !bail) {
        if (RACE && race.on() && (total_sweeps & 3) == 3) {  // (every two to four microseconds)
          stop = __builtin_amdgcn_readfirstlane(answer) != 0;
          answer = race.ask();
          if (stop) break;
        }
        const int head = done & 63;
        // this lane's token of the window [done, done + 64)
        const int f_lane = done + ((lane - head) & 63);
        const bool enters = f_lane < avail && cur_f != f_lane;
        if (enters) {
          ridx += 64;
          ridx = ridx >= kSpecRing ? ridx - kSpecRing : ridx;
          const SpecTok<CP>* src = &ring[ridx];
          const uint4 ids = src->ids;
          const unsigned idw[4] = {ids.x, ids.y, ids.z, ids.w};
          sel = 0;
#pragma unroll
          for (int j = 0; j < CP; ++j) {
            ex[j] = (idw[j >> 2] >> (8 * (j & 3))) & 255;
            b[j] = src->b[j];
          }
          cur_f = f_lane;
        }
        const bool valid = cur_f == f_lane;
        if (!valid) sel = 0;
        const unsigned long long hb = lanes_below(head);
        const unsigned long long earlier = lane >= head ? (lb & ~hb) : (~hb | lb);
        unsigned key[CP];
#pragma unroll
        for (int j = 0; j < CP; ++j) {
          const uint4 m = *reinterpret_cast<const uint4*>(&M[ex[j]]);  // mask lo, hi, G, -
          const unsigned cnt = (unsigned)(__builtin_popcount(m.x & (unsigned)earlier) +
                                          __builtin_popcount(m.y & (unsigned)(earlier >> 32)));
          key[j] = ((b[j] + m.z + cnt) << 4) | (unsigned)j;
        }
        unsigned newsel = smallest_k_slots<CP, KK>(key, k);
        newsel = valid ? newsel : 0u;
        const unsigned diff = sel ^ newsel;
        const unsigned long long bal = __builtin_amdgcn_ballot_w64(diff != 0u);
        if (bal != 0ull) {
          // flip this lane's bit in the masks of the experts whose choice changed
#pragma unroll
          for (int j = 0; j < CP; ++j)
            if ((diff >> j) & 1u) flip_lane_bit(&M[ex[j]].mask, lane);
        }
        sel = newsel;
        // tokens up to the first changed one are final
        const unsigned long long rot = rotr64(bal, head);
        const int q = rot ? __builtin_ctzll(rot) : 64;
        // (more than 32 is rare: a token needs a sweep to get a choice)
        const int fin = min(min(q + 1, avail - done), 32);
        lds_wave_fence();
        __builtin_amdgcn_wave_barrier();
        {  // lane = expert
          unsigned long long mk = M[lane].mask;
          const unsigned long long finmask = rotl64((1ull << fin) - 1ull, head);
          const unsigned long long fbits = mk & finmask;
          G += __builtin_popcountll(fbits);
          mk &= ~finmask;
          const unsigned ob = (unsigned)rotr64(fbits, head);  // bit i: token done + i
          pend |= (unsigned long long)ob << pn;               // pn < 32 bits were held
          pn += fin;
          if (pn >= 32) {
            const unsigned word = (unsigned)pend;
            gflushed += __builtin_popcount(word);
            ws.chain_bits[(size_t)w * 64 + lane] = word;
            ws.chain_cum[(size_t)(w + 1) * 64 + lane] = gflushed;
            pend >>= 32;
            pn -= 32;
            ++w;
          }
          M[lane].mask = mk;
          M[lane].G = G;
        }
        lds_wave_fence();
        __builtin_amdgcn_wave_barrier();
        done += fin;
        ++total_sweeps;
        if (CP <= 8 && total_sweeps == kSpecWarmUp) {
          sweeps = 0;
          done_mark = done;
        } else if (++sweeps == kSpecCheckSweeps) {
          // (the switch is one-way)
          const int progress = done - done_mark, left = nflex_tok - done;
          if (CP <= 8) {
            constexpr int line = spec_break_even(CP);
            const int lost = total_sweeps * line / kSpecCheckSweeps - done;  // in tokens walked
            if (left > 64 && progress < line && lost > (progress < line / 2 ? 0 : left / 8)) bail = true;
          } else if (progress < kSpecMinProgress && done * kSpecCheckSweeps < kSpecMinProgress * total_sweeps &&
                     left > 2 * kSpecSeg) {
            bail = true;
          }
          sweeps = 0;
          done_mark = done;
        }
      }
      if (lane == 0) {
        sh_done[ep & 1] = done;
        sh_bail[ep & 1] = stop ? 2 : bail ? 1 : 0;
      }
    }
    __syncthreads();
    decided = __builtin_amdgcn_readfirstlane(sh_done[ep & 1]);
    const int why = __builtin_amdgcn_readfirstlane(sh_bail[ep & 1]);
    if (RACE && why == 2) return -1;
    if (why != 0) break;
  }
  if (wave == 0) {
    gflex = G;
    hist = (unsigned)pend;  // the decided % 32 bits of the unfinished word
    if (decided == nflex_tok && pn > 0) ws.chain_bits[(size_t)w * 64 + lane] = (unsigned)pend;
    if constexpr (RACE)
      nsweeps = total_sweeps;
    else if (lane == 0)
      ws.status[kStatusSweeps] = total_sweeps;
  }
  __syncthreads();  // the ring is dead: the sequential walk may reuse the LDS
  return decided;
}

// ---- window of 256 tokens, four wavefronts -----------------------------------------------
//
// Where tokens rarely compete (many experts behind each candidate) a sweep retires most of its
// window, so a wide window decides more tokens for the same chain of dependent steps.  The four
// wavefronts hold 64 of the 256 window positions each (position = flexible token number mod 256; wave =
// position / 64, lane = position mod 64) and evaluate them as above.  A wave owns the masks of its
// positions; what the tokens of the other waves chose enters as one number per expert, summed up
// once per sweep, so an evaluation costs as much as in the window of 64.
//
// A sweep:
//   count     lane = expert: the masks of all waves, for the wave's own tokens the choices before them
//   evaluate  lane = token
//   -- barrier: every wave finds the same first changed token --
//   retire    lane = expert: the choices up to that token are final, its own being the new one
//   enter     lane = token: the next tokens, with the choice by the counters as they stand as first
//             guess (any guess gives the same result); the choices of the wave's tokens become its masks,
//             in the other of two copies (the other waves still read this one)
//   stage     a token per thread goes to a ring in LDS, the three dependent loads of a token (its slot, its
//             record, the counters of its candidates) spread over three sweeps so that none is waited for
//   -- barrier --
// Decided bits go to a small ring of output words in LDS; wave 3 writes out the words that are complete.
// What bounds it: 1.5 / 2.0 / 2.8 us per sweep (4 / 8 / 16 candidates), about 450 instructions, two barriers
// and, where tokens are staged, their scattered loads.
// (Before: a window of 128 with two wavefronts that staged tokens and two that evaluated against
// both masks: 1.65 us per sweep.  12345 tokens, 1214 of them load-dependent: 18 sweeps, 29 us, now 10
// sweeps, 22 us; a prefill of 131072 tokens, 13150 load-dependent, the call 317 -> 286 us.)
constexpr int kWinTokens = 256;

// 64 x 64 bits, a row (lo, hi) per lane -> a column per lane.  Blocks of 32, 16, ... 1 bits change places
// with those of the lane 32, 16, ... 1 away: no LDS, about 40 instructions, and as fast as
// LDS atomics, a bit per chosen expert, that then need no second copy of the choices.
struct Transpose64 {
  unsigned pick16, pick8, mask4, mask2, mask1;
  int rot4, rot2, rot1;
  __device__ __forceinline__ explicit Transpose64(int lane)
      : pick16((lane & 16) ? 0x07060302u : 0x05040100u),
        pick8((lane & 8) ? 0x03070105u : 0x06020400u),
        mask4((lane & 4) ? 0xF0F0F0F0u : 0x0F0F0F0Fu),
        mask2((lane & 2) ? 0xCCCCCCCCu : 0x33333333u),
        mask1((lane & 1) ? 0xAAAAAAAAu : 0x55555555u),
        rot4((lane & 4) ? 4 : 28),
        rot2((lane & 2) ? 2 : 30),
        rot1((lane & 1) ? 1 : 31) {}
  __device__ __forceinline__ unsigned within32(unsigned x) const {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    constexpr int kRowRor8 = 0x128, kQuadReverse = 3 | (2 << 2) | (1 << 4) | (0 << 6);
    const u32x2 p = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = __builtin_amdgcn_perm(p[1], p[0], pick16);
    x = __builtin_amdgcn_perm((unsigned)dpp_int<kRowRor8>((int)x), x, pick8);
    auto merge = [](unsigned x, unsigned other, unsigned mask, int rot) {
      return (x & mask) | (__builtin_amdgcn_alignbit(other, other, rot) & ~mask);
    };
    x = merge(x, (unsigned)dpp_int<kQuadReverse>(dpp_int<kRowHalfMirror>((int)x)), mask4, rot4);
    x = merge(x, (unsigned)dpp_int<kQuadXor2>((int)x), mask2, rot2);
    return merge(x, (unsigned)dpp_int<kQuadXor1>((int)x), mask1, rot1);
  }
  __device__ __forceinline__ unsigned long long operator()(unsigned long long row) const {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 p = __builtin_amdgcn_permlane32_swap((unsigned)row, (unsigned)(row >> 32), false, false);
    return ((unsigned long long)within32(p[1]) << 32) | within32(p[0]);
  }
};

// Given up where the walk is faster, judged as in the window of 64: a sweep costs as much as 28, 38 and 21
// steps of the walk with up to 4, 8 and 16 candidates; the lines are lower, because the first sweeps
// of a call, and those that end it, retire less than the others.
constexpr int win_break_even(int cp) { return cp <= 4 ? 190 : cp <= 8 ? 230 : 130; }  // per kSpecCheckSweeps
constexpr int win_ring(int cp) { return cp <= 8 ? 768 : 512; }                        // tokens in the LDS ring
constexpr int kWinWords = 16;                                                         // output ring

template <int CP>
struct WinShared {
  uint4 b[CP / 4][win_ring(CP)];       // counters of the candidates without flexible choices
  unsigned ids[win_ring(CP)][CP / 4];  // their experts, a byte each
  uint4 chose[2][kChainWaves][64];     // [copy][wave][expert] positions that tentatively chose it (x, y), and
                                       // choices that became final in the sweep before (z)
  uint4 count[kChainWaves][64];        // [wave][expert] its positions, choices before the wave's positions, and
                                       // before those behind the end of the ring
  unsigned out[kWinWords][64];         // per expert: chosen bits of 32 flexible tokens, not yet written out
  int4 changed[2];                     // [copy] per wave: the first token that changed, from the window's head on
  unsigned long long first[2][kChainWaves];  // [copy][wave] experts that token chooses now
};
static_assert(sizeof(WinShared<4>) <= kChainLdsBytes && sizeof(WinShared<8>) <= kChainLdsBytes &&
                  sizeof(WinShared<16>) <= kChainLdsBytes,
              "ring and state fit the chain LDS");

// What a thread has under way of the tokens it stages.
template <int CP>
struct WinStage {
  int base[CP];                         // of the next token to be staged: assignments in the tiles before its tile
  unsigned ids[CP / 4], pref[CP / 4];   // ... its candidates
  unsigned ids1[CP / 4], pref1[CP / 4]; // of the one behind that
  int slot, slot1, slot2;               // of all three
};
template <int CP>
__device__ __forceinline__ void win_records(unsigned (&ids)[CP / 4], unsigned (&pref)[CP / 4], int slot,
                                            const Workspace& ws) {
#pragma unroll
  for (int i = 0; i < CP / 4; ++i) {
    ids[i] = reinterpret_cast<const unsigned*>(ws.rec_cids)[(size_t)slot * 4 + i];
    pref[i] = reinterpret_cast<const unsigned*>(ws.rec_pref)[(size_t)slot * 4 + i];
  }
}
template <int CP>
__device__ __forceinline__ void win_counters(int (&base)[CP], const unsigned (&ids)[CP / 4], int slot,
                                             const Workspace& ws) {
#pragma unroll
  for (int j = 0; j < CP; ++j)
    base[j] = ws.tile_base[(size_t)(slot >> 6) * 64 + ((ids[j >> 2] >> (8 * (j & 3))) & 255u)];
}

// The positions before x (0..64) of a wave.
__device__ __forceinline__ unsigned long long below64(int x) { return x >= 64 ? ~0ull : (1ull << x) - 1ull; }

// Runs the window evaluation from flexible token 0 (see spec_walk for the contract).
template <int CP, int KK, bool RACE>
__device__ __forceinline__ int window_walk(uint8_t* lds, int nflex_tok, const RouteArgs& a, const Workspace& ws,
                                           int wave, int lane, int lin, int& gflex, unsigned& hist, int& nsweeps,
                                           Race<RACE> race) {
  own_lane(lane);
  nflex_tok = __builtin_amdgcn_readfirstlane(nflex_tok);
  WinShared<CP>& S = *reinterpret_cast<WinShared<CP>*>(lds);
  constexpr int kRing = win_ring(CP);
  const int k = KK > 0 ? KK : a.k;
  const int tid = 64 * wave + lane;
  const unsigned long long lb = lanes_below(lane);
  const Transpose64 transpose(lane);
  int G = 0;               // lane = expert: final flexible choices, as of the sweep before
  // tokens decided, in the ring, and of these not behind the window (as all that decides the course: the
  // same in every wave)
  int done = 0, avail = 0, inside = 0;
  int sweeps = 0, done_mark = 0, total_sweeps = 0;
  bool bail = false;
  int wout = 0, gflushed = 0;  // wave 3, lane = expert: output words written, their bits so far

  // ---- staging ------------------------------------------------------------------------------
  // (loads without conditions stay in flight: the last token stands in for none)
  WinStage<CP> st;
  int nb = 0, at = tid;  // tokens 256 nb + tid are staged next, at this place of the ring
  auto slot_of = [&](int n) { return ws.flex_slot[min(kWinTokens * n + tid, nflex_tok - 1)]; };
  auto stage = [&]() {
    unsigned b[CP];
#pragma unroll
    for (int j = 0; j < CP; ++j) {
      const int e = (int)((st.ids[j >> 2] >> (8 * (j & 3))) & 255u);
      const unsigned pf = (st.pref[j >> 2] >> (8 * (j & 3))) & 255u;
      const unsigned before = (unsigned)(st.base[j] + __builtin_amdgcn_ds_bpermute(4 * e, lin)) + pf;
      b[j] = pf == 0xFFu ? kSpecInvalid : before;
    }
#pragma unroll
    for (int i = 0; i < CP / 4; ++i) {
      S.b[i][at] = make_uint4(b[4 * i], b[4 * i + 1], b[4 * i + 2], b[4 * i + 3]);
      S.ids[at][i] = st.ids[i];
      st.ids[i] = st.ids1[i];
      st.pref[i] = st.pref1[i];
    }
    at = at + kWinTokens >= kRing ? at + kWinTokens - kRing : at + kWinTokens;
    win_counters<CP>(st.base, st.ids, st.slot1, ws);
    win_records<CP>(st.ids1, st.pref1, st.slot2, ws);
    st.slot1 = st.slot2;
    st.slot2 = slot_of(nb + 3);
    ++nb;
  };
  st.slot = slot_of(0);
  st.slot1 = slot_of(1);
  st.slot2 = slot_of(2);
  win_records<CP>(st.ids, st.pref, st.slot, ws);
  win_records<CP>(st.ids1, st.pref1, st.slot1, ws);
  win_counters<CP>(st.base, st.ids, st.slot, ws);
  for (int i = tid; i < kWinWords * 64; i += kTailThreads) (&S.out[0][0])[i] = 0u;
  S.count[wave][lane] = make_uint4(0u, 0u, 0u, 0u);
  stage();
  avail = min(nflex_tok, kWinTokens);
  __syncthreads();

  // ---- the window ---------------------------------------------------------------------------
  unsigned ids[CP / 4];  // candidate experts by rank, a byte each
  unsigned b[CP];        // their counters without flexible choices
  unsigned long long choice = 0ull;  // experts
  int cur_f = tid - kWinTokens;      // token whose data this lane holds ...
  int place = tid - kWinTokens;      // ... and its place in the ring (advances by 256 per token)
#pragma unroll
  for (int j = 0; j < CP; ++j) b[j] = kSpecInvalid;
#pragma unroll
  for (int i = 0; i < CP / 4; ++i) ids[i] = 0u;
  auto ex = [&](int j) { return (int)((ids[j >> 2] >> (8 * (j & 3))) & 255u); };
  auto experts = [&](unsigned sel) {
    unsigned long long m = 0ull;
#pragma unroll
    for (int j = 0; j < CP; ++j) m |= (unsigned long long)((sel >> j) & 1u) << (ex(j) & 63);
    return m;
  };
  // The tokens of the window [done, done + 256) that are not in it yet; the wave's masks, and what it
  // retired, to copy `to`.
  auto enter = [&](int to, int retired) {
    const int f = done + ((tid - done) & (kWinTokens - 1));
    if (cur_f != f) choice = 0ull;
    if (f < avail && cur_f != f) {
      cur_f = f;
      place = place + kWinTokens >= kRing ? place + kWinTokens - kRing : place + kWinTokens;
      unsigned key[CP];
#pragma unroll
      for (int i = 0; i < CP / 4; ++i) {
        const uint4 bb = S.b[i][place];
        ids[i] = S.ids[place][i];
        b[4 * i] = bb.x;
        b[4 * i + 1] = bb.y;
        b[4 * i + 2] = bb.z;
        b[4 * i + 3] = bb.w;
      }
#pragma unroll
      for (int j = 0; j < CP; ++j) key[j] = ((b[j] + S.count[wave][ex(j)].w) << 4) | (unsigned)j;
      choice = experts(smallest_k_slots<CP, KK>(key, k));
    }
    const unsigned long long m = transpose(choice);
    S.chose[to][wave][lane] = make_uint4((unsigned)m, (unsigned)(m >> 32), (unsigned)retired, 0u);
  };
  int par = 0;
  int answer = RACE && wave == kChainWaves - 1 ? race.ask() : 0;
  enter(0, 0);
  inside = avail;
  lds_barrier();
  for (;;) {
    const int head = done & (kWinTokens - 1), hw = head >> 6, ho = head & 63;
    unsigned long long own = 0ull;  // lane = expert: the wave's positions that tentatively chose it
    {  // ---- count: lane = expert
      int before = 0, wrap = 0;
#pragma unroll
      for (int i = 0; i < kChainWaves; ++i) {
        // (in the order of the window: the head's wave from the head on, the others)
        const int w = (hw + i) & (kChainWaves - 1);
        const uint4 x = S.chose[par][w][lane];
        const unsigned long long m = ((unsigned long long)x.y << 32) | x.x;
        const int n = __builtin_popcountll(i == 0 ? m & ~below64(ho) : m);
        if (w == wave) own = m;
        if (i < ((wave - hw) & (kChainWaves - 1))) before += n;
        wrap += n;
        G += (int)x.z;
      }
      S.count[wave][lane] = make_uint4((unsigned)own, (unsigned)(own >> 32), (unsigned)(G + before), (unsigned)(G + wrap));
    }
    if (done >= nflex_tok || bail) break;
    lds_wave_fence();
    __builtin_amdgcn_wave_barrier();
    // ---- evaluate: lane = token
    {
      const bool behind = wave == hw && lane < ho;  // (behind the end of the ring)
      const unsigned long long earlier = wave == hw && lane >= ho ? lb & ~below64(ho) : lb;
      unsigned key[CP];
#pragma unroll
      for (int j = 0; j < CP; ++j) {
        const uint4 m = S.count[wave][ex(j)];
        const unsigned cnt = (unsigned)(__builtin_popcount(m.x & (unsigned)earlier) +
                                        __builtin_popcount(m.y & (unsigned)(earlier >> 32)));
        key[j] = ((b[j] + (behind ? m.w : m.z) + cnt) << 4) | (unsigned)j;
      }
      unsigned long long now = experts(smallest_k_slots<CP, KK>(key, k));
      now = cur_f >= done ? now : 0ull;
      const unsigned long long bal = __builtin_amdgcn_ballot_w64(now != choice);
      choice = now;
      const unsigned long long head_part = wave == hw ? bal & ~below64(ho) : bal;
      const unsigned long long c = head_part != 0ull ? head_part : bal;
      const int pos = c != 0ull ? __builtin_ctzll(c) : 0;
      const unsigned lo = __builtin_amdgcn_readlane((unsigned)choice, pos);
      const unsigned hi = __builtin_amdgcn_readlane((unsigned)(choice >> 32), pos);
      if (lane == 0) {
        reinterpret_cast<int*>(&S.changed[par])[wave] =
            c != 0ull ? (64 * wave + pos - head) & (kWinTokens - 1) : kWinTokens;
        S.first[par][wave] = ((unsigned long long)hi << 32) | lo;
      }
    }
    lds_barrier();
    // ---- retire: tokens up to the first changed one are final (every wave works it out)
    const int4 cq = S.changed[par];
    const int q = __builtin_amdgcn_readfirstlane(min(min(cq.x, cq.y), min(cq.z, cq.w)));
    const int fin = min(min(q + 1, kWinTokens), inside - done);
    int retired;
    {  // lane = expert
      // the wave's positions among head .. head + fin - 1, cyclically
      const int from = head - 64 * wave, to = from + fin;
      const unsigned long long ret =
          (below64(min(max(to, 0), 64)) & ~below64(min(max(from, 0), 64))) | below64(min(max(to - kWinTokens, 0), 64));
      unsigned long long mine = own & ret;
      const int qpos = head + q;
      if (q < fin && ((qpos >> 6) & (kChainWaves - 1)) == wave) {
        // (the changed token's bits are the old ones in the mask: it goes by its new choice)
        const unsigned long long bit = 1ull << (qpos & 63);
        mine = (S.first[par][wave] >> lane) & 1ull ? mine | bit : mine & ~bit;
      }
      retired = __builtin_popcountll(mine);
      // 32 positions are bit-aligned with the output word of their tokens; only those around the
      // head can hold tokens of two words
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int quarter = 2 * wave + h;
        const unsigned bits = (unsigned)(mine >> (32 * h));
        const int cut = (head >> 5) == quarter ? (head & 31) : 0;
        const int word = (done + ((32 * quarter + cut - head) & (kWinTokens - 1))) >> 5;
        const unsigned behind_cut = ~((1u << cut) - 1u);
        S.out[word & (kWinWords - 1)][lane] |= bits & behind_cut;
        if (cut != 0) S.out[(word + kWinTokens / 32) & (kWinWords - 1)][lane] |= bits & ~behind_cut;
      }
    }
    done += fin;
    ++total_sweeps;
    if (total_sweeps == kSpecWarmUp) {
      sweeps = 0;
      done_mark = done;
    } else if (++sweeps == kSpecCheckSweeps) {
      // (the switch is one-way)
      constexpr int line = win_break_even(CP);
      const int progress = done - done_mark, left = nflex_tok - done;
      const int lost = total_sweeps * line / kSpecCheckSweeps - done;  // in tokens walked
      if (left > 64 && progress < line && lost > (progress < line / 2 ? 0 : left / 8)) bail = true;
      sweeps = 0;
      done_mark = done;
    }
    par ^= 1;
    enter(par, retired);
    inside = avail;
    // (a token's place is free once the token has entered the window, which 256 tokens fit)
    if (kWinTokens * nb < nflex_tok && kWinTokens * (nb + 1) <= done + kRing) stage();
    if (RACE && wave == kChainWaves - 1) {
      race.hand_out(answer, lane);
      answer = race.ask();
    }
    lds_barrier();
    if (RACE && race.over()) return -1;
    avail = min(nflex_tok, kWinTokens * nb);
    // ---- output words that are complete (lane = expert) -----------------------------------------
    if (wave == kChainWaves - 1) {
      while (32 * (wout + 1) <= done) {
        unsigned* word = &S.out[wout & (kWinWords - 1)][lane];
        const unsigned bits = *word;
        *word = 0u;
        gflushed += __builtin_popcount(bits);
        ws.chain_bits[(size_t)wout * 64 + lane] = bits;
        ws.chain_cum[(size_t)(wout + 1) * 64 + lane] = gflushed;
        ++wout;
      }
    }
  }
  if (wave == 0) {
    gflex = G;
    hist = (done & 31) != 0 ? S.out[(done >> 5) & (kWinWords - 1)][lane] : 0u;  // the decided bits of the unfinished word
    if (done == nflex_tok && (done & 31) != 0) ws.chain_bits[(size_t)(done >> 5) * 64 + lane] = hist;
    if constexpr (RACE)
      nsweeps = total_sweeps;
    else if (lane == 0)
      ws.status[kStatusSweeps] = total_sweeps;
  }
  __syncthreads();  // (the LDS is free again)
  return done;
}

// ---- the chain in blocks, side by side ---------------------------------------------------
//
// A long chain of load-dependent tokens is cut into blocks of consecutive ones, a workgroup
// each.  A block is walked from a guess of the choices before it, and the guesses are mended
// in rounds until every block has begun where the one before it ended: then, block by block from
// the first (whose beginning is known), all of it is what one walk would have decided.  Nothing
// but that equality, expert by expert, ends the rounds, so the guesses decide about time only;
// every round makes at least one more block final.
//
// Nobody depends on the blocks.  The chain workgroup walks such a call like any other one, the blocks write
// their choices to arrays of their own beside it, and whoever is through first claims the call, writes
// the totals and raises the last flag; the others see the claim and leave.  So a call whose rounds are
// many takes what one walk takes, and one whose blocks are not even on the GPU (other calls', other streams'
// workgroups in the way) waits for none of them: the chain workgroup waits for nobody.
//
// The guess.  Block q says where it began (I_q), where it ended (N_q) and how closely its tokens were
// decided.  A correction d_q of I_q moves N_q by A_q d_q, so the correction of the next block is
//     d_(q+1) = A_q d_q + (N_q - I_(q+1)),     d_0 = 0
// (Newton's method for "every block begins where the one before ends").  A_q: an expert whose
// counter is far from those it is compared with keeps a correction; experts whose counters are
// level with one another forget it, because whoever is ahead is passed over until it is not, and only
// what all of them got together stays.  With g_e in [0, 1] for how far expert e is of the second kind,
//     (A d)_e = (1 - g_e) d_e + g_e (sum_i g_i d_i) / (sum_i g_i).
// g comes from a sample of the block's tokens: how often the expert was chosen or passed over with at
// most one to spare.
// (Rounds until 16384 load-dependent tokens of 64 experts are decided, k = 6, c = 8, blocks of 256: 6 to 12 where
// the gate is skewed and the counters begin at zero, without A 62 to 64 in a simulation; 30 to 42 where
// the counters begin random in 0..2000 or the gate is flat, because several groups of experts are then level
// at heights of their own and A takes them for one.)
// What bounds a round of that call, 20 us: the walk of 256 tokens 15, the sample 1.7, the rows' way
// through memory and what is made of them 3, the correction 1.  The call from logits: 888 us in one piece, 172
// to 238 in 6 to 9 rounds; with c = 10, 2194 and 383; 8192 tokens of 64 candidates, one round, 777 and 70; 3072
// tokens, c = 8, seven rounds, 206 and 132.  Where the chain workgroup is first the blocks cost the call 2 to 9 %,
// and up to 20 % (7 to 37 us) where it is through in windows: they leave between two of their walks
// only, and the kernel ends with them.
constexpr int kChainBlocks = 64;         // blocks of a call, at most
constexpr int kChainBlockMin = 128;      // tokens of a block, at least
// A call is walked in blocks where at least this many of its tokens, and three quarters, are
// load-dependent.  The other tokens' choices set experts apart that the load-dependent ones hardly ever
// compare: blocks forget less of their beginning and the rounds are more.  The line lies where a call of up to 8
// candidates stops gaining (16384 tokens, 64 experts, k = 6, c = 8, skewed gate; in one piece and with blocks
// beside it: no other tokens 888 and 238 us, 10 % of them 808 and 172, 24 % 690 and 694, 26 % 674 and 704, 40 %
// 559 and 587).  Longer calls and more candidates would still gain beyond it (60000 tokens, 26 %: 2325 and 1824;
// c = 10, 26 %: 1632 and 1408; 33 experts, k = 3, c = 9, 26 %: 1630 and 345), which is given away here.
constexpr int kChainBlocksMinTokens = 3072;
__device__ __forceinline__ bool chain_in_blocks(int nflex_tok, int T) {
  return nflex_tok >= kChainBlocksMinTokens && 4ll * nflex_tok >= 3ll * T;
}
constexpr int kBlockSamples = 32;        // tokens of a block that are looked at for g
constexpr int kSamplesPerWave = kBlockSamples / kChainWaves;
constexpr float kForgetHalf = 4.0f;      // close decisions per block that make g one half (2 to 5: the same within 3 %; 8: a sixth more rounds)

// What a block tells the others, per expert: where it began (27 bits), what it added (11), close
// decisions among its samples (6), the round (20; 0: nothing yet, kBlockFinal: it stays so).  Whole
// words travel at once, a row of them that shows one round in all of its words is of one piece.
constexpr unsigned kBlockFinal = 0xFFFFFu;
static_assert(kSelfPrefixTiles * kTile < (1 << 27), "where a block begins, at most a choice per token, fits its field");
static_assert(kSelfPrefixTiles * kTile / kChainBlocks < (1 << 11), "what a block adds fits its field");
__device__ __forceinline__ unsigned long long block_word(int begin, int added, int close, unsigned round) {
  return ((unsigned long long)(unsigned)begin << 37) | ((unsigned long long)(unsigned)added << 26) |
         ((unsigned long long)(unsigned)close << 20) | round;
}
__device__ __forceinline__ unsigned block_round(unsigned long long w) { return (unsigned)w & 0xFFFFFu; }
__device__ __forceinline__ int block_close(unsigned long long w) { return (int)((unsigned)w >> 20) & 63; }
__device__ __forceinline__ int block_added(unsigned long long w) { return (int)(w >> 26) & 2047; }
__device__ __forceinline__ int block_begin(unsigned long long w) { return (int)(w >> 37); }

// The rows stand where the logits were: nothing reads those any more.  Behind the rows of
// all blocks: per expert the assignments of all tokens that are not load-dependent, then how many
// blocks have written out their final choices, and the claim; then the choices of the blocks, as in
// Workspace::chain_bits and chain_cum.
__device__ __forceinline__ unsigned long long* block_rows(const Workspace& ws) {
  return reinterpret_cast<unsigned long long*>(ws.logits);
}
__device__ __forceinline__ int* blocks_done(const Workspace& ws) {
  return reinterpret_cast<int*>(block_rows(ws) + kChainBlocks * 64 + 64);
}
__device__ __forceinline__ int* chain_claim(const Workspace& ws) { return blocks_done(ws) + 1; }
constexpr int kBlockRowsBytes = ((kChainBlocks * 64 + 64 + 1) * 8 + 255) / 256 * 256;
// (the finishing pass reads up to two words beyond that of a token)
__host__ __device__ constexpr size_t block_words(int T) { return (size_t)T / 32 + 3; }
__device__ __forceinline__ uint32_t* block_bits(const Workspace& ws) {
  return reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(ws.logits) + kBlockRowsBytes);
}
__device__ __forceinline__ int32_t* block_cum(const Workspace& ws, int T) {
  return reinterpret_cast<int32_t*>(block_bits(ws)) + block_words(T) * 64;
}
// (9 experts at least; 36 bytes of logits per token, 16 of choices)
static_assert(kBlockRowsBytes + 2 * 64 * 4 * block_words(kChainBlocksMinTokens) <= kChainBlocksMinTokens * 9 * 4,
              "the rows and choices fit the logits");
// (by the chain workgroup, before the first flag; fixed: lane = expert, every wave the same)
__device__ __forceinline__ void clear_block_rows(const Workspace& ws, int T, int lane, int wave, int fixed) {
  unsigned long long* const rows = block_rows(ws);
  for (int i = threadIdx.x; i < kChainBlocks * 64; i += kTailThreads)
    __hip_atomic_store(&rows[i], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (wave == 0) {
    __hip_atomic_store(&rows[kChainBlocks * 64 + lane], (unsigned long long)fixed, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    block_cum(ws, T)[lane] = 0;
  }
  if (threadIdx.x == 0) {
    __hip_atomic_store(blocks_done(ws), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(chain_claim(ws), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}
// (one wavefront) Whether the call is this workgroup's to finish.
__device__ __forceinline__ bool claim_chain(const Workspace& ws, int lane) {
  int before = 0;
  if (lane == 0) before = atomicExch(chain_claim(ws), 1);
  return __builtin_amdgcn_readfirstlane(before) == 0;
}
__device__ __forceinline__ int chain_block_tokens(int nflex_tok) {
  return max(kChainBlockMin, ((nflex_tok + kChainBlocks - 1) / kChainBlocks + 31) & ~31);
}

// Sum over the wavefront, as a scalar: inside the rows of 16 lanes as in wave_min_u32, then along the rows.
__device__ __forceinline__ float wave_sum(float v) {
  constexpr int kRowMirror = 0x140, kRowBcast15 = 0x142, kRowBcast31 = 0x143;
  v += dpp_float<kQuadXor1>(v);
  v += dpp_float<kQuadXor2>(v);
  v += dpp_float<kRowHalfMirror>(v);
  v += dpp_float<kRowMirror>(v);
  v += dpp_float<kRowBcast15>(v);
  v += dpp_float<kRowBcast31>(v);
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Inclusive prefix sum over the wavefront.
__device__ __forceinline__ float wave_prefix(float v) {
  auto moved = [](float x, auto ctrl, auto rows) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, decltype(rows)::value, 0xF, false));
  };
  typedef std::integral_constant<int, 0xF> AllRows;
  v += moved(v, std::integral_constant<int, 0x111>{}, AllRows{});  // within a row of 16: from 1, 2, 4, 8 lanes before
  v += moved(v, std::integral_constant<int, 0x112>{}, AllRows{});
  v += moved(v, std::integral_constant<int, 0x114>{}, AllRows{});
  v += moved(v, std::integral_constant<int, 0x118>{}, AllRows{});
  v += moved(v, std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xA>{});  // the row before
  v += moved(v, std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xC>{});  // the two rows before
  return v;
}

// k choices of each of `tokens` tokens poured on the levels of the first E lanes: what each of them gets, at
// most one per token.  (What the bound cuts off is left out.  Poured on the others instead: a round
// less for some calls, one or two more for others, 64 experts, c = 10, one of them far below: 299 -> 384 us.)
__device__ __forceinline__ int first_guess(float level, int lane, int E, int k, int tokens) {
  const float units = (float)(k * tokens);
  bool in = lane < E;
  float surface = 0.0f;
  for (int it = 0; it < E; ++it) {
    const float n = (float)__builtin_popcountll(__builtin_amdgcn_ballot_w64(in));
    surface = (units + wave_sum(in ? level : 0.0f)) / n;
    const bool out = in && level > surface;
    if (__builtin_amdgcn_ballot_w64(out) == 0ull) break;
    in = in && !out;
  }
  const int sum = (int)floorf(wave_prefix(in ? surface - level : 0.0f) + 0.5f);  // (whole numbers, of the same sum)
  const int before = __shfl_up(sum, 1, 64);
  return min(max(sum - (lane > 0 ? before : 0), 0), tokens);
}

// What a block's workgroup keeps in LDS beside that of the walks.
struct BlockLds {
  float inv[64];               // of each group of blocks before this one: 1 / (sum of g)
  unsigned open[kChainWaves];  // bit u of wave w's: the boundary behind block 16 w + u does not match
  int first_begin[kChainWaves][64];  // where the first block of a wave began
  int begin[64], begin_next[64];
  int close[kChainWaves][64];
  int ok, state;                // state: 0 go on, 1 the next walk is the last one, 2 this one was
};
// In the LDS of the walks, between two of them, for every group of blocks before this one what they do to
// a correction, { added, g }: fewer of the dependent steps, 60 ns each (eight shapes of calls, 4 seeds
// each, 16384 and 6000 tokens: block by block 324 us on the average, by twos 306, by fours and eights 296).
constexpr int kBlockGroup = 8;
typedef float2 BlockRow[64];
static_assert((kChainBlocks + 8) * sizeof(BlockRow) <= kChainLdsBytes, "the rows of all blocks, and read-ahead, fit the LDS of a walk");

// How often the decisions of the block's samples were close, lane = expert; wave w looks at samples
// 8 w .. 8 w + 7 (`slots`: lane i the record of the wave's i-th sample).
__device__ __forceinline__ int block_close_decisions(int f0, int n, int slots, int begin, const RouteArgs& a,
                                                     const Workspace& ws, int wave, int lane, int lin) {
  const int shift = a.cw > kMaxC ? 6 : 4;
  unsigned rec[kSamplesPerWave], bits[kSamplesPerWave];
  int base[kSamplesPerWave], cum[kSamplesPerWave];
  auto token = [&](int u) { return f0 + (int)((unsigned)((wave * kSamplesPerWave + u) * n) / kBlockSamples); };
#pragma unroll
  for (int u = 0; u < kSamplesPerWave; ++u) {
    const int slot = __builtin_amdgcn_readlane(slots, u);
    const int word = token(u) >> 5;
    rec[u] = (ws.rec_lane + (size_t)slot * a.EP)[(unsigned)min(lane, a.EP - 1)];
    base[u] = ws.tile_base[(size_t)(slot >> 6) * 64 + lane];
    bits[u] = ws.chain_bits[(size_t)word * 64 + lane];
    cum[u] = ws.chain_cum[(size_t)word * 64 + lane];
  }
  int close = 0;
#pragma unroll
  for (int u = 0; u < kSamplesPerWave; ++u) {
    const int f = token(u);
    const bool cand = lane < a.EP && rec[u] != 0xFFFFu;
    const bool chosen = ((bits[u] >> (f & 31)) & 1u) != 0u;
    const int so_far = ((f >> 5) == (f0 >> 5) ? begin : cum[u]) + __builtin_popcount(bits[u] & ((1u << (f & 31)) - 1u));
    const unsigned load = (unsigned)(lin + base[u] + (int)(rec[u] >> shift) + so_far);
    const unsigned least_out = wave_min_u32(cand && !chosen ? load : 0x7FFFFFFFu);
    const unsigned most_in = 0x7FFFFFFFu - wave_min_u32(chosen ? 0x7FFFFFFFu - load : 0x7FFFFFFFu);
    close += cand && (chosen ? least_out <= load + 1u : load <= most_in + 1u) ? 1 : 0;
  }
  return close;
}

// After a walk of the block [f0, f0 + n) from `begin` to `end` (wave 0, lane = expert), which was walk
// number `round`: tells the others, waits for the blocks before this one to have come as far, and
// works out the next beginning.  (tokens: of every block but the last.)  Returns the state (see BlockLds), or -1
// where the call has been claimed or a wait ran out.
__device__ __forceinline__ int block_round_end(BlockLds& S, BlockRow* row, int blk, int tokens, unsigned round,
                                               bool last_walk, int f0, int n, int slots, int end, const RouteArgs& a, const Workspace& ws, int wave,
                                               int lane, int lin) {
  own_lane(lane);
  unsigned long long* const rows = block_rows(ws);
  __syncthreads();  // (the walk's choices are written; begin[] was)
  const int begin = S.begin[lane];
  auto tell = [&](int close, unsigned r) {
    __hip_atomic_store(&rows[(size_t)blk * 64 + lane], block_word(begin, end - begin, close, r), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  };
  if (last_walk) {
    if (wave == 0) tell(0, kBlockFinal);
    return 2;
  }
  const int mine = block_close_decisions(f0, n, slots, begin, a, ws, wave, lane, lin);
  S.close[wave][lane] = mine;
  if (threadIdx.x == 0) S.ok = 1;
  __syncthreads();
  if (wave == 0) {
    int close = 0;
#pragma unroll
    for (int w = 0; w < kChainWaves; ++w) close += S.close[w][lane];
    tell(min(close, 63), round);
  }
  // ---- the rows of the blocks before, and the boundaries behind them: wave w those from 16 w on ---
  constexpr int kPer = kChainBlocks / kChainWaves;
  const int r0 = wave * kPer, r1 = min(blk, r0 + kPer);
  int last_end = 0;
  if (r0 < r1) {
    unsigned long long v[kPer];
    bool there = false;
    int claimed = 0;
    for (long long it = 0; it < a.spin_limit && !there; ++it) {
      // (the last of them first: it is the one that is waited for)
      const unsigned long long probe =
          __hip_atomic_load(&rows[(size_t)(r1 - 1) * 64 + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      // (with every look, it cost 1 % of the call)
      if ((it & 3) == 0) claimed = __hip_atomic_load(chain_claim(ws), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__builtin_amdgcn_ballot_w64(block_round(probe) < round) != 0ull) {
        // (a block that has seen the claim tells no more)
        if (__builtin_amdgcn_readfirstlane(claimed) != 0) break;
        __builtin_amdgcn_s_sleep(2);
        continue;
      }
#pragma unroll
      for (int u = 0; u < kPer; ++u)
        v[u] = __hip_atomic_load(&rows[(size_t)min(r0 + u, r1 - 1) * 64 + lane], __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
      bool whole = true;
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const unsigned r = block_round(v[u]);
        whole = whole && r >= round && r == (unsigned)__builtin_amdgcn_readfirstlane(r);
      }
      there = __builtin_amdgcn_ballot_w64(!whole) == 0ull;
      if (__builtin_amdgcn_readfirstlane(claimed) != 0) break;
    }
    if (!there || __builtin_amdgcn_readfirstlane(claimed) != 0) {
      S.ok = 0;
#pragma unroll
      for (int u = 0; u < kPer; ++u) v[u] = 0ull;
    }
    // (one reading of every row: a row that is written again meanwhile must not be seen as two)
    S.first_begin[wave][lane] = block_begin(v[0]);
    unsigned open = 0;
    const float close_scale = (float)tokens / kBlockSamples;
#pragma unroll
    for (int u0 = 0; u0 < kPer; u0 += kBlockGroup) {
      // a group in one step: what a boundary adds passes the group's blocks behind it
      // (blocks that do not exist change nothing; the gap behind the wave's last one comes below)
      float x = 0.0f, keep = 1.0f;
#pragma unroll
      for (int u = u0; u < u0 + kBlockGroup; ++u) {
        const bool there_is = r0 + u < r1;
        const int end = block_begin(v[u]) + block_added(v[u]);
        const int gap = r0 + u + 1 < r1 ? end - block_begin(v[u + 1 < kPer ? u + 1 : u]) : 0;
        const float close = (float)block_close(v[u]) * close_scale;
        const float g = there_is ? close * __builtin_amdgcn_rcpf(close + kForgetHalf) : 0.0f;
        if (u != u0) {
          const float sum = wave_sum(g), mean = wave_sum(g * x) * (sum > 0.0f ? __builtin_amdgcn_rcpf(sum) : 0.0f);
          x += g * (mean - x);
        }
        x += (float)gap;
        keep *= 1.0f - g;
        last_end = there_is ? end : last_end;
        open |= (__builtin_amdgcn_ballot_w64(gap != 0) != 0ull ? 1u : 0u) << u;
      }
      const float sum = wave_sum(1.0f - keep);
      if (r0 + u0 < r1) {
        row[(r0 + u0) / kBlockGroup][lane] = make_float2(x, 1.0f - keep);
        if (lane == 0) S.inv[(r0 + u0) / kBlockGroup] = sum > 0.0f ? __builtin_amdgcn_rcpf(sum) : 0.0f;
      }
    }
    if (lane == 0) S.open[wave] = open;
  } else if (lane == 0) {
    S.open[wave] = 0u;
  }
  __syncthreads();
  if (S.ok == 0) return -1;
  if (r0 < r1) {
    // (of the wave's last row the one behind is another wave's, or this block's own)
    const int gap = last_end - (r1 == blk ? begin : S.first_begin[min(wave + 1, kChainWaves - 1)][lane]);
    row[(r1 - 1) / kBlockGroup][lane].x += (float)gap;
    const unsigned open = __builtin_amdgcn_ballot_w64(gap != 0) != 0ull ? 1u : 0u;
    if (lane == 0) S.open[wave] |= open << (r1 - 1 - r0);
  }
  __syncthreads();
  // ---- the correction of this block's beginning ------------------------------------------------
  if (wave == 0) {
    unsigned long long open = 0ull;
#pragma unroll
    for (int w = 0; w < kChainWaves; ++w) open |= (unsigned long long)S.open[w] << (kPer * w);
    open = ((unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(open >> 32)) << 32) |
           (unsigned)__builtin_amdgcn_readfirstlane((unsigned)open);
    int state = 0, next = begin;
    if (open == 0ull) {
      state = 2;  // (everything before this block is decided, and it began there)
    } else {
      const int q0 = __builtin_ctzll(open);
      const unsigned inv = __float_as_uint(S.inv[lane]);
      float d = 0.0f;
      // what bounds a step: the 8 dependent instructions of the sum and the waits between them
      auto step = [&](const float2& x, int q) {
        const float share = x.y * __uint_as_float(__builtin_amdgcn_readlane(inv, q));
        const float keep = fmaf(-x.y, d, d + x.x);
        d = fmaf(share, wave_sum(x.y * d), keep);
      };
      // (four rows ahead; behind the last one: read and not used)
      const int groups = (blk + kBlockGroup - 1) / kBlockGroup;
      int q = q0 / kBlockGroup;
      const float2* from = &row[q][lane];
      float2 x0 = from[0], x1 = from[64], x2 = from[128], x3 = from[192];
      for (; q + 4 <= groups; q += 4) {
        from += 256;
        const float2 y0 = from[0], y1 = from[64], y2 = from[128], y3 = from[192];
        __builtin_amdgcn_sched_barrier(0);
        step(x0, q);
        step(x1, q + 1);
        step(x2, q + 2);
        step(x3, q + 3);
        __builtin_amdgcn_sched_barrier(0);
        x0 = y0;
        x1 = y1;
        x2 = y2;
        x3 = y3;
      }
      if (q < groups) step(x0, q);
      if (q + 1 < groups) step(x1, q + 1);
      if (q + 2 < groups) step(x2, q + 2);
      if (q0 == blk - 1) {
        state = 1;  // (the block before ended where everything is decided: this is no guess)
        next = begin + (int)d;
      } else {
        // whole numbers, of the same sum; a correction that is one stays as it is; nobody has more
        // choices than there are tokens before the block
        const int sum = (int)floorf(wave_prefix(d) + 0.5f);
        const int before = __shfl_up(sum, 1, 64);
        next = min(max(begin + sum - (lane > 0 ? before : 0), 0), f0);
      }
    }
    S.begin_next[lane] = next;
    if (lane == 0) S.state = state;
    if (state == 2) tell(0, kBlockFinal);
  }
  __syncthreads();
  const int state = __builtin_amdgcn_readfirstlane(S.state);
  const int next = S.begin_next[lane];
  __syncthreads();
  if (wave == 0) S.begin[lane] = next;
  return state;
}

// The call's totals (one wave, lane = expert): the counters, and the exclusive prefix over the experts.
__device__ __forceinline__ void chain_totals(int lane, int lin, int cnt, int E, int32_t* __restrict__ loads_inout,
                                             int32_t* __restrict__ expert_offsets) {
  if (lane < E) loads_inout[lane] = lin + cnt;
  int incl = cnt;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int up = __shfl_up(incl, d, 64);
    if (lane >= d) incl += up;
  }
  if (lane < E) expert_offsets[lane] = incl - cnt;
  if (lane == E - 1) expert_offsets[E] = incl;
}

// One segment of a pipelined call, as chain_workgroup sees it: `a` and `ws` are then the
// segment's own view (tile 0 = the segment's first tile, flexible token 0 = its first
// flexible token), and what the earlier segments did comes in through here.
struct ChainSeg {
  bool on;        // false: the whole call in one go (everything below unused)
  int carry0;     // lane = expert: assignments in the earlier segments
  int fbase;      // number of the segment's first flexible token in the call's numbering
  int* out;       // LDS, 66 words: [lane] assignments up to the segment's end, [64] its tiles
                  // with flexible tokens, [65] its flexible tokens
};

// EP: the padded number of experts where it is known (the gate kernel of a pipelined call, whose
// registers the walks that cannot occur would cost), else 0.  BLOCKS: a long chain is walked by the
// workgroups of its blocks (chain_block) as well, once the lists of tokens are there.
template <int EP, bool BLOCKS>
__device__ __forceinline__ void chain_workgroup(uint8_t* lds, const RouteArgs& a, const Workspace& ws,
                                int32_t* __restrict__ loads_inout,
                                int32_t* __restrict__ expert_offsets, const ChainSeg seg) {
  __shared__ int wave_tot[kChainWaves][64];
  __shared__ __align__(16) int tb_rows[kChainWaves][4 * 64];
  __shared__ int wave_flex[kChainWaves], wave_tok[kChainWaves];
  __shared__ SpecShared spec_sh;
  // (as a scalar: branches on the wave number are then uniform for the compiler, and
  // values carried around them stay in scalar registers)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int ntiles = a.ntiles;
  // (a call without tokens has no analysis kernel that would have cleared the status
  // words, and no finishing workgroup that polls them)
  if (!seg.on && ntiles == 0 && threadIdx.x < 4) ws.status[threadIdx.x] = 0;
  // Everything the workgroup reads first is requested before anything is consumed:
  // the counters, the first super-batch of byte counts, the flexible-tile masks.
  int lin = 0;
  if (lane < a.E) lin = loads_inout[lane];
  uint8_t* stage = lds;
  uint4 sv[8];  // 8 loads in flight per thread
  auto stage_load = [&](int sb0, int i0) {
    const int nt = min(kChainStageTiles, ntiles - sb0);
    const uint4* src = reinterpret_cast<const uint4*>(ws.tile_fixed_cnt + (size_t)sb0 * 64);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u * kTailThreads;
      sv[u] = i < nt * 4 ? src[i] : make_uint4(0, 0, 0, 0);
    }
  };
  auto stage_store = [&](int sb0, int i0) {
    const int nt = min(kChainStageTiles, ntiles - sb0);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u * kTailThreads;
      if (i < nt * 4) reinterpret_cast<uint4*>(stage)[i] = sv[u];
    }
  };
  if (ntiles > 0) stage_load(0, threadIdx.x);

  // ---- which tiles hold flexible tokens (groups of 64 tiles per ballot) ------
  const int groups = (ntiles + 63) >> 6;
  const int gper = (groups + kChainWaves - 1) / kChainWaves;
  const int ga = min(wave * gper, groups), gb = min(ga + gper, groups);
  int nfl = 0, ntok = 0;
  // masks of this lane's tiles in the wave's first two groups (kept for the second pass
  // over the groups below: a segment of a pipelined call has no more per wave)
  unsigned long long first_fm = 0ull, second_fm = 0ull;
  for (int g = ga; g < gb; ++g) {
    const int tile = g * 64 + lane;
    const unsigned long long fm = tile < ntiles ? ws.flexmask[tile] : 0ull;
    if (g == ga) first_fm = fm;
    if (g == ga + 1) second_fm = fm;
    nfl += __builtin_popcountll(__builtin_amdgcn_ballot_w64(fm != 0ull));
    ntok += __builtin_popcountll(fm);
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) ntok += __shfl_xor(ntok, d, 64);
  if (lane == 0) {
    wave_flex[wave] = nfl;
    wave_tok[wave] = ntok;
  }
  __syncthreads();
  int nflex_tiles = 0, tokbefore = 0, nflex_tok = 0;  // nflex_tok: flexible tokens of the call
  for (int w = 0; w < kChainWaves; ++w) {
    const int fl = wave_flex[w], tk = wave_tok[w];
    tokbefore += w < wave ? tk : 0;
    nflex_tiles += fl;
    nflex_tok += tk;
  }
  // a handful of flexible tokens: the finishing workgroups resolve them themselves and
  // write the totals; nothing to do here
  // (never in a pipelined call: the finishing workgroups judge by the whole call's sizes)
  if (!seg.on && fast_path_applies(ntiles, nflex_tiles, nflex_tok, a.cw)) return;
  // Without flexible tokens, small problems are finished without tile_base (the
  // finishing workgroups sum the byte counts themselves): only the totals are needed.
  // (A segment cannot know what the later segments hold.)
  const bool need_tile_base = seg.on || nflex_tiles > 0 || ntiles > kSelfPrefixTiles;

  // ---- prefix over tiles of the fixed tokens' counts -------------------------
  // The byte counts are staged through LDS in super-batches with wide loads; wave
  // w then scans a contiguous run of tiles for its lane's expert.
  int carry = seg.on ? seg.carry0 : 0;  // assignments before this super-batch (lane's expert)
  for (int sb0 = 0; sb0 < ntiles; sb0 += kChainStageTiles) {
    const int nt = min(kChainStageTiles, ntiles - sb0);
    for (int i0 = threadIdx.x; i0 < nt * 4; i0 += kTailThreads * 8) {
      if (sb0 != 0 || i0 != (int)threadIdx.x) stage_load(sb0, i0);  // the very first batch is in flight
      stage_store(sb0, i0);
    }
    __syncthreads();
    const int per_wave = (nt + kChainWaves - 1) / kChainWaves;
    const int ta = min(wave * per_wave, nt), tb = min(ta + per_wave, nt);
    int tot = 0;
#pragma unroll 16
    for (int tile = ta; tile < tb; ++tile) tot += stage[tile * 64 + lane];
    wave_tot[wave][lane] = tot;
    __syncthreads();
    int run = carry;
    for (int w = 0; w < kChainWaves; ++w) {
      const int v = wave_tot[w][lane];
      run += w < wave ? v : 0;
      carry += v;
    }
    if (need_tile_base) {
      // Four tiles per store: a wavefront has at most 64 memory operations in flight, and
      // with one store per tile a long run of tiles (a segment of a pipelined call: 128
      // per wave) would wait for memory round trips.  The four rows meet in a wave-private
      // piece of LDS, laid out like the rows of tile_base, and leave as 16 bytes per lane.
      int* rows = tb_rows[wave];
      int tile = ta;
      for (; tile + 4 <= tb; tile += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          rows[u * 64 + lane] = run;
          run += stage[(tile + u) * 64 + lane];
        }
        const int4 v = reinterpret_cast<const int4*>(rows)[lane];
        reinterpret_cast<int4*>(ws.tile_base + (size_t)(sb0 + tile) * 64)[lane] = v;
      }
      for (; tile < tb; ++tile) {
        ws.tile_base[(size_t)(sb0 + tile) * 64 + lane] = run;
        run += stage[tile * 64 + lane];
      }
    }
    // stage and wave_tot are reused by the next super-batch (after the last one nothing
    // writes LDS before the next barrier, and that barrier then waits for the stores
    // above once, together with those below)
    if (sb0 + kChainStageTiles < ntiles) __syncthreads();
  }
  const int total_fixed = carry;

  nflex_tiles = __builtin_amdgcn_readfirstlane(nflex_tiles);
  nflex_tok = __builtin_amdgcn_readfirstlane(nflex_tok);
  const bool wide = a.cw > kMaxC;
  const bool use_spec = nflex_tok >= kSpecMinTokens && !wide;
  // for every tile the number of flexible tokens before it, and the list of those tokens
  const int fbase = seg.on ? seg.fbase : 0;
  for (int g = ga; g < gb && (nflex_tiles > 0 || seg.on); ++g) {
    const int tile = g * 64 + lane;
    const unsigned long long fm =
        g == ga ? first_fm : g == ga + 1 ? second_fm : (tile < ntiles ? ws.flexmask[tile] : 0ull);
    const int np = __builtin_popcountll(fm);
    int incl = np;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int up = __shfl_up(incl, d, 64);
      if (lane >= d) incl += up;
    }
    if (tile < ntiles) {
      ws.flex_tok_base[tile] = fbase + tokbefore + incl - np;  // (read by the finishing pass only)
      if (tile == ntiles - 1 && !seg.on) ws.flex_tok_base[ntiles] = tokbefore + incl;
    }
    // slot (tile * 64 + rank among the tile's flexible tokens) of every flexible token: every
    // lane lists its own tile's
    const int mybase = tokbefore + incl - np;
    for (int i = 0; __builtin_amdgcn_ballot_w64(i < np) != 0ull; ++i)
      if (i < np) ws.flex_slot[mybase + i] = (tile << 6) + i;
    tokbefore += __shfl(incl, 63, 64);
  }

  int gflex = 0;  // flexible assignments so far (meaningful in wave 0)

  auto write_totals = [&]() {  // wave 0
    chain_totals(lane, lin, lane < a.E ? total_fixed + gflex : 0, a.E, loads_inout, expert_offsets);
  };

  // A segment hands its results to the caller instead of publishing anything.
  auto segment_result = [&]() {  // wave 0
    seg.out[lane] = total_fixed + gflex;
    if (lane == 0) {
      seg.out[64] = nflex_tiles;
      seg.out[65] = nflex_tok;
    }
  };

  if (wave == 0 && (nflex_tiles > 0 || seg.on)) ws.chain_cum[lane] = 0;  // nothing chosen before flexible token 0
  bool blocks = false;
  if (seg.on) {
    if (nflex_tiles == 0) {
      if (wave == 0) segment_result();
      return;
    }
    __syncthreads();  // tile_base, flex_slot written by every wave
  } else {
    if (nflex_tiles == 0 && wave == 0) write_totals();  // already final
    blocks = BLOCKS && chain_in_blocks(nflex_tok, a.T);
    if (blocks) clear_block_rows(ws, a.T, lane, wave, total_fixed);
    __syncthreads();  // tile_base, flex_slot (and the totals) written by every wave
    if (threadIdx.x == 0) {
      ws.status[kStatusFlexTiles] = blocks ? -nflex_tiles : nflex_tiles;
      __hip_atomic_store(&ws.status[kStatusPhase], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (nflex_tiles == 0) return;
  }

  Race<BLOCKS> race = {};
  if constexpr (BLOCKS) {
    __shared__ int race_stop[2];
    race.claim = blocks ? chain_claim(ws) : nullptr;
    race.stop = race_stop;
  }
  int decided = 0, nsweeps = 0;
  unsigned hist0 = 0;
  if (use_spec && EP != 8 && a.EP != 8) {
    // With many experts per candidate tokens rarely compete: the window of 256.
    // With fewer a sweep may end at an early conflict: the window of 64, which is given up where the
    // walk is faster.  (Up to 8 experts the walk always is, or nearly: 17.7 ns per token against at least 16.)
    if (a.c <= 4) {
      if (a.E >= 16)
        decided = a.k == 2 ? window_walk<4, 2>(lds, nflex_tok, a, ws, wave, lane, lin, gflex, hist0, nsweeps, race)
                           : window_walk<4, 0>(lds, nflex_tok, a, ws, wave, lane, lin, gflex, hist0, nsweeps, race);
      else if (EP == 0 || EP == 16)
        decided = a.k == 2 ? spec_walk<4, 2>(lds, spec_sh, nflex_tok, a, ws, wave, lane, lin, gflex, hist0, nsweeps, race)
                           : spec_walk<4, 0>(lds, spec_sh, nflex_tok, a, ws, wave, lane, lin, gflex, hist0, nsweeps, race);
    } else if (a.c <= 8) {
      if ((EP == 0 || EP >= 32) && a.E >= 32)
        decided = a.k == 6 ? window_walk<8, 6>(lds, nflex_tok, a, ws, wave, lane, lin, gflex, hist0, nsweeps, race)
                           : window_walk<8, 0>(lds, nflex_tok, a, ws, wave, lane, lin, gflex, hist0, nsweeps, race);
      else if (EP <= 32)
        decided = a.k == 6 ? spec_walk<8, 6>(lds, spec_sh, nflex_tok, a, ws, wave, lane, lin, gflex, hist0, nsweeps, race)
                           : spec_walk<8, 0>(lds, spec_sh, nflex_tok, a, ws, wave, lane, lin, gflex, hist0, nsweeps, race);
    } else if ((EP == 0 || EP == 64) && a.E == 64) {
      decided = window_walk<16, 0>(lds, nflex_tok, a, ws, wave, lane, lin, gflex, hist0, nsweeps, race);
    } else {
      decided = spec_walk<16, 0>(lds, spec_sh, nflex_tok, a, ws, wave, lane, lin, gflex, hist0, nsweeps, race);
    }
  }
  if (BLOCKS && decided < 0) return;  // (the blocks were first)
  bool whole = true;
  if (decided < nflex_tok) {
    // the rest (or everything) one token after the other
    if (EP == 8 || (EP == 0 && a.EP == 8))  // (nothing is decided yet)
      chain_walk_pairs(lds, nflex_tok, ws, a.k, wave, lane, lin, gflex);
    else if (a.c <= 8)
      whole = chain_walk_lag(lds, decided, hist0, nflex_tok, a, ws, wave, lane, lin, gflex, race);
    else if (EP == 0 && wide)
      whole = chain_walk<0>(lds, decided, hist0, nflex_tok, a, ws, wave, lane, lin, gflex, race);
    else
      whole = chain_walk<16>(lds, decided, hist0, nflex_tok, a, ws, wave, lane, lin, gflex, race);
  }
  if (BLOCKS && !whole) return;
  if (seg.on) {
    if (wave == 0) segment_result();
    return;
  }
  const bool mine = !blocks || wave != 0 || claim_chain(ws, lane);
  if (wave == 0 && mine) {
    write_totals();
    if (BLOCKS && lane == 0) ws.status[kStatusSweeps] = nsweeps;
  }
  __syncthreads();
  if (threadIdx.x == 0 && mine)
    __hip_atomic_store(&ws.status[kStatusPhase], kPhaseWalked, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// Block `blk` of a chain of nflex_tok tokens (kTailThreads threads), see "the chain in blocks".
__device__ __forceinline__ void chain_block(uint8_t* lds, const RouteArgs& a, const Workspace& call,
                                            int32_t* __restrict__ loads_inout, int32_t* __restrict__ expert_offsets,
                                            int blk, int nflex_tok) {
  __shared__ BlockLds S;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int tokens = chain_block_tokens(nflex_tok);  // of every block but the last
  const int f0 = blk * tokens, f1 = min(nflex_tok, f0 + tokens);
  if (f0 >= nflex_tok) return;
  // (a claim is looked for between the walks: looks inside them cost the blocks 4 to 8 %, and a walk of
  // a block is a 64th of the claimant's, a 24th where the call is short)
  const Race<false> no_race = {};
  Workspace ws = call;  // (with the blocks' own choices)
  ws.chain_bits = block_bits(call);
  ws.chain_cum = block_cum(call, a.T);
  const int lin = ws.lin_copy[lane];
  // the lists of tokens, from the chain workgroup
  // (a wait that runs out is no error: the chain workgroup walks the call)
  if (wave == 0) {
    const bool ok = poll_flag(&ws.status[kStatusPhase], 1, a.spin_limit) != 0;
    if (lane == 0) S.ok = ok ? 1 : 0;
    S.begin[lane] = 0;
  }
  __syncthreads();
  if (S.ok == 0) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  const int sample = wave * kSamplesPerWave + min(lane, kSamplesPerWave - 1);
  const int slots = ws.flex_slot[f0 + (int)((unsigned)(sample * (f1 - f0)) / kBlockSamples)];
  int gflex = 0;  // wave 0, lane = expert: choices by the tokens before the block, then by those of the block too
  if (wave == 0 && blk != 0) {
    // the first guess: all choices before the block have gone to whoever was lowest
    gflex = first_guess(lane < a.E ? (float)(lin + ws.tile_base[(size_t)(ws.flex_slot[f0] >> 6) * 64 + lane]) : 0.0f, lane,
                        a.E, a.k, f0);
    S.begin[lane] = gflex;
  }
  __syncthreads();
  bool last_walk = blk == 0;
  unsigned round = 1;
  for (;; ++round) {
    if (a.c <= 8)
      chain_walk_lag(lds, f0, 0u, f1, a, ws, wave, lane, lin, gflex, no_race);
    else if (a.cw > kMaxC)
      chain_walk<0>(lds, f0, 0u, f1, a, ws, wave, lane, lin, gflex, no_race);
    else
      chain_walk<16>(lds, f0, 0u, f1, a, ws, wave, lane, lin, gflex, no_race);
    const int state = block_round_end(S, reinterpret_cast<BlockRow*>(lds), blk, tokens, round, last_walk, f0, f1 - f0,
                                      slots, gflex, a, ws, wave, lane, lin);
    if (state < 0) return;
    if (state == 2) break;
    last_walk = state == 1;
    gflex = S.begin_next[lane];
  }
  __syncthreads();  // (the choices are written)
  int* const done = blocks_done(ws);
  if (f1 < nflex_tok) {
    if (threadIdx.x == 0) __hip_atomic_fetch_add(done, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  // the last block, when all the others have written their choices: the totals and the last flag
  if (wave == 0) {
    const int fixed = (int)__hip_atomic_load(&block_rows(ws)[kChainBlocks * 64 + lane], __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
    bool ok = false;
    for (long long it = 0; it < a.spin_limit; ++it) {
      const int n = __hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int claimed = __hip_atomic_load(chain_claim(ws), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      ok = __builtin_amdgcn_readfirstlane(n) >= blk;
      if (ok || __builtin_amdgcn_readfirstlane(claimed) != 0) break;
      __builtin_amdgcn_s_sleep(2);
    }
    ok = ok && claim_chain(ws, lane);
    if (ok) {
      chain_totals(lane, lin, lane < a.E ? fixed + gflex : 0, a.E, loads_inout, expert_offsets);
      if (lane == 0) ws.status[kStatusSweeps] = (int)round;
    }
    if (lane == 0) S.ok = ok ? 1 : 0;
  }
  __syncthreads();
  if (S.ok != 0 && threadIdx.x == 0)
    __hip_atomic_store(&ws.status[kStatusPhase], kPhaseBlocks, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// ---- pipelined calls: the chain segment by segment ---------------------------------
//
// Algorithm 1 orders the tokens of a batch, so the chain over tiles [0, n) needs nothing
// of the tiles behind them.  A large call is therefore cut into segments of a.seg_tiles
// tiles; the chain over a segment starts as soon as the gate kernel has analysed the
// segment's tiles, inside that kernel (workgroup 0 of its grid), while the other
// workgroups go on streaming the later tiles.  Every wavefront of an analysis workgroup
// counts itself into its tile's word of ws.seg when its records are written and
// acknowledged (what the chain reads is stored write-through); the chain workgroup waits
// for all tiles of a segment to be complete and then invalidates its caches (acquire).
// The wait is bounded: should it ever give up, the tail kernel's chain workgroup takes
// over where it stopped, behind the kernel boundary; otherwise the tail kernel's finds
// every segment done and only writes the totals and raises the flags.
// What is carried from segment to segment (ws.seg) is small: per expert the assignments
// so far, and where the numbering of flexible tokens and tiles goes on.  A segment's
// flexible tokens are numbered from a multiple of 32 (words of chain_bits / chain_cum
// are not shared between segments), chain_cum restarts at 0 in every segment, and
// tile_base carries the earlier segments' choices -- the finishing pass reads all of it
// exactly as in a call that is not pipelined.

// The chain numbers the tiles and the flexible tokens of a segment from 0.  `v` becomes the
// view of the arrays in which those are dtiles tiles and dflex flexible tokens (a multiple of
// 32) further on than in `v`.
// (Advanced in place from segment to segment: one set of pointers in scalar registers.)
__device__ __forceinline__ void advance_view(Workspace& v, const RouteArgs& a, int dtiles, int dflex) {
  const size_t tok = (size_t)dtiles * kTile;  // tokens and record slots
  v.rec_cstar += tok;
  v.rec_ids += tok * a.cw;
  v.rec_p += tok * a.cw;
  v.rec_Z += tok;
  v.rec_lane += tok * a.EP;
  v.flexmask += dtiles;
  v.tile_fixed_cnt += (size_t)dtiles * 64;
  v.tile_mask += (size_t)dtiles * 64;
  v.tile_base += (size_t)dtiles * 64;
  v.rec_cids += tok * 16;
  v.rec_pref += tok * 16;
  v.flex_tok_base += dtiles;
  v.flex_slot += dflex;
  v.chain_bits += (size_t)(dflex >> 5) * 64;
  v.chain_cum += (size_t)(dflex >> 5) * 64;
}

// Polls of a segment's counter before the chain workgroup inside the gate kernel leaves
// the rest to the tail kernel (a poll is a memory round trip plus a short sleep).
constexpr long long kSegPollLimit = 1ll << 20;
// Every wavefront of an analysis workgroup counts itself into its tile's word.
constexpr int kGateSignals = 8;

// The chain of a call, by the chain workgroup (kTailThreads threads) of the gate kernel
// (IN_GATE: as far as the analysed tiles allow, nothing is published) or of the tail
// kernel (the rest, then the totals and the flags the finishing workgroups wait for).
template <bool IN_GATE, int EP, bool BLOCKS = false>  // EP, BLOCKS: see chain_workgroup
__device__ __forceinline__ void chain_segments(uint8_t* lds, const RouteArgs& a, const Workspace& ws,
                                               int32_t* __restrict__ loads_inout,
                                               int32_t* __restrict__ expert_offsets) {
  ChainSeg sg;
  sg.on = a.nseg > 0;  // (not pipelined: one round over the whole call, which publishes for itself)
  sg.carry0 = 0;
  sg.fbase = 0;
  __shared__ int seg_out[66];
  __shared__ int seg_ready;
  sg.out = seg_out;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int32_t* const status = ws.status;
  int32_t* const segw = ws.seg;
  int j = 0, fbase = 0, ordbase = 0, carry = 0;
  RouteArgs av = a;
  Workspace wv = ws;
  if (sg.on) {
    // (written by the kernel before this one: the clearing kernel, or the gate kernel)
    j = __builtin_amdgcn_readfirstlane(segw[kSegNext]);
    fbase = __builtin_amdgcn_readfirstlane(segw[kSegFlexBase]);
    ordbase = __builtin_amdgcn_readfirstlane(segw[kSegOrdBase]);
    carry = segw[kSegCarry + lane];
    advance_view(wv, a, min(segment_start(a, j), a.ntiles), fbase);
  }
  const int rounds = sg.on ? a.nseg : 1;
  for (; j < rounds; ++j) {
    if (sg.on) {
      const int tile0 = segment_start(a, j);
      const int nt = min(segment_start(a, j + 1), a.ntiles) - tile0;
      if (IN_GATE) {
        // every thread waits for some of the segment's tiles (all of their wavefronts
        // counted in), then the workgroup agrees on whether all of them are there
        if (threadIdx.x == 0) seg_ready = 1;
        __syncthreads();
        bool mine = true;
        for (int i = threadIdx.x; i < nt && mine; i += kTailThreads)
          mine = poll_word(&segw[kSegDone + tile0 + i], kGateSignals, kSegPollLimit);
        if (!mine) seg_ready = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        __syncthreads();
        const bool ready = seg_ready != 0;
        __syncthreads();  // (seg_ready is written again in the next round)
        if (!ready) break;
      }
      av.ntiles = nt;
      av.T = min(a.T - tile0 * kTile, nt * kTile);
      sg.carry0 = carry;
      sg.fbase = fbase;
    }
    chain_workgroup<EP, BLOCKS>(lds, av, wv, loads_inout, expert_offsets, sg);
    if (!sg.on) return;
    __syncthreads();  // seg_out written (wave 0); the chain's LDS is free again
    carry = seg_out[lane];
    // (as scalars: the next segment's view is then computed in scalar registers)
    const int dord = __builtin_amdgcn_readfirstlane(seg_out[64]);
    const int dflex = (__builtin_amdgcn_readfirstlane(seg_out[65]) + 32) & ~31;
    advance_view(wv, a, av.ntiles, dflex);
    ordbase += dord;
    fbase += dflex;
    __syncthreads();  // (seg_out is written again in the next round)
  }
  if (IN_GATE) {
    // for the tail kernel, behind the kernel boundary
    if (wave == 0) segw[kSegCarry + lane] = carry;
    if (threadIdx.x == 0) {
      segw[kSegNext] = j;
      segw[kSegFlexBase] = fbase;
      segw[kSegOrdBase] = ordbase;
    }
    return;
  }
  // the totals, and the flags of the finishing workgroups
  if (wave == 0) {
    const int lin = lane < a.E ? loads_inout[lane] : 0;
    chain_totals(lane, lin, lane < a.E ? carry : 0, a.E, loads_inout, expert_offsets);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    status[kStatusFlexTiles] = ordbase;
    __hip_atomic_store(&status[kStatusPhase], kPhaseWalked, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// ---- a handful of flexible tokens: every finishing workgroup resolves them itself ----
//
// With thresholds like the paper's, a layer of a skewed gate has no or very few
// flexible tokens.  Waiting for the chain workgroup then costs several dependent
// memory round trips and two flag hand-overs for one or two chain steps.  Instead,
// when the call has at most kFastTokens flexible tokens in at most kFastTiles tiles
// (and at most kFastMaxTiles tiles in all, so that one batch of loads covers every
// tile's counts), every finishing workgroup sums, beside its own prefix, the fixed
// assignments before each flexible tile, fetches the few records and walks them with
// the same step as the sequential chain.  All workgroups compute the same choices;
// nobody waits for anybody, and the chain workgroup has nothing to do.
struct FastShared {
  unsigned long long bal[kChainWaves];          // wave w: which of tiles 64w .. 64w+63 are flexible
  unsigned long long fmtile[kFastMaxTiles];     // flexible-token mask of a flexible tile
  int fbefore[kFastTiles][kChainWaves][64];     // per wave: fixed assignments in the tiles before
                                                // the f-th flexible tile, per expert
  // the n-th flexible token of the call:
  unsigned rec[kFastTokens][64];                // its record row (lane = expert)
  uint4 cids[kFastTokens];                      // candidate experts by rank, padded
  uint8_t rids[kFastTokens][kMaxC];             // candidate experts by rank
  float p[kFastTokens][kMaxC];                  // their probabilities
  float Z[kFastTokens];                         // the softmax denominator
  int tok[kFastTokens];                         // token index
  int tokf[kFastTokens];                        // index of its flexible tile
  unsigned long long emask[kFastTokens];        // the experts chosen for it
};

// LDS of a finishing workgroup beside the dynamic part.
struct FinishShared {
  int sh_before[kChainWaves][64], sh_all[kChainWaves][64];
  int own_base[kChainWaves][64], own_offsets[64];
  int sh_anyflex[kChainWaves];  // per wave: some tile it looked at holds flexible tokens
  FastShared fs;
};

struct FinishLds {
  unsigned long long mask64[64];
  int before[64];  // per expert: slots of all earlier experts + of this expert in earlier tiles
  unsigned bits[3][64];  // per expert: the chain's words in which the tile's flexible tokens are
  uint8_t ids[kTile][kMaxC];
};

// What a finishing wave can read before anything else of the tail kernel has run.
struct FinishPrologue {
  int cstar;               // working-set size of a flexible token, else 0
  unsigned long long fm;   // the tile's flexible-token mask
  unsigned long long tmask;  // lane = expert: the tile's non-flexible tokens assigned to it
  int ids[kMaxC];          // experts of the token as the analysis left them (k entries)
};

// Requests the loads only; nothing here waits for them.
__device__ __forceinline__ FinishPrologue finish_prologue(int tile, const RouteArgs& a, const Workspace& ws,
                                                          const int32_t* __restrict__ expert_ids) {
  const int lane = threadIdx.x & 63;
  const int t = tile * kTile + lane;
  const bool live = t < a.T;
  FinishPrologue p;
  p.cstar = live ? ws.rec_cstar[t] : 0;
  p.fm = ws.flexmask[tile];
  p.tmask = ws.tile_mask[(size_t)tile * 64 + lane];
#pragma unroll
  for (int j = 0; j < kMaxC; ++j) p.ids[j] = (live && j < a.k) ? expert_ids[(size_t)t * a.k + j] : 0;
  return p;
}

// experts of the tokens that are final already go to LDS (rows of flexible tokens hold
// stale data; they are overwritten in finish_row)
__device__ __forceinline__ void finish_commit(FinishLds* fl, const FinishPrologue& p, int k) {
  const int lane = threadIdx.x & 63;
  fl->mask64[lane] = p.tmask;  // the flexible tokens add themselves in finish_row
#pragma unroll
  for (int j = 0; j < kMaxC; ++j)
    if (j < k) fl->ids[lane][j] = (uint8_t)p.ids[j];
}

// A flexible token (lane = token) whose choice is known: its experts in score order and their weights,
// and its bit in the masks of those experts.  `chosen(j)`, `id(j)`, `p(j)`: of rank j < cstar, of which
// n_ranks are looked at (the loop is the same in every lane).
template <typename Chosen, typename Id, typename P>
__device__ __forceinline__ void finish_row(FinishLds* fl, int t, int cstar, int n_ranks, float Z, const RouteArgs& a,
                                           int32_t* __restrict__ expert_ids, float* __restrict__ weights, Chosen chosen,
                                           Id id, P p) {
  const int lane = threadIdx.x & 63;
  const int k = a.k;
  float denom = Z;
  if (a.renormalize) {
    bool first = true;
#pragma unroll
    for (int j = 0; j < kMaxC; ++j) {
      if (j >= n_ranks) break;
      if (j < cstar && chosen(j)) {
        denom = first ? p(j) : denom + p(j);
        first = false;
      }
    }
  }
  int n = 0;
#pragma unroll
  for (int j = 0; j < kMaxC; ++j) {
    if (j >= n_ranks) break;
    if (j < cstar && chosen(j) && n < k) {  // (exactly k are chosen; n < k keeps the row)
      const int e = id(j);
      expert_ids[(size_t)t * k + n] = e;
      weights[(size_t)t * k + n] = p(j) / denom;
      fl->ids[lane][n] = (uint8_t)e;
      atomicOr(&fl->mask64[e], 1ull << lane);
      ++n;
    }
  }
}

// LDS traffic of one wavefront is processed in order; this only stops the compiler from moving reads
// above the other lanes' writes.  (A fence would also wait for the rows' stores: a microsecond.)
__device__ __forceinline__ void finish_fence() {
  lds_wave_fence();
  __builtin_amdgcn_wave_barrier();
}

// One wavefront, one tile; `fl` is this wave's private LDS, complete: every slot of the tile.
__device__ __forceinline__ void finish_slots(FinishLds* fl, int t, const RouteArgs& a, const Workspace& ws,
                                             int32_t* __restrict__ permutation) {
  const int lane = threadIdx.x & 63;
  const int k = a.k;
  finish_fence();
  if (t < a.T) {
    const unsigned long long below = lanes_below(lane);
    for (int j = 0; j < k; ++j) {
      const int e = fl->ids[lane][j];
      const int pos = fl->before[e] + __builtin_popcountll(fl->mask64[e] & below);
      // (pos is a slot number by construction; the check turns any inconsistency of
      // the inputs into a missing entry instead of a stray store)
      if ((unsigned)pos < (unsigned)(a.T * k))
        permutation[pos] = t * k + j;
      else
        ws.status[kStatusError] = kErrorInconsistent;
    }
  }
}

// A tile of a call without flexible tokens, or (fast_n > 0) with a handful of them that this workgroup has
// decided itself: the caller has computed, for every expert, the number of assignments in earlier
// tiles (own_base, LDS, 64 words) and the exclusive prefix over experts of the totals (own_offsets).
__device__ __forceinline__ void finish_tile(FinishLds* fl, int tile, const FinishPrologue& pro, const RouteArgs& a,
                                            const Workspace& ws, int32_t* __restrict__ expert_ids,
                                            float* __restrict__ weights, int32_t* __restrict__ permutation,
                                            const int* own_base, const int* own_offsets, int fast_n,
                                            const FastShared* fast) {
  const int lane = threadIdx.x & 63;
  const int t = tile * kTile + lane;
  fl->before[lane] = own_offsets[lane] + own_base[lane];
  if (__builtin_expect(fast_n > 0, 0)) {
    finish_fence();
    if (pro.cstar > 0) {
      int n = 0;
      for (int i = 0; i < fast_n; ++i) n = fast->tok[i] == t ? i : n;
      const unsigned long long emask = fast->emask[n];
      finish_row(fl, t, pro.cstar, a.c, fast->Z[n], a, expert_ids, weights,
                 [&](int j) { return ((emask >> fast->rids[n][j]) & 1ull) != 0ull; },
                 [&](int j) { return (int)fast->rids[n][j]; }, [&](int j) { return fast->p[n][j]; });
    }
  }
  finish_slots(fl, t, a, ws, permutation);
}

// A tile of a call whose chain runs in another workgroup.  What does not depend on the chain's choices
// is asked for before they are waited for; what does comes in one round trip, a row of experts per
// load: the tile's flexible tokens are in at most three words of 32.  (A byte and a word per candidate, one
// after the other, before: 3001 tokens, 287 flexible, from the flag to the last store 7.3 -> 4.3 us.)
// (BLOCKS: the choices may be those of the chain's blocks)
template <bool BLOCKS>
__device__ __forceinline__ void finish_tile_of_chain(FinishLds* fl, int tile, const FinishPrologue& pro,
                                                     const RouteArgs& a, const Workspace& ws,
                                                     const int32_t* __restrict__ expert_offsets,
                                                     int32_t* __restrict__ expert_ids, float* __restrict__ weights,
                                                     int32_t* __restrict__ permutation) {
  const int lane = threadIdx.x & 63;
  const int t = tile * kTile + lane;
  const int cstar = pro.cstar;
  const bool narrow = a.cw == kMaxC;
  // records of up to 16 candidates: in registers
  uint4 ids = make_uint4(0, 0, 0, 0);
  float p[kMaxC] = {};
  float Z = 0.0f;
  if (cstar > 0) {
    Z = ws.rec_Z[t];
    if (narrow) {
      ids = reinterpret_cast<const uint4*>(ws.rec_ids)[t];
#pragma unroll
      for (int i = 0; i < kMaxC / 4; ++i) {
        if (4 * i >= a.c) break;
        const float4 v = reinterpret_cast<const float4*>(ws.rec_p)[(size_t)t * (kMaxC / 4) + i];
        p[4 * i] = v.x;
        p[4 * i + 1] = v.y;
        p[4 * i + 2] = v.z;
        p[4 * i + 3] = v.w;
      }
    }
  }
  if (!poll_flag(&ws.status[kStatusPhase], 1, a.spin_limit)) {
    ws.status[kStatusError] = kErrorTimeout;
    return;
  }
  const int flex_tiles = load_published(&ws.status[kStatusFlexTiles]);
  // lane = expert: where this tile's first slot of the expert goes.  With flexible
  // tokens about, the choices made for the f0 flexible tokens of earlier tiles are
  // the running count at the last 32-token boundary plus the bits since.
  int before = load_published(&ws.tile_base[(size_t)tile * 64 + lane]);
  if (flex_tiles != 0) {
    const int f0 = load_published(&ws.flex_tok_base[tile]);
    const int phase = poll_flag(&ws.status[kStatusPhase], kPhaseWalked, a.spin_limit);
    if (phase == 0) {
      ws.status[kStatusError] = kErrorTimeout;
      return;
    }
    const bool by_blocks = BLOCKS && phase == kPhaseBlocks;
    const uint32_t* const chain_bits = by_blocks ? block_bits(ws) : ws.chain_bits;
    const int32_t* const chain_cum = by_blocks ? block_cum(ws, a.T) : ws.chain_cum;
    const size_t w = (size_t)(f0 >> 5) * 64 + lane;
    unsigned bits[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) bits[u] = load_published(&chain_bits[w + 64 * u]);
    const int cum = load_published(&chain_cum[w]);
    const int offset = lane < a.E ? load_published(&expert_offsets[lane]) : 0;
    fl->before[lane] = offset + before + cum + __builtin_popcount(bits[0] & ((1u << (f0 & 31)) - 1u));
#pragma unroll
    for (int u = 0; u < 3; ++u) fl->bits[u][lane] = bits[u];
    finish_fence();
    if (cstar > 0) {
      const int f = (f0 & 31) + __builtin_popcountll(pro.fm & lanes_below(lane));
      const unsigned* row = fl->bits[f >> 5];
      if (narrow) {
        const unsigned idw[4] = {ids.x, ids.y, ids.z, ids.w};
        auto id = [&](int j) { return (int)((idw[j >> 2] >> (8 * (j & 3))) & 255u); };
        unsigned chosen = 0;
#pragma unroll
        for (int j = 0; j < kMaxC; ++j) {
          if (j >= a.c) break;
          chosen |= ((row[id(j) & 63] >> (f & 31)) & 1u) << j;
        }
        finish_row(fl, t, cstar, a.c, Z, a, expert_ids, weights, [&](int j) { return ((chosen >> j) & 1u) != 0u; }, id,
                   [&](int j) { return p[j]; });
      } else {
        // which ranks are chosen, then those k of them
        const uint8_t* wide_ids = ws.rec_ids + (size_t)t * kWideC;
        unsigned long long ranks = 0ull;
        for (int i = 0; 16 * i < cstar; ++i) {
          const uint4 v = reinterpret_cast<const uint4*>(wide_ids)[i];
          const unsigned w[4] = {v.x, v.y, v.z, v.w};
          unsigned some = 0;
#pragma unroll
          for (int j = 0; j < 16; ++j)
            some |= ((row[(w[j >> 2] >> (8 * (j & 3))) & 63u] >> (f & 31)) & 1u) << j;
          ranks |= (unsigned long long)some << (16 * i);
        }
        if (cstar < 64) ranks &= (1ull << cstar) - 1ull;
        float wp[kMaxK];
        int we[kMaxK];
#pragma unroll
        for (int n = 0; n < kMaxK; ++n) {
          if (n >= a.k) break;
          const int j = ranks != 0ull ? __builtin_ctzll(ranks) : 0;  // (exactly k are chosen)
          ranks &= ranks - 1ull;
          wp[n] = ws.rec_p[(size_t)t * kWideC + j];
          we[n] = wide_ids[j];
        }
        float denom = Z;
        if (a.renormalize) {
          denom = wp[0];
#pragma unroll
          for (int n = 1; n < kMaxK; ++n) {
            if (n >= a.k) break;
            denom = denom + wp[n];
          }
        }
#pragma unroll
        for (int n = 0; n < kMaxK; ++n) {
          if (n >= a.k) break;
          expert_ids[(size_t)t * a.k + n] = we[n];
          weights[(size_t)t * a.k + n] = wp[n] / denom;
          fl->ids[lane][n] = (uint8_t)we[n];
          atomicOr(&fl->mask64[we[n] & 63], 1ull << lane);
        }
      }
    }
  } else {
    fl->before[lane] = before + (lane < a.E ? load_published(&expert_offsets[lane]) : 0);
  }
  finish_slots(fl, t, a, ws, permutation);
}

// Per-expert assignment counts of the tiles before `t0` and of all tiles, summed by
// the whole workgroup straight from the analysis kernel's byte counts.  Only valid
// when no tile holds a flexible token (then the fixed counts are all there is).
// Lane l of a load takes experts 4*(l%16)..+3 of tile 4*j + l/16; bytes are
// accumulated pairwise in 16-bit fields (at most 64 per tile, ntiles <= 1024).
__device__ __forceinline__ void self_prefix(int t0, const RouteArgs& a, const Workspace& ws, int (*sh_before)[64],
                            int (*sh_all)[64], int* sh_anyflex, unsigned long long& fm_first) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int ntiles = a.ntiles;
  const int sub = lane >> 4;  // which of the 4 tiles of a load
  const unsigned* cnt32 = reinterpret_cast<const unsigned*>(ws.tile_fixed_cnt);
  unsigned b02 = 0, b13 = 0, a02 = 0, a13 = 0;
  // flexible-tile masks first (ntiles <= kSelfPrefixTiles: at most 4 per thread), so that
  // their latency overlaps the count loads
  unsigned long long fmv[kSelfPrefixTiles / kTailThreads];
#pragma unroll
  for (int u = 0; u < kSelfPrefixTiles / kTailThreads; ++u) {
    const int i = threadIdx.x + u * kTailThreads;
    fmv[u] = i < ntiles ? ws.flexmask[i] : 0ull;
  }
  const int nload = (ntiles + 3) >> 2;
  constexpr int kBatch = 16;  // loads issued together: the loop is bound by latency, not by volume
  for (int j0 = wave; j0 < nload; j0 += kChainWaves * kBatch) {
    unsigned wd[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int tile = 4 * (j0 + u * kChainWaves) + sub;
      wd[u] = tile < ntiles ? cnt32[(size_t)tile * 16 + (lane & 15)] : 0u;
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int tile = 4 * (j0 + u * kChainWaves) + sub;
      const unsigned lo = wd[u] & 0x00FF00FFu, hi = (wd[u] >> 8) & 0x00FF00FFu;
      a02 += lo;
      a13 += hi;
      b02 += tile < t0 ? lo : 0u;
      b13 += tile < t0 ? hi : 0u;
    }
  }
  // fold the 4 tile sub-groups of the wave (lanes l, l+16, l+32, l+48)
#pragma unroll
  for (int d = 16; d < 64; d <<= 1) {
    a02 += __shfl_xor(a02, d, 64);
    a13 += __shfl_xor(a13, d, 64);
    b02 += __shfl_xor(b02, d, 64);
    b13 += __shfl_xor(b13, d, 64);
  }
  if (lane < 16) {
    const int e = 4 * lane;
    sh_all[wave][e] = a02 & 0xFFFF;
    sh_all[wave][e + 1] = a13 & 0xFFFF;
    sh_all[wave][e + 2] = a02 >> 16;
    sh_all[wave][e + 3] = a13 >> 16;
    sh_before[wave][e] = b02 & 0xFFFF;
    sh_before[wave][e + 1] = b13 & 0xFFFF;
    sh_before[wave][e + 2] = b02 >> 16;
    sh_before[wave][e + 3] = b13 >> 16;
  }
  fm_first = fmv[0];  // the mask of tile threadIdx.x
  bool flex = false;
#pragma unroll
  for (int u = 0; u < kSelfPrefixTiles / kTailThreads; ++u) flex |= fmv[u] != 0ull;
  const bool any = __builtin_amdgcn_ballot_w64(flex) != 0ull;  // (all lanes take part)
  if (lane == 0) sh_anyflex[wave] = any ? 1 : 0;
}

// Called by a whole finishing workgroup once it knows that some tile holds flexible
// tokens (ntiles <= kFastMaxTiles: thread i looked at tile i's flexible mask, fm_mine).
// Returns 0, having done nothing but look, if there are too many; otherwise the
// number of flexible tokens, with own_base / own_offsets and the choices (fs.emask,
// fs.tok) ready for finish_tile.  sh_before / sh_all hold the four waves' partial sums
// of the fixed counts before this workgroup's tiles / of all tiles.  A lone wavefront
// issues an instruction every few cycles only, so the point here is few instructions:
// per-token state lives in LDS and the loops over tokens are not unrolled.  (Inlined
// by force, like every helper of this kernel: a real call gives the kernel a stack,
// and every wave of it a slower start.)
__device__ __forceinline__ int finish_fast(int group, FastShared& fs, unsigned long long fm_mine,
                                           const int (&wg_cnt)[kChainWaves - 1], int (*sh_before)[64],
                                           int (*sh_all)[64], int (*own_base)[64], int* own_offsets,
                                           const RouteArgs& a, const Workspace& ws,
                                           int32_t* __restrict__ loads_inout,
                                           int32_t* __restrict__ expert_offsets) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int ntiles = a.ntiles;
  const int t0 = group * kChainWaves;
  const int tile = t0 + wave;

  // ---- the flexible tiles (wave w looked at tiles 64w .. 64w+63) ---------------------
  {
    const unsigned long long bal = __builtin_amdgcn_ballot_w64(fm_mine != 0ull);
    if (fm_mine != 0ull) fs.fmtile[threadIdx.x] = fm_mine;
    if (lane == 0) fs.bal[wave] = bal;
  }
  __syncthreads();
  unsigned long long bal[kChainWaves];
  int nft = 0;
#pragma unroll
  for (int w = 0; w < kChainWaves; ++w) {
    const unsigned long long b = fs.bal[w];
    bal[w] = ((unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(b >> 32)) << 32) |
             (unsigned)__builtin_amdgcn_readfirstlane((unsigned)b);
    nft += __builtin_popcountll(bal[w]);
  }
  if (nft > kFastTiles) return 0;
  // in ascending order, with their masks and the number of flexible tokens
  int ftile[kFastTiles];
  unsigned long long fmask[kFastTiles];
  int ntok = 0;
#pragma unroll
  for (int f = 0; f < kFastTiles; ++f) {
    ftile[f] = 0x7fffffff;
    fmask[f] = 0ull;
    if (f < nft) {
      int tl = 0;
      bool found = false;
#pragma unroll
      for (int w = 0; w < kChainWaves; ++w) {
        if (!found && bal[w] != 0ull) {
          tl = 64 * w + __builtin_ctzll(bal[w]);
          bal[w] &= bal[w] - 1ull;
          found = true;
        }
      }
      ftile[f] = tl;
      const unsigned long long m = fs.fmtile[tl];
      fmask[f] = ((unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(m >> 32)) << 32) |
                 (unsigned)__builtin_amdgcn_readfirstlane((unsigned)m);
      ntok += __builtin_popcountll(fmask[f]);
    }
  }
  if (!fast_path_applies(ntiles, nft, ntok, a.cw)) return 0;

  // ---- lane n < ntok: the n-th flexible token of the call ---------------------------
  int my_tok = 0, my_slot = 0, my_f = 0;
  {
    int r = lane;
#pragma unroll
    for (int f = 0; f < kFastTiles - 1; ++f) {
      const int pc = __builtin_popcountll(fmask[f]);
      if (my_f == f && r >= pc) {
        r -= pc;
        my_f = f + 1;
      }
    }
    unsigned long long m = fmask[0];
    int tl = ftile[0];
#pragma unroll
    for (int f = 1; f < kFastTiles; ++f) {
      m = my_f == f ? fmask[f] : m;
      tl = my_f == f ? ftile[f] : tl;
    }
    if (lane < ntok) {
      for (int i = 0; i < r; ++i) m &= m - 1ull;  // (r < kFastTokens)
      my_tok = tl * kTile + __builtin_ctzll(m);
      my_slot = tl * kTile + r;
    }
  }

  // ---- loads: wave w fetches what belongs to tokens w and w + 4; every wave the
  // tiles' counts once more (one batch; they are near, having just been read) ----------
  static_assert(kFastTokens <= 2 * kChainWaves, "two tokens per wave");
  static_assert(kFastMaxTiles == kTailThreads, "thread i looks at tile i");
  unsigned rv[2];
  float pv[2];
  int tk[2], tf[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int n = wave + h * kChainWaves;
    rv[h] = 0xFFFFu;
    pv[h] = 0.0f;
    tk[h] = tf[h] = 0;
    if (n < ntok) {
      const int slot = __builtin_amdgcn_readlane(my_slot, n);
      tk[h] = __builtin_amdgcn_readlane(my_tok, n);
      tf[h] = __builtin_amdgcn_readlane(my_f, n);
      // lanes 0..EP-1: the record row; then 4 lanes each for the two id rows, 16 for the
      // probabilities, one for the denominator -- as bits, sorted out after the wait
      if (lane < a.EP) rv[h] = ws.rec_lane[(size_t)slot * a.EP + lane];
      const unsigned* extra = lane < 4    ? reinterpret_cast<const unsigned*>(ws.rec_cids) + (size_t)slot * 4 + lane
                              : lane < 8  ? reinterpret_cast<const unsigned*>(ws.rec_ids) + (size_t)tk[h] * 4 + (lane - 4)
                              : lane < 24 ? reinterpret_cast<const unsigned*>(ws.rec_p) + (size_t)tk[h] * 16 + (lane - 8)
                                          : reinterpret_cast<const unsigned*>(ws.rec_Z) + tk[h];
      if (lane < 25) pv[h] = __uint_as_float(*extra);
    }
  }
  const int lin = ws.lin_copy[lane];
  const int sub = lane >> 4;  // which of the 4 tiles of a count load
  const unsigned* cnt32 = reinterpret_cast<const unsigned*>(ws.tile_fixed_cnt);
  constexpr int kBatch = kFastMaxTiles / (4 * kChainWaves);  // 16 loads cover 256 tiles
  unsigned wd[kBatch];
#pragma unroll
  for (int u = 0; u < kBatch; ++u) {
    const int tl = 4 * (wave + u * kChainWaves) + sub;
    wd[u] = tl < ntiles ? cnt32[(size_t)tl * 16 + (lane & 15)] : 0u;
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int n = wave + h * kChainWaves;
    if (n < ntok) {
      fs.rec[n][lane] = rv[h];
      const unsigned bits = __float_as_uint(pv[h]);
      if (lane < 4) reinterpret_cast<unsigned*>(&fs.cids[n])[lane] = bits;
      else if (lane < 8) reinterpret_cast<unsigned*>(fs.rids[n])[lane - 4] = bits;
      else if (lane < 24) fs.p[n][lane - 8] = pv[h];
      else if (lane == 24) fs.Z[n] = pv[h];
      if (lane == 0) {
        fs.tok[n] = tk[h];
        fs.tokf[n] = tf[h];
      }
    }
  }

  // ---- fixed assignments before each flexible tile -----------------------------------
#pragma unroll
  for (int f = 0; f < kFastTiles; ++f) {
    if (f < nft) {
      unsigned c02 = 0u, c13 = 0u;
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int tl = 4 * (wave + u * kChainWaves) + sub;
        c02 += tl < ftile[f] ? (wd[u] & 0x00FF00FFu) : 0u;
        c13 += tl < ftile[f] ? ((wd[u] >> 8) & 0x00FF00FFu) : 0u;
      }
#pragma unroll
      for (int d = 16; d < 64; d <<= 1) {
        c02 += __shfl_xor(c02, d, 64);
        c13 += __shfl_xor(c13, d, 64);
      }
      if (lane < 16) {
        const int e = 4 * lane;
        fs.fbefore[f][wave][e] = c02 & 0xFFFF;
        fs.fbefore[f][wave][e + 1] = c13 & 0xFFFF;
        fs.fbefore[f][wave][e + 2] = c02 >> 16;
        fs.fbefore[f][wave][e + 3] = c13 >> 16;
      }
    }
  }
  __syncthreads();

  // ---- wave 0 walks the flexible tokens (lane = expert), as the sequential chain does ----
  if (wave == 0) {
    int gflex = 0;
    for (int n = 0; n < ntok; ++n) {
      const int f = __builtin_amdgcn_readfirstlane(fs.tokf[n]);
      int base = lin + gflex;
#pragma unroll
      for (int w = 0; w < kChainWaves; ++w) base += fs.fbefore[f][w][lane];
      const unsigned rec = fs.rec[n][lane];
      const bool cand = lane < a.EP && rec != 0xFFFFu;
      const unsigned key = cand ? (((unsigned)base << 4) + rec) : 0xFFFFFFFFu;
      const bool chosen = chain_step(key, cand, fs.cids[n], a.k);
      gflex += chosen ? 1 : 0;
      const unsigned long long em = __builtin_amdgcn_ballot_w64(chosen);
      if (lane == 0) fs.emask[n] = em;
    }
  }
  __syncthreads();

  // ---- as on the path without flexible tokens, plus the flexible choices ------------
  int before = 0, all = 0, flex_before = 0, flex_all = 0;  // lane = expert
#pragma unroll
  for (int w = 0; w < kChainWaves; ++w) {
    before += sh_before[w][lane];
    all += sh_all[w][lane];
  }
#pragma unroll
  for (int j = 0; j < kChainWaves - 1; ++j) before += wg_cnt[j];
  for (int n = 0; n < ntok; ++n) {
    const int bit = (int)((fs.emask[n] >> lane) & 1ull);
    flex_all += bit;
    flex_before += (fs.tok[n] < tile * kTile) ? bit : 0;
  }
  own_base[wave][lane] = before + flex_before;
  const int cnt = lane < a.E ? all + flex_all : 0;
  if (wave == 0) {
    int incl = cnt;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int up = __shfl_up(incl, d, 64);
      if (lane >= d) incl += up;
    }
    own_offsets[lane] = incl - cnt;
    if (group == 0) {
      // the chain workgroup leaves such calls alone: the totals are written here
      if (lane < a.E) {
        loads_inout[lane] = lin + cnt;
        expert_offsets[lane] = incl - cnt;
      }
      if (lane == a.E - 1) expert_offsets[a.E] = incl;
    }
  }
  __syncthreads();
  return ntok;
}

// Load-dependent tokens of a call of at most kSelfPrefixTiles tiles, by the whole workgroup.
__device__ __forceinline__ int count_flexible(int ntiles, const Workspace& ws) {
  __shared__ int found[kChainWaves];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  int n = 0;
#pragma unroll
  for (int u = 0; u < kSelfPrefixTiles / kTailThreads; ++u) {
    const int tile = threadIdx.x + u * kTailThreads;
    n += __builtin_popcountll(tile < ntiles ? ws.flexmask[tile] : 0ull);
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) n += __shfl_xor(n, d, 64);
  if (lane == 0) found[wave] = n;
  __syncthreads();
  n = 0;
  for (int w = 0; w < kChainWaves; ++w) n += found[w];
  return __builtin_amdgcn_readfirstlane(n);
}

// Finishing workgroup `group` of the tail grid (kTailThreads threads): tiles kChainWaves * group ... .
// tail_lds: kChainLdsBytes of LDS.  BLOCKS: see finish_tile_of_chain.
template <bool BLOCKS>
__device__ __forceinline__ void finish_role(int group, uint8_t* tail_lds, FinishShared& S, const RouteArgs& a,
                                           const Workspace& ws, int32_t* __restrict__ loads_inout,
                                           int32_t* __restrict__ expert_offsets,
                                           int32_t* __restrict__ expert_ids, float* __restrict__ weights,
                                           int32_t* __restrict__ permutation) {
  auto& sh_before = S.sh_before;
  auto& sh_all = S.sh_all;
  auto& own_base = S.own_base;
  auto& own_offsets = S.own_offsets;
  auto& sh_anyflex = S.sh_anyflex;
  FastShared& fs = S.fs;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int t0 = group * kChainWaves;
  const int tile = t0 + wave;
  // Small problems without flexible tokens need nothing from the chain workgroup:
  // every finishing workgroup sums the byte counts itself.
  FinishLds* fl = reinterpret_cast<FinishLds*>(tail_lds) + wave;
  const bool small = a.ntiles <= kSelfPrefixTiles;
  // (no barrier from here to the end of self_prefix: a barrier waits for every load in
  // flight, and the point is to have all of this workgroup's loads in flight at once)
  FinishPrologue pro;
  pro.cstar = 0;
  pro.fm = 0ull;
  pro.tmask = 0ull;
  if (tile < a.ntiles) pro = finish_prologue(tile, a, ws, expert_ids);
  bool self = false;
  int fast_n = 0;  // flexible tokens resolved by this workgroup itself
  // fixed counts of the workgroup's earlier tiles (needed by the self path)
  int wg_cnt[kChainWaves - 1];
#pragma unroll
  for (int j = 0; j < kChainWaves - 1; ++j)
    wg_cnt[j] = (small && j < wave && t0 + j < a.ntiles) ? ws.tile_fixed_cnt[(size_t)(t0 + j) * 64 + lane] : 0;
  if (__builtin_expect(small, 1)) {
    unsigned long long fm_mine = 0ull;
    self_prefix(t0, a, ws, sh_before, sh_all, sh_anyflex, fm_mine);
    if (tile < a.ntiles) finish_commit(fl, pro, a.k);
    __syncthreads();
    self = (sh_anyflex[0] | sh_anyflex[1] | sh_anyflex[2] | sh_anyflex[3]) == 0;
    if (__builtin_expect(self, 1)) {
      int before = 0, all = 0;
      for (int w = 0; w < kChainWaves; ++w) {
        before += sh_before[w][lane];
        all += sh_all[w][lane];
      }
      int wg_before = 0;
#pragma unroll
      for (int j = 0; j < kChainWaves - 1; ++j) wg_before += wg_cnt[j];
      own_base[wave][lane] = before + wg_before;  // this wave's tile: plus the workgroup's earlier tiles
      if (wave == 0) {
        int incl = lane < a.E ? all : 0;
        const int cnt = incl;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const int up = __shfl_up(incl, d, 64);
          if (lane >= d) incl += up;
        }
        own_offsets[lane] = incl - cnt;
      }
    }
    __syncthreads();
    // a handful of flexible tokens: resolved here, by every workgroup for itself
    // (not in a pipelined call: there the chain workgroup walks every flexible token)
    if (__builtin_expect(!self && a.ntiles <= kFastMaxTiles && a.nseg == 0, 0)) {
      fast_n = finish_fast(group, fs, fm_mine, wg_cnt, sh_before, sh_all, own_base, own_offsets, a, ws, loads_inout,
                           expert_offsets);
      self = fast_n > 0;
    }
  } else if (tile < a.ntiles) {
    finish_commit(fl, pro, a.k);
  }
  if (tile >= a.ntiles) return;
  if (__builtin_expect(self, 1))
    finish_tile(fl, tile, pro, a, ws, expert_ids, weights, permutation, own_base[wave], own_offsets, fast_n, &fs);
  else
    finish_tile_of_chain<BLOCKS>(fl, tile, pro, a, ws, expert_offsets, expert_ids, weights, permutation);
}

}  // namespace laser
