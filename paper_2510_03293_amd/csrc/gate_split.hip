// The bf16 gate projection and analysis of small calls: the contraction axis of a tile
// cut over several workgroups (see the comment above the kernel).
#include <atomic>

#include "gate_tile.h"
#include "tail.h"

namespace laser {

// ---- small calls (at most a quarter as many tiles as the chip has compute units) ------
//
// In gate_analyse_bf16_kernel one workgroup streams the 64 rows of its tile and all of W
// through one compute unit; with a handful of tiles the rest of the chip idles while that
// unit pulls its half megabyte at what one unit can pull.  Here the eight wavefront roles
// of that kernel -- role r owns the chunks r, r + 8, ... of the contraction axis, from
// load to MFMA, in the same order -- go to `split` workgroups of 8 / split roles each.
// Every workgroup leaves its roles' partial tiles in the workspace (stored write-through)
// and, all stores acknowledged, counts itself into the tile's counter; the workgroup that
// finds the count complete fetches the eight partial tiles (agent-scope loads), and goes on
// exactly as the other kernel does: the analysis adds the same eight partial tiles in the
// same order, so the logits, and with them everything else, are bit for bit those of a
// call that is not split.  Nobody waits for anybody.
//
// The counters must be zero before the first workgroup arrives and the caller's workspace
// holds whatever it held, so they live in the library's own memory: an array that is part
// of the code object (zero when it is loaded) of which every workspace address gets a slice
// on first sight.  The last workgroup of a tile sets the tile's counter back to zero.  Calls
// that share a workspace must not overlap anyway, so a slice has one user at a time.

// The load-dependent tokens of a one-tile call, by the workgroup that analysed it.
struct OneTile {
  unsigned rec[kTile + 1][64];         // the n-th one's record row (lane = expert); kSeqNoCand: no candidate
  uint8_t cids[kTile + 1][16];         // its candidates by rank, padded (one row of read-ahead)
  __align__(16) uint8_t rids[kTile][16];  // its experts by rank
  __align__(16) float p[kTile][16];    // their probabilities
  float Z[kTile];                      // the softmax denominator
  int cstar[kTile], tok[kTile];        // candidates, token
  unsigned long long chosen[kTile];    // the experts chosen for it
};
static_assert(sizeof(OneTile) <= kGateLdsBytes, "the partial tiles are dead by then");

// `fm`: those tokens; `lin` (wave 0, lane = expert): the counters before token 0.  Writes their
// ids and weights and adds them to mask64.  All 512 threads; ends with a barrier.
__device__ __forceinline__ void finish_flexible(OneTile& ot, unsigned long long fm, unsigned long long* mask64, int lin,
                                                const RouteArgs& a, const Workspace& ws,
                                                int32_t* __restrict__ expert_ids, float* __restrict__ weights) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int n_flex = __builtin_popcountll(fm);
  // ---- the records, wave w those of tokens number w, w + 8, ..., all in flight together ----
  {
    constexpr int kPer = kTile / kGateWaves;
    unsigned rec[kPer], more[kPer];
    int tok[kPer];
    unsigned long long left = fm;
    for (int i = 0; i < wave; ++i) left &= left - 1ull;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int n = wave + u * kGateWaves;  // (the slot of a one-tile call's n-th flexible token)
      rec[u] = 0xFFFFu;
      more[u] = 0u;
      tok[u] = 0;
      if (n < n_flex) {
        tok[u] = __builtin_ctzll(left);
        for (int i = 0; i < kGateWaves; ++i) left &= left - 1ull;
        if (lane < a.EP) rec[u] = ws.rec_lane[(size_t)n * a.EP + lane];
        // lanes 0..3 and 4..7: the two id rows, 8..23: the probabilities, 24: the denominator
        const unsigned* src = lane < 4    ? reinterpret_cast<const unsigned*>(ws.rec_cids) + n * 4 + lane
                              : lane < 8  ? reinterpret_cast<const unsigned*>(ws.rec_ids) + tok[u] * 4 + (lane - 4)
                              : lane < 24 ? reinterpret_cast<const unsigned*>(ws.rec_p) + tok[u] * 16 + (lane - 8)
                                          : reinterpret_cast<const unsigned*>(ws.rec_Z) + tok[u];
        if (lane < 25) more[u] = *src;
        if (lane == 25) more[u] = ws.rec_cstar[tok[u]];
      }
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int n = wave + u * kGateWaves;
      if (n < n_flex) {
        ot.rec[n][lane] = rec[u] == 0xFFFFu ? kSeqNoCand : rec[u];
        if (lane < 4) reinterpret_cast<unsigned*>(ot.cids[n])[lane] = more[u];
        else if (lane < 8) reinterpret_cast<unsigned*>(ot.rids[n])[lane - 4] = more[u];
        else if (lane < 24) ot.p[n][lane - 8] = __uint_as_float(more[u]);
        else if (lane == 24) ot.Z[n] = __uint_as_float(more[u]);
        else if (lane == 25) ot.cstar[n] = (int)more[u];
        else if (lane == 26) ot.tok[n] = tok[u];
      }
    }
  }
  __syncthreads();
  // ---- token after token, lane = expert -------------------------------------------------
  // What bounds it is one wavefront's chain of dependent instructions, as in the walks of the tail
  // kernel, so the next token's record is read while this one's keys are exchanged.  (64 tokens,
  // all load-dependent, 64 experts, c = 8, H = 2048: the call 37.7 -> 28.7 us, with 8 experts, c = 4,
  // H = 4096 31.6 -> 24.8.)
  if (wave == 0) {
    unsigned base = (unsigned)lin;  // (the fixed tokens before a token are in its record)
    unsigned em_lo = 0, em_hi = 0;  // lane n: the experts chosen for token n
    unsigned rec = ot.rec[0][lane];
    auto keep = [&](int n, bool chosen) {
      const unsigned long long em = __builtin_amdgcn_ballot_w64(chosen);
      em_lo = lane == n ? (unsigned)em : em_lo;
      em_hi = lane == n ? (unsigned)(em >> 32) : em_hi;
      base += chosen ? 1u : 0u;
    };
    if (a.c <= 8) {
      // all pairs of candidates by rank (i, j) = (lane / 8, lane % 8) at once: byte i of the
      // comparisons has fewer than k bits
      unsigned ai = ot.cids[0][lane >> 3], aj = ot.cids[0][lane & 7];
      for (int n = 0; n < n_flex; ++n) {
        const unsigned key = (base << 4) + rec;
        const unsigned ki = (unsigned)__builtin_amdgcn_ds_bpermute((int)(4 * ai), (int)key);
        const unsigned kj = (unsigned)__builtin_amdgcn_ds_bpermute((int)(4 * aj), (int)key);
        __builtin_amdgcn_sched_barrier(0);
        const unsigned rec_n = ot.rec[n + 1][lane];
        const unsigned ai_n = ot.cids[n + 1][lane >> 3], aj_n = ot.cids[n + 1][lane & 7];
        const int shift = 8 * (int)(rec & 7u), none = (int)rec < 0 ? 64 : 0;
        __builtin_amdgcn_sched_barrier(0);
        const unsigned long long less = __builtin_amdgcn_ballot_w64(kj < ki);
        const int before = __builtin_popcount((unsigned)(less >> shift) & 0xFFu) + none;
        keep(n, before < a.k);
        rec = rec_n;
        ai = ai_n;
        aj = aj_n;
      }
    } else {
      uint4 ids = *reinterpret_cast<const uint4*>(ot.cids[0]);
      for (int n = 0; n < n_flex; ++n) {
        const unsigned key = (base << 4) + rec;
        const bool cand = (int)rec >= 0;
        rec = ot.rec[n + 1][lane];
        const uint4 ids_n = *reinterpret_cast<const uint4*>(ot.cids[n + 1]);
        keep(n, chain_step(key, cand, ids, a.k));
        ids = ids_n;
      }
    }
    ot.chosen[lane] = ((unsigned long long)em_hi << 32) | em_lo;
  }
  __syncthreads();
  // ---- ids, weights, masks: thread = (token, one of eight), which has ranks q and q + 8 -----
  {
    const int n = threadIdx.x >> 3, q = threadIdx.x & 7;
    if (n < n_flex) {
      const unsigned long long em = ot.chosen[n];
      const int cs = ot.cstar[n], tok = ot.tok[n];
      const size_t row = (size_t)tok * a.k;
      const uint4 ids4 = *reinterpret_cast<const uint4*>(ot.rids[n]);
      const unsigned idw[4] = {ids4.x, ids4.y, ids4.z, ids4.w};
      unsigned ranks = 0;  // the chosen ranks
      float sum = 0.0f;    // their probabilities, added in the order of the ranks
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const unsigned e = (idw[j >> 2] >> (8 * (j & 3))) & 63u;
        const bool chosen = j < cs && ((em >> e) & 1ull) != 0ull;
        ranks |= chosen ? 1u << j : 0u;
        sum = chosen ? sum + ot.p[n][j] : sum;
      }
      const float denom = a.renormalize ? sum : ot.Z[n];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int j = q + 8 * h;
        const int at = __builtin_popcount(ranks & ((1u << j) - 1u));
        if (((ranks >> j) & 1u) != 0u && at < a.k) {  // (exactly k are chosen; at < k keeps the row)
          const int e = ot.rids[n][j];
          expert_ids[row + at] = e;
          weights[row + at] = ot.p[n][j] / denom;
          atomicOr(&mask64[e], 1ull << tok);
        }
      }
    }
  }
  __syncthreads();
}

template <int EB, int NE, int NR, bool STATS, bool BATCH>  // NR: wavefront roles per workgroup, 1 or 2
__global__ __launch_bounds__(kGateThreads) void gate_split_bf16_kernel(
    const uint16_t* __restrict__ hidden, const uint16_t* __restrict__ w, int H, const RouteArgs a0,
    const Workspace ws0, int32_t* __restrict__ expert_ids, float* __restrict__ weights,
    float* __restrict__ logits_out, size_t logits_stride) {
  static_assert(NR == 1 || NR == 2, "one or two roles per workgroup");
  extern __shared__ __align__(16) unsigned char gate_lds[];
  __shared__ unsigned long long mask64[64];
  __shared__ unsigned long long flex_lds;
  __shared__ int sh_last;
  // (blockIdx.y: the problem of a batched call)
  const int prob = BATCH ? blockIdx.y : 0;
  RouteArgs a = BATCH ? problem_args(a0, prob) : a0;
  const Workspace ws = BATCH ? problem_workspace(ws0, (size_t)prob * a0.ws_stride) : ws0;
  if (STATS && a.pool_in_ws) a.st_pool = ws.pool;
  if (BATCH) {
    hidden += (size_t)prob * a.T * H;
    w += (size_t)prob * a.E * H;
    expert_ids += (size_t)prob * a.T * a.k;
    weights += (size_t)prob * a.T * a.k;
    logits_out = logits_out != nullptr ? logits_out + (size_t)prob * logits_stride : nullptr;
  }
  const int T = a.T, E = a.E;
  constexpr int split = kGateWaves / NR;  // workgroups per tile (the launcher sees to a.split == split)
  constexpr int nroles = NR;
  // (the workgroups of a tile are ntiles apart in the grid)
  const int tile = (int)blockIdx.x % a.ntiles;
  const int part_of_tile = (int)blockIdx.x / a.ntiles;
  const int wave = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);

  // The chunks of role r are those of wave r of the unsplit kernel, in its order: chunk i
  // is (start + 8 i) mod nfull.  Here the chunks of the workgroup's roles form one list
  // (role by role); wave v of the workgroup loads and stages item v + 8 n in round n, so
  // that all items of a round are in flight at once (the projection shapes with 2048 or
  // 4096 columns are one or two rounds).  Then four waves per role multiply the round's
  // chunks of that role, in the role's order, each into its own 16x16 blocks of the role's
  // partial tile (a 2x2 patch of blocks for 64 experts: two operands of each kind per
  // product step instead of three for two blocks).  Block (eb, tb) accumulates exactly the
  // products it accumulates in the unsplit kernel, in the same order, whoever runs the
  // instructions.
  constexpr int EBW = EB >= 4 ? 2 : 1;  // expert blocks per multiplying wave
  constexpr int TBW = EB >= 2 ? 2 : 1;  // token blocks per multiplying wave
  const int mrole = NR == 2 ? wave_u >> 2 : 0;       // the role this wave multiplies for ...
  const bool multiplies = NR == 2 || wave_u < 4;     // ... if it does
  const int mq = wave_u & 3;
  const int eb0 = EB >= 4 ? 2 * (mq >> 1) : EB == 2 ? (mq >> 1) : 0;
  const int tb0 = EB >= 2 ? 2 * (mq & 1) : mq;
  f32x4 acc[EBW][TBW];
#pragma unroll
  for (int e = 0; e < EBW; ++e)
#pragma unroll
    for (int t = 0; t < TBW; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[e][t][r] = 0.0f;

  const int lrow = lane >> 3, lpiece = lane & 7;
  const size_t row_bytes = (size_t)H * 2;
  const unsigned char* hbase = reinterpret_cast<const unsigned char*>(hidden) + (size_t)tile * kTile * row_bytes;
  const unsigned char* wbase = reinterpret_cast<const unsigned char*>(w);
  const int last_row = T - 1 - tile * kTile;  // >= 0
  unsigned hoff[8], woff[2 * EB];
#pragma unroll
  for (int q = 0; q < 8; ++q) hoff[q] = (unsigned)(min(q * 8 + lrow, last_row) * row_bytes) + lpiece * 16;
#pragma unroll
  for (int q = 0; q < 2 * EB; ++q) woff[q] = (unsigned)(min(q * 8 + lrow, E - 1) * row_bytes) + lpiece * 16;
  unsigned char* st_wr = gate_lds + wave_u * kStripBytes + lrow * kRowBytes + lpiece * 16;
  const unsigned rd_lane = (lane & 15) * kRowBytes + (lane >> 4) * 16;

  const int nfull = H >> 6;
  // per role: its full chunks, where it starts, and whether the ragged end of the
  // contraction axis (H % 64 != 0) is its to take, after its full chunks, as in the unsplit
  // kernel (pieces past H are read from the start of the row instead and replaced by zeros)
  int nmine[NR], start[NR], nitem[NR];
#pragma unroll
  for (int rr = 0; rr < NR; ++rr) {
    const int role = part_of_tile * NR + rr;
    nmine[rr] = (nfull - role + kGateWaves - 1) / kGateWaves;
    start[rr] = nfull > 0 ? (tile * 5 + role) % nfull : 0;
    nitem[rr] = nmine[rr] + (((H & 63) != 0 && role == (nfull & (kGateWaves - 1))) ? 1 : 0);
  }
  const int nitems = nitem[0] + (NR == 2 ? nitem[NR - 1] : 0);
  const u32x4 zero4 = {0u, 0u, 0u, 0u};

  u32x4 rh[8], rw[2 * EB];
  auto load_item = [&](int it) {
    const int rr = (NR == 2 && it >= nitem[0]) ? 1 : 0;
    const int i = it - (rr ? nitem[0] : 0);
    if (i < nmine[rr]) {  // chunk i of the role
      const int koff = ((start[rr] + kGateWaves * i) % nfull) * 128;
      GATE_GH(rh, koff)
      GATE_GW(rw, koff)
    } else {  // the ragged end
      const bool kin = nfull * 64 + lpiece * 8 < H;  // H % 8 == 0: a piece is all in or all out
      const int off = kin ? nfull * 128 : -lpiece * 16;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const u32x4 v = load_global_16(hbase + hoff[q] + off);
        rh[q] = kin ? v : zero4;
      }
#pragma unroll
      for (int q = 0; q < 2 * EB; ++q) {
        const u32x4 v = load_global_16(wbase + woff[q] + off);
        rw[q] = kin ? v : zero4;
      }
    }
  };
  // the item in strip j, if it is one of this wave's role
  auto multiply = [&](int j) {
    const unsigned char* st_rd = gate_lds + j * kStripBytes + rd_lane;
#pragma unroll
    for (int s_ = 0; s_ < 2; ++s_) {
      u32x4 a_[EBW], b_[TBW];
#pragma unroll
      for (int t = 0; t < TBW; ++t) b_[t] = *(lds_u4_ptr)(st_rd + (tb0 + t) * 16 * kRowBytes + s_ * 64);
#pragma unroll
      for (int e = 0; e < EBW; ++e)
        a_[e] = *(lds_u4_ptr)(st_rd + kTile * kRowBytes + (eb0 + e) * 16 * kRowBytes + s_ * 64);
#pragma unroll
      for (int e = 0; e < EBW; ++e)
#pragma unroll
        for (int t = 0; t < TBW; ++t)
          acc[e][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a_[e]),
                                                              __builtin_bit_cast(bf16x8, b_[t]), acc[e][t], 0, 0, 0);
    }
  };
  if (wave_u < nitems) load_item(wave_u);
  for (int r0 = 0; r0 < nitems; r0 += kGateWaves) {
    if (r0 + wave_u < nitems) {
      GATE_S(rh, rw)  // (waits for the loads)
    }
    __syncthreads();
    // the next round's loads travel while this round is multiplied
    if (r0 + kGateWaves + wave_u < nitems) load_item(r0 + kGateWaves + wave_u);
    if (multiplies) {
      // strips [j0, j1) hold this wave's role's items of the round
      const int lo = mrole == 0 ? 0 : nitem[0], hi = mrole == 0 ? nitem[0] : nitems;
      const int j0 = max(lo - r0, 0), j1 = min(min(hi - r0, kGateWaves), nitems - r0);
      // (written out for the usual sizes, so that the operand reads of a chunk do not wait
      // for the products of the chunk before)
      if (j1 - j0 == 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) multiply(j0 + j);
      } else if (j1 - j0 == 8) {
#pragma unroll
        for (int j = 0; j < 8; ++j) multiply(j);
      } else {
        for (int j = j0; j < j1; ++j) multiply(j);
      }
    }
    __syncthreads();  // the strips are free again (after the last round: dead, the partial tiles reuse the space)
  }
  if (nitems == 0) __syncthreads();

  float* part = reinterpret_cast<float*>(gate_lds);  // [roles][64][kPartStride]
  if (multiplies) {
    const int n = lane & 15, kgrp = lane >> 4;
    float* mine = part + (size_t)mrole * kTile * kPartStride;
#pragma unroll
    for (int e = 0; e < EBW; ++e)
#pragma unroll
      for (int t = 0; t < TBW; ++t) {
        const float4 v = make_float4(acc[e][t][0], acc[e][t][1], acc[e][t][2], acc[e][t][3]);
        *reinterpret_cast<float4*>(mine + ((tb0 + t) * 16 + n) * kPartStride + (eb0 + e) * 16 + 4 * kgrp) = v;
      }
  }
  __syncthreads();

  // ---- this workgroup's partial tiles -> workspace, 64 x 64 floats per role ------------
  // (element j of a role's tile, 8 bytes: row j / 32, columns 2 (j % 32) and the next)
  constexpr int kPairs = kTile * 64 / 2;  // 8-byte elements per partial tile
  auto lds_pair = [&](int r, int jj) {
    return reinterpret_cast<unsigned long long*>(part + ((size_t)r * kTile + (jj >> 5)) * kPartStride + 2 * (jj & 31));
  };
  unsigned long long* const tile_parts =
      reinterpret_cast<unsigned long long*>(ws.split_part) + (size_t)tile * kGateWaves * kPairs;
  {
    unsigned long long* dst = tile_parts + (size_t)part_of_tile * nroles * kPairs;
    for (int j = threadIdx.x; j < nroles * kPairs; j += kGateThreads)
      __hip_atomic_store(dst + j, *lds_pair(j / kPairs, j % kPairs), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // every store acknowledged ...
  __syncthreads();                                   // ... by every wavefront
  if (threadIdx.x == 0) {
    int32_t* counter = a.split_cnt + (size_t)prob * a.ntiles + tile;
    const int before = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int last = before == split - 1;
    if (last) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // for the next call
    sh_last = last;
  }
  __syncthreads();
  if (sh_last == 0) return;

  // ---- the last workgroup of the tile: all eight partial tiles -> LDS, then the analysis ----
  // Wave w fetches the tile of role w: 16 loads of 16 bytes per lane, 1 KiB per instruction
  // (with 8-byte loads the fetch took twice as long: the memory pipeline takes a wave's
  // instruction every 16 cycles whatever its width).  Agent-scope loads of 16 bytes exist
  // only as instructions, so they are written out, all of them and the wait for them in one
  // block: the compiler takes an output of a block as valid when the block ends.
  {
    const unsigned char* src = reinterpret_cast<const unsigned char*>(tile_parts) + (size_t)wave * (kPairs * 8) + lane * 16;
    const unsigned char *s0 = src, *s1 = src + 4096, *s2 = src + 8192, *s3 = src + 12288;
    u32x4 v[16];
    asm volatile(
        "global_load_dwordx4 %0, %16, off sc1\n\t"
        "global_load_dwordx4 %1, %16, off offset:1024 sc1\n\t"
        "global_load_dwordx4 %2, %16, off offset:2048 sc1\n\t"
        "global_load_dwordx4 %3, %16, off offset:3072 sc1\n\t"
        "global_load_dwordx4 %4, %17, off sc1\n\t"
        "global_load_dwordx4 %5, %17, off offset:1024 sc1\n\t"
        "global_load_dwordx4 %6, %17, off offset:2048 sc1\n\t"
        "global_load_dwordx4 %7, %17, off offset:3072 sc1\n\t"
        "global_load_dwordx4 %8, %18, off sc1\n\t"
        "global_load_dwordx4 %9, %18, off offset:1024 sc1\n\t"
        "global_load_dwordx4 %10, %18, off offset:2048 sc1\n\t"
        "global_load_dwordx4 %11, %18, off offset:3072 sc1\n\t"
        "global_load_dwordx4 %12, %19, off sc1\n\t"
        "global_load_dwordx4 %13, %19, off offset:1024 sc1\n\t"
        "global_load_dwordx4 %14, %19, off offset:2048 sc1\n\t"
        "global_load_dwordx4 %15, %19, off offset:3072 sc1\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7]),
          "=&v"(v[8]), "=&v"(v[9]), "=&v"(v[10]), "=&v"(v[11]), "=&v"(v[12]), "=&v"(v[13]), "=&v"(v[14]),
          "=&v"(v[15])
        : "v"(s0), "v"(s1), "v"(s2), "v"(s3)
        : "memory");
    // bytes 1024 u + 16 lane of the tile = row 4 u + lane / 16, columns 4 (lane % 16) ...
#pragma unroll
    for (int u = 0; u < 16; ++u)
      *reinterpret_cast<u32x4*>(part + ((size_t)wave * kTile + 4 * u + (lane >> 4)) * kPartStride + 4 * (lane & 15)) = v[u];
  }
  __syncthreads();
  analyse_tile<NE, kGateWaves, STATS>(part, kPartStride, mask64, &flex_lds, tile, a, ws, expert_ids, weights,
                                      logits_out);

  // ---- a call of one tile ends here ------------------------------------------------------
  // Everything the rest needs is in this workgroup: the records of the load-dependent tokens,
  // per expert the other tokens assigned to it (mask64) and, just written, the tokens' experts
  // in rank order.  What follows is what the tail kernel would do, without its launch and the
  // way of all of this through memory.  (64 tokens, 64 experts, H = 2048: split kernel and tail
  // 10.5 + 4.4 us, now 10.1; 27 such layers replayed from a graph 355 -> 301 us.)
  if (a.one_permutation != nullptr) {  // (a.ntiles == 1)
    int32_t* const permutation = a.one_permutation + (size_t)prob * T * a.k;
    int32_t* const expert_offsets = a.one_expert_offsets + (size_t)prob * (E + 1);
    int32_t* const loads = a.one_loads + (size_t)prob * E;
    __shared__ int sh_off[64];
    int lin = 0;
    if (wave == 0 && lane < E) lin = loads[lane];
    __syncthreads();  // expert ids and records are stored, mask64 and flex_lds are final
    const unsigned long long fm = ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(flex_lds >> 32)) << 32) |
                                  (unsigned)__builtin_amdgcn_readfirstlane((int)flex_lds);
    // (out of the way of calls without any: 16 such problems in one call, 12.8 us with this code in the
    // middle, 12.3 with it at the end)
    if (__builtin_expect(fm != 0ull, 0))
      finish_flexible(*reinterpret_cast<OneTile*>(gate_lds), fm, mask64, lin, a, ws, expert_ids, weights);
    if (wave == 0) {  // lane = expert
      const int cnt = lane < E ? __builtin_popcountll(mask64[lane]) : 0;
      int incl = cnt;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_up(incl, d, 64);
        if (lane >= d) incl += up;
      }
      sh_off[lane] = incl - cnt;
      if (lane < E) {
        expert_offsets[lane] = incl - cnt;
        loads[lane] = lin + cnt;
      }
      if (lane == E - 1) expert_offsets[E] = incl;
    }
    __syncthreads();
    const int k = a.k;
    bool kept = true;
    for (int slot = threadIdx.x; slot < T * k; slot += kGateThreads) {
      const int t = slot / k;
      const int e = expert_ids[slot];
      // (an expert's number, and a slot's, by construction; the checks turn any inconsistency of
      // the inputs into a missing entry instead of a stray store)
      const int pos = sh_off[e & 63] + __builtin_popcountll(mask64[e & 63] & lanes_below(t));
      const bool ok = (unsigned)e < (unsigned)E && (unsigned)pos < (unsigned)(T * k);
      if (ok) permutation[pos] = slot;
      kept = kept && ok;
    }
    if (!kept) ws.status[kStatusError] = kErrorInconsistent;
  }
}

// ---- the counters ---------------------------------------------------------------------
constexpr int kSplitSlices = 1024;
static __device__ int32_t split_counters[kSplitSlices * kSplitMaxTiles];

struct SplitTable {
  std::atomic<uintptr_t> key[kSplitSlices];  // workspace address that owns the slice, 0: free
  std::atomic<int32_t*> base;                // the array's address on this device
};
static SplitTable g_split[kMaxDevices];

int32_t* split_counters_for(const void* workspace) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  SplitTable& t = g_split[dev];
  int32_t* base = t.base.load(std::memory_order_acquire);
  if (base == nullptr) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(split_counters)) != hipSuccess || p == nullptr) {
      (void)hipGetLastError();
      return nullptr;
    }
    base = static_cast<int32_t*>(p);
    t.base.store(base, std::memory_order_release);
  }
  const uintptr_t k = reinterpret_cast<uintptr_t>(workspace);
  const unsigned h = (unsigned)((k >> 8) * 0x9E3779B1u);
  for (int probe = 0; probe < 64; ++probe) {
    const unsigned i = (h + (unsigned)probe) % kSplitSlices;
    uintptr_t cur = t.key[i].load(std::memory_order_acquire);
    if (cur == 0) {
      if (t.key[i].compare_exchange_strong(cur, k, std::memory_order_acq_rel)) cur = k;
      // (on failure `cur` holds what another thread put there)
    }
    if (cur == k) return base + (size_t)i * kSplitMaxTiles;
  }
  return nullptr;  // the table is crowded: the call runs without the split
}

template <int EB, int NE, int NR, bool STATS, bool BATCH>
static hipError_t launch_split(const void* hidden, const void* w, int H, const RouteArgs& a, const Workspace& ws,
                               int32_t* expert_ids, float* weights, float* logits_out, size_t logits_stride,
                               hipStream_t s) {
  static LdsAttr allowed;
  const void* fn = reinterpret_cast<const void*>(&gate_split_bf16_kernel<EB, NE, NR, STATS, BATCH>);
  const hipError_t e = allow_dynamic_lds(fn, kGateLdsBytes, allowed);
  if (e != hipSuccess) return e;
  if (a.split * NR != kGateWaves || a.ntiles * a.nbatch > kSplitMaxTiles) return hipErrorInvalidValue;
  clear_stale_error();
  hipLaunchKernelGGL((gate_split_bf16_kernel<EB, NE, NR, STATS, BATCH>), dim3(a.ntiles * a.split, a.nbatch),
                     dim3(kGateThreads), kGateLdsBytes, s, static_cast<const uint16_t*>(hidden),
                     static_cast<const uint16_t*>(w), H, a, ws, expert_ids, weights, logits_out, logits_stride);
  return hipGetLastError();
}

template <int EB, int NE, int NR>
static hipError_t launch_split_nr(const void* hidden, const void* w, int H, const RouteArgs& a, const Workspace& ws,
                                  int32_t* expert_ids, float* weights, float* logits_out, size_t logits_stride,
                                  hipStream_t s) {
  const bool st = wants_stats(a);
  if (a.nbatch > 1) {
    if (st) return launch_split<EB, NE, NR, true, true>(hidden, w, H, a, ws, expert_ids, weights, logits_out, logits_stride, s);
    return launch_split<EB, NE, NR, false, true>(hidden, w, H, a, ws, expert_ids, weights, logits_out, logits_stride, s);
  }
  if (st) return launch_split<EB, NE, NR, true, false>(hidden, w, H, a, ws, expert_ids, weights, logits_out, logits_stride, s);
  return launch_split<EB, NE, NR, false, false>(hidden, w, H, a, ws, expert_ids, weights, logits_out, logits_stride, s);
}

template <int EB, int NE>
static hipError_t launch_split_one(const void* hidden, const void* w, int H, const RouteArgs& a, const Workspace& ws,
                                   int32_t* expert_ids, float* weights, float* logits_out, size_t logits_stride,
                                   hipStream_t s) {
  if (a.split == kGateWaves)
    return launch_split_nr<EB, NE, 1>(hidden, w, H, a, ws, expert_ids, weights, logits_out, logits_stride, s);
  return launch_split_nr<EB, NE, 2>(hidden, w, H, a, ws, expert_ids, weights, logits_out, logits_stride, s);
}

hipError_t launch_gate_split_bf16(const void* hidden, const void* w, int H, const RouteArgs& a, const Workspace& ws,
                                  int32_t* expert_ids, float* weights, float* logits_out, size_t logits_stride,
                                  hipStream_t s) {
  switch (a.EP) {
    case 8: return launch_split_one<1, 1>(hidden, w, H, a, ws, expert_ids, weights, logits_out, logits_stride, s);
    case 16: return launch_split_one<1, 2>(hidden, w, H, a, ws, expert_ids, weights, logits_out, logits_stride, s);
    case 32: return launch_split_one<2, 4>(hidden, w, H, a, ws, expert_ids, weights, logits_out, logits_stride, s);
    default: return launch_split_one<4, 8>(hidden, w, H, a, ws, expert_ids, weights, logits_out, logits_stride, s);
  }
}

}  // namespace laser
