// Per-token analysis for Algorithm 1 with trimming mode RANDOM (Method: Final
// assignment, "trimming can be ... randomized (sampling c uniformly)"; appendix Pseudo
// Code, the RANDOM branch): a pool larger than c is cut down to a uniform sample of c
// of its members instead of its c best.  Everything else (scores, order, top-k mass
// test, pool, records for the chain, dispatch) is as in the deterministic analysis, in
// the same binary32 arithmetic and the same workspace layout, so the chain and the
// finishing pass do not know the difference.
//
// The sample must be reproducible, so it is defined by a counter-based generator:
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC 2011) with key = seed and counter =
// (token index low, token index high, stream, block); draw i of a token is word i % 4
// of block i / 4.  A partial Fisher-Yates shuffle of the pool's positions [0, m) in
// the score order swaps position i with i + floor(r_i * (m - i) / 2^32) for
// i = 0..c-1; the first c positions, in ascending order, are the candidates.
//
// Two kernels.  analyse_general_kernel is the whole analysis in either trimming mode.  It is
// used for RANDOM trimming where c == k (a sampled token is then not load-dependent, but its
// experts are the sample), and in both modes for trimming sizes above the 16 candidates that
// the fast analysis carries ("wide" calls: up to 64 candidates per token, e.g. the load-only
// baseline of the paper's evaluation, c = n).  Where 16 >= c > k the deterministic analysis
// already gives everything but the candidates of the tokens it trimmed, and
// random_resample_kernel only redoes those.
//
// Both give a token to one wavefront, lane = expert: the rank of the lane's expert is counted
// against the 64 logits read out one after the other (a lane read, a compare, an add each);
// the shuffle's positions are lanes, its draws and swaps scalars; the sample is a mask of
// positions, so that its ascending order costs nothing.  What bounds them is the issue of those
// instructions, about 400 per token, and waves enough to fill it: 16 per tile (see
// random_resample_kernel for calls of many tiles), which take up to four tokens at a time, whose logits
// are all on their way together and whose random blocks are drawn at once.  (12345 tokens, a tenth of them sampled, the call: 114 us with lane = token, one wavefront
// per tile behind a counting pass over E^2 values in LDS; 72 with four waves per tile, a token after the
// other; now 68.  64 tokens, all sampled, 16 experts: 44, 60, 42 us.  The whole analysis of 8192 tokens,
// 64 experts: 65 us with lane = token, now 17.)
#include "analyse.h"
#include "laser_internal.h"

namespace laser {

__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t (&out)[4]) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
    const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  out[0] = c0;
  out[1] = c1;
  out[2] = c2;
  out[3] = c3;
}

// Lane = expert: the number of experts before this lane's in the score order (logit
// descending, equal logits by lower index); lanes without an expert get their own number.
// Counted with bare logits (against the keys of the analysis, a lane read and a double comparison more per
// expert: the general analysis of 8192 tokens 20.2 -> 16.9 us, resampling 1214 tokens 8.0 -> 7.2).  Where
// two are equal, which shows in the sum of the counts, their counts are too, and the lanes below of the
// same count are added, which six ballots find.  (Logits rounded to bf16, 40000 tokens of 64 experts,
// c = k, the call: 77 us by keys, 104 when the keys were counted again for them, now 66; distinct ones 62.)
__device__ __forceinline__ int rank_of(float z, bool real, int lane, int E) {
  const float zr = real ? z : -__builtin_inff();
  int before = 0;
  for (int j0 = 0; j0 < E; j0 += 8) {
#pragma unroll
    for (int u = 0; u < 8; ++u)
      before += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(zr), j0 + u)) > zr ? 1 : 0;
  }
  before = real ? before : lane;
  constexpr int kRowMirror = 0x140, kRowBcast15 = 0x142, kRowBcast31 = 0x143;
  int sum = before;
  sum += dpp_int<kQuadXor1>(sum);
  sum += dpp_int<kQuadXor2>(sum);
  sum += dpp_int<kRowHalfMirror>(sum);
  sum += dpp_int<kRowMirror>(sum);
  sum += dpp_int<kRowBcast15>(sum);
  sum += dpp_int<kRowBcast31>(sum);
  if (__builtin_amdgcn_readlane(sum, 63) == 64 * 63 / 2) return before;
  unsigned long long same = ~0ull;  // lanes that counted as many
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    const bool set = ((before >> i) & 1) != 0;
    const unsigned long long m = __builtin_amdgcn_ballot_w64(set);
    same &= set ? m : ~m;
  }
  return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(same >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)same, (unsigned)before));
}

// Block lane % 16 of a token's generator (`g`: its number in the caller's numbering; at most
// 64 draws, so 16 blocks are all it can need).
__device__ __forceinline__ void draw_blocks(const RandomArgs& rnd, unsigned long long g, int lane, uint32_t (&w)[4]) {
  philox4x32_10((uint32_t)g, (uint32_t)(g >> 32), rnd.stream, (uint32_t)(lane & 15), (uint32_t)rnd.seed,
                (uint32_t)(rnd.seed >> 32), w);
}

// The sample of a token whose blocks are in lanes first, first + 1, ...: c of the positions
// [0, m), m <= 64, as a mask.
__device__ __forceinline__ unsigned long long sample_positions(const uint32_t (&w)[4], int first, int m, int c, int lane) {
  int at = lane;  // lane = place in the shuffled array: the position it holds
  unsigned long long picked = 0ull;
  for (int i = 0; i < c; ++i) {
    const int q = i & 3;
    const unsigned r = (unsigned)__builtin_amdgcn_readlane((int)(q == 0 ? w[0] : q == 1 ? w[1] : q == 2 ? w[2] : w[3]), first + (i >> 2));
    const int j = i + (int)(((unsigned long long)r * (unsigned)(m - i)) >> 32);  // i <= j < m
    // (place i is not looked at again: what it held goes to place j, what j held is drawn)
    const int ai = __builtin_amdgcn_readlane(at, i), aj = __builtin_amdgcn_readlane(at, j);
    at = lane == j ? ai : at;
    picked |= 1ull << aj;
  }
  return picked;
}

// Wave-uniform 64-bit value as a scalar.
__device__ __forceinline__ unsigned long long scalar64(unsigned long long x) {
  return ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32) |
         (unsigned)__builtin_amdgcn_readfirstlane((int)x);
}

// The records of a flexible token, lane = expert: `in` the expert is candidate number j (its
// position among the `ncand` candidates in score order) with the softmax numerator p; `pref`
// fixed tokens of the tile before the token were assigned to it.
__device__ __forceinline__ void write_records(const RouteArgs& a, const Workspace& ws, int t, int slot, int lane, bool in,
                                              int j, float p, int pref, int ncand) {
  const int cw = a.cw;
  const bool wide = cw > kMaxC;  // (the wide chain reads the per-expert rows only)
  // ranks beyond the working set point the chain at a lane that holds no candidate
  // (at most 16 of the 32 low experts are candidates unless the call is wide)
  const unsigned low = (unsigned)__builtin_amdgcn_ballot_w64(in);
  const int padlane = a.E < 64 ? a.E : wide ? 0 : __builtin_ctz(~low);
  if (in) {
    ws.rec_ids[(size_t)t * cw + j] = (uint8_t)lane;
    ws.rec_p[(size_t)t * cw + j] = p;
    if (!wide) {
      ws.rec_cids[(size_t)slot * 16 + j] = (uint8_t)lane;
      ws.rec_pref[(size_t)slot * 16 + j] = (uint8_t)pref;
    }
  }
  if (lane >= ncand && lane < cw) {
    ws.rec_ids[(size_t)t * cw + lane] = 0;
    ws.rec_p[(size_t)t * cw + lane] = 0.0f;
    if (!wide) {
      ws.rec_cids[(size_t)slot * 16 + lane] = (uint8_t)padlane;
      ws.rec_pref[(size_t)slot * 16 + lane] = 0xFF;
    }
  }
  if (lane < a.EP)
    ws.rec_lane[(size_t)slot * a.EP + lane] = in ? (uint16_t)((pref << (wide ? 6 : 4)) | j) : (uint16_t)0xFFFF;
}

constexpr int kGeneralWaves = 16;
constexpr int kGeneralTokens = kTile / kGeneralWaves;  // tokens of a wavefront

// SAMPLE: trimming mode RANDOM (otherwise the c best of the pool are kept).
template <bool SAMPLE>
__global__ __launch_bounds__(64 * kGeneralWaves) void analyse_general_kernel(const float* __restrict__ logits,
                                                            size_t logits_stride, const RouteArgs a0,
                                                            const Workspace ws0, const RandomArgs rnd0,
                                                            int32_t* __restrict__ expert_ids,
                                                            float* __restrict__ weights) {
  // blockIdx.y: the problem of a batched call; it draws with its own stream id
  const int prob = blockIdx.y;
  const RouteArgs a = problem_args(a0, prob);
  const Workspace ws = problem_workspace(ws0, (size_t)prob * a0.ws_stride);
  RandomArgs rnd = rnd0;
  rnd.stream += (uint32_t)prob;
  logits += (size_t)prob * logits_stride;
  expert_ids += (size_t)prob * a.T * a.k;
  weights += (size_t)prob * a.T * a.k;
  __shared__ unsigned long long maskl[64], flexl;
  const int tile = blockIdx.x, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int E = a.E, k = a.k, c = a.c;

  // the tail kernel of this call polls these words; they are cleared here, one
  // kernel earlier on the same stream
  if (tile == 0 && threadIdx.x < 4) ws.status[threadIdx.x] = 0;
  if (tile == 0 && threadIdx.x < 64) ws.lin_copy[threadIdx.x] = (int)threadIdx.x < a.E ? a.loads_in[threadIdx.x] : 0;
  if (threadIdx.x < 64) maskl[threadIdx.x] = 0ull;
  if (threadIdx.x == 0) flexl = 0ull;

  // wave w has the tokens w, w + 16, ... of the tile
  const bool real = lane < E;
  float z[kGeneralTokens];
#pragma unroll
  for (int n = 0; n < kGeneralTokens; ++n) {
    const int t = tile * kTile + wave + n * kGeneralWaves;
    z[n] = (real && t < a.T) ? logits[(size_t)t * E + lane] : 0.0f;
  }
  // what the second half of the kernel needs of a token
  int rank[kGeneralTokens], ncand[kGeneralTokens];   // (ncand 0: not load-dependent)
  float p[kGeneralTokens];
  unsigned long long picked[kGeneralTokens];         // the candidates' positions in the score order
  unsigned long long mine = 0ull;                    // the wave's fixed tokens assigned to the lane's expert
  unsigned long long fm = 0ull;
  __syncthreads();
#pragma unroll
  for (int n = 0; n < kGeneralTokens; ++n) {
    const int itok = wave + n * kGeneralWaves, t = tile * kTile + itok;
    rank[n] = ncand[n] = 0;
    p[n] = 0.0f;
    picked[n] = 0ull;
    if (t < a.T) {
      // ---- scores, normaliser (fixed tree over the expert index), top-k mass, pool ----
      rank[n] = rank_of(z[n], real, lane, E);
      const int best = __builtin_ctzll(__builtin_amdgcn_ballot_w64(real && rank[n] == 0));
      const float d = z[n] - __int_as_float(__builtin_amdgcn_readlane(__float_as_int(z[n]), best));
      p[n] = real ? exp_fixed(clamp_exp_arg(d)) : 0.0f;
      float tr = p[n];
#pragma unroll
      for (int s = 32; s >= 1; s >>= 1) tr = tr + __shfl_down(tr, s, 64);  // (lane 0 holds the tree's sum)
      const float zsum = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(tr)));
      // lane = rank
      const float ranked = __int_as_float(__builtin_amdgcn_ds_permute(4 * rank[n], __float_as_int(p[n])));
      auto at_rank = [&](int r) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ranked), r)); };
      float sk = at_rank(0);
      for (int i = 1; i < k; ++i) sk = sk + at_rank(i);
      const bool mass_ok = sk >= a.eps_high * zsum;
      const int inpool = __builtin_popcountll(__builtin_amdgcn_ballot_w64(real && d >= a.tau_ln));
      const int m = inpool > k ? inpool : k;
      const int cstar = mass_ok ? k : (c < m ? c : m);
      // ---- candidates ------------------------------------------------------------------
      if (SAMPLE && !mass_ok && m > c) {
        uint32_t w[4];
        draw_blocks(rnd, rnd.token_offset + (unsigned long long)t, lane, w);
        picked[n] = sample_positions(w, 0, m, c, lane);
      } else {
        picked[n] = cstar >= 64 ? ~0ull : (1ull << cstar) - 1ull;
      }
      const bool flex = !mass_ok && cstar > k;
      const bool in = real && ((picked[n] >> rank[n]) & 1ull) != 0ull;
      if (flex) {
        ncand[n] = cstar;
        fm |= 1ull << itok;
      } else {  // (exactly k positions are picked)
        float denom = zsum;
        if (a.renormalize) {
          unsigned long long left = picked[n];
          denom = at_rank(__builtin_ctzll(left));
          for (left &= left - 1ull; left != 0ull; left &= left - 1ull) denom = denom + at_rank(__builtin_ctzll(left));
        }
        if (in) {
          const int j = __builtin_popcountll(picked[n] & lanes_below(rank[n]));
          expert_ids[(size_t)t * k + j] = lane;
          weights[(size_t)t * k + j] = p[n] / denom;
          mine |= 1ull << itok;
        }
      }
      if (lane == 0) {
        ws.rec_cstar[t] = (uint8_t)ncand[n];
        ws.rec_Z[t] = zsum;
      }
    }
  }
  if (mine != 0ull) atomicOr(&maskl[lane], mine);
  if (lane == 0 && fm != 0ull) atomicOr(&flexl, fm);
  __syncthreads();
  const unsigned long long all = maskl[lane];  // per expert: the fixed tokens of the tile assigned to it
  fm = scalar64(flexl);
  if (wave == 0) {
    ws.tile_fixed_cnt[(size_t)tile * 64 + lane] = (uint8_t)__builtin_popcountll(all);
    ws.tile_mask[(size_t)tile * 64 + lane] = all;
    if (lane == 0) ws.flexmask[tile] = fm;
  }
  // ---- records of the flexible tokens -------------------------------------------
#pragma unroll
  for (int n = 0; n < kGeneralTokens; ++n) {
    if (ncand[n] > 0) {
      const int itok = wave + n * kGeneralWaves;
      const bool in = real && ((picked[n] >> rank[n]) & 1ull) != 0ull;
      write_records(a, ws, tile * kTile + itok, tile * kTile + __builtin_popcountll(fm & lanes_below(itok)), lane, in,
                    __builtin_popcountll(picked[n] & lanes_below(rank[n])), p[n],
                    __builtin_popcountll(all & lanes_below(itok)), ncand[n]);
    }
  }
}

// RANDOM trimming with c > k, behind the deterministic analysis.  That analysis has
// written, for every token, what the RANDOM mode would write too -- except the
// candidates of the tokens it trimmed: load-dependent tokens whose pool is larger than c
// (working-set size c in both modes).  Those are found here by (rec_cstar > 0, pool
// size > c); their c candidates are drawn instead of taken from the top, and their
// records are written again.  Fixed tokens, masks, counts and the flexible-token masks
// are not touched: none of them depends on which candidates a flexible token has.
// One workgroup per tile; tiles without such a token cost two loads per lane.  WAVES: 16 in a call
// of few tiles, where a tile's sampled tokens are the call's time; 4 beyond that, where the tiles' wavefronts
// fill the chip by themselves and starting them is what a call with few such tokens pays for (55184 tokens
// of 32 experts, none sampled: the call 23.2 us with 16, 22.2 with 4).
constexpr int kResampleFewTiles = 512;
constexpr int kResampleTokens = 4;  // of a wavefront at a time: 16 lanes draw the blocks of each

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void random_resample_kernel(const float* __restrict__ logits,
                                                             size_t logits_stride, const RouteArgs a0,
                                                             const Workspace ws0, const RandomArgs rnd0) {
  const int prob = blockIdx.y;  // the problem of a batched call; it draws with its own stream id
  const RouteArgs a = problem_args(a0, prob);
  const Workspace ws = problem_workspace(ws0, (size_t)prob * a0.ws_stride);
  RandomArgs rnd = rnd0;
  rnd.stream += (uint32_t)prob;
  logits += (size_t)prob * logits_stride;
  const int tile = blockIdx.x, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int E = a.E, c = a.c;
  const int32_t* pool = a.pool_in_ws ? ws.pool : a.st_pool;

  // lane = token
  const bool live = tile * kTile + lane < a.T;
  const int cst = live ? (int)ws.rec_cstar[tile * kTile + lane] : 0;
  const int m_lane = live ? pool[tile * kTile + lane] : 0;
  // (then cst == c)
  const unsigned long long todo = __builtin_amdgcn_ballot_w64(cst > 0 && m_lane > c);  // the same in all waves
  const int total = __builtin_popcountll(todo);
  if (wave >= total) return;
  const int number = ((todo >> lane) & 1ull) != 0ull ? __builtin_popcountll(todo & lanes_below(lane)) : -1;

  // lane = expert
  const bool real = lane < E;
  const float* src = logits + (size_t)tile * kTile * E + min(lane, E - 1);
  const unsigned long long fm_lane = ws.flexmask[tile];
  const unsigned long long all = ws.tile_mask[(size_t)tile * 64 + lane];
  // wave w takes the sampled tokens number w, w + WAVES, ...
  for (int n0 = wave; n0 < total; n0 += WAVES * kResampleTokens) {
    int itok[kResampleTokens];  // (-1: none)
#pragma unroll
    for (int u = 0; u < kResampleTokens; ++u) {
      const unsigned long long at = __builtin_amdgcn_ballot_w64(number == n0 + u * WAVES);
      itok[u] = at != 0ull ? __builtin_ctzll(at) : -1;
    }
    float z[kResampleTokens];  // (all on their way together; loads without conditions stay in flight)
#pragma unroll
    for (int u = 0; u < kResampleTokens; ++u) z[u] = src[max(itok[u], 0) * E];
    // lanes 16 u .. 16 u + 15: the blocks of token u
    uint32_t w[4];
    int mine = itok[0];
#pragma unroll
    for (int u = 1; u < kResampleTokens; ++u) mine = (lane >> 4) == u ? itok[u] : mine;
    draw_blocks(rnd, rnd.token_offset + (unsigned long long)(tile * kTile + max(mine, 0)), lane, w);
    const unsigned long long fm = scalar64(fm_lane);
#pragma unroll
    for (int u = 0; u < kResampleTokens; ++u) {
      if (itok[u] < 0) break;
      const int t = tile * kTile + itok[u];
      const int m = __builtin_amdgcn_readlane(m_lane, itok[u]);
      const int rank = rank_of(z[u], real, lane, E);
      const int best = __builtin_ctzll(__builtin_amdgcn_ballot_w64(real && rank == 0));
      const float zmax = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(z[u]), best));
      const unsigned long long picked = sample_positions(w, 16 * u, m, c, lane);
      const bool in = real && ((picked >> rank) & 1ull) != 0ull;
      write_records(a, ws, t, tile * kTile + __builtin_popcountll(fm & lanes_below(itok[u])), lane, in,
                    __builtin_popcountll(picked & lanes_below(rank)), exp_fixed(clamp_exp_arg(z[u] - zmax)),
                    __builtin_popcountll(all & lanes_below(itok[u])), c);
    }
  }
}

hipError_t launch_random_resample(const float* logits, size_t logits_stride, const RouteArgs& a,
                                  const Workspace& ws, const RandomArgs& rnd, hipStream_t s) {
  if (a.ntiles == 0) return hipSuccess;
  clear_stale_error();
  if ((long long)a.ntiles * a.nbatch <= kResampleFewTiles)
    hipLaunchKernelGGL(random_resample_kernel<16>, dim3(a.ntiles, a.nbatch), dim3(64 * 16), 0, s, logits, logits_stride,
                       a, ws, rnd);
  else
    hipLaunchKernelGGL(random_resample_kernel<4>, dim3(a.ntiles, a.nbatch), dim3(64 * 4), 0, s, logits, logits_stride,
                       a, ws, rnd);
  return hipGetLastError();
}

hipError_t launch_analyse_general(const float* logits, size_t logits_stride, const RouteArgs& a,
                                  const Workspace& ws, bool sample, const RandomArgs& rnd,
                                  int32_t* expert_ids, float* weights, hipStream_t s) {
  if (a.ntiles == 0) return hipSuccess;
  clear_stale_error();
  if (sample)
    hipLaunchKernelGGL(analyse_general_kernel<true>, dim3(a.ntiles, a.nbatch), dim3(64 * kGeneralWaves), 0, s,
                       logits, logits_stride, a, ws, rnd, expert_ids, weights);
  else
    hipLaunchKernelGGL(analyse_general_kernel<false>, dim3(a.ntiles, a.nbatch), dim3(64 * kGeneralWaves), 0, s,
                       logits, logits_stride, a, ws, rnd, expert_ids, weights);
  return hipGetLastError();
}

}  // namespace laser
