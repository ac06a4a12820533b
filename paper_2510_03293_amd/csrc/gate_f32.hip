// The single-precision gate projection, logits[t,e] = sum_h hidden[t,h] * w[e,h].
//
// A logit is one chain of fused multiply-adds in the order of h, starting from zero: the
// routing decisions behind it are taken in binary32 and compared bit for bit, so the order is
// part of the result and the contraction axis cannot be cut.  What can be done side by side
// are the logits, and v_mfma_f32_16x16x4_f32 advances 256 of them by four links of their
// chains: its result is that of four fused multiply-adds in slot order, each rounded on its own
// (tests/test_gpu_f32.py compares whole chains bit for bit with fmaf, with exponents
// far apart, cancellation and subnormal numbers among them).
//
// Bound: the chain.  H / 4 dependent matrix instructions of 32 cycles (H = 2048: 6.9 us), as
// long as there are no more blocks of 16 x 16 logits than SIMDs.  So a workgroup takes only two
// blocks -- 16 tokens x 32 experts, or 32 x 16 where there are no more experts -- one per
// wavefront on SIMDs of their own, which puts 2048 tokens of 64 experts on all 256 compute
// units; the other two wavefronts help to bring the rows in.  Rows travel memory ->
// registers, two chunks of 128 columns in flight, -> LDS (rows padded by four words: 16 rows x
// 4 slots then read 64 different banks), so that a wavefront's memory instruction takes 512
// contiguous bytes of each of two rows.  The operands of eight products are read while the eight
// before them are multiplied.
// One thread per logit walking its two rows with 16-byte loads -- 64 lanes on up to 64 different
// rows, a quarter of which a memory instruction serves per cycle -- took 143 us; the whole call
// (2048 tokens, 64 experts, H = 2048) went from 158 to 28 us.
#include "laser_internal.h"

namespace laser {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kF32Chunk = 128;             // columns staged at a time
constexpr int kF32Row = kF32Chunk + 4;     // floats per staged row
constexpr int kF32Rows = 48;               // rows of a workgroup: (1 + 2) x 16
constexpr int kF32Pieces = kF32Rows * (kF32Chunk / 4) / 256;  // 16-byte pieces per thread and chunk, ...
constexpr int kF32PieceRows = kF32Rows / kF32Pieces;          // ... that many rows apart
constexpr int kF32Depth = 2;               // chunks in flight

// NTB blocks of 16 tokens times NEB blocks of 16 experts per workgroup, NTB * NEB == 2.
template <int NTB, int NEB>
__global__ __launch_bounds__(256) void gate_f32_kernel(const float* __restrict__ hidden, const float* __restrict__ w,
                                                       int T, int H, int E, int token_groups,
                                                       float* __restrict__ logits, size_t logits_stride) {
  static_assert(NTB * NEB == 2 && 16 * (NTB + NEB) == kF32Rows && 16 % kF32PieceRows == 0, "two blocks, one per multiplying wavefront");
  __shared__ __align__(16) float stage[2][kF32Rows * kF32Row];
  hidden += (size_t)blockIdx.y * T * H;
  w += (size_t)blockIdx.y * E * H;
  logits += (size_t)blockIdx.y * logits_stride;
  // The workgroups that share token rows follow each other on one XCD (workgroups go to the
  // eight XCDs in turn): eight token groups, all of their expert groups, the next eight.
  const int expert_groups = (E + 16 * NEB - 1) / (16 * NEB);
  const int oct = (int)blockIdx.x / (8 * expert_groups), in_oct = (int)blockIdx.x - oct * 8 * expert_groups;
  const int tg = 8 * oct + (in_oct & 7), eg = in_oct >> 3;
  if (tg >= token_groups) return;
  const int t0 = tg * 16 * NTB, e0 = eg * 16 * NEB;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Load side: thread i takes piece i % 32 of rows i / 32, i / 32 + 8, ... (rows 0 .. 16 NTB - 1:
  // tokens, then experts; rows past the end repeat the last one, unused).
  const int piece = threadIdx.x & (kF32Chunk / 4 - 1), row0 = threadIdx.x / (kF32Chunk / 4);
  const float* row[kF32Pieces];
#pragma unroll
  for (int u = 0; u < kF32Pieces; ++u) {
    const int r = row0 + kF32PieceRows * u;
    row[u] = kF32PieceRows * u < 16 * NTB ? hidden + (size_t)min(t0 + r, T - 1) * H
                                          : w + (size_t)min(e0 + r - 16 * NTB, E - 1) * H;
  }
  float* const put = &stage[0][0] + row0 * kF32Row + piece * 4;
  // Multiply side: wavefront v < 2 has one block; lane l holds row l % 16 of both operands,
  // slot l / 16.
  const int tb = NTB == 2 ? wave & 1 : 0, eb = NEB == 2 ? wave & 1 : 0;
  const float* const get_t = &stage[0][0] + (16 * tb + (lane & 15)) * kF32Row + (lane >> 4);
  const float* const get_e = &stage[0][0] + (16 * (NTB + eb) + (lane & 15)) * kF32Row + (lane >> 4);

  const int nchunks = (H + kF32Chunk - 1) / kF32Chunk;
  f32x4_t in[kF32Depth][kF32Pieces];
  // (without a condition, so that the loads stay in flight: behind a branch the compiler would
  // wait for them at its end.  H % 4 == 0: a piece is all in or all out; out: read and not used)
  auto load = [&](f32x4_t (&x)[kF32Pieces], int c) {
    const int col = c * kF32Chunk + piece * 4;
#pragma unroll
    for (int u = 0; u < kF32Pieces; ++u)
      x[u] = *reinterpret_cast<const f32x4_t*>(row[u] + (col < H ? col : 0));
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int d = 0; d < kF32Depth; ++d) load(in[d], d);
  f32x4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int c0 = 0; c0 < nchunks; c0 += kF32Depth) {
#pragma unroll
    for (int d = 0; d < kF32Depth; ++d) {
      const int c = c0 + d;
      // (two staging buffers and one barrier per chunk: whoever writes buffer c % 2 again,
      // two chunks on, has passed the barrier that follows everybody's products of chunk c)
      constexpr int kBuf = kF32Rows * kF32Row;
      const int buf = (d & 1) * kBuf;  // (kF32Depth is even)
#pragma unroll
      for (int u = 0; u < kF32Pieces; ++u) *reinterpret_cast<f32x4_t*>(put + buf + kF32PieceRows * u * kF32Row) = in[d][u];
      __builtin_amdgcn_sched_barrier(0);
      load(in[d], c + kF32Depth);
      lds_barrier();
      const int steps = min(kF32Chunk, H - c * kF32Chunk) >> 2;  // (<= 0 behind the last chunk)
      if (wave < 2) {
        constexpr int kG = 8;  // products whose operands are read while the group before is multiplied
        if (steps == kF32Chunk / 4) {
          float a[2][kG], b[2][kG];
          auto read = [&](int g) {
#pragma unroll
            for (int s = 0; s < kG; ++s) {
              a[g & 1][s] = get_e[buf + 4 * (kG * g + s)];
              b[g & 1][s] = get_t[buf + 4 * (kG * g + s)];
            }
            __builtin_amdgcn_sched_barrier(0);
          };
          read(0);
#pragma unroll
          for (int g = 0; g < kF32Chunk / 4 / kG; ++g) {
            if (g + 1 < kF32Chunk / 4 / kG) read(g + 1);
#pragma unroll
            for (int s = 0; s < kG; ++s)
              acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[g & 1][s], b[g & 1][s], acc, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
          }
        } else {
          for (int s = 0; s < steps; ++s)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(get_e[buf + 4 * s], get_t[buf + 4 * s], acc, 0, 0, 0);
        }
      }
    }
  }
  if (wave < 2) {
    // register r of lane l: expert 4 (l / 16) + r, token l % 16 of the block
    const int t = t0 + 16 * tb + (lane & 15), e = e0 + 16 * eb + 4 * (lane >> 4);
    if (t < T) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (e + r < E) logits[(size_t)t * E + e + r] = acc[r];
    }
  }
}

hipError_t launch_gate_f32(const float* hidden, const float* w, int T, int H, int E, int nbatch,
                           float* logits, size_t logits_stride, hipStream_t s) {
  if (T == 0) return hipSuccess;
  clear_stale_error();
  // (up to 16 experts there is one block of them)
  const int ntb = E <= 16 ? 2 : 1, neb = 2 / ntb;
  const int token_groups = (T + 16 * ntb - 1) / (16 * ntb), expert_groups = (E + 16 * neb - 1) / (16 * neb);
  const dim3 grid((token_groups + 7) / 8 * 8 * expert_groups, nbatch);
  if (ntb == 2)
    hipLaunchKernelGGL((gate_f32_kernel<2, 1>), grid, dim3(256), 0, s, hidden, w, T, H, E, token_groups, logits,
                       logits_stride);
  else
    hipLaunchKernelGGL((gate_f32_kernel<1, 2>), grid, dim3(256), 0, s, hidden, w, T, H, E, token_groups, logits,
                       logits_stride);
  return hipGetLastError();
}

}  // namespace laser
