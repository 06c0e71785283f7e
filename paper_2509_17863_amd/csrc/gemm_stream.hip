// Grouped expert GEMMs for batches that give an expert a few rows (decode):
// every wave streams its own weight rows straight into registers.
//
// Such a launch is bound by the weight stream from HBM (each weight byte is
// used for a handful of rows), so what counts is how many bytes the whole
// chip keeps in flight.  The LDS-tiled kernels of gemm.hip need 256 or 512
// weight rows per workgroup and a whole CU per workgroup: with few active
// experts most CUs hold nothing, and with many the start and the end of every
// tile leave its CU idle.  Here a wave owns 32 weight rows (gate/up: 16 gate
// rows and the matching 16 up rows) and a ring of D K tiles of 4 KiB in
// registers, so 8 to 32 KiB are in flight per wave, and four (wide4) or eight
// waves share a CU:
//
//   grouped_gemm_stream_kernel  one wave per workgroup, token rows loaded like
//                               the weights; no LDS, no barrier (a row or two
//                               per expert: latency is everything)
//   grouped_gemm_shared_kernel  four or eight waves share the token rows of a
//                               row block through LDS, a chunk of channels at
//                               a time (loading them per wave costs L2 traffic
//                               that slows the weights: 16 rows of 7 168
//                               channels a quarter)
//
// Both operands reach v_mfma_f32_16x16x32_bf16 in its own layout (lane l: row
// l%16, 8 channels at 8*(l/16) of a 32-channel k-step; src0 = weight rows,
// src1 = token rows).  That instruction's sums are those of two 32x32x16 steps
// in ascending k, bit for bit, and the K tiles are walked in ascending order
// by one wave, so a token's result is the one the tiled kernels give (fp8
// weights: likewise per 128-channel scale block).
//
// Measured (one MI355X, HIP kernel times, tiled kernel -> this file; dsv3: H
// 7168, I 2048, E 32, k 8; qwen3: H 2048, I 768, E 128, k 8; mixtral: H 4096,
// I 14336, E 8, k 2):
//   dsv3, 1 token, fp8 tiled      gate/up 121 -> 39 us, down 30 -> 22 us
//   dsv3, 32 tokens, fp8 tiled    gate/up 169 -> 146, down 97 -> 81
//   dsv3, 64 tokens, bf16         gate/up 288 -> 285, down 226 -> 187
//   qwen3, 16 tokens, bf16        gate/up 129 -> 107, down 60 -> 45
//   qwen3, 192 tokens, bf16       gate/up 181 -> 152, down 86 -> 81
//   dsv3, 256 tokens, fp8 tiled   gate/up 209 -> 182 (wide8; 5.2 TB/s)
//   mixtral, 445 tokens, fp8      gate/up 394 -> 306 (wide8), down 227 -> 187 (wide4)
#include <algorithm>

#include "gemm_common.h"

namespace eaas {
namespace {

// Non-temporal: a weight byte is read once in the launch, and without the hint
// the stream runs 5% slower (dsv3, 1 token: 78 against 74 us per step).
// (The pointer says that it is global memory: a flat load would count against
// the LDS reads' waits too and drain the ring at every fragment read.)
__device__ __forceinline__ u32x4 load_weights(const GLOBAL_AS uint8_t* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const GLOBAL_AS u32x4*>(p));
}

// Exchanges a bit of the register index (lo, hi) with bit 3 of the lane
// index: lo keeps its lanes with bit 3 clear and takes hi's in the others'
// place, hi the other way round.
__device__ __forceinline__ void swap_reg_lane3(uint32_t& lo, uint32_t& hi) {
  constexpr int kRor8 = 0x128;  // rotate by 8 inside a row of 16 lanes
  const uint32_t a = lo, b = hi;
  lo = __builtin_amdgcn_update_dpp(a, b, kRor8, 0xf, 0xc, false);
  hi = __builtin_amdgcn_update_dpp(b, a, kRor8, 0xf, 0x3, false);
}
// The same with bit 4 of the lane index.
__device__ __forceinline__ void swap_reg_lane4(uint32_t& lo, uint32_t& hi) {
  const auto r = __builtin_amdgcn_permlane16_swap(lo, hi, false, false);
  lo = r[0];
  hi = r[1];
}

// Weight layouts: bf16 rows, fp8 rows, fp8 tiled; fp8 rows times fp8 activations.
enum StreamWeights { kBf16Rows = 0, kFp8Rows = 1, kFp8Tiled = 2, kFp8A8 = 3 };

// A K tile is 128 bytes of each weight row.  MFMA wants lane l to hold row
// l%16 and 16-byte chunks l/16, l/16 + 4 (bf16) or 8-byte pieces l/16,
// l/16 + 4, ... (fp8) of those 128 bytes, but a load in that order asks memory for 64
// or 32 bytes of 16 rows at a time.  So each load takes whole 128-byte lines
// (8 rows; tiled fp8: 16 rows of 64 contiguous bytes, 1 KiB in all), and the
// chunks are put in place by swapping register-index bits with lane-index
// bits just before the MFMAs.  (fp8 activations: v_mfma_scale_f32_16x16x128
// takes the whole K tile, chunks 2*(l/16) and 2*(l/16) + 1 in lane l.)
constexpr int kBlocks = 2;  // 16-row weight blocks of a wave

template <int W, int MB, int D>
struct StreamLoop {
  static constexpr bool FP8 = W != kBf16Rows, kTiled = W == kFp8Tiled, A8 = W == kFp8A8;
  static constexpr int KT = FP8 ? 128 : 64;  // channels per K tile
  static constexpr int KS = A8 ? 2 : KT / 32;  // MFMA k-steps per K tile (A8: 16-byte chunks)

  struct Weights {
    const GLOBAL_AS uint8_t* w;  // the expert's (wave-uniform)
    uint32_t step;           // bytes to the next K tile
    uint32_t second;         // bytes from the first to the second load of a block
    uint32_t off[kBlocks];   // per lane
    const CONST_AS float* sc[kBlocks];  // fp8: scales of the block's rows
  };
  struct Rows {
    const uint8_t* x;        // wave-uniform
    uint32_t off[MB];        // per lane
    const float* xs;         // A8: row scales, wave-uniform
    uint32_t soff[MB];       // A8: per lane, index of the row's first scale
  };
  struct Stage {
    u32x4 w[kBlocks][2];
    float sc[kBlocks];
    bf16x8 x[MB][KS];        // not used where the rows come through LDS
    float xs[MB];            // A8
  };

  // Byte offset inside the K tile and row that lane l loads for block row 0.
  static __device__ __forceinline__ int lane_row(int lane) {
    return W == kFp8Tiled ? lane & 15 : lane & 7;
  }
  static __device__ __forceinline__ int lane_byte(int lane) {
    const int b3 = (lane >> 3) & 1, b4 = (lane >> 4) & 1, b5 = lane >> 5;
    if (W == kFp8Tiled) return 16 * (2 * b4 + b5);          // lane bits 5,4 = piece bits 1,2
    if (W == kFp8Rows) return 16 * (4 * b4 + 2 * b3 + b5);  // bits 5,4,3 = piece bits 1,3,2
    if (A8) return 16 * (4 * b5 + 2 * b4 + b3);             // bits 5,4,3 = chunk bits 2,1,0
    return 16 * (4 * b3 + 2 * b5 + b4);                     // bits 5,4,3 = chunk bits 1,0,2
  }

  static __device__ __forceinline__ void load_w(const Weights& s, int kt, Stage& f) {
    const GLOBAL_AS uint8_t* wk = s.w + (size_t)kt * s.step;
#pragma unroll
    for (int j = 0; j < kBlocks; ++j) {
      f.w[j][0] = load_weights(wk + s.off[j]);
      f.w[j][1] = load_weights(wk + s.second + s.off[j]);
    }
    if (FP8) {
#pragma unroll
      for (int j = 0; j < kBlocks; ++j) f.sc[j] = s.sc[j][kt];
    }
  }
  static __device__ __forceinline__ void load_x(const Rows& x, int kt, Stage& f) {
    const uint8_t* xk = x.x + (size_t)kt * (A8 ? KT : KT * 2);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int i = 0; i < MB; ++i)
        f.x[i][ks] = *reinterpret_cast<const bf16x8*>(xk + ks * (A8 ? 16 : 64) + x.off[i]);
    if constexpr (A8) {
#pragma unroll
      for (int i = 0; i < MB; ++i) f.xs[i] = x.xs[x.soff[i] + (uint32_t)kt];
    }
  }

  // The block's weight fragment of each k-step.
  static __device__ __forceinline__ void fragments(const u32x4 (&w)[2], bf16x8 (&f)[KS]) {
    u32x4 a = w[0], b = w[1];
    if constexpr (W == kBf16Rows || A8) {
      // register = row bit 3, lane bit 3 = chunk bit 2 (A8: 0)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t lo = a[i], hi = b[i];
        swap_reg_lane3(lo, hi);
        a[i] = lo;
        b[i] = hi;
      }
      f[0] = __builtin_bit_cast(bf16x8, a);
      f[1] = __builtin_bit_cast(bf16x8, b);
    } else {
      // piece bit 0 = which 8-byte half of a load
      uint32_t v[2][2][2];  // [load][half][word]
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        v[0][0][c] = a[c];
        v[0][1][c] = a[2 + c];
        v[1][0][c] = b[c];
        v[1][1][c] = b[2 + c];
        swap_reg_lane4(v[0][0][c], v[0][1][c]);
        swap_reg_lane4(v[1][0][c], v[1][1][c]);
        if (W == kFp8Rows) {
          swap_reg_lane3(v[0][0][c], v[1][0][c]);
          swap_reg_lane3(v[0][1][c], v[1][1][c]);
        }
      }
      // rows: the load index now is piece bit 2 and the half piece bit 3;
      // tiled: the load index is piece bit 3 and the half piece bit 2
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int ld = W == kFp8Rows ? ks & 1 : ks >> 1, half = W == kFp8Rows ? ks >> 1 : ks & 1;
        f[ks] = fp8x8_to_bf16(u32x2{v[ld][half][0], v[ld][half][1]});
      }
    }
  }

  static __device__ __forceinline__ i32x8 chunk_pair(const bf16x8 (&c)[KS]) {
    const u32x4 lo = __builtin_bit_cast(u32x4, c[0]), hi = __builtin_bit_cast(u32x4, c[1]);
    return i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3],
                 (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
  }
  static __device__ __forceinline__ void multiply(const Stage& f, f32x4 (&acc)[MB][kBlocks]) {
    if constexpr (A8) {
      i32x8 w[kBlocks];
#pragma unroll
      for (int j = 0; j < kBlocks; ++j) {
        bf16x8 c[KS];
        fragments(f.w[j], c);
        w[j] = chunk_pair(c);
      }
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        const i32x8 x = chunk_pair(f.x[i]);
#pragma unroll
        for (int j = 0; j < kBlocks; ++j) {
          const f32x4 part = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
              w[j], x, f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0, 127, 0, 127);
          const float s = f.xs[i] * f.sc[j];
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[i][j][v] += s * part[v];
        }
      }
    } else if constexpr (FP8) {
#pragma unroll
      for (int j = 0; j < kBlocks; ++j) {
        bf16x8 w[KS];
        fragments(f.w[j], w);
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          f32x4 part = {};
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
            part = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks], f.x[i][ks], part, 0, 0, 0);
          acc[i][j] += f.sc[j] * part;
        }
      }
    } else {
      bf16x8 w[kBlocks][KS];
#pragma unroll
      for (int j = 0; j < kBlocks; ++j) fragments(f.w[j], w[j]);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < kBlocks; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[j][ks], f.x[i][ks], acc[i][j],
                                                                0, 0, 0);
    }
  }

  // The scheduling barriers keep the compiler from sinking a load to its use
  // D tiles later.  Loads that the loop skips near the end come after it: a
  // skipped load inside would make the compiler's wait counts assume the worst.
  static __device__ __forceinline__ void start(const Weights& s, int nk, Stage (&st)[D]) {
#pragma unroll
    for (int d = 0; d < D; ++d) load_w(s, min(d, nk - 1), st[d]);
    __builtin_amdgcn_sched_barrier(0);
  }
  static __device__ __forceinline__ void run(const Weights& s, const Rows& x, int nk,
                                             Stage (&st)[D], f32x4 (&acc)[MB][kBlocks]) {
#pragma unroll
    for (int d = 0; d < D; ++d) load_x(x, min(d, nk - 1), st[d]);
    __builtin_amdgcn_sched_barrier(0);
    int k0 = 0;
    for (; k0 + 2 * D <= nk; k0 += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        multiply(st[d], acc);
        load_w(s, k0 + d + D, st[d]);
        load_x(x, k0 + d + D, st[d]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (k0 + d < nk) multiply(st[d], acc);
      if (k0 + d + D < nk) {
        load_w(s, k0 + d + D, st[d]);
        load_x(x, k0 + d + D, st[d]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
      if (k0 + d + D < nk) multiply(st[d], acc);
  }
};

// Weight source of wave `wt` of expert e: output columns from c0 on.
template <int KIND, class Loop>
__device__ __forceinline__ typename Loop::Weights weight_source(const GemmParams& p, int e,
                                                                int c0) {
  constexpr bool GATEUP = KIND == kGateUp;
  constexpr int ESZ = Loop::FP8 ? 1 : 2;
  const int lane = __lane_id();
  typename Loop::Weights s;
  s.w = (const GLOBAL_AS uint8_t*)wave_uniform(group_weights(p, e, ESZ));
  // tiled: stages of bn rows x 64 bytes, stored one after the other along K
  const int bn = GATEUP && p.N % 512 == 0 ? 512 : 256;
  s.step = Loop::kTiled ? bn * 128 : 128;
  s.second = Loop::kTiled ? bn * 64 : 8u * (uint32_t)(p.K * ESZ);
#pragma unroll
  for (int j = 0; j < kBlocks; ++j) {
    const int row = GATEUP ? j * p.I + c0 : c0 + j * 16;  // first weight row of the block
    if (Loop::kTiled) {
      const int tn = GATEUP ? c0 / (bn / 2) : c0 / bn;
      const int jr = GATEUP ? c0 % (bn / 2) + j * (bn / 2) : c0 % bn + j * 16;
      s.off[j] = (uint32_t)tn * (uint32_t)(p.K / 64) * (bn * 64) +
                 (jr + Loop::lane_row(lane)) * 64 + Loop::lane_byte(lane);
    } else {
      s.off[j] =
          (uint32_t)(row + Loop::lane_row(lane)) * (uint32_t)(p.K * ESZ) + Loop::lane_byte(lane);
    }
    s.sc[j] = Loop::FP8 ? (const CONST_AS float*)wave_uniform(
                              group_scales(p, e) + (size_t)(row / 128) * (p.K / 128))
                        : nullptr;
  }
  return s;
}

// The rows of a block: m of [0, rows) is permuted row r0 + m.  Their slots are
// in perm, or (self: a launch that routes its rows itself) in LDS.
struct BlockRows {
  int r0, rows;
  bool self;
  const LDS_AS int* slots;
};
// The row of the A operand and the row of the output (m clamped into the block).
template <int KIND>
__device__ __forceinline__ int source_row(const GemmParams& p, const BlockRows& b, int m) {
  m = m < b.rows ? m : 0;
  if (KIND != kGateUp) return b.r0 + m;
  const int slot = b.self ? b.slots[m] : min(max(p.perm[b.r0 + m], 0), p.R - 1);
  return slot / p.k;
}
template <int KIND>
__device__ __forceinline__ int output_row(const GemmParams& p, const BlockRows& b, int m) {
  m = m < b.rows ? m : 0;
  return KIND == kDownBySlotK ? min(max(p.perm[b.r0 + m], 0), p.R - 1) : b.r0 + m;
}

// acc[i][j][v]: token row 16i + lane%16 of the block's `rows`, weight row
// 4*(lane/16) + v of block j.
template <int KIND, int MB>
__device__ __forceinline__ void store_rows(const GemmParams& p, int rows, int c0,
                                           const int (&orow)[MB],
                                           const f32x4 (&acc)[MB][kBlocks]) {
  const int lane = __lane_id();
  const int l16 = lane & 15, q = lane >> 4;
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    if (i * 16 + l16 >= rows) continue;
    if constexpr (KIND == kGateUp) {
      const f32x4 g = acc[i][0], u = acc[i][1];
      u32x2 v;
      v[0] = pack_bf16x2(silu_mul(g[0], u[0]), silu_mul(g[1], u[1]));
      v[1] = pack_bf16x2(silu_mul(g[2], u[2]), silu_mul(g[3], u[3]));
      *reinterpret_cast<u32x2*>(p.h + (size_t)orow[i] * p.I + c0 + 4 * q) = v;
    } else {
#pragma unroll
      for (int j = 0; j < kBlocks; ++j)
        *reinterpret_cast<f32x4*>(p.y + (size_t)orow[i] * p.N + c0 + j * 16 + 4 * q) = acc[i][j];
    }
  }
}

// fp8 activations, gate/up: h quantized per row and 128 columns, which are the
// workgroup's eight waves' (red: [16 * MB][8] in LDS).
constexpr int kA8Waves = 8;
template <int MB>
__device__ __forceinline__ void store_rows_a8(const GemmParams& p, int rows, int c0,
                                              const int (&orow)[MB],
                                              const f32x4 (&acc)[MB][kBlocks],
                                              LDS_AS float* red) {
  const int lane = __lane_id();
  const int l16 = lane & 15, q = lane >> 4;
  const int wave = c0 / 16 % kA8Waves;
  float hv[MB][4];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    float m = 0.0f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float h = silu_mul(acc[i][0][v], acc[i][1][v]);
      hv[i][v] = __uint_as_float(f32_to_bf16_bits(h) << 16);
      m = fmaxf(m, fabsf(hv[i][v]));
    }
    m = fmaxf(m, __shfl_xor(m, 16));
    m = fmaxf(m, __shfl_xor(m, 32));
    if (q == 0) red[(i * 16 + l16) * kA8Waves + wave] = m;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const int m0 = i * 16 + l16;
    if (m0 >= rows) continue;
    float m = 0.0f;
#pragma unroll
    for (int w = 0; w < kA8Waves; ++w) m = fmaxf(m, red[m0 * kA8Waves + w]);
    const float s = m > 0.0f ? m / 448.0f : 1.0f;
    *reinterpret_cast<uint32_t*>(p.hq + (size_t)orow[i] * p.I + c0 + 4 * q) =
        pack_e4m3x4(hv[i][0] / s, hv[i][1] / s, hv[i][2] / s, hv[i][3] / s);
    if (wave == 0 && q == 0) p.hs[(size_t)orow[i] * (p.I / 128) + c0 / 128] = s;
  }
}

// A block of expert e (rows <= 16*MB) times this wave's weights.
template <int KIND, int W, int MB, int D>
__device__ __forceinline__ void stream_tile(const GemmParams& p, int e, const BlockRows& b,
                                            int wt, LDS_AS float* red) {
  using Loop = StreamLoop<W, MB, D>;
  const int lane = __lane_id();
  const int l16 = lane & 15, q = lane >> 4;
  const int c0 = wt * (KIND == kGateUp ? 16 : 32);
  const typename Loop::Weights s = weight_source<KIND, Loop>(p, e, c0);
  const int nk = p.K / Loop::KT;
  typename Loop::Stage st[D];
  Loop::start(s, nk, st);
  typename Loop::Rows x;
  x.x = Loop::A8 ? p.a8 : reinterpret_cast<const uint8_t*>(p.a);
  x.xs = p.a_scale;
  int orow[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    orow[i] = output_row<KIND>(p, b, i * 16 + l16);
    const uint32_t row = (uint32_t)source_row<KIND>(p, b, i * 16 + l16);
    x.off[i] = row * (uint32_t)(Loop::A8 ? p.lda : p.lda * 2) + q * (Loop::A8 ? 32 : 16);
    x.soff[i] = row * (uint32_t)nk;
  }
  f32x4 acc[MB][kBlocks];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < kBlocks; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  Loop::run(s, x, nk, st, acc);
  if constexpr (Loop::A8 && KIND == kGateUp) store_rows_a8<MB>(p, b.rows, c0, orow, acc, red);
  else store_rows<KIND, MB>(p, b.rows, c0, orow, acc);
}

// All rows of an expert, 32 at a time, times one wave's weights.  (bf16: a ring
// of 8 K tiles with 16 rows, 5 with 32: 4 and 3 were within 3%; past 256
// registers fewer waves would fit.)
template <int KIND, int W>
__device__ __forceinline__ void stream_rows(const GemmParams& p, int e, const BlockRows& all,
                                            int wt) {
  constexpr bool FP8 = W != kBf16Rows;
  for (int m0 = 0; m0 < all.rows; m0 += 32) {
    const BlockRows b{all.r0 + m0, min(32, all.rows - m0), all.self, all.slots + m0};
    if (b.rows <= 16) stream_tile<KIND, W, 1, FP8 ? 5 : 8>(p, e, b, wt, nullptr);
    else stream_tile<KIND, W, 2, FP8 ? 3 : 5>(p, e, b, wt, nullptr);
  }
}

// ---------------------------------------------------------------------------
// Routing inside the gate/up launch, for batches of at most kSelfSlots slots.
// The routing launch is 4 to 5 us of such a step (a sixth of the tiny
// workload's, 7% of one dsv3 token's), and its result is a few ballots away:
// every wave reads all ids (2 KiB at most), takes the slots of its expert and
// counts those of the experts before it.  One more workgroup writes the
// routing arrays that the down projection and the combine read.
constexpr int kSelfWords = kSelfSlots / kWave;

__device__ __forceinline__ int slot_id(const GemmParams& p, int w) {
  const int s = w * kWave + __lane_id();
  const int id = s < p.R ? p.ids[s] : -1;
  return (unsigned)id < (unsigned)p.E ? id : -1;
}

// Group g of min(E, R): expert g, or (more experts than slots) the expert of
// slot g if that is its first slot.  False if the group has no rows.  The
// expert's slots go to `slots` (written where `writes`) in ascending order.
__device__ __forceinline__ bool route_self(const GemmParams& p, int g, int* slots, bool writes,
                                           int& e, BlockRows& b) {
  int id[kSelfWords];
#pragma unroll
  for (int w = 0; w < kSelfWords; ++w) id[w] = w * kWave < p.R ? slot_id(p, w) : -1;
  e = g;
  if (p.E > p.R) {
    e = -1;
#pragma unroll
    for (int w = 0; w < kSelfWords; ++w)
      if (w == g / kWave) e = __builtin_amdgcn_readlane(id[w], g % kWave);
    if (e < 0) return false;
  }
  b.r0 = 0;
  b.rows = 0;
  b.self = true;
  b.slots = (const LDS_AS int*)slots;
  const uint64_t lt = lanemask_lt();
  bool first = true;
#pragma unroll
  for (int w = 0; w < kSelfWords; ++w) {
    if (w * kWave >= p.R) break;
    const uint64_t m = ballot(id[w] == e);
    if (p.E > p.R && m && b.rows == 0) first = w * kWave + __builtin_ctzll(m) == g;
    if (writes && id[w] == e) slots[b.rows + __popcll(m & lt)] = w * kWave + __lane_id();
    b.rows += __popcll(m);
    b.r0 += __popcll(ballot(id[w] >= 0 && id[w] < e));
  }
  // the wave's own LDS writes are read back in order
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  return first && b.rows > 0;
}

// The routing of launch_route_permute, by one wave.
__device__ __forceinline__ void write_routing(const GemmParams& p, int* next) {
  const int lane = __lane_id();
  const uint64_t lt = lanemask_lt();
  int32_t* offsets = const_cast<int32_t*>(p.offsets);
  int32_t* active = const_cast<int32_t*>(p.active);
  int32_t* perm = const_cast<int32_t*>(p.perm);
  auto wave_sync = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };
  for (int e = lane; e < p.E; e += kWave) next[e] = 0;
  wave_sync();
  for (int w = 0; w * kWave < p.R; ++w) {
    const int id = slot_id(p, w);
    if (id >= 0) atomicAdd(&next[id], 1);
  }
  wave_sync();
  // counts, offsets and the active experts, 64 experts at a time
  int row = 0, n_active = 0;
  for (int e0 = 0; e0 < p.E; e0 += kWave) {
    const int e = e0 + lane;
    const int c = e < p.E ? next[e] : 0;
    int incl = c;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const int o = __shfl_up(incl, d, kWave);
      if (lane >= d) incl += o;
    }
    const uint64_t act = ballot(c > 0);
    if (e < p.E) {
      p.counts[e] = c;
      offsets[e] = row + incl - c;
      next[e] = row + incl - c;
      if (c > 0) active[1 + n_active + __popcll(act & lt)] = e;
    }
    row += __shfl(incl, kWave - 1, kWave);
    n_active += __popcll(act);
  }
  if (lane == 0) {
    offsets[p.E] = row;
    active[0] = n_active;
  }
  for (int a = n_active + lane; a < p.E; a += kWave) active[1 + a] = 0;
  wave_sync();
  // stable ranks, 64 slots per step, steps in slot order
  for (int w = 0; w * kWave < p.R; ++w) {
    const int s = w * kWave + lane;
    const int id = slot_id(p, w);
    uint64_t peers = ballot(id >= 0);
    for (int bit = 1; bit < p.E; bit <<= 1) {
      const uint64_t m = ballot(id & bit);
      peers &= (id & bit) ? m : ~m;
    }
    const int rank = __popcll(peers & lt);
    if (id >= 0) {
      const int r = next[id] + rank;
      perm[r] = s;
      p.inv[s] = r;
    } else if (s < p.R) {
      p.inv[s] = -1;
    }
    wave_sync();
    if (id >= 0 && rank == 0) next[id] += __popcll(peers);
    wave_sync();
  }
  for (int r = row + lane; r < p.R; r += kWave) perm[r] = -1;
}

// grid: min(E, R) * N / 32 waves, one per workgroup: wave wt of the a-th active
// expert.
template <int KIND, int W>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(2, 2)))
void grouped_gemm_stream_kernel(GemmParams p) {
  const int waves_n = p.N / 32;
  const int a = blockIdx.x / waves_n;
  const int wt = blockIdx.x - a * waves_n;
  // routing arrays may come from the caller: clamp every index taken from them
  if (a >= min(max(p.active[0], 0), p.E)) return;
  const int e = min(max(p.active[1 + a], 0), p.E - 1);
  const int r0 = min(max(p.offsets[e], 0), p.R);
  const int end = min(max(p.offsets[e + 1], r0), p.R);
  stream_rows<KIND, W>(p, e, BlockRows{r0, end - r0, false, nullptr}, wt);
}

// Gate/up of a small batch that routes its rows itself (route_self): block 0
// writes the routing, the others find their own rows.
template <int W>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(2, 2)))
void grouped_gemm_stream_self_kernel(GemmParams p) {
  __shared__ int table[kMaxExperts];
  if (blockIdx.x == 0) return write_routing(p, table);
  const int waves_n = p.N / 32;
  const int g = (blockIdx.x - 1) / waves_n;
  const int wt = blockIdx.x - 1 - g * waves_n;
  int e;
  BlockRows all;
  if (!route_self(p, g, table, true, e, all)) return;
  stream_rows<kGateUp, W>(p, e, all, wt);
}

// ---------------------------------------------------------------------------
// The same streams with the token rows shared through LDS: a row block's
// channels are staged in chunks of CHB bytes per row, double-buffered, one
// barrier per chunk.  The next chunk's loads are issued a whole chunk before
// they are stored to LDS; since loads return in order, that wait leaves the
// weight tiles issued since (TPC per wave) in flight.
template <int W, int MB, int NW, int CHB, int D>
struct SharedLoop {
  using S = StreamLoop<W, 1, D>;  // weight loads and fragments
  static constexpr bool FP8 = S::FP8;
  static constexpr int KT = S::KT, KS = S::KS;
  static constexpr int TPC = CHB / (KT * 2);  // K tiles per chunk of token rows
  static_assert(TPC >= 1 && D % TPC == 0, "ring slots are compile-time indexes");
  static constexpr int LPR = CHB / 16;        // lanes per row when staging
  static constexpr int RP = NW * kWave / LPR; // rows per staging pass
  static_assert(MB * 16 % RP == 0, "whole staging passes");
  static constexpr int NP = MB * 16 / RP;
  static constexpr int XROW = CHB + 16;       // 16-byte pad: a fragment read hits every bank once

  struct Rows {
    const uint8_t* x;    // wave-uniform
    uint32_t off[NP];    // per thread: byte offset of its row of each pass
    uint32_t kbyte, kmax;  // this thread's 16 bytes inside a chunk; last 16 bytes of a row
    LDS_AS char* dst;    // this thread's place in pass 0 of buffer 0
    uint32_t buf;        // bytes of one buffer
    u32x4 r[NP];         // the chunk on its way
  };
  static __device__ __forceinline__ void load_x(Rows& x, int c) {
    const uint32_t kb = min((uint32_t)(c * CHB) + x.kbyte, x.kmax);
#pragma unroll
    for (int p = 0; p < NP; ++p)
      x.r[p] = *reinterpret_cast<const u32x4*>(x.x + (size_t)(x.off[p] + kb));
  }
  static __device__ __forceinline__ void store_x(const Rows& x, int c) {
    LDS_AS char* d = x.dst + (c & 1) * x.buf;
#pragma unroll
    for (int p = 0; p < NP; ++p)
      *reinterpret_cast<LDS_AS u32x4*>(d + p * RP * XROW) = x.r[p];
  }

  static __device__ __forceinline__ void multiply(const typename S::Stage& f,
                                                  const LDS_AS char* xs,
                                                  f32x4 (&acc)[MB][kBlocks]) {
    bf16x8 w[kBlocks][KS];
#pragma unroll
    for (int j = 0; j < kBlocks; ++j) S::fragments(f.w[j], w[j]);
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      bf16x8 x[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        x[ks] = *reinterpret_cast<const LDS_AS bf16x8*>(xs + i * 16 * XROW + ks * 64);
      f32x4 part[kBlocks];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int j = 0; j < kBlocks; ++j) {
          f32x4& to = FP8 ? part[j] : acc[i][j];
          to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[j][ks], x[ks],
                                                       FP8 && ks == 0 ? f32x4{} : to, 0, 0, 0);
        }
      if (FP8) {
#pragma unroll
        for (int j = 0; j < kBlocks; ++j) acc[i][j] += f.sc[j] * part[j];
      }
    }
  }

  // Chunk c has been read: the next one goes into the other buffer, which
  // every wave finished reading before the last barrier.
  static __device__ __forceinline__ void next_chunk(Rows& x, int c, int nch) {
    store_x(x, c + 1);
    load_x(x, min(c + 2, nch - 1));
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  }

  static __device__ __forceinline__ void run(const typename S::Weights& s, Rows& x, int nk,
                                             typename S::Stage (&st)[D], const LDS_AS char* xs,
                                             f32x4 (&acc)[MB][kBlocks]) {
    const int nch = (nk + TPC - 1) / TPC;
    load_x(x, 0);
    store_x(x, 0);
    load_x(x, min(1, nch - 1));
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    int k0 = 0;
    for (; k0 + 2 * D <= nk; k0 += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const int c = (k0 + d) / TPC;
        multiply(st[d], xs + (c & 1) * x.buf + (d % TPC) * (KT * 2), acc);
        S::load_w(s, k0 + d + D, st[d]);
        if ((d + 1) % TPC == 0) next_chunk(x, c, nch);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int d = 0; d < 2 * D - 1; ++d) {
      const int kt = k0 + d, c = kt / TPC;
      if (kt < nk) multiply(st[d % D], xs + (c & 1) * x.buf + (d % TPC) * (KT * 2), acc);
      if (d < D && kt + D < nk) S::load_w(s, kt + D, st[d % D]);
      if ((d + 1) % TPC == 0 && c + 1 < nch) next_chunk(x, c, nch);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
};

template <int KIND, int W, int MB, int NW, int CHB, int D>
__device__ __forceinline__ void shared_tile(const GemmParams& p, int e, const BlockRows& b,
                                            int wt, LDS_AS char* lds) {
  using Loop = SharedLoop<W, MB, NW, CHB, D>;
  using S = typename Loop::S;
  const int lane = __lane_id();
  const int l16 = lane & 15, q = lane >> 4;
  const int c0 = wt * (KIND == kGateUp ? 16 : 32);
  const typename S::Weights s = weight_source<KIND, S>(p, e, c0);
  const int nk = p.K / Loop::KT;
  typename S::Stage st[D];
  S::start(s, nk, st);
  typename Loop::Rows x;
  x.x = reinterpret_cast<const uint8_t*>(p.a);
  x.kbyte = (threadIdx.x % Loop::LPR) * 16;
  x.kmax = (uint32_t)p.K * 2 - 16;
  x.buf = MB * 16 * Loop::XROW;
  x.dst = lds + (threadIdx.x / Loop::LPR) * Loop::XROW + x.kbyte;
#pragma unroll
  for (int i = 0; i < Loop::NP; ++i) {
    const int m = threadIdx.x / Loop::LPR + i * Loop::RP;
    x.off[i] = (uint32_t)source_row<KIND>(p, b, m) * (uint32_t)(p.lda * 2);
  }
  int orow[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) orow[i] = output_row<KIND>(p, b, i * 16 + l16);
  f32x4 acc[MB][kBlocks];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < kBlocks; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  Loop::run(s, x, nk, st, lds + l16 * Loop::XROW + q * 16, acc);
  store_rows<KIND, MB>(p, b.rows, c0, orow, acc);
}

// Row block of a workgroup: the experts' rows in blocks of at most BM rows
// (an expert's blocks are of equal height, rounded up to 16 rows), expert
// major, then weight tile major and row block minor.  Every wave finds its
// block by itself: 64 experts at a time, one per lane.
struct RowBlock {
  int e, r0, rows, tn;
};
template <int BM>
__device__ __forceinline__ bool locate_rows(const GemmParams& p, int tile, int tiles_n,
                                            RowBlock& b) {
  const int lane = threadIdx.x & (kWave - 1);
  const int n_active = min(max(p.active[0], 0), p.E);
  int before = 0;
  for (int a0 = 0; a0 < n_active; a0 += kWave) {
    // routing arrays may come from the caller: clamp every index taken from them
    const int a = a0 + lane;
    int e = 0, beg = 0, rows = 0;
    if (a < n_active) {
      e = min(max(p.active[1 + a], 0), p.E - 1);
      beg = min(max(p.offsets[e], 0), p.R);
      rows = min(max(p.offsets[e + 1], beg), p.R) - beg;
    }
    const int blocks = (rows + BM - 1) / BM;
    int incl = blocks;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const int o = __shfl_up(incl, d, kWave);
      if (lane >= d) incl += o;
    }
    const int end = (before + incl) * tiles_n;
    const uint64_t past = ballot(tile < end);
    if (past) {
      const int l = __builtin_ctzll(past);
      const int first = before + __builtin_amdgcn_readlane(incl - blocks, l);
      const int nb = __builtin_amdgcn_readlane(blocks, l);
      const int local = tile - first * tiles_n;
      b.e = __builtin_amdgcn_readlane(e, l);
      const int all = __builtin_amdgcn_readlane(rows, l);
      const int height = ((all + nb - 1) / nb + 15) & ~15;
      b.tn = local / nb;
      const int m0 = (local - b.tn * nb) * height;
      b.r0 = __builtin_amdgcn_readlane(beg, l) + m0;
      b.rows = min(height, all - m0);
      return b.rows > 0;
    }
    before += __builtin_amdgcn_readlane(incl, kWave - 1);
  }
  return false;
}

// Geometry of a launch: NW waves (32 weight rows each), row blocks of up to
// 16*MBX rows, a ring of D K tiles per wave, OCC waves per SIMD.  512-byte
// chunks of token rows (256-byte ones, with twice the barriers, were 3-25%
// slower).
//   few    four waves, 64 rows, two workgroups per CU.  (32 rows with three or
//          four per CU were within 4% up to 24 rows per expert and read the
//          weights twice past 32.)
//   wide8  eight waves, 144 rows (what two chunks of LDS hold), one workgroup
//          per CU: one block for the 50 to 130 rows that a decode batch of some
//          hundred tokens gives an expert, in steps of 16 rows, where the
//          tiled fp8 kernel steps by 32 and needs two tiles past 96.  A ring
//          of 2: 4 leave too few registers to read fragments ahead (+6%).
//   wide4  the same with four waves: twice the workgroups, for matrices that
//          have too few 256-row tiles for the chip.
template <int W>
struct Few {
  static constexpr int NW = 4, MBX = 4, D = 4, OCC = 2;
};
struct Wide8 {  // fp8 gate/up
  static constexpr int NW = 8, MBX = 9, D = 2, OCC = 2;
};
template <int W>
struct Wide4 {
  static constexpr int NW = 4, MBX = 9, D = W == kBf16Rows ? 4 : 2, OCC = 1;
};
constexpr int kChunk = 512;

// The smallest of shared_tile's row counts that holds the block.
template <int KIND, int W, class G, int MB>
__device__ __forceinline__ void tile_of_height(const GemmParams& p, int e, const BlockRows& b,
                                               int wt, LDS_AS char* lds) {
  if (MB == 1 || b.rows > 16 * (MB - 1))
    shared_tile<KIND, W, MB, G::NW, kChunk, G::D>(p, e, b, wt, lds);
  else if constexpr (MB > 1)
    tile_of_height<KIND, W, G, MB - 1>(p, e, b, wt, lds);
}

// grid: row blocks x N tiles of 32 * NW weight rows, from tile tn0 on.
template <int KIND, int W, class G>
__global__ __launch_bounds__(kWave * G::NW) __attribute__((amdgpu_waves_per_eu(G::OCC, G::OCC)))
void grouped_gemm_shared_kernel(GemmParams p) {
  constexpr int ROWS = 16 * G::MBX;
  __shared__ __attribute__((aligned(16))) char smem[2 * ROWS * (kChunk + 16)];
  if (not_this_launch(p)) return;
  RowBlock b;
  const int tile = xcd_window_remap(blockIdx.x, gridDim.x);
  if (!locate_rows<ROWS>(p, tile, p.N / (32 * G::NW) - p.tn0, b)) return;
  const int wt = (p.tn0 + b.tn) * G::NW + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  tile_of_height<KIND, W, G, G::MBX>(p, b.e, BlockRows{b.r0, b.rows, false, nullptr}, wt,
                                     (LDS_AS char*)smem);
}

// Gate/up of a small batch that routes its rows itself: block 0 writes the
// routing; workgroup tn of group g takes all of its expert's rows.
template <int W, class G>
__global__ __launch_bounds__(kWave * G::NW) __attribute__((amdgpu_waves_per_eu(G::OCC, G::OCC)))
void grouped_gemm_shared_self_kernel(GemmParams p) {
  constexpr int ROWS = 16 * G::MBX;
  __shared__ __attribute__((aligned(16))) char smem[2 * ROWS * (kChunk + 16)];
  __shared__ int table[kMaxExperts];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  if (blockIdx.x == 0) {
    if (wave == 0) write_routing(p, table);
    return;
  }
  const int tiles_n = p.N / (32 * G::NW);
  const int g = (blockIdx.x - 1) / tiles_n;
  const int tn = blockIdx.x - 1 - g * tiles_n;
  int e;
  BlockRows all;
  if (!route_self(p, g, table, wave == 0, e, all)) return;  // the same answer in every wave
  for (int m0 = 0; m0 < all.rows; m0 += ROWS) {
    __syncthreads();  // the slots are written; the last block's rows are read
    tile_of_height<kGateUp, W, G, G::MBX>(
        p, e, BlockRows{all.r0 + m0, min(ROWS, all.rows - m0), true, all.slots + m0}, tn * G::NW + wave,
        (LDS_AS char*)smem);
  }
}

template <int KIND, int W, class G>
hipError_t launch_shared(const GemmParams& p, int R, int E, hipStream_t stream) {
  constexpr int ROWS = 16 * G::MBX;
  if (p.N % (32 * G::NW)) return hipErrorInvalidValue;
  long long blocks = (long long)(R + ROWS - 1) / ROWS + std::min(E, R);
  if (p.choice && !p.tiled_launch) blocks = std::min<long long>(blocks, p.most_blocks);
  const long long grid = blocks * (p.N / (32 * G::NW) - p.tn0);
  if (grid <= 0) return hipSuccess;
  if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((grouped_gemm_shared_kernel<KIND, W, G>), dim3((unsigned)grid),
                     dim3(kWave * G::NW), 0, stream, p);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// fp8 weights and activations, one row block of 16 rows: every wave loads its
// token rows like its weights (half the bytes of bf16 rows, read through L2);
// the eight waves of a gate/up workgroup own the 128 columns of h that share a
// scale.  (Blocks of 32 and 64 rows, for batches of up to 24 slots per expert,
// gained 3 to 20% on even routing but lost up to 3.5x where a few experts get
// most of the rows: qwen3, 384 tokens, Zipf 1.2: 126 -> 444 us.)
constexpr int kA8Rows = 16;
template <int KIND>
__device__ __forceinline__ void stream_rows_a8(const GemmParams& p, int e, const BlockRows& all,
                                               int wt, LDS_AS float* red) {
  for (int m0 = 0; m0 < all.rows; m0 += kA8Rows) {
    const BlockRows b{all.r0 + m0, min(kA8Rows, all.rows - m0), all.self, all.slots + m0};
    if (KIND == kGateUp) __syncthreads();  // the slots are written; the last block's maxima are read
    stream_tile<KIND, kFp8A8, 1, 5>(p, e, b, wt, red);
  }
}

// grid: min(E, R) experts x N / (32 * waves) workgroups; SELF (gate/up): block
// 0 writes the routing, the others find their own rows.
template <int KIND, bool SELF>
__global__ __launch_bounds__(kWave * (KIND == kGateUp ? kA8Waves : 1))
__attribute__((amdgpu_waves_per_eu(2, 2)))
void grouped_gemm_stream_a8_kernel(GemmParams p) {
  constexpr int NW = KIND == kGateUp ? kA8Waves : 1;
  __shared__ float red[KIND == kGateUp ? kA8Rows * kA8Waves : 1];
  __shared__ int table[SELF ? kMaxExperts : 1];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  if (SELF && blockIdx.x == 0) {
    if (wave == 0) write_routing(p, table);
    return;
  }
  const int bid = blockIdx.x - SELF;
  const int tiles_n = p.N / (32 * NW);
  const int a = bid / tiles_n;
  const int wt = (bid - a * tiles_n) * NW + wave;
  int e;
  BlockRows all;
  if constexpr (SELF) {
    if (!route_self(p, a, table, wave == 0, e, all)) return;  // the same answer in every wave
  } else {
    // routing arrays may come from the caller: clamp every index taken from them
    if (a >= min(max(p.active[0], 0), p.E)) return;
    e = min(max(p.active[1 + a], 0), p.E - 1);
    const int r0 = min(max(p.offsets[e], 0), p.R);
    all = BlockRows{r0, min(max(p.offsets[e + 1], r0), p.R) - r0, false, nullptr};
  }
  stream_rows_a8<KIND>(p, e, all, wt, (LDS_AS float*)red);
}

template <int KIND, int W>
hipError_t enqueue(const GemmParams& p, int R, int E, GemmPath path, hipStream_t stream) {
  if constexpr (KIND == kGateUp && W != kBf16Rows) {
    if (path == kPathWide8) return launch_shared<KIND, W, Wide8>(p, R, E, stream);
  }
  if (path == kPathWide4) return launch_shared<KIND, W, Wide4<W>>(p, R, E, stream);
  const bool self = KIND == kGateUp && p.ids != nullptr;
  if (path == kPathFew && !self) return launch_shared<KIND, W, Few<W>>(p, R, E, stream);
  const int waves = path == kPathFew ? Few<W>::NW : 1;
  const long long grid = (long long)std::min(E, R) * (p.N / (32 * waves)) + self;
  if (grid <= 0) return hipSuccess;
  if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
  if (!self)
    hipLaunchKernelGGL((grouped_gemm_stream_kernel<KIND, W>), dim3((unsigned)grid), dim3(kWave), 0,
                       stream, p);
  else if (waves == 1)
    hipLaunchKernelGGL((grouped_gemm_stream_self_kernel<W>), dim3((unsigned)grid), dim3(kWave), 0,
                       stream, p);
  else
    hipLaunchKernelGGL((grouped_gemm_shared_self_kernel<W, Few<W>>), dim3((unsigned)grid),
                       dim3(kWave * waves), 0, stream, p);
  return hipGetLastError();
}

}  // namespace

template <int KIND>
hipError_t launch_gemm_stream_a8(const GemmParams& p, int R, int E, hipStream_t stream) {
  constexpr int NW = KIND == kGateUp ? kA8Waves : 1;
  const bool self = KIND == kGateUp && p.ids != nullptr;
  if (p.N % (32 * NW)) return hipErrorInvalidValue;
  const long long grid = (long long)std::min(E, R) * (p.N / (32 * NW)) + self;
  if (grid <= 0) return hipSuccess;
  if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
  if (self)
    hipLaunchKernelGGL((grouped_gemm_stream_a8_kernel<KIND, KIND == kGateUp>),
                       dim3((unsigned)grid), dim3(kWave * NW), 0, stream, p);
  else
    hipLaunchKernelGGL((grouped_gemm_stream_a8_kernel<KIND, false>), dim3((unsigned)grid),
                       dim3(kWave * NW), 0, stream, p);
  return hipGetLastError();
}
template hipError_t launch_gemm_stream_a8<kGateUp>(const GemmParams&, int, int, hipStream_t);
template hipError_t launch_gemm_stream_a8<kDownPlainK>(const GemmParams&, int, int, hipStream_t);
template hipError_t launch_gemm_stream_a8<kDownBySlotK>(const GemmParams&, int, int, hipStream_t);

template <int KIND, bool FP8>
hipError_t launch_gemm_stream(const GemmParams& p, int R, int E, GemmPath path,
                              hipStream_t stream) {
  if constexpr (!FP8) return enqueue<KIND, kBf16Rows>(p, R, E, path, stream);
  else if (p.tiled) return enqueue<KIND, kFp8Tiled>(p, R, E, path, stream);
  else return enqueue<KIND, kFp8Rows>(p, R, E, path, stream);
}

template hipError_t launch_gemm_stream<kGateUp, false>(const GemmParams&, int, int, GemmPath,
    hipStream_t);
template hipError_t launch_gemm_stream<kGateUp, true>(const GemmParams&, int, int, GemmPath,
    hipStream_t);
template hipError_t launch_gemm_stream<kDownPlainK, false>(const GemmParams&, int, int, GemmPath,
    hipStream_t);
template hipError_t launch_gemm_stream<kDownPlainK, true>(const GemmParams&, int, int, GemmPath,
    hipStream_t);
template hipError_t launch_gemm_stream<kDownBySlotK, false>(const GemmParams&, int, int, GemmPath,
    hipStream_t);
template hipError_t launch_gemm_stream<kDownBySlotK, true>(const GemmParams&, int, int, GemmPath,
    hipStream_t);

}  // namespace eaas
