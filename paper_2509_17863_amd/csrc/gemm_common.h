// Device-side parts shared by the grouped GEMM kernels (gemm.hip,
// gemm_stream.hip): the launch parameters and the lookups of a group's
// weights and scales.
#pragma once

#include "common.h"
#include "dispatch.h"

namespace eaas {

#define LDS_AS __attribute__((address_space(3)))
#define CONST_AS __attribute__((address_space(4)))  // read-only global data, scalar loads
#define GLOBAL_AS __attribute__((address_space(1)))

typedef int i32x8 __attribute__((ext_vector_type(8)));

enum GemmKind { kGateUp = 0, kDownPlainK = 1, kDownBySlotK = 2 };

struct GemmParams {
  const uint16_t* a;      // gate/up: x [T, lda]; down: h [R, lda]
  const int32_t* perm;    // [R]
  int k;                  // slots per token
  int lda;                // K of this GEMM
  const uint8_t* b;       // weights [E, N, K] (bf16 or fp8 bytes)
  const float* b_scale;   // [E, N/128, K/128] (fp8)
  int N;                  // weight rows per expert
  int K;                  // reduction length
  int I;                  // intermediate size (gate/up: up rows start at I)
  const int32_t* offsets; // [E+1]
  const int32_t* active;  // [E+1]
  uint16_t* h;            // gate/up output [R, I]
  float* y;               // down output [R, N]
  int R;                  // slots (T*k)
  int E;                  // resident experts (groups)
  // server step over several layers: group e is expert e % e_layer of layer
  // e / e_layer, whose weights come from that layer's record instead of b
  const eaas_layer_weights* layers;  // nullptr: one weight array (b, b_scale)
  int e_layer;
  bool down;              // the records' down-projection members
  // fp8 activations: A is fp8 (a8, rows of K bytes) with one fp32 scale per
  // row and 128 channels (a_scale [rows, K/128]); the gate/up epilogue writes
  // h quantized the same way (hq [R, I], hs [R, I/128])
  const uint8_t* a8;
  const float* a_scale;
  uint8_t* hq;
  float* hs;
  // fp8 weights in the tiled layout of tile_weights_fp8 (the ring kernels'
  // weight stages stored contiguously) instead of [E, N, K] row-major
  bool tiled;
  int tn0;                // streaming kernels: first N tile of the launch
  // a small batch's gate/up launch that routes its rows itself: the slots'
  // expert ids [R]; it writes counts, offsets, perm, inv and active
  const int32_t* ids;
  int32_t* counts;
  int32_t* inv;
  // one of two launches of which the batch's rows let one run: where the choice
  // stands, this GEMM's bit in it, and whether this is the tiled launch
  const int32_t* choice;
  int choice_bit;
  bool tiled_launch;
  int most_blocks;        // row blocks of the streaming launch, if it runs
};

// Whether the batch is the other launch's.
__device__ __forceinline__ bool not_this_launch(const GemmParams& p) {
  if (p.choice == nullptr) return false;
  return ((*(const CONST_AS int32_t*)p.choice & p.choice_bit) != 0) == p.tiled_launch;
}

// Weights of group e ([N, K], bf16 or fp8 bytes of esz each).
__device__ __forceinline__ const uint8_t* group_weights(const GemmParams& p, int e, int esz) {
  if (p.layers == nullptr) return p.b + (size_t)e * p.N * p.K * esz;
  const int L = e / p.e_layer;
  const eaas_layer_weights& lw = p.layers[L];
  return static_cast<const uint8_t*>(p.down ? lw.w_down : lw.w_gate_up) +
         (size_t)(e - L * p.e_layer) * p.N * p.K * esz;
}

// fp8 block scales of group e ([N/128, K/128]).
__device__ __forceinline__ const float* group_scales(const GemmParams& p, int e) {
  const size_t per = (size_t)(p.N / 128) * (p.K / 128);
  if (p.layers == nullptr) return p.b_scale + (size_t)e * per;
  const int L = e / p.e_layer;
  const eaas_layer_weights& lw = p.layers[L];
  return (p.down ? lw.w_down_scale : lw.w_gate_up_scale) + (size_t)(e - L * p.e_layer) * per;
}

constexpr int kNumXcd = 8;

// Workgroups are dispatched in id order and round-robin over the XCDs
// (XCD = id mod 8).  The k-th workgroup of XCD x takes tile
//   (k / 32) * 256 + x * 32 + k % 32,
// so the 32 workgroups an XCD runs at once hold 32 consecutive tiles (they
// share token and weight tiles in its L2) and the 256 running on the whole
// GPU hold one window of 256 consecutive tiles, which keeps the weights the
// XCDs re-read within the window in the shared MALL.  Tiles past the last
// whole window keep their ids.
__device__ __forceinline__ int xcd_window_remap(int bid, int total) {
  constexpr int kChunk = 32;
  constexpr int window = kNumXcd * kChunk;
  if (bid >= (total / window) * window) return bid;
  const int x = bid % kNumXcd, kk = bid / kNumXcd;
  return (kk / kChunk) * window + x * kChunk + (kk % kChunk);
}

struct Tile {
  int e;           // expert
  int tn;          // weight (N) tile
  int r0;          // first permuted row of the tile
  int rows_valid;  // rows of the tile that belong to the expert
};

// silu(g) * u with the hardware exp and reciprocal (a few ulp from the
// correctly rounded value, which moves rare h roundings by one bf16 ulp).
__device__ __forceinline__ float silu_mul(float g, float u) {
  return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;
}

__device__ __forceinline__ void lds_barrier() { asm volatile("s_barrier" ::: "memory"); }

// 8 fp8-e4m3 values -> 8 bf16 (exact).
__device__ __forceinline__ bf16x8 fp8x8_to_bf16(u32x2 q) {
  bf16x2 v0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(q[0], 1.0f, false);
  bf16x2 v1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(q[0], 1.0f, true);
  bf16x2 v2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(q[1], 1.0f, false);
  bf16x2 v3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(q[1], 1.0f, true);
  return bf16x8{v0[0], v0[1], v1[0], v1[1], v2[0], v2[1], v3[0], v3[1]};
}

// A wave-uniform pointer held in SGPRs even where the compiler cannot prove it
// uniform (free when it already is).
__device__ __forceinline__ const void* wave_uniform(const void* p) {
  const uint64_t v = reinterpret_cast<uintptr_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const void*>(((uint64_t)hi << 32) | lo);
}

// The register-streaming kernels (gemm_stream.hip) of the given path.
template <int KIND, bool FP8>
hipError_t launch_gemm_stream(const GemmParams& p, int R, int E, GemmPath path,
                              hipStream_t stream);
// The same for fp8 weights times fp8 activations (row-major weights).
template <int KIND>
hipError_t launch_gemm_stream_a8(const GemmParams& p, int R, int E, hipStream_t stream);

}  // namespace eaas
