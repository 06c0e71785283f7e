// Which kernels a batch's two grouped GEMMs take: a function of sizes and
// weight dtype alone, so that it can be asked without a GPU
// (eaas_internal_gemm_plan).
#pragma once

#include "internal.h"

namespace eaas {

enum GemmPath {
  kPathTiled = 0,     // gemm.hip: LDS-DMA tiles
  kPathOneWave = 1,   // gemm_stream.hip: one wave per workgroup
  kPathFew = 2,       // 64-row blocks, four waves
  kPathWide8 = 3,     // 144-row blocks, eight waves
  kPathWide4 = 4,     // 144-row blocks, four waves
  kPathTiledA8 = 5,   // gemm.hip: fp8 activations
  kPathStreamA8 = 6,  // gemm_stream.hip: fp8 activations
};

struct GemmPlan {
  GemmPath path;
  bool routes;   // gate/up: the launch routes the batch itself if it has the ids
  RowRule rule;  // between this path and the tiled kernels
};

// Most slots of a batch whose gate/up launch routes its rows itself.
constexpr int kSelfSlots = 512;
// Rows that a one-wave workgroup, and a self-routing one of four waves, takes
// at once; it walks an expert's further rows in series.
constexpr int kOneWaveRows = 32, kFewRows = 64;
// Rows of the tallest streamed block.
constexpr int kWideRows = 144;

// Which batches the streaming kernels of gemm_stream.hip may take, by the slots
// per resident expert.  The host knows the slots, which other servers' experts
// and (dynamic batches pass their capacity) unused room share, but not the rows
// of each expert; where the answer hangs on those, row_rule below lets the
// device choose.
//
// Few rows: step times, tiled kernels -> streaming (us), by slots per expert:
//   bf16: qwen3 shape 2: 226 -> 190, 32: 284 -> 261, 48: 298 -> 289, 64: 312 ->
//         370; with Zipf 1.1 routing 16: 185 -> 187, 32: 230 -> 252
//         dsv3 shape 16: 503 -> 466, 32: 519 -> 500, 48: 529 -> 530
//         mixtral shape 2: 571 -> 444, 32: 626 -> 517
//   fp8:  dsv3 shape 8: 264 -> 233, 32: 278 -> 268, 48: 293 -> 304; with Zipf
//         1.2 routing 32: 375 -> 330
//         mixtral shape 8: 411 -> 259, 48: 469 -> 358
// One wave per workgroup up to two rows per expert on average: with the waves
// of 1 to 16 tokens its start-up is shorter (qwen3, 1 token: gate/up 25 -> 16
// us, 16 tokens 108 -> 102); from 2 rows on they are equal, and past 4 the rows
// that every wave loads by itself cost more.
// The one-wave kernel takes no batch of more than 32 tokens, and a launch routes
// itself for no more than 64: an expert then has one block of rows (a token's
// slots name different experts).  Past that a hot expert's blocks follow one
// another in each workgroup, where the routing launch's row blocks go to
// different ones (k 1, whole step, tiled / in series / row blocks: H 2048, I
// 512, E 256, 512 tokens of one expert, bf16: 66 / 196 / 47 us; 512 tokens,
// Zipf 1.2: 71 / 160 / 50; H 4096, I 2048, E 32, 512 tokens, Zipf 1.2, fp8: 165
// / 218 / 133).
// Row blocks are found 64 active experts at a time, about 1 us a step, so a long
// list needs a long K (whole step, tiled / row blocks: H 1024, I 256, E 1024,
// k 1, 2048 tokens: fp8 210 / 294 us, bf16 306 / 340; H 4096, I 1024, E 512,
// k 8, 96 tokens, fp8: 954 / 809).
// One 144-row block per expert: the fp8 gate/up GEMM, whose tiled kernel needs a
// second tile past 96 rows: dsv3 shape 64 slots 209 -> 182 us, 64 with Zipf 1.2
// 302 -> 264, 96: 327 -> 239; at 128 it is 336 -> 355.  (The down GEMM's smaller
// tiled workgroups are as fast: 64: 132 -> 129, 96: 163 -> 159.)
// The same where 128-row tiles at most fill the chip once, so that the tiled
// kernels' 256-row ones leave half of it idle: down GEMM, mixtral shape, bf16
// 64 slots 281 -> 185 us, 128: 288 -> 222, fp8 111: 227 -> 187; a bf16 gate/up
// of 8 experts x 1 024 rows, 64 slots: 33 -> 27.
// N no multiple of 256: the streaming kernel alone up to 350 slots per expert or
// two rounds of its blocks, past that the tiled kernel for N / 256 tiles and the
// streaming one for the rest (whole step, H 1920, I 640, E 24, k 6, alone / both,
// bf16: 250 slots 109 / 112 us, 300: 120 / 125, 350: 138 / 135, 500: 214 / 201;
// fp8: 250: 127 / 128, 300: 142 / 141, 350: 161 / 153; H 384, I 128, E 5, k 2,
// 280 slots: 32 / 43).
inline GemmPath stream_path(const FfnArgs& a, bool gateup) {
  const long long R = (long long)a.T * a.k, N = gateup ? 2LL * a.I : a.H;
  const bool few = R <= (a.capacity ? 48 : a.fp8 ? 32 : 24) * (long long)a.E;
  if (few && R <= 2LL * a.E && a.T <= kOneWaveRows) return kPathOneWave;
  const long long steps = ((R < a.E ? R : a.E) + 63) / 64;
  const bool short_k = (gateup ? a.H : a.I) < 128 * (steps - 1);
  if (few && !short_k) return kPathFew;
  if (N % 256 && (R <= 350LL * a.E || (R / 144 + a.E) * (N / 128) <= 512)) return kPathWide4;
  if (R > (a.capacity ? 1024 : 120) * (long long)a.E || short_k) return kPathTiled;
  if (a.E * (N / 128) <= 256) return kPathWide4;
  return a.fp8 && gateup ? kPathWide8 : kPathTiled;
}

// When the rows decide.  (Times of one GEMM, tiled -> streamed, in us.)
//   64-row blocks: up to 64 tokens an expert has one block, and up to 256 tokens
//     and 16 slots per expert further blocks cost about what the choice does.
//     Past that each block re-reads its weights: qwen3 shape bf16, gate/up, 512
//     tokens, even (one block an expert) 185 -> 157, Zipf 1.2 (124 blocks of 77
//     experts) 122 -> 130, 384 equal tokens (48 blocks of 8) 51 -> 66.  fp8 has
//     96-row tiles to beat: dsv3 shape, 192 tokens, Zipf 1.2 (45 of 32) 275 ->
//     219.  With many rows a block the tiled MFMAs win: the same, 48 rows per
//     expert, even, 171 -> 175.  Blocks that fill the chip once win all the same:
//     mixtral shape fp8, down, 128 equal tokens (4 blocks of 2) 190 -> 110.
//   144-row blocks, eight waves: an expert's second block is a second pass over
//     its weights: dsv3 shape fp8, gate/up, 384 tokens, even 301 -> 221, Zipf 0.8
//     (39 of 32) 289 -> 323, 960 tokens (64 of 32) 473 -> 504.
//   144-row blocks, four waves: one workgroup per CU, so a second round doubles
//     the time: mixtral shape bf16, down, 480 tokens (256 workgroups) 276 -> 211,
//     320 with Zipf 0.8 (288) 278 -> 348, 960 (512) 323 -> 374.
// The launch that is not chosen costs 2 to 3 us.
inline RowRule row_rule(const FfnArgs& a, bool gateup, GemmPath path) {
  const long long R = (long long)a.T * a.k;
  const int N = gateup ? 2 * a.I : a.H;
  if (N % 256) return {0, 0, 0, 0};
  RowRule r{0, 0, 0, 0};
  if (path == kPathFew && a.T > kFewRows && (a.T > 256 || R > 16LL * a.E))
    r = a.fp8 ? RowRule{kFewRows, 512 / (N / 128), 3, 40} : RowRule{kFewRows, 256 / (N / 128), 4, 32};
  if (path == kPathWide8 && a.T > kWideRows) r = {kWideRows, 256 / (N / 256), 5, kWideRows};
  if (path == kPathWide4 && a.T > kWideRows) r = {kWideRows, 256 / (N / 128), 0, 0};
  // no routing of these slots has more blocks than the chip holds
  if (r.height > 0 && R / r.height + a.E <= r.one_round) r.height = 0;
  return r;
}

// fp8 activations: the streaming kernel takes the gate/up GEMM of up to 4
// tokens and the down GEMM of up to 16, where an expert has one 16-row block.
// Gate/up has the same workgroups per 128 columns of h either way, so what it
// gains is the routing launch, and it loses where every wave's loads of long
// rows are many (step, tiled / streamed gate/up, both with a streamed down: qwen3
// shape, 4 tokens, 42.7 / 39.1 us; mixtral shape, H 4096, not routed inside: 3
// tokens 199 / 190, 4 tokens 207 / 205; dsv3 shape, H 7168, not routed inside: 3
// tokens with ids of 8 servers 77 / 81, 4 tokens Zipf 1.2 176 / 186, 4 equal
// tokens 90 / 98, against 92 with nothing streamed).  So: where it routes, or up
// to H 4096.  From 5 tokens on (down streamed alone, nothing streamed / that):
// dsv3 shape, 5 tokens 209 / 196, 8 tokens 217 / 205, with ids of 8 servers 98 /
// 93, Zipf 1.2 186 / 179, 16 tokens 247 / 230, Zipf 1.2 212 / 206, 16 equal tokens
// 94 / 97; qwen3 shape, 8 tokens 81 / 73; mixtral shape, 8 tokens 332 / 298.
inline GemmPlan gemm_plan(const FfnArgs& a, bool gateup) {
  const long long R = (long long)a.T * a.k;
  if (!a.act8) {
    const GemmPath path = stream_path(a, gateup);
    // Routing inside the launch saves the routing launch (3 to 5 us), but groups
    // without rows are not compacted away, and where four-wave workgroups are
    // more than the chip holds at once (two on each CU) those that have work
    // pile up on some CUs (whole step, routed by a launch / inside: dsv3 shape
    // bf16, 16 tokens with ids of 8 servers, Zipf 1.2, 4 096 waves: 112 / 158 us;
    // H 2048, I 768, E 256, k 8, 48 equal tokens, 12 288 waves: 49 / 60).
    // One-wave workgroups are short enough to even out on most batches (4 096
    // waves, dsv3 shape, 4 tokens: 158 / 156, Zipf 1.2: 137 / 132, ids of 8
    // servers: 49 / 54; qwen3 shape bf16, 8 tokens, 3 072 waves: 104 / 92).
    const long long waves = (R < a.E ? R : a.E) * (2 * a.I / 32);
    return {path, gateup && R <= kSelfSlots && a.T <= kFewRows &&
                      (path == kPathOneWave || (path == kPathFew && waves <= 2048)),
            row_rule(a, gateup, path)};
  }
  // Routing inside the launch only where one workgroup per CU covers every
  // slot's columns: the groups without rows are not compacted away, and with
  // more workgroups than CUs the ones that have work pile up on some of them
  // (dsv3 shape, 16 tokens with ids of 8 servers: 167 us, compacted by the
  // routing launch 119, tiled 125; qwen3 shape, 16 tokens, Zipf 1.2: 59, tiled
  // 51).
  const bool routes = gateup && a.T <= 4 && R <= kSelfSlots && R <= a.E && R * (2 * a.I / 256) <= 256;
  const bool stream = gateup ? a.T <= 4 && (routes || a.H <= 4096) : a.T <= 16;
  return {stream ? kPathStreamA8 : kPathTiledA8, routes, RowRule{0, 0, 0, 0}};
}

}  // namespace eaas
