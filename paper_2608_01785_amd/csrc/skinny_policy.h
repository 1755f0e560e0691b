// Work split of the skinny (decode-sized) GEMM, shared by the launcher and the
// workspace planner.  Pure C++; no HIP types.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace hs {

constexpr int kSkinnyMaxRows = 128;      // M at or below this takes the skinny GEMM
constexpr int kSkinnyBK = 64;            // K per pipeline stage
constexpr int kSkinnyTargetBlocks = 128; // blocks wanted per launch
constexpr int kSkinnyMaxSplits = 8;
constexpr int kSkinnyMinStages = 8;      // K stages per split at least
constexpr int kSkinnySplitBelow = 128;   // only GEMMs with fewer strips split K ...
constexpr int kSkinnySplitFrom = 32;     // ... and only when K has this many stages
constexpr int kSkinnyMaxNormParts = 64;  // folded RMSNorm: partial sums per row a consumer prefetches

// 32-row activation subtiles covering M rows (1, 2 or 4).
inline int skinny_m_tiles(int M) { return M <= 32 ? 1 : (M <= 64 ? 2 : 4); }

// K stages of a block up to which its waves load weight fragments straight
// from memory; beyond, whole lines through LDS (skinny_unit.h).  ns and
// m_tiles: 32-row subtiles of weights and activations per block.
//
// Whole lines are cheaper per byte (a CU's address unit takes 17 cycles per
// 1 KB against 93); fragments are in MFMA layout when they arrive and come in
// finer chunks, which is what a short K, and a block with more products per
// byte, waits for.  bf16 fragments lie further apart than those of a prepared
// fp16 panel.  Time with fragments over time with lines, weights in the
// last-level cache, 128 CUs (N = 256 / 4096 gate+up):
//          rows      K 256       K 512       K 768       K 1024      K 1536
//   fp16   1-32    .97 / .91   .99 / .95  1.01 / .98  1.03 / 1.04 1.08 / 1.07
//          33-64   .92 / .87   .97 / .92   .96 / .91  1.01 / .97  1.05 / 1.00
//          65-128  .87 / .87   .92 / .89   .91 / .86   .96 / .92   .99 / .96
//   bf16   1-32    .99 / .97  1.06 / 1.06 1.11 / 1.14 1.17 / 1.25 1.23 / 1.43
//          33-64   .97 / .91  1.04 / 1.01 1.08 / 1.05 1.15 / 1.14 1.17 / 1.27
//          65-128  .89 / .87   .98 / .94   .98 / .96  1.06 / 1.05 1.13 / 1.15
// Weights that stream from memory move the line down: lines ask for it in
// order.  `resident`: the weights of all the call's layers fit the last-level
// cache (256 MB) beside its other data.  Layers of 33.6 MB, 90 rows, fp16, K =
// 1024 as fragments / lines: four 194 / 202 us, six 285 / 297, eight 425 / 416,
// twelve 673 / 650; 128 rows: six 294 / 304, seven 367 / 353.
constexpr int64_t kSkinnyResidentBytes = int64_t(208) << 20;
inline int skinny_frag_stages(int ns, int m_tiles, bool w_f16, bool resident) {
  if (w_f16) return !resident || m_tiles == 1 ? 12 : m_tiles == 2 ? 16 : 24;
  return m_tiles == 4 ? 12 : m_tiles == 2 && ns == 2 ? 8 : 4;
}

// Activations of decode-sized batches are stored k-group-major with this many
// (padded) rows: element (m, k) at ((k / 8) * rows + m) * 8 + k % 8.  Rows
// M .. rows - 1 are never written; the GEMM discards their products.
inline int skinny_k8_rows(int M) { return 32 * skinny_m_tiles(M); }

struct SkinnySplit {
  int splits;  // blocks along K per weight strip
  int per;     // K stages per split (the last split may hold fewer)
};

// GEMMs with few weight strips split K until strips * splits reaches the
// target, keeping at least kSkinnyMinStages stages per split (a split's
// partial sums cost one extra round trip to memory) and no empty split.
inline SkinnySplit skinny_split(int strips, int k_stages) {
  if (strips >= kSkinnySplitBelow || k_stages < kSkinnySplitFrom) return {1, k_stages};
  int s = (kSkinnyTargetBlocks + strips - 1) / strips;
  s = std::min(s, kSkinnyMaxSplits);
  s = std::min(s, std::max(1, k_stages / kSkinnyMinStages));
  s = std::max(s, 1);
  const int per = (k_stages + s - 1) / s;
  s = (k_stages + per - 1) / per;
  return {s, per};
}

// Weight strips per GEMM: 32 output rows (residual GEMMs), 32 gate + 32 up
// rows (SwiGLU), 16 dimensions of one head and their RoPE partners (QKV).
inline int skinny_strips_resid(int n_out) { return n_out / 32; }
inline int skinny_strips_swiglu(int ffn) { return ffn / 32; }
inline int skinny_strips_qkv(int hq, int hkv, int dh) { return (hq + 2 * hkv) * (dh / 32); }

// fp32 partial sums of one split of one strip: NS x MT accumulator images of
// 16 registers x 64 lanes.
inline size_t skinny_partial_bytes(int ns, int m_tiles) { return size_t(ns) * m_tiles * 16 * 64 * 4; }

}  // namespace hs
