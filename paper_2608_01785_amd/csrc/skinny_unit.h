// One block's unit of the skinny (decode-sized) fp16 MFMA GEMM.
//
// Decode re-reads every weight for a handful of rows, so the unit streams W
// rather than reusing it: a block owns a thin strip of weight rows (32, or 64
// when the epilogue needs RoPE or gate/up pairs), all M rows and one K range.
// The four waves split the range among them and load their weights and
// activations into registers two steps ahead, so no wave waits on another
// until the end, where partial accumulators are summed through LDS and the
// fused epilogues run (residual add into fp32, SwiGLU, or RoPE + key/value
// store).  A K split publishes fp32 partial sums; the last split of a strip to
// arrive adds them in split order.
//
// The weights come in one of two ways (FRAG).  A short K: as fragments in MFMA
// layout, straight from memory, in chunks of one or two 32-wide panels.  A
// long K: stages of 64 as whole lines, through an LDS image of the wave's own
// into MFMA layout.  skinny_frag_stages() draws the line.
//
// What bounds it, for large weights and up to 32 rows, is memory, once the
// loads are whole lines: fragments put adjacent lanes in different weight
// rows, which costs a CU's address unit about 93 cycles per 1 KB against 17
// (gate/up of a 3584-wide layer, 272 MB on 256 CUs: 55 us, 4.9 TB/s).  Small
// weights take a launch's latencies: 7 to 9 us for 2 to 17 MB on 128 CUs.  With
// 65 to 128 rows (MT = 4) it is neither: every strip reads the same activations
// again, 16 KB a stage beside 4 or 8 KB of weights, and registers and LDS leave
// one block a CU: 10 to 15 us for the same weights.
//
// Weights are bf16 row-major or prepared fp16 panel-major ([K / 32][N][32]).
// The weight strip is the MFMA A operand and activation rows the B operand, so
// each lane of a 32x32 accumulator owns one activation row and 4 consecutive
// output columns per register group.
#pragma once

#include <type_traits>

#include "hs_device.h"
#include "hs_kernels.h"

namespace hs {
namespace skinny {

constexpr int BK = kSkinnyBK;           // K per stage
constexpr int kLdsBytes = 160 * 1024;
constexpr int kThreads = 256;
constexpr int kDeviceScope = 16;        // buffer cache-policy bit sc1: device-coherent access

// Weight row held in row r of strip `tile` (NR rows per strip).
//   SWIGLU: [gate 32 | up 32] for output columns 32 tile .. + 31.
//   QKV: strip s of head h (DH / 32 strips per head) holds dimensions
//     16 s .. 16 s + 15 then their rotation partners DH / 2 + 16 s .. + 15,
//     so an accumulator lane's registers 4 g + e and 4 (g + 2) + e (g < 2)
//     hold a RoPE pair.
template <int EPI, int NR, int DH>
__device__ __forceinline__ uint32_t strip_row(int tile, int r, int ffn) {
  if constexpr (EPI == EPI_SWIGLU) {
    return uint32_t((r >> 5) * ffn + tile * 32 + (r & 31));
  } else if constexpr (EPI == EPI_QKV) {
    constexpr int SPH = DH / 32;  // strips per head
    const int head = tile / SPH, sub = tile % SPH;
    return uint32_t(head * DH + (r < 16 ? 16 * sub + r : DH / 2 + 16 * sub + (r - 16)));
  } else {
    return uint32_t(tile * NR + r);
  }
}

// LDS of one block: the waves' stage images or the cross-wave reduction
// buffer, and an arrival flag.  A stage image holds two 32-wide panels of
// 32 NS rows.
template <int NS, int MT>
struct SkinnyShape {
  static constexpr int IMAGE = 2 * NS * 32 * 64;
  static constexpr int RED = 4 * NS * MT * 16 * 64 * 4;
  static constexpr int SMEM = (RED > 4 * IMAGE ? RED : 4 * IMAGE) + 16;
};

constexpr int kSets = 2;  // stages in flight per wave, and walked per iteration

// One weight strip (`tile`) and one K split (`ks`) of a skinny GEMM, by one
// block of kThreads threads, in LDS `smem` (SkinnyShape::SMEM bytes, 1 KB
// aligned).
template <int EPI, int DH, bool W_F16, int NS, int MT, bool FRAG>
__device__ __forceinline__ void skinny_unit(const GemmArgs& a, int tile, int ks, uint8_t* smem) {
  constexpr int NR = 32 * NS;                 // weight rows per block
  constexpr int S = kSets;
  constexpr int SMEM = SkinnyShape<NS, MT>::SMEM;
  static_assert(SMEM <= kLdsBytes, "LDS");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = lane & 31, fh = lane >> 5;
  const int n_split = a.n_split;
  const int m_own = wave * 32 + fr;
  const bool row_own = wave < MT && m_own < a.M;
  // Folded RMSNorm: this lane's row's partial sums of squares, half of them in
  // each of the row's two lanes, loaded now and summed in the epilogue (wave w
  // owns rows 32 w .. 32 w + 31 there).  Rows past M fall outside the buffer
  // range and read zero.
  constexpr int kPre = (EPI == EPI_RESID) ? 1 : kSkinnyMaxNormParts / 8;
  u32x4 pre[kPre];
  const bool want_rs = EPI != EPI_RESID && a.row_sumsq && wave < MT;
  if (want_rs) {
    const __amdgpu_buffer_rsrc_t pr = make_rsrc(a.row_sumsq, uint32_t(a.M) * a.row_parts * 4);
    const uint32_t row_off = uint32_t(m_own * a.row_parts + 4 * fh) * 4;
#pragma unroll
    for (int u = 0; u < kPre; ++u)
      if (8 * u < a.row_parts)
        pre[u] = __builtin_amdgcn_raw_buffer_load_b128(pr, row_off + uint32_t(u * 32), 0, 0);
  }
  // Operands of the epilogue that do not depend on the product, loaded now
  // so that they are in registers by then (wave w owns rows 32 w .. 32 w + 31
  // there): RESID the residual and the next norm's gains; QKV the row's
  // position, cache offsets and RoPE table entries (issued after the first
  // stages' loads, see below).
  f32x4 res_pre[EPI == EPI_RESID ? NS : 1][4];
  f32x4 gain_pre[EPI == EPI_RESID ? NS : 1][4];
  if constexpr (EPI == EPI_RESID) {
    if (row_own) {
#pragma unroll
      for (int i = 0; i < NS; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int n = tile * NR + i * 32 + 8 * g + 4 * fh;
          if (a.resid_f32) {
            res_pre[i][g] = *reinterpret_cast<const f32x4*>(a.resid_f32 + int64_t(m_own) * a.ldo + n);
          } else {
            float r4[4];
            load_bf16x4(a.resid + int64_t(m_own) * a.ldo + n, r4);
            res_pre[i][g] = f32x4{r4[0], r4[1], r4[2], r4[3]};
          }
          if (a.scaled_out) {
            float gm[4];
            load_bf16x4(a.gain + n, gm);
            gain_pre[i][g] = f32x4{gm[0], gm[1], gm[2], gm[3]};
          }
        }
    }
  }
  int64_t qkv_koff = 0, qkv_voff = 0;
  if constexpr (EPI == EPI_QKV) {
    if (row_own) {
      qkv_koff = a.k_off[m_own];
      qkv_voff = a.v_off[m_own];
    }
  }
  const int kt0 = ks * a.k_per_split;
  const int KT = min(a.K / BK - kt0, a.k_per_split);  // stages of this split
  const uint32_t row_bytes = uint32_t(a.K) * 2;

  const uint32_t w_rows = (EPI == EPI_SWIGLU) ? uint32_t(2 * a.ffn) : uint32_t(a.n_tiles_n * 256);
  const __amdgpu_buffer_rsrc_t wres = make_rsrc(a.W, w_rows * row_bytes);
  const __amdgpu_buffer_rsrc_t xres =
      make_rsrc(a.A, a.k8_rows ? uint32_t(a.K) * uint32_t(a.k8_rows) * 2 : uint32_t(a.M) * row_bytes);

  // Whole lines: wave w takes stages w, w + 4, w + 8, ... of the split, in
  // pairs, S of them in flight.  A stage past the range is read through an
  // empty buffer resource (zeros, no traffic), so every iteration issues the
  // same loads and the wait counts stay exact; the second of an odd last pair
  // is not multiplied.
  //   weight fragment (A operand): rows strip_row(i * 32 + fr), K 16 s + 8 fh .. + 7
  //   activation fragment (B operand): rows j * 32 + fr, the same K
  // Every weight load of a wave covers 1 KB in runs of 64 bytes or more: 16
  // rows of one 32-wide panel of prepared weights, or 8 rows x 128 bytes.
  static_assert(NS <= 2 && MT <= 4, "fragment slots");
  constexpr int WL = 4 * NS;  // 1 KB weight loads of a stage
  const __amdgpu_buffer_rsrc_t zres = make_rsrc(a.W, 0);
  const uint32_t panel_bytes = w_rows * 64;
  uint8_t* image = smem + wave * SkinnyShape<NS, MT>::IMAGE;
  // 16-byte chunk c of row r of panel q sits in image row r ^ q at physical
  // chunk c ^ (r / 4 % 4): a 16-lane pass of fragment reads takes one logical
  // chunk of 16 consecutive 64-byte rows, which need the four rows of each
  // bank quarter apart; eight writing lanes hold two rows of a panel, or one
  // row of both.
  auto phys = [](int q, int r, int c) { return uint32_t((q * NS * 32 + (r ^ q)) * 64 + (c ^ ((r >> 2) & 3)) * 16); };
  uint32_t w_off[WL], w_lds[WL];
#pragma unroll
  for (int l = 0; l < WL; ++l) {
    if constexpr (W_F16) {
      const int q = l & 1, r = 16 * (l >> 1) + (lane >> 2), c = lane & 3;
      w_off[l] = strip_row<EPI, NR, DH>(tile, r, a.ffn) * 64u + uint32_t(q) * panel_bytes + uint32_t(c * 16);
      w_lds[l] = phys(q, r, c);
    } else {
      const int r = 8 * l + (lane >> 3), c = lane & 7;
      w_off[l] = strip_row<EPI, NR, DH>(tile, r, a.ffn) * row_bytes + uint32_t(c * 16);
      w_lds[l] = phys(c >> 2, r, c & 3);
    }
  }
  const uint32_t w_stage = W_F16 ? 2 * panel_bytes : 128u;
  // Activations row-major: a step is 32 bytes along the row.  k-group-major
  // (k8_rows padded rows): a fragment is 512 contiguous bytes, a step 2
  // k-groups.
  uint32_t x_off[MT];
  const int k8 = a.k8_rows;
#pragma unroll
  for (int j = 0; j < MT; ++j)
    x_off[j] = k8 ? uint32_t((fh * k8 + j * 32 + fr) * 16) : uint32_t(j * 32 + fr) * row_bytes + uint32_t(fh * 16);
  const uint32_t x_step = k8 ? uint32_t(2 * k8 * 16) : 32u;
  const int my_stages = KT > wave ? (KT - wave + 3) / 4 : 0;

  f32x16 acc[NS][MT];
#pragma unroll
  for (int i = 0; i < NS; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  struct Stage {
    u32x4 w[WL];
    u32x4 x[4][MT];
  };
  auto load_w = [&](int i, Stage& b) {
    const __amdgpu_buffer_rsrc_t wr = i < my_stages ? wres : zres;
    const uint32_t P = uint32_t(kt0 + wave + 4 * i);  // stage of the matrix
#pragma unroll
    for (int l = 0; l < WL; ++l) b.w[l] = __builtin_amdgcn_raw_buffer_load_b128(wr, w_off[l], P * w_stage, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto load_x = [&](int i, Stage& b) {
    const __amdgpu_buffer_rsrc_t xr = i < my_stages ? xres : zres;
    const uint32_t P = uint32_t(kt0 + wave + 4 * i);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int j = 0; j < MT; ++j)
        b.x[s][j] = __builtin_amdgcn_raw_buffer_load_b128(xr, x_off[j] + x_step * s, P * 4 * x_step, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // Stage i: its weights through the wave's image, the loads of stage i + S
  // into the registers it leaves (`next`: its pair has one), its products.
  // Nothing here waits for stage i + 1, so a wave with four stages (K = 1024)
  // takes two memory latencies.  Passing stage i + 1 through LDS ahead of
  // stage i's products hides the LDS latency, but then the activations of
  // stage i + 2 are not asked for before the weights of stage i + 1 are
  // there: three latencies, and loads past the end besides (talker step of
  // one row, two layers, 64 CUs: 83.3 us against 76.7; 16 layers of 32 rows on
  // 128 CUs 880 against 850; one thinker layer of 4 rows 195 against 192).
  // The lanes read each other's chunks: LDS accesses of a wave complete in
  // order, so keeping the program order is enough.
  auto stage = [&](int i, Stage& b, auto next) {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int l = 0; l < WL; ++l) *reinterpret_cast<u32x4*>(image + w_lds[l]) = b.w[l];
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (decltype(next)::value) load_w(i + S, b);
    u32x4 f[4][NS];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int n = 0; n < NS; ++n)
        f[s][n] = *reinterpret_cast<const u32x4*>(image + phys(s >> 1, fr, 2 * (s & 1) + fh) + n * 32 * 64);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int n = 0; n < NS; ++n) {
        const u32x4 wh = W_F16 ? f[s][n] : bf8_to_h8(f[s][n]);
#pragma unroll
        for (int j = 0; j < MT; ++j) acc[n][j] = mfma32(wh, b.x[s][j], acc[n][j]);
      }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (decltype(next)::value) load_x(i + S, b);
  };

  // FRAG: the wave's 32-wide panels w, w + 4, w + 8, ... of the split, as
  // fragments, in chunks of CH panels: chunk c + 1 is loaded while chunk c is
  // multiplied, chunk 0 always (a panel past the range reads zeros), later
  // ones only when they hold panels, so the wait counts stay exact.
  constexpr int CH = NS + MT <= 3 ? 2 : 1;
  const int n_panels = 2 * KT;
  const int my_panels = n_panels > wave ? (n_panels - wave + 3) / 4 : 0;
  const int n_chunks = (my_panels + CH - 1) / CH;
  struct Chunk {
    u32x4 w[CH][2][NS];
    u32x4 x[CH][2][MT];
  };
  uint32_t f_off[NS];
#pragma unroll
  for (int n = 0; n < NS; ++n)
    f_off[n] = strip_row<EPI, NR, DH>(tile, n * 32 + fr, a.ffn) * (W_F16 ? 64u : row_bytes) + uint32_t(fh * 16);
  auto load_chunk = [&](int c, Chunk& b) {
#pragma unroll
    for (int q = 0; q < CH; ++q) {
      const int p = wave + 4 * (c * CH + q);  // panel of this split
      const __amdgpu_buffer_rsrc_t wr = p < n_panels ? wres : zres;
      const __amdgpu_buffer_rsrc_t xr = p < n_panels ? xres : zres;
      const uint32_t P = uint32_t(2 * kt0 + p);  // panel of the matrix
#pragma unroll
      for (int s = 0; s < 2; ++s) {
#pragma unroll
        for (int n = 0; n < NS; ++n)
          b.w[q][s][n] = __builtin_amdgcn_raw_buffer_load_b128(wr, f_off[n] + 32 * s, P * (W_F16 ? panel_bytes : 64u), 0);
#pragma unroll
        for (int j = 0; j < MT; ++j)
          b.x[q][s][j] = __builtin_amdgcn_raw_buffer_load_b128(xr, x_off[j] + x_step * s, P * 2 * x_step, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto mma_chunk = [&](const Chunk& b) {
#pragma unroll
    for (int q = 0; q < CH; ++q)
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int n = 0; n < NS; ++n) {
          const u32x4 wh = W_F16 ? b.w[q][s][n] : bf8_to_h8(b.w[q][s][n]);
#pragma unroll
          for (int j = 0; j < MT; ++j) acc[n][j] = mfma32(wh, b.x[q][s][j], acc[n][j]);
        }
    __builtin_amdgcn_sched_barrier(0);
  };

  Stage st[S];
  Chunk b0, b1;
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (FRAG) {
    load_chunk(0, b0);
  } else {
#pragma unroll
    for (int u = 0; u < S; ++u) {
      load_w(u, st[u]);
      load_x(u, st[u]);
    }
  }
  // QKV: the RoPE table entries of this lane's dimension pairs and, with a
  // bias, the bias of its columns (registers 4 g + e: dimension
  // 16 sub + 8 g + 4 fh + e, registers 4 (g + 2) + e: that plus DH / 2).
  float2 rope_pre[EPI == EPI_QKV ? 8 : 1];
  float bias_pre[EPI == EPI_QKV ? 16 : 1];
  if constexpr (EPI == EPI_QKV) {
    if (row_own) {
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        // Pairs j .. j + 3 share one RoPE section (sections are multiples of 4 pairs).
        const int j = 16 * (tile % (DH / 32)) + 8 * g + 4 * fh;
        const float2* rt = a.rope + int64_t(rope_pos(a, m_own, j)) * (DH / 2) + j;
#pragma unroll
        for (int e = 0; e < 4; ++e) rope_pre[4 * g + e] = rt[e];
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) bias_pre[r] = 0.0f;
    if (a.bias && wave < MT) {
      const uint16_t* bp = a.bias + (tile / (DH / 32)) * DH + 16 * (tile % (DH / 32)) + 4 * fh;
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        load_bf16x4(bp + 8 * g, &bias_pre[4 * g]);
        load_bf16x4(bp + 8 * g + DH / 2, &bias_pre[4 * (g + 2)]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (FRAG) {
    int c = 0;
    for (; c + 2 < n_chunks; c += 2) {
      load_chunk(c + 1, b1);
      mma_chunk(b0);
      load_chunk(c + 2, b0);
      mma_chunk(b1);
    }
    if (n_chunks - c == 2) {
      load_chunk(c + 1, b1);
      mma_chunk(b0);
      mma_chunk(b1);
    } else if (n_chunks - c == 1) {
      mma_chunk(b0);
    }
  } else {
    constexpr std::true_type more{};
    constexpr std::false_type done{};
    int i = 0;
    for (; i + S < my_stages; i += S) {
      stage(i, st[0], more);
      stage(i + 1, st[1], more);
    }
    stage(i, st[0], done);
    if (i + 1 < my_stages) stage(i + 1, st[1], done);
  }

  // Sum the four waves' partial accumulators through LDS ([wave][i][j][lane]
  // images of 16 floats, moved 16 bytes at a time); wave w then owns row
  // subtile j = w (MT <= 4).
  __syncthreads();
  f32x4* red = reinterpret_cast<f32x4*>(smem);
#pragma unroll
  for (int i = 0; i < NS; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        red[(((wave * NS + i) * MT + j) * 64 + lane) * 4 + q] =
            f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
  __syncthreads();
  const int j = wave;
  const bool owner = j < MT;
  f32x16 c[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
      if (owner) {
#pragma unroll
        for (int w = 0; w < 4; ++w) v += red[(((w * NS + i) * MT + j) * 64 + lane) * 4 + q];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) c[i][4 * q + e] = v[e];
    }

  if (n_split > 1) {
    // Publish this split's sums; the last split of the strip to arrive adds
    // all splits in split order (the same order whoever arrives last) and
    // runs the epilogue.  Partial sums move with device-scope (sc1) vector
    // accesses, which write through to and read from the coherent level, so
    // no agent-scope fence (a full L2 write-back and invalidate) is needed.
    constexpr int IMG = NS * MT * 16 * 64;  // floats per split image: [i][j][lane][16]
    const __amdgpu_buffer_rsrc_t pres =
        make_rsrc(a.part + size_t(tile) * n_split * IMG, uint32_t(n_split) * IMG * 4);
    if (owner) {
#pragma unroll
      for (int i = 0; i < NS; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 v = {c[i][4 * q], c[i][4 * q + 1], c[i][4 * q + 2], c[i][4 * q + 3]};
          const uint32_t off = uint32_t(((ks * NS + i) * MT + j) * 1024 + lane * 16 + 4 * q) * 4;
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), pres, off, 0, kDeviceScope);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // stores complete before the arrival count
    __syncthreads();
    int* last = reinterpret_cast<int*>(smem + SMEM - 16);  // past the reduction buffer
    if (tid == 0) {
      const int arrived = atomicAdd(a.counters + tile, 1);
      *last = arrived == n_split - 1;
      if (*last) __hip_atomic_store(a.counters + tile, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!*last) return;
    // All threads add the split images (every load in flight at once), then
    // the owners pick their registers up from LDS.
    f32x4* red4 = reinterpret_cast<f32x4*>(smem);
    for (int e = tid; e < IMG / 4; e += kThreads) {
      // Splits past n_split lie outside the buffer resource and read zero.
      u32x4 x[kSkinnyMaxSplits];
#pragma unroll
      for (int sp = 0; sp < kSkinnyMaxSplits; ++sp)
        x[sp] = __builtin_amdgcn_raw_buffer_load_b128(pres, uint32_t((sp * IMG + 4 * e) * 4), 0, kDeviceScope);
      f32x4 v = __builtin_bit_cast(f32x4, x[0]);
#pragma unroll
      for (int sp = 1; sp < kSkinnyMaxSplits; ++sp) v += __builtin_bit_cast(f32x4, x[sp]);
      red4[e] = v;
    }
    __syncthreads();
    if (owner) {
#pragma unroll
      for (int i = 0; i < NS; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) c[i][r] = reinterpret_cast<const float*>(red4)[((i * MT + j) * 64 + lane) * 16 + r];
    }
  }

  const int m = j * 32 + fr;
  if constexpr (EPI == EPI_RESID) {
    const int strips = a.n_tiles_n * 256 / NR;
    if (owner && m < a.M) {
      float* orow = a.out_f32 + int64_t(m) * a.ldo;
      float ss = 0.0f;
#pragma unroll
      for (int i = 0; i < NS; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int n = tile * NR + i * 32 + 8 * g + 4 * fh;
          f32x4 v = {c[i][4 * g], c[i][4 * g + 1], c[i][4 * g + 2], c[i][4 * g + 3]};
          v += res_pre[i][g];
          *reinterpret_cast<f32x4*>(orow + n) = v;
          ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
          if (a.scaled_out) {
            const f32x4 gm = gain_pre[i][g];
            store_h4(a.scaled_out + act_index(m, n, a.ldo, a.k8_rows), v[0] * gm[0], v[1] * gm[1], v[2] * gm[2],
                     v[3] * gm[3]);
          }
        }
      if (a.sumsq_out) {
        // The lane pair (fh = 0, 1) holds this row's NR columns of the strip.
        ss += __shfl_xor(ss, 32, 64);
        if (fh == 0) st_f32<false>(a.sumsq_out + int64_t(m) * strips + tile, ss);
      }
    }
    return;
  } else {
    if (!owner) return;
    if (want_rs) {
      float sum = 0.0f;
#pragma unroll
      for (int u = 0; u < kPre; ++u) {
        if (8 * u >= a.row_parts) break;
        const f32x4 f = __builtin_bit_cast(f32x4, pre[u]);
        if (8 * u + 4 * fh < a.row_parts) sum += f[0] + f[1] + f[2] + f[3];
      }
      sum += __shfl_xor(sum, 32, 64);
      const float rs = rsqrtf(sum / float(a.K) + a.eps);
#pragma unroll
      for (int i = 0; i < NS; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) c[i][r] *= rs;
    }
    if (m >= a.M) return;
    if constexpr (EPI == EPI_QKV) {
#pragma unroll
      for (int r = 0; r < 16; ++r) c[0][r] += bias_pre[r];
    }
  }
  if constexpr (EPI == EPI_SWIGLU) {
    static_assert(EPI != EPI_SWIGLU || NS == 2, "gate/up strips hold 32 + 32 rows");
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = silu(c[0][4 * g + e]) * c[1][4 * g + e];
      store_h4(a.out + act_index(m, tile * 32 + 8 * g + 4 * fh, a.ldo, a.k8_rows), v[0], v[1], v[2], v[3]);
    }
  } else {  // EPI_QKV: a strip holds 16 dimensions of one head and their RoPE partners
    static_assert(EPI != EPI_QKV || NS == 1, "QKV strips are 32 rows");
    constexpr int SPH = DH / 32;
    const int head = tile / SPH, sub = tile % SPH;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const int d = 16 * sub + 8 * g + 4 * fh;  // < DH / 2; partner d + DH / 2
      if (head < a.hq + a.hkv) {
        float rl[4], rh[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float2 cs = rope_pre[4 * g + e];
          const float lo = c[0][4 * g + e], hi = c[0][4 * (g + 2) + e];
          rl[e] = fmaf(lo, cs.x, -(hi * cs.y));
          rh[e] = fmaf(hi, cs.x, lo * cs.y);
        }
        uint16_t* dst = (head < a.hq) ? a.q + (int64_t(m) * a.hq + head) * DH
                                      : a.kstore + qkv_koff + int64_t(head - a.hq) * a.kv_head_stride;
        store_h4(dst + d, rl[0], rl[1], rl[2], rl[3]);
        store_h4(dst + d + DH / 2, rh[0], rh[1], rh[2], rh[3]);
      } else {
        const int gh = head - a.hq - a.hkv;
        uint16_t* dst = a.vstore + qkv_voff + int64_t(gh) * a.kv_head_stride;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          dst[(d + e) * kv_tile_keys] = f2h(c[0][4 * g + e]);
          dst[(d + DH / 2 + e) * kv_tile_keys] = f2h(c[0][4 * (g + 2) + e]);
        }
      }
    }
  }
}

}  // namespace skinny
}  // namespace hs
