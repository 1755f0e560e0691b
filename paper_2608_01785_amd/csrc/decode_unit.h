// Single-row (decode) attention unit.
//
// A unit is one key range (a "split" of unit_keys keys, inside one page of
// the cache) of one row r and one key/value head g; the group's G query heads
// are columns of one 16-wide MFMA (G <= 8 valid), so the keys and values of
// the head are read once for the whole group.  The range is cut into tiles
// (kDecTileKeys keys); wave w takes tiles w, w + 4, w + 8, ... and keeps its
// own running softmax state over them.  A tile is loaded as whole lines into
// registers one tile ahead and passes through a private LDS image of the wave
// (no barrier; keys, then values in their place) into MFMA layout.  The four
// waves' states are merged through LDS.  A row with one split writes its
// output directly; otherwise every split publishes its state and the last
// split of (r, g) to arrive merges them in split order.
//
// What bounds it is memory: the split's keys and values, read once.  MFMA
// fragments fetched straight from the cache put adjacent lanes in different
// key rows, which occupies a CU's address unit for about 93 cycles per 1 KB
// against 17 for whole lines, and 32-wide score tiles spend twice the softmax
// work on columns that hold no query: a talker step (32 rows of 128 .. 1024
// keys, 128 CUs, 16 layers) went from 929 to 909 us without, one of 128 rows
// on 160 CUs from 2068 to 2013.  One register set and half the LDS instead of
// two sets (four blocks a CU instead of three) and non-temporal loads, which
// leave the last-level cache to the weights, brought these to 885 and 1913.
// Five or six blocks a CU spill or gain nothing.  A launch of the first now
// takes 20.4 us for 71 MB, of the second 62 us, one of 8 rows of 16 to 128
// keys 4.1 (4.5 with fragments loaded straight from the cache).
#pragma once

#include "hs_device.h"
#include "hs_kernels.h"

namespace hs {
namespace decode {

constexpr int kUnitThreads = 256;  // threads per block running a unit

template <int DH>
struct DecodeSmem {
  static constexpr int kTile = kDecTileKeys * DH * 2;  // bytes of a tile's keys, and of its values
  union {
    uint8_t tile[4][kTile];  // [wave] a tile's keys, then its values
    struct {
      float red_m[4][8], red_l[4][8];
      float red_o[4][DH][9];  // [wave][d][query head], G <= 8
      int last;
    };
  };
};

// Largest and total value over the four lanes that hold one query's keys
// (lanes l, l ^ 16, l ^ 32, l ^ 48): a swap of a value with itself leaves a
// lane's own value in one result and its partner's in the other.
__device__ __forceinline__ float quarter_max(float v) {
  const uint32_t u = __float_as_uint(v);
  const auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const uint32_t w = __float_as_uint(fmaxf(__uint_as_float(h[0]), __uint_as_float(h[1])));
  const auto q = __builtin_amdgcn_permlane16_swap(w, w, false, false);
  return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
__device__ __forceinline__ float quarter_sum(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

// One work item (a key range of one row) for one key/value head g, by one
// block of 256 threads.
template <int DH>
__device__ __forceinline__ void decode_attn_unit(const DecodeAttnArgs& a, int item, int g, DecodeSmem<DH>& sm) {
  constexpr int TK = kDecTileKeys;        // keys per tile
  constexpr int NKB = DH / 32;                 // 32-wide K steps of q.k
  constexpr int NDS = DH / 16;                 // output subtiles along dh
  constexpr int kTile = DecodeSmem<DH>::kTile;
  constexpr int NL = kTile / 1024;             // 1 KB loads of a tile's keys, and of its values
  static_assert(TK == 32 && TK == kv_tile_keys, "a tile is one value tile of the cache");
  auto& red_m = sm.red_m;
  auto& red_l = sm.red_l;
  auto& red_o = sm.red_o;
  int& last = sm.last;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = lane & 15, fh = lane >> 4;
  const DecItem it = a.items[item];
  const int t = it.t, n_keys = it.n_keys, split = it.split, n_split = it.n_split;
  const int G = a.hq / a.hkv;
  const int k_begin = split * a.unit_keys;
  const int k_end = min(n_keys, k_begin + a.unit_keys);  // keys past it belong to the next range or to none
  const int n_tiles = (k_end - k_begin + TK - 1) / TK;
  // The range lies in one page (of a slot or the packed buffer): its first
  // key sits at key0 = k_begin rounded down to the page size.
  const int key0 = k_begin - k_begin % a.page_keys;
  const int my_tiles = n_tiles > wave ? (n_tiles - wave + 3) / 4 : 0;
  const int qh = min(fr, G - 1);  // query head of this lane's column (padding lanes repeat the last)
  const int64_t kbase = it.kbase + int64_t(g) * a.kv_head_stride;
  const int64_t vbase = it.vbase + int64_t(g) * a.kv_head_stride;

  // Keys and values of tile `ti` of the range, each one contiguous run of
  // kTile bytes: every load of a wave covers 1 KB of whole lines.  Keys past
  // the last one stay inside the page (ranges are whole tiles of a page whose
  // length is a multiple of 64); their scores are masked below.  A tile past
  // the wave's last is read through an empty resource: zeros, no traffic, so
  // every iteration issues the same loads and the wait counts stay exact.
  const __amdgpu_buffer_rsrc_t kres =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.kstore + kbase), 0, 0x7ffffff0, 0x00020000);
  const __amdgpu_buffer_rsrc_t vres =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.vstore + vbase), 0, 0x7ffffff0, 0x00020000);
  const __amdgpu_buffer_rsrc_t zres =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.kstore + kbase), 0, 0, 0x00020000);
  struct {
    u32x4 k[NL], v[NL];
  } tl;
  auto load_k = [&](int i) {
    const __amdgpu_buffer_rsrc_t res = i < my_tiles ? kres : zres;
    const uint32_t so = uint32_t(k_begin + (wave + 4 * i) * TK - key0) * uint32_t(DH * 2);
#pragma unroll
    for (int l = 0; l < NL; ++l)
      tl.k[l] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(res, uint32_t(lane * 16 + l * 1024), so, kNt));
    __builtin_amdgcn_sched_barrier(0);
  };
  auto load_v = [&](int i) {
    const __amdgpu_buffer_rsrc_t res = i < my_tiles ? vres : zres;
    const uint32_t so = uint32_t(k_begin + (wave + 4 * i) * TK - key0) * uint32_t(DH * 2);
#pragma unroll
    for (int l = 0; l < NL; ++l)
      tl.v[l] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(res, uint32_t(lane * 16 + l * 1024), so, kNt));
    __builtin_amdgcn_sched_barrier(0);
  };

  u32x4 qf[NKB];  // B operand of S^T = K Q^T: 32 dimensions per step
  {
    const uint16_t* qp = a.q + (int64_t(t) * a.hq + g * G + qh) * DH + fh * 8;
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) qf[kb] = *reinterpret_cast<const u32x4*>(qp + kb * 32);
  }
  __builtin_amdgcn_sched_barrier(0);
  load_k(0);
  load_v(0);
  float m_run = -INFINITY, l_run = 0.0f;
  f32x4 o[NDS];
#pragma unroll
  for (int i = 0; i < NDS; ++i) o[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  // The wave's LDS tile.  Chunk c (16 bytes) of key row r sits at physical
  // chunk c ^ kswz(r), of value row d at c ^ vswz(d).  A 16-lane pass of
  // fragment reads takes one logical chunk of 16 key rows 8 (i / 4) + i % 4
  // (+ 4): 256-byte rows all start on bank 0 and need 16 different chunks,
  // 128-byte rows 8 per parity; or of 16 consecutive 64-byte value rows,
  // which need the four rows of each bank quarter apart.
  uint8_t* ks = sm.tile[wave];
  uint8_t* vs = ks;  // the values take the keys' place
  auto kphys = [](int r, int c) {
    const int i = ((r >> 3) << 2) | (r & 3);
    return c ^ (DH == 128 ? i : (i >> 1));
  };
  auto vphys = [](int d, int c) { return c ^ ((d >> 2) & 3); };
  constexpr int KCH = DH / 8;  // chunks per key row
  // The swizzles depend on the lane and few of the load's bits: these
  // addresses plus constants reach every chunk.
  constexpr int kPer = NL / 4;  // key loads that share an address
  uint32_t kw[4], kr[NKB];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int ch = q * kPer * 64 + lane, r = ch / KCH, c = ch % KCH;
    kw[q] = uint32_t(r * DH * 2 + kphys(r, c) * 16);
  }
#pragma unroll
  for (int kb = 0; kb < NKB; ++kb) {
    const int r = 8 * (fr >> 2) + (fr & 3);
    kr[kb] = uint32_t(r * DH * 2 + kphys(r, 4 * kb + fh) * 16);
  }
  const uint32_t vw = uint32_t((lane >> 2) * 64 + vphys(lane >> 2, lane & 3) * 16);
  const uint32_t vr = uint32_t(fr * 64 + vphys(fr, fh) * 16);
  // The lanes read each other's chunks: LDS accesses of a wave complete in
  // order, so keeping the program order is enough.
  auto stage_k = [&]() {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int l = 0; l < NL; ++l)
      *reinterpret_cast<u32x4*>(ks + kw[l / kPer] + (l % kPer) * 1024) = tl.k[l];
    asm volatile("" ::: "memory");
  };
  auto stage_v = [&](int ti) {
    asm volatile("" ::: "memory");
    // Values past the range: P is 0 there; keep 0 * garbage out.
    const int v_left = k_end - (k_begin + ti * TK) - 8 * (lane & 3);
    if (k_begin + (ti + 1) * TK > k_end) {
      u32x4 keep;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        keep[e] = (2 * e < v_left ? 0x0000ffffu : 0u) | (2 * e + 1 < v_left ? 0xffff0000u : 0u);
#pragma unroll
      for (int l = 0; l < NL; ++l) *reinterpret_cast<u32x4*>(vs + vw + l * 1024) = tl.v[l] & keep;
    } else {
#pragma unroll
      for (int l = 0; l < NL; ++l) *reinterpret_cast<u32x4*>(vs + vw + l * 1024) = tl.v[l];
    }
    asm volatile("" ::: "memory");
  };
  // Online softmax over this wave's tiles, in the exp2 domain.  Score row i
  // of subtile st is key 8 (i / 4) + 4 st + i % 4, which leaves every lane
  // with keys 8 fh .. 8 fh + 7 of its query: the B operand of O^T = V^T P^T.
  auto do_tile = [&](int i) {
    const int ti = wave + 4 * i;
    const int kv0 = k_begin + ti * TK;
    stage_k();
    load_k(i + 1);
    f32x4 sc[2];
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      sc[st] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
        sc[st] = mfma16(*reinterpret_cast<const u32x4*>(ks + kr[kb] + st * 4 * DH * 2), qf[kb], sc[st]);
    }
    if (kv0 + TK > k_end) {
      const int left = k_end - kv0 - 8 * fh;  // valid keys from the lane's first on
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (4 * st + r >= left) sc[st][r] = -INFINITY;
    }
    // The maximum is taken on the raw scores (the scale is positive) and the
    // scale folded into the exponent's FMA.  Every tile holds at least one
    // valid key, so m_new is finite.
    float mx = fmaxf(sc[0][0], sc[1][0]);
#pragma unroll
    for (int r = 1; r < 4; ++r) mx = fmaxf(mx, fmaxf(sc[0][r], sc[1][r]));
    const float m_new = fmaxf(m_run, quarter_max(mx) * a.scale_log2);
    const float alpha = exp2_raw(m_run - m_new);  // 0 on the first tile
    float psum = 0.0f;
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float p = exp2_raw(fmaf(sc[st][r], a.scale_log2, -m_new));
        sc[st][r] = p;
        psum += p;
      }
    l_run = l_run * alpha + psum;
    m_run = m_new;
#pragma unroll
    for (int i = 0; i < NDS; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) o[i][r] *= alpha;
    __builtin_amdgcn_sched_barrier(0);
    stage_v(ti);
    load_v(i + 1);
    u32x4 pf;
#pragma unroll
    for (int e = 0; e < 4; ++e) pf[e] = pack2h_rne(sc[e >> 1][2 * (e & 1)], sc[e >> 1][2 * (e & 1) + 1]);
#pragma unroll
    for (int i = 0; i < NDS; ++i) o[i] = mfma16(*reinterpret_cast<const u32x4*>(vs + vr + i * 1024), pf, o[i]);
    __builtin_amdgcn_sched_barrier(0);
  };

  for (int i = 0; i < my_tiles; ++i) do_tile(i);

  // Merge the four waves.  Lane (fr, fh) holds query column fr; its four
  // lanes share the maximum, each holds part of the sum.  Waves without a
  // tile hold -inf and weigh zero.
  const float l_tot = quarter_sum(l_run);
  __syncthreads();  // the states take the tiles' place
  if (fh == 0 && fr < 8) {
    red_m[wave][fr] = m_run;
    red_l[wave][fr] = l_tot;
  }
  if (fr < 8) {
#pragma unroll
    for (int i = 0; i < NDS; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) red_o[wave][16 * i + 4 * fh + r][fr] = o[i][r];
  }
  __syncthreads();

  const int pf_stride = dec_part_floats(G, DH);
  const int64_t row_item0 = item - split;  // first split of this row
  for (int idx = tid; idx < G * DH; idx += kUnitThreads) {
    const int q = idx / DH, d = idx % DH;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) M = fmaxf(M, red_m[w][q]);
    float num = 0.0f, den = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float sc = exp2f(red_m[w][q] - M);
      num += sc * red_o[w][d][q];
      den += sc * red_l[w][q];
    }
    if (n_split == 1) {
      a.o[act_index(t, (g * G + q) * DH + d, a.hq * DH, a.o_k8_rows)] = f2h(num / den);
    } else {
      // Publish (unnormalised output, maximum, sum) with device-scope stores.
      float* st = a.part + (int64_t(item) * a.hkv + g) * pf_stride;
      __hip_atomic_store(st + idx, num, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (d == 0) {
        __hip_atomic_store(st + G * DH + q, M, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(st + G * DH + G + q, den, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
  if (n_split == 1) return;

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // partial state complete before the arrival count
  __syncthreads();
  if (tid == 0) {
    int32_t* cnt = a.counters + row_item0 * a.hkv + g;
    last = atomicAdd(cnt, 1) == n_split - 1;
    if (last) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!last) return;

  // Last arrival: combine the splits of (r, g) in split order, eight at a
  // time (all loads of a batch in flight), with a running maximum.
  const float* base = a.part + (row_item0 * a.hkv + g) * pf_stride;
  const int64_t split_stride = int64_t(a.hkv) * pf_stride;
  for (int idx = tid; idx < G * DH; idx += kUnitThreads) {
    const int q = idx / DH;
    float M = -INFINITY, num = 0.0f, den = 0.0f;
    for (int sp0 = 0; sp0 < n_split; sp0 += 8) {
      float mv[8], lv[8], ov[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float* st = base + min(sp0 + k, n_split - 1) * split_stride;
        mv[k] = __hip_atomic_load(st + G * DH + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        lv[k] = __hip_atomic_load(st + G * DH + G + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ov[k] = __hip_atomic_load(st + idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      float bm = M;
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (sp0 + k < n_split) bm = fmaxf(bm, mv[k]);
      const float rescale = exp2f(M - bm);  // M = -inf on the first batch: 0
      num *= rescale;
      den *= rescale;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (sp0 + k < n_split) {
          const float sc = exp2f(mv[k] - bm);
          num += sc * ov[k];
          den += sc * lv[k];
        }
      }
      M = bm;
    }
    a.o[act_index(t, (g * G + q) * DH + idx % DH, a.hq * DH, a.o_k8_rows)] = f2h(num / den);
  }
}

}  // namespace decode
}  // namespace hs
