// fp16 MFMA GEMM in small tiles for gfx950: the shapes whose 256 x 256 tiles
// would leave most of the budget's CUs idle (gemm_policy.h says which).
//
// Same contraction and epilogues as the persistent GEMM (gemm.hip), and the
// same accumulation order per output element (K ascending in 16-wide MFMA
// steps, residual first), so which of the two runs changes no bit
// (tests/test_gpu_gemm_kernels.py).
//
// A block is WN x WM waves over a tile of 32 NS WN weight rows x 32 MT WM
// activation rows; K advances in stages of 64 through two LDS buffers, fetched
// two to three stages ahead into registers.  What bounds it is the path into
// the CU, not the matrix pipe: a 128 x 128 tile needs 32 KB a stage for 512
// MFMA cycles, and a CU takes about 58 bytes a cycle from its L2 and 20 from
// HBM.  Measured on the way here (389 x 3584 x 18944, 112 tiles of 128 x 128
// on 160 CUs): weight fragments straight from memory into registers 212 us
// (rows 64 bytes apart cost the address unit a cycle each: 93 cycles per 1 KB
// load against 17 for whole lines), through LDS 166, with each step's
// accesses pinned between its MFMAs and conflict-free writes 120.
#include "hs_device.h"
#include "hs_kernels.h"

namespace hs {
namespace {

constexpr int BK = 64;               // K per stage
constexpr int kRowBytes = BK * 2;    // 128 bytes = 8 chunks of 16
constexpr int kKk = BK / 16;         // MFMA steps per stage
constexpr int kGroupM = 8;

// Weight row held in row r of a strip; SWIGLU and QKV strips hold 16 rows and
// their 16 partners (gate / up, rotation pairs), so registers 4 g + e and
// 4 (g + 2) + e (g < 2) of a lane are a pair.
template <int EPI, int DH>
__device__ __forceinline__ uint32_t strip_row(int strip, int r, int ffn) {
  if constexpr (EPI == EPI_SWIGLU) {
    return uint32_t((r >> 4) * ffn + strip * 16 + (r & 15));
  } else if constexpr (EPI == EPI_QKV) {
    constexpr int SPH = DH / 32;
    const int head = strip / SPH, sub = strip % SPH;
    return uint32_t(head * DH + (r >> 4) * (DH / 2) + 16 * sub + (r & 15));
  } else {
    return uint32_t(strip * 32 + r);
  }
}

// 16-byte chunk c of tile row r sits at physical chunk c ^ swz(r).  Reads move
// 256 bytes a cycle: a pass takes one logical chunk of eight even and eight
// odd rows, and odd rows start on bank 32, so swz is a permutation of bits
// 1 .. 3 of r.  Writes move 128 bytes a cycle: eight lanes hold a whole row,
// or four chunks of rows r and r + 1 of a panel, which bit 0 of r keeps in
// different halves.
__device__ __forceinline__ int phys(int r, int c) { return c ^ ((r >> 1) & 7) ^ ((r & 1) << 2); }

// One row subtile's outputs: accumulator c of strip `strip`, activation row m.
template <int EPI, int DH>
__device__ __forceinline__ void store_rows(const GemmArgs& a, const f32x16& c, int strip, int m, int fh) {
  if constexpr (EPI == EPI_RESID) {
    float* orow = a.out_f32 + int64_t(m) * a.ldo + strip * 32 + 4 * fh;
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<f32x4*>(orow + 8 * g) = f32x4{c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]};
  } else if constexpr (EPI == EPI_GATED) {
    const int n = strip * 32 + 4 * fh;
    float* orow = a.out_f32 + int64_t(m) * a.ldo + n;
    const float* grow = a.gate + int64_t(a.row_seq[m]) * a.gate_stride + n;
    const uint16_t* brow = a.bias + n;
    float r[4][4], b[4][4];
    f32x4 gt[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      load_bf16x4(brow + 8 * g, b[g]);
      gt[g] = *reinterpret_cast<const f32x4*>(grow + 8 * g);
      if (a.resid_f32) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(a.resid_f32 + int64_t(m) * a.ldo + n + 8 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) r[g][e] = v[e];
      } else {
        load_bf16x4(a.resid + int64_t(m) * a.ldo + n + 8 * g, r[g]);
      }
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = gated(r[g][e], gt[g][e], c[4 * g + e], b[g][e]);
      *reinterpret_cast<f32x4*>(orow + 8 * g) = v;
    }
  } else if constexpr (EPI == EPI_GELU) {
    uint16_t* orow = a.out + int64_t(m) * a.ldo + strip * 32;
    const uint16_t* brow = a.bias + strip * 32 + 4 * fh;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      float v[2][4];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float b[4];
        load_bf16x4(brow + 16 * p + 8 * h, b);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[h][e] = gelu(c[8 * p + 4 * h + e] + b[e]);
      }
      store_h8_pair(orow + 16 * p, fh, v[0], v[1]);
    }
  } else if constexpr (EPI == EPI_SWIGLU) {
    float v[2][4];
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[g][e] = silu(c[4 * g + e]) * c[4 * (g + 2) + e];
    store_h8_pair(a.out + int64_t(m) * a.ldo + strip * 16, fh, v[0], v[1]);
  } else {  // EPI_QKV
    constexpr int SPH = DH / 32;
    const int head = strip / SPH, sub = strip % SPH;
    float lo[2][4], hi[2][4];
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        lo[g][e] = c[4 * g + e];
        hi[g][e] = c[4 * (g + 2) + e];
      }
    if (a.bias) {
      const uint16_t* bp = a.bias + head * DH + 16 * sub + 4 * fh;
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        float bl[4], bh[4];
        load_bf16x4(bp + 8 * g, bl);
        load_bf16x4(bp + 8 * g + DH / 2, bh);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          lo[g][e] += bl[e];
          hi[g][e] += bh[e];
        }
      }
    }
    if (head >= a.hq + a.hkv) {
      uint16_t* dst = a.vstore + a.v_off[m] + int64_t(head - a.hq - a.hkv) * a.kv_head_stride;
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int d = 16 * sub + 8 * g + 4 * fh + e;
          dst[d * kv_tile_keys] = f2h(lo[g][e]);
          dst[(d + DH / 2) * kv_tile_keys] = f2h(hi[g][e]);
        }
      return;
    }
    if (a.rope) {
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        // Pairs d .. d + 3 share one RoPE section (sections are multiples of 4 pairs).
        const int d = 16 * sub + 8 * g + 4 * fh;
        const float2* rt = a.rope + int64_t(rope_pos(a, m, d)) * (DH / 2) + d;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = lo[g][e], y = hi[g][e];
          rope_rotate(x, y, rt[e], lo[g][e], hi[g][e]);
        }
      }
    }
    uint16_t* dst = head < a.hq ? a.q + (int64_t(m) * a.hq + head) * DH
                                : a.kstore + a.k_off[m] + int64_t(head - a.hq) * a.kv_head_stride;
    store_h8_pair(dst + 16 * sub, fh, lo[0], lo[1]);
    store_h8_pair(dst + 16 * sub + DH / 2, fh, hi[0], hi[1]);
  }
}

// Wave grid WN x WM; each wave NS weight strips x MT row subtiles of 32.
template <int EPI, int DH, bool W_F16, int WN, int WM, int NS, int MT>
__global__ __launch_bounds__(WN * WM * 64, 2) void tile_kernel(GemmArgs a) {
  constexpr int kWaves = WN * WM;
  constexpr int kThreads = kWaves * 64;
  constexpr int BN = 32 * NS * WN, BM = 32 * MT * WM;
  constexpr int kWBytes = BN * kRowBytes, kABytes = BM * kRowBytes;
  constexpr int kStage = kWBytes + kABytes;
  constexpr int WL = kWBytes / (1024 * kWaves), AL = kABytes / (1024 * kWaves);  // 1 KB loads per wave and stage
  static_assert(WL * 1024 * kWaves == kWBytes && AL * 1024 * kWaves == kABytes, "tile split");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * kStage];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave % WN, wm = wave / WN;
  const int fr = lane & 31, fh = lane >> 5;

  // Tiles in groups of kGroupM row tiles, rows fastest; block b runs on XCD
  // b % 8, and each XCD takes a contiguous range of tiles, so the tiles that
  // share operands meet in one L2.  The grid is padded to whole rounds.
  const int tiles_m = (a.M + BM - 1) / BM;
  const int tiles_n = a.n_tiles_n * 256 / BN;
  const int L = int(blockIdx.x % kNumXcd) * int(gridDim.x / kNumXcd) + int(blockIdx.x / kNumXcd);
  if (L >= tiles_m * tiles_n) return;
  TileClock clk;
  clk.begin(a.clock);
  const int per_group = kGroupM * tiles_n;
  const int first_m = (L / per_group) * kGroupM;
  const int gsize = min(tiles_m - first_m, kGroupM);
  const int tile_m = first_m + (L % per_group) % gsize;
  const int strip0 = (L % per_group) / gsize * (BN / 32);  // first strip of the tile
  const int my_strip = strip0 + wn * NS;
  const int my_m = tile_m * BM + wm * MT * 32 + fr;  // this lane's first row

  f32x16 acc[NS][MT];
#pragma unroll
  for (int i = 0; i < NS; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
  if constexpr (EPI == EPI_RESID) {
    // The accumulators start from the residual (rows past M, never stored,
    // read the last valid row).  Issued first, so that waiting for them
    // leaves the operand loads in flight.
#pragma unroll
    for (int i = 0; i < NS; ++i)
#pragma unroll
      for (int j = 0; j < MT; ++j) {
        const int64_t ro = int64_t(min(my_m + j * 32, a.M - 1)) * a.ldo + (my_strip + i) * 32 + 4 * fh;
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          float r[4];
          if (a.resid_f32) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(a.resid_f32 + ro + 8 * g4);
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = v[e];
          } else {
            load_bf16x4(a.resid + ro + 8 * g4, r);
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[i][j][4 * g4 + e] = r[e];
        }
      }
    __builtin_amdgcn_sched_barrier(0);
  }

  const int KT = a.K / BK;  // even, at least 2
  const uint32_t row_bytes = uint32_t(a.K) * 2;
  const uint32_t w_rows = (EPI == EPI_SWIGLU) ? uint32_t(2 * a.ffn) : uint32_t(a.n_tiles_n * 256);
  const __amdgpu_buffer_rsrc_t wres = make_rsrc(a.W, w_rows * row_bytes);
  const __amdgpu_buffer_rsrc_t ares = make_rsrc(a.A, uint32_t(a.M) * row_bytes);  // rows >= M read zero
  const uint32_t panel_bytes = w_rows * 64;

  // Every load instruction of a wave covers 1 KB in runs of 64 bytes or more:
  // 8 rows x 128 bytes of a row-major operand, or 16 rows of one 32-wide
  // panel of prepared weights.
  uint32_t a_off[AL], a_lds[AL], w_off[WL], w_lds[WL];
#pragma unroll
  for (int l = 0; l < AL; ++l) {
    const int r = 8 * (wave + kWaves * l) + (lane >> 3), c = lane & 7;
    a_off[l] = uint32_t(tile_m * BM + r) * row_bytes + uint32_t(c * 16);
    a_lds[l] = uint32_t(kWBytes + r * kRowBytes + phys(r, c) * 16);
  }
#pragma unroll
  for (int l = 0; l < WL; ++l) {
    const int q = wave + kWaves * l;
    int r, c;
    if constexpr (W_F16) {
      r = 16 * (q >> 1) + (lane >> 2);
      c = 4 * (q & 1) + (lane & 3);
      w_off[l] = strip_row<EPI, DH>(strip0 + (r >> 5), r & 31, a.ffn) * 64u + uint32_t(q & 1) * panel_bytes +
                 uint32_t((lane & 3) * 16);
    } else {
      r = 8 * q + (lane >> 3);
      c = lane & 7;
      w_off[l] = strip_row<EPI, DH>(strip0 + (r >> 5), r & 31, a.ffn) * row_bytes + uint32_t(c * 16);
    }
    w_lds[l] = uint32_t(r * kRowBytes + phys(r, c) * 16);
  }
  const uint32_t w_step = W_F16 ? 2 * panel_bytes : uint32_t(kRowBytes);

  // Load or LDS write l (0 .. NL - 1, weights first) of a stage, through the
  // registers of slot `slot`.
  constexpr int NM = NS * MT, NR = NS + MT, NL = WL + AL;
  u32x4 gr[2][NL];
  auto load = [&](int kt, int slot, int l) {
    gr[slot][l] = __builtin_bit_cast(
        u32x4, l < WL ? __builtin_amdgcn_raw_buffer_load_b128(wres, w_off[l < WL ? l : 0], uint32_t(kt) * w_step, 0)
                      : __builtin_amdgcn_raw_buffer_load_b128(ares, a_off[l < WL ? 0 : l - WL], uint32_t(kt * kRowBytes), 0));
  };
  auto put = [&](int buf, int slot, int l) {
    *reinterpret_cast<u32x4*>(smem + buf * kStage + (l < WL ? w_lds[l < WL ? l : 0] : a_lds[l < WL ? 0 : l - WL])) =
        gr[slot][l];
  };
  struct Frag {
    u32x4 w[NS], a[MT];
  };
  Frag f[2];
  // Fragment x (0 .. NR - 1, activations first) of step kk.
  auto read = [&](int buf, int kk, int x, Frag& d) {
    const uint8_t* base = smem + buf * kStage + fr * kRowBytes + phys(fr, 2 * kk + fh) * 16;
    if (x < MT)
      d.a[x < MT ? x : 0] = *reinterpret_cast<const u32x4*>(base + kWBytes + (wm * MT + x) * 32 * kRowBytes);
    else
      d.w[x < MT ? 0 : x - MT] = *reinterpret_cast<const u32x4*>(base + (wn * NS + x - MT) * 32 * kRowBytes);
  };
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int l = 0; l < NL; ++l) load(t, t, l);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int l = 0; l < NL; ++l) put(0, 0, l);
#pragma unroll
  for (int l = 0; l < NL; ++l) load(min(2, KT - 1), 0, l);
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int x = 0; x < NR; ++x) read(0, 0, x, f[0]);
  __builtin_amdgcn_sched_barrier(0);

  // Stage t multiplies buffer t % 2, writes stage t + 1 to the other one in
  // its first two steps and loads stage t + 3 into the registers that held it
  // in the middle two.  Each step's fragments are read during the step before.
  // One barrier per stage, inside the last step, whose fragments have been
  // read by then: it follows every wave's writes of stage t + 1 (whose first
  // fragments are read next) and its reads of buffer t % 2 (which the next
  // stage overwrites).  Loads past the end repeat the last stage (in bounds,
  // never used).  Every MFMA is issued with its share of the LDS accesses and
  // loads, pinned by scheduling barriers: a wave issues in order, and eight
  // writes in a row keep its MFMAs from issuing for 300 cycles.
  constexpr int H = (NL + 1) / 2, HB = NM / 2;
  for (int kt = 0; kt < KT; kt += 2) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int tn = min(kt + u + 3, KT - 1);
#pragma unroll
      for (int kk = 0; kk < kKk; ++kk) {
        const bool last = kk + 1 == kKk;
        const int nw = kk == 0 ? H : kk == 1 ? NL - H : 0;  // writes: 0 .. H - 1, then the rest
        const int nl = kk == 1 ? H : kk == 2 ? NL - H : 0;  // loads likewise, one step later
        u32x4 wh[NS];
#pragma unroll
        for (int q = 0; q < NM; ++q) {
          if (last && q == HB) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
          }
          if (!last) {
#pragma unroll
            for (int x = q * NR / NM; x < (q + 1) * NR / NM; ++x) read(u, kk + 1, x, f[(kk + 1) & 1]);
          } else if (q >= HB) {
#pragma unroll
            for (int x = (q - HB) * NR / (NM - HB); x < (q - HB + 1) * NR / (NM - HB); ++x) read(1 - u, 0, x, f[0]);
          }
#pragma unroll
          for (int x = q * nw / NM; x < (q + 1) * nw / NM; ++x) put(1 - u, 1 - u, kk * H + x);
          const int i = q / MT, j = q % MT;
          if (j == 0) wh[i] = W_F16 ? f[kk & 1].w[i] : bf8_to_h8(f[kk & 1].w[i]);
          acc[i][j] = mfma32(wh[i], f[kk & 1].a[j], acc[i][j]);
#pragma unroll
          for (int x = q * nl / NM; x < (q + 1) * nl / NM; ++x) load(tn, 1 - u, (kk - 1) * H + x);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  }

#pragma unroll
  for (int j = 0; j < MT; ++j) {
    const int m = my_m + j * 32;
    if (m < a.M) {
#pragma unroll
      for (int i = 0; i < NS; ++i) store_rows<EPI, DH>(a, acc[i][j], my_strip + i, m, fh);
    }
  }
  clk.end(a.clock);
}

template <int EPI, int DH, int WN, int WM, int NS, int MT>
hipError_t launch_tile(const GemmArgs& a, hipStream_t s) {
  constexpr int BN = 32 * NS * WN, BM = 32 * MT * WM;
  const int tiles = ((a.M + BM - 1) / BM) * (a.n_tiles_n * 256 / BN);
  const int grid = (tiles + kNumXcd - 1) / kNumXcd * kNumXcd;
  if (a.w_f16)
    hipLaunchKernelGGL((tile_kernel<EPI, DH, true, WN, WM, NS, MT>), dim3(grid), dim3(WN * WM * 64), 0, s, a);
  else
    hipLaunchKernelGGL((tile_kernel<EPI, DH, false, WN, WM, NS, MT>), dim3(grid), dim3(WN * WM * 64), 0, s, a);
  return hipGetLastError();
}

// The tile shapes of kGemmTileShapes, in order.
template <int EPI, int DH>
hipError_t launch_shape(const GemmArgs& a, int tile, hipStream_t s) {
  switch (tile) {
    case 0: return launch_tile<EPI, DH, 2, 2, 1, 1>(a, s);
    case 1: return launch_tile<EPI, DH, 2, 2, 2, 1>(a, s);
    case 2: return launch_tile<EPI, DH, 4, 1, 1, 3>(a, s);
    case 3: return launch_tile<EPI, DH, 2, 2, 2, 2>(a, s);
    case 4: return launch_tile<EPI, DH, 4, 1, 1, 5>(a, s);
    case 5: return launch_tile<EPI, DH, 2, 2, 2, 3>(a, s);
    case 6: return launch_tile<EPI, DH, 4, 2, 2, 3>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_gemm_tile(int epi, const GemmArgs& a, int tile, hipStream_t s) {
  switch (epi) {
    case EPI_RESID: return launch_shape<EPI_RESID, 128>(a, tile, s);
    case EPI_SWIGLU: return launch_shape<EPI_SWIGLU, 128>(a, tile, s);
    case EPI_GATED: return launch_shape<EPI_GATED, 128>(a, tile, s);
    case EPI_GELU: return launch_shape<EPI_GELU, 128>(a, tile, s);
    case EPI_QKV: return a.dh == 64 ? launch_shape<EPI_QKV, 64>(a, tile, s) : launch_shape<EPI_QKV, 128>(a, tile, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace hs
