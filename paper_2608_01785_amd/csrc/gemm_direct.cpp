// One GEMM by itself, on the kernel the caller names.  Internal to the
// library and its tests (not declared in horizon.h): it lets a test run every
// kernel that an epilogue can be sent to on the same operands, whatever the
// dispatch would choose for their sizes.
#include <cstdint>

#include "gemm_policy.h"
#include "horizon.h"
#include "hs_kernels.h"
#include "plan.h"

namespace {

// The caller's values, in order; pointers are device addresses or 0.
enum Field {
  kA, kW, kWF16, kM, kK, kN, kOut, kOutF32, kLdo, kResid, kResidF32, kFfn, kQ, kKeys, kValues, kPos, kPosStride,
  kSec1, kSec2, kKOff, kVOff, kKvHeadStride, kRope, kBias, kGate, kGateStride, kRowSeq, kHq, kHkv, kDh, kPart,
  kCounters, kK8Rows, kClock,
  kWResident, kFields
};

constexpr int kSkinnyKernel = -2, kPersistentKernel = -1;  // tile shapes count from 0

}  // namespace

extern "C" {

// epi: an Epilogue.  kernel: -2 the skinny GEMM, -1 the persistent one, else
// a shape of kGemmTileShapes.  cus: the persistent kernel's blocks.
hs_status hs_gemm_direct(int32_t epi, int32_t kernel, int32_t cus, const int64_t* v, int32_t n, void* stream) {
  hs::clear_error();
  if (!v || n != kFields) return hs::fail(HS_ERR_INVALID_ARG, "%d fields, expected %d", n, int(kFields));
  auto u16 = [&](Field f) { return reinterpret_cast<uint16_t*>(v[f]); };
  auto f32 = [&](Field f) { return reinterpret_cast<float*>(v[f]); };
  auto i32 = [&](Field f) { return reinterpret_cast<int32_t*>(v[f]); };
  hs::GemmArgs a{};
  a.A = u16(kA);
  a.W = u16(kW);
  a.w_f16 = int(v[kWF16]);
  a.M = int(v[kM]);
  a.K = int(v[kK]);
  a.n_tiles_n = int(v[kN] / 256);
  a.out = u16(kOut);
  a.out_f32 = f32(kOutF32);
  a.ldo = int(v[kLdo]);
  a.resid = u16(kResid);
  a.resid_f32 = f32(kResidF32);
  a.ffn = int(v[kFfn]);
  a.q = u16(kQ);
  a.kstore = u16(kKeys);
  a.vstore = u16(kValues);
  a.pos = i32(kPos);
  a.pos_stride = int(v[kPosStride]);
  a.sec1 = int(v[kSec1]);
  a.sec2 = int(v[kSec2]);
  a.k_off = reinterpret_cast<int64_t*>(v[kKOff]);
  a.v_off = reinterpret_cast<int64_t*>(v[kVOff]);
  a.kv_head_stride = v[kKvHeadStride];
  a.rope = reinterpret_cast<float2*>(v[kRope]);
  a.bias = u16(kBias);
  a.gate = f32(kGate);
  a.gate_stride = int(v[kGateStride]);
  a.row_seq = i32(kRowSeq);
  a.hq = int(v[kHq]);
  a.hkv = int(v[kHkv]);
  a.dh = int(v[kDh]);
  a.part = f32(kPart);
  a.counters = i32(kCounters);
  a.k8_rows = int(v[kK8Rows]);
  a.clock = reinterpret_cast<uint64_t*>(v[kClock]);
  a.w_resident = int(v[kWResident]);

  const bool skinny = kernel == kSkinnyKernel;
  const int64_t limit = int64_t(1) << 32;
  if (!a.A || !a.W || v[kM] < 1 || v[kK] < 128 || v[kK] % 128 != 0 || v[kN] < 256 || v[kN] % 256 != 0 ||
      v[kM] * v[kK] * 2 >= limit || v[kN] * v[kK] * 2 >= limit || cus < 1)
    return hs::fail(HS_ERR_INVALID_ARG, "operands or sizes");
  bool ok = false;
  switch (epi) {
    case hs::EPI_RESID: ok = a.out_f32 && (a.resid || a.resid_f32) && v[kLdo] >= v[kN]; break;
    case hs::EPI_SWIGLU: ok = a.out && v[kFfn] * 2 == v[kN] && v[kLdo] >= v[kFfn]; break;
    case hs::EPI_GELU: ok = a.out && a.bias && v[kLdo] >= v[kN]; break;
    case hs::EPI_GATED:
      ok = a.out_f32 && a.bias && a.gate && a.row_seq && (a.resid || a.resid_f32) && v[kLdo] >= v[kN];
      break;
    case hs::EPI_QKV:
      ok = a.q && a.kstore && a.vstore && a.pos && a.k_off && a.v_off && (a.dh == 64 || a.dh == 128) && a.hq > 0 &&
           a.hkv > 0 && int64_t(a.hq + 2 * a.hkv) * a.dh == v[kN];
      break;
    default: break;
  }
  if (!ok) return hs::fail(HS_ERR_INVALID_ARG, "operands of epilogue %d", epi);
  if (skinny ? !hs::skinny_supported(epi, a) || (a.k8_rows && a.k8_rows != hs::skinny_k8_rows(a.M)) : a.k8_rows != 0)
    return hs::fail(HS_ERR_UNSUPPORTED, "kernel %d does not take these sizes", kernel);
  if (kernel < kSkinnyKernel || kernel >= hs::kGemmTiles) return hs::fail(HS_ERR_INVALID_ARG, "kernel %d", kernel);

  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const hipError_t e = skinny                        ? hs::launch_gemm_skinny(epi, a, s)
                       : kernel == kPersistentKernel ? hs::launch_gemm_persistent(epi, a, cus, s)
                                                     : hs::launch_gemm_tile(epi, a, kernel, s);
  return e == hipSuccess ? HS_OK : hs::fail(HS_ERR_HIP, "launch: %s", hipGetErrorString(e));
}

// The kernel launch_gemm() sends an [M, K] x [N, K]^T product to: -1 or a
// tile shape.
int32_t hs_gemm_choice(int32_t M, int32_t N, int32_t K, int32_t cus) {
  return M < 1 || N < 256 || K < 1 || cus < 1 ? -1 : hs::gemm_tile_choice(M, N, K, cus);
}

}  // extern "C"
