// Matrix-core building blocks shared by the multi-class scoring kernels
// (gfx950, wave64).
#pragma once

#include "nb.h"
#include "nb_device.hpp"

namespace nb {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  // exact for the small integers, FP8 values and truncated parts packed here:
  // keep the upper halves of the two FP32 images
  return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}

// 16 feature bytes -> 16 BF16 values (two MFMA A operands) and their FP32 images.
template <int XT, bool BIN>
__device__ __forceinline__ void to_bf16(const dev::u32x4& v, dev::u32x4& a0, dev::u32x4& a1, float (&g)[16]) {
  uint32_t o[8];
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const uint32_t u = v[d];
    if (XT == NB_X_U8) {
      g[4 * d] = (float)(u & 0xFFu);
      g[4 * d + 1] = (float)((u >> 8) & 0xFFu);
      g[4 * d + 2] = (float)((u >> 16) & 0xFFu);
      g[4 * d + 3] = (float)(u >> 24);
    } else {
      const auto lo = __builtin_amdgcn_cvt_pk_f32_fp8(u, false);
      const auto hi = __builtin_amdgcn_cvt_pk_f32_fp8(u, true);
      g[4 * d] = lo[0];
      g[4 * d + 1] = lo[1];
      g[4 * d + 2] = hi[0];
      g[4 * d + 3] = hi[1];
    }
    if (BIN) {   // presence: a clamp to [0, 1] for byte counts (folds into the conversion), a compare for FP8
#pragma unroll
      for (int e = 0; e < 4; ++e)
        g[4 * d + e] = (XT == NB_X_U8) ? __builtin_amdgcn_fmed3f(g[4 * d + e], 0.0f, 1.0f) : (g[4 * d + e] > 0.0f ? 1.0f : 0.0f);
    }
    o[2 * d] = pack_bf16(g[4 * d], g[4 * d + 1]);
    o[2 * d + 1] = pack_bf16(g[4 * d + 2], g[4 * d + 3]);
  }
  a0 = dev::u32x4{o[0], o[1], o[2], o[3]};
  a1 = dev::u32x4{o[4], o[5], o[6], o[7]};
}

__device__ __forceinline__ f32x4 mfma(const dev::u32x4& a, const dev::u32x4& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                 0, 0, 0);
}

// Granule (16 bytes) p of file r in a wave's stage: the granules of a file are
// XOR-swizzled so that both the line-shaped writes and the operand-shaped reads
// fall in distinct banks.
template <int NG>
__device__ __forceinline__ int stage_granule(int r, int p) {
  return NG == 8 ? r * 8 + (p ^ ((r >> 1) & 7)) : r * NG + (p ^ (r & 15));
}

}  // namespace
}  // namespace nb
