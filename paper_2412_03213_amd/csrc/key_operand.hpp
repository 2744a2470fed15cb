// Keys as an MFMA operand of the assignment kernels.
#pragma once
#include "ck_common.hpp"

namespace ck {

// v_mfma_f32_32x32x16_bf16 wants lane (half, col) = (l / 32, l % 32) to hold the 16 bytes
// 2 kk + half of key `col` in step kk.  Loaded that way every lane of a quarter wavefront touches
// another row, and the address unit takes four times as long as for 64 consecutive bytes: 33 MB by
// 256 workgroups of eight wavefronts 4.9 us against 2.6 (launch included), whether they come from a
// cache or not, and while it is busy no wavefront of the compute unit gets its next load out.  So
// four lanes load 64 consecutive bytes of a key, and the keys change lanes through a
// wavefront-private piece of LDS, 64 bytes of 32 keys at a time.
constexpr int KEY_STAGE_ROW = 40;                         // bf16 elements: 80 B, no bank conflicts
constexpr int KEY_STAGE_ELEMS = 32 * KEY_STAGE_ROW;       // of one wavefront

template <int NKB>
struct KeyTile {
  uint4 w[NKB][8];        // as loaded, then the operands of the steps

  // keys [t0, t0 + 32 NKB) of K, those beyond tok_count re-read the last one
  __device__ __forceinline__ void load(const bf16* K, int64_t t0, int64_t tok_count, int lane) {
    const bf16* p[NKB][2];
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        int64_t t = t0 + kb * 32 + x * 16 + (lane >> 2);
        t = t < tok_count ? t : tok_count - 1;
        p[kb][x] = K + t * D + (lane & 3) * 8;
      }
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int x = 0; x < 2; ++x)
          w[kb][2 * q + x] = *reinterpret_cast<const uint4*>(p[kb][x] + q * 32);
  }
  // LDS serves one wavefront in order, so nothing waits between writing and reading
  __device__ __forceinline__ void to_operand(bf16* stage, int lane) {
    bf16* in = stage + (lane >> 2) * KEY_STAGE_ROW + (lane & 3) * 8;
    const bf16* out = stage + (lane & 31) * KEY_STAGE_ROW + (lane >> 5) * 8;
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        wave_lds_order();
        *reinterpret_cast<uint4*>(in) = w[kb][2 * q];
        *reinterpret_cast<uint4*>(in + 16 * KEY_STAGE_ROW) = w[kb][2 * q + 1];
        wave_lds_order();
        w[kb][2 * q] = *reinterpret_cast<const uint4*>(out);
        w[kb][2 * q + 1] = *reinterpret_cast<const uint4*>(out + 16);
      }
    wave_lds_order();
  }
  // the same through half of the room, sixteen keys at a time
  __device__ __forceinline__ void to_operand_16(bf16* stage, int lane) {
    bf16* in = stage + (lane >> 2) * KEY_STAGE_ROW + (lane & 3) * 8;
    const bf16* out = stage + (lane & 15) * KEY_STAGE_ROW + (lane >> 5) * 8;
    const bool upper = (lane & 16) != 0;
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint4 o[2][2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          wave_lds_order();
          *reinterpret_cast<uint4*>(in) = w[kb][2 * q + x];
          wave_lds_order();
          o[x][0] = *reinterpret_cast<const uint4*>(out);
          o[x][1] = *reinterpret_cast<const uint4*>(out + 16);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
          w[kb][2 * q + i] = make_uint4(upper ? o[1][i].x : o[0][i].x, upper ? o[1][i].y : o[0][i].y,
                                        upper ? o[1][i].z : o[0][i].z, upper ? o[1][i].w : o[0][i].w);
      }
    wave_lds_order();
  }
  __device__ __forceinline__ bf16x8 operand(int kb, int kk) const {
    return __builtin_bit_cast(bf16x8, w[kb][kk]);
  }
};

}  // namespace ck
