// Epilogues of the two 16-bit GEMM kernels.
#pragma once
#include "bf16_common.h"

namespace fsv_bf16 {

enum { EPI_PARTIAL = 0, EPI_SWIGLU = 1, EPI_F32 = 2 };

typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_t;

// The barrier as an opaque statement: memory operations do not move across it, and no counter wait is attached.
#define FSV_BARRIER() asm volatile("s_barrier" ::: "memory")

// Stores one wave's result: for row tiles mt < mtc of the block starting at tile mt0, lane holds, for batch row
// m = tile*32 + lane%32, features nt*32 + 8*(v/4) + 4*h + v%4 of strip nt.
template <int MT, int EPI, bool F16>
__device__ __forceinline__ void store_strip(f32x16_t (&acc)[MT], void *__restrict__ out, int nt, int mt0, int mtc, int lane,
                                            int h, int split, int M, int Mpad, int N, int KBo, float oscale) {
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    if (mt >= mtc) continue;
    if constexpr (F16) {   // undo the power of two the weights carry (exact)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[mt][v] *= oscale;
    }
    const int m = (mt0 + mt) * 32 + (lane & 31);
    if constexpr (EPI == EPI_PARTIAL) {
      if (m >= M) continue;  // the consumers read rows below M only
      float *dst = (float *)out + ((size_t)split * Mpad + m) * N;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int n0 = nt * 32 + 8 * g + 4 * h;
        if (n0 + 3 < N) {
          *reinterpret_cast<float4 *>(dst + n0) =
              make_float4(acc[mt][4 * g], acc[mt][4 * g + 1], acc[mt][4 * g + 2], acc[mt][4 * g + 3]);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (n0 + r < N) dst[n0 + r] = acc[mt][4 * g + r];
        }
      }
    } else if constexpr (EPI == EPI_F32) {
      if (m < M) {
        float *dst = (float *)out + (size_t)m * N;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int n0 = nt * 32 + 8 * g + 4 * h;
          if (n0 + 3 < N) {
            *reinterpret_cast<f32x4_any *>(dst + n0) =
                (f32x4_any){acc[mt][4 * g], acc[mt][4 * g + 1], acc[mt][4 * g + 2], acc[mt][4 * g + 3]};
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (n0 + r < N) dst[n0 + r] = acc[mt][4 * g + r];
          }
        }
      }
    } else {  // SwiGLU: regs 0-3 gate / 4-7 up of features 16*nt + 4h + r, regs 8-11 / 12-15 of 16*nt + 8 + 4h + r
      if (nt < KBo) {
        uint16_t *base = (uint16_t *)out;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          uint16_t o4[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float gte = acc[mt][8 * j + r], up = acc[mt][8 * j + 4 + r];
            o4[r] = f2bf(gte / (1.0f + __expf(-gte)) * up);
          }
          const size_t unit = ((size_t)(mt0 + mt) * KBo + nt) * 64 + (lane & 31) + 32 * j;
          uint2 pk = make_uint2((uint32_t)o4[0] | ((uint32_t)o4[1] << 16), (uint32_t)o4[2] | ((uint32_t)o4[3] << 16));
          *reinterpret_cast<uint2 *>(base + unit * 8 + 4 * h) = pk;
        }
      }
    }
  }
}

}  // namespace fsv_bf16
