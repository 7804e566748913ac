// The 16-bit GEMM of the FSV_BF16 path for many rows (bf16 or fp16 operands, fp32 sums); gemm_bf16.hip has the one for fewer.  Built without
// -amdgpu-mfma-vgpr-form: the sums of a wave (up to 256 registers) live in the accumulation half of the register file.
#include <hip/hip_ext.h>
#include <type_traits>

#include "gemm_store.h"

using namespace fsv_bf16;

namespace {

// ---------------------------------------------------------------------------------------------
// Many rows (more than 256): the matrix cores are the bound
// ---------------------------------------------------------------------------------------------
// The weight-streaming kernel stops at 0.36 of the matrix-core peak: its 128 x 128 block has to move 64 bytes per clock into the
// compute unit to keep the matrix cores busy, all a unit can take.  Here a block is 256 features x 64 MT rows (MT = 2, 3, 4: 128,
// 192, 256 rows) and both operands arrive through LDS: half to three quarters of the bytes per product.  The contraction advances in
// stages of 32 (two k blocks); a ring of five or six stages in LDS (140 .. 160 KiB, one block per compute unit) is filled by direct
// loads, every wave its share of every stage, three to four stages ahead.  The operands being in the order the matrix cores take them,
// every load, LDS write and LDS read is 1 KiB of consecutive 16-byte units: no bank conflicts, no address arithmetic.
// MT = 3, 4: four waves of 128 features x 32 MT rows, one to a SIMD, with their sums in the accumulation registers: 4 + MT operands
// read from LDS for 4 MT products, where eight waves of 64 features read 2 + MT for 2 MT.  MT = 2 keeps eight waves
// of 64 features x 64 rows, two to a SIMD.
// A wave interleaves the LDS reads of the next k block and its loads with the products, so the issue slots of these fall into their
// shadow.  Operands of the next k block are read across the barrier: the barrier before stage it certifies that stage it + 1 has
// landed, too.
// With every unit at work the clock falls from 2.36 to about 1.9 GHz.  2048 x 28672 x 4096: products alone 1.41 PFLOP/s, without the direct
// loads 1.30, without the LDS reads 1.20, whole 1.14; the library's fp16 product of 8192^3 reaches 1.42 with all of its loads, so that
// power alone is not the bound: every block fills its ring from nothing and stores its result with no load in flight (kWideFixed, 5 us in
// each of three to five rounds), and the last round is partly filled.  Fewer LDS reads for a product pay although
// their slots are free: 192-row blocks 5 .. 7 % faster than with eight waves, 256-row blocks 0 .. 1 %; gate|up, 2048 rows 447 -> 427 us.
// MT = 4 with bf16 operands fills all 512 registers; sixteen are spilled and read back once, in the epilogue.

template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

constexpr int WSB = 2;      // 16-wide k blocks per stage
constexpr int WSTRIPS = 8;  // weight strips per block: 256 features
template <int MT>
struct wide_geo {
  static constexpr int NSW = MT >= 3 ? 4 : 2, WF = WSTRIPS / NSW, WR = 2, NW = WF * WR;   // strips per wave; waves along features and rows
  static constexpr int RT = WR * MT, UNITS = (WSTRIPS + RT) * WSB, NS = MT == 2 ? 6 : 5;   // row tiles, KiB per stage, stages of the ring
  static constexpr int STAGE = UNITS * 1024, LDS = NS * STAGE, LJ = UNITS / NW;            // LJ: loads per wave and stage
  static_assert(UNITS % NW == 0 && LDS <= 160 * 1024 && LJ * (NS - 2) <= 63, "");
};

template <int MT, int EPI, bool F16>
__global__ __launch_bounds__(64 * wide_geo<MT>::NW) void k_gemm_wide(const char *__restrict__ Wp, const char *__restrict__ Ap, void *__restrict__ out,
                                                   int N, int KB, int Mt_total, int M, int Mpad, int S, int nchunks, int KBo,
                                                   int NBv, int MB, float oscale, int NT, uint32_t strip_bytes) {
  extern __shared__ uint4 lds[];
  using G = wide_geo<MT>;
  constexpr int NS = G::NS, RT = G::RT, STAGE = G::STAGE, LJ = G::LJ, NSW = G::NSW, NW = G::NW, WF = G::WF;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, h = lane >> 5;
  int nblk, split, zb;
  {
    const int L = blockIdx.x, x = L & 7, a = L >> 3;
    zb = a % MB;
    const int a2 = a / MB;
    if ((S & 7) == 0) {
      const int s8 = S >> 3;
      split = x + 8 * (a2 % s8);
      nblk = a2 / s8;
    } else {
      split = a2 % S;
      nblk = (a2 / S) * 8 + x;
    }
  }
  if (nblk >= NBv) return;
  const int mt0 = zb * RT, mlast = min(RT, Mt_total - mt0) - 1;
  const int g0 = split * nchunks / S, g1 = (split + 1) * nchunks / S;   // 256-element granules
  constexpr int SPG = 256 / (16 * WSB);                                  // stages per granule
  const int n = (g1 - g0) * SPG;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)lds;

  // this wave's loads of a stage: unit u = NW j + w; units 0 .. 15 are (strip u / 2, k block u % 2), the rest row tiles alike
  const char *src[LJ];
  const uint32_t lane_off = (uint32_t)lane * 16u;
#pragma unroll
  for (int j = 0; j < LJ; ++j) {
    const int u = NW * j + w, kb = u % WSB, q = u / WSB;
    if (q < WSTRIPS) {
      const int strip = min(nblk * WSTRIPS + q, NT - 1);
      src[j] = Wp + (size_t)strip * strip_bytes + ((size_t)g0 * 16 + kb) * 1024;
    } else {
      const int mt = mt0 + min(q - WSTRIPS, mlast);
      src[j] = Ap + ((size_t)mt * KB + (size_t)g0 * 16 + kb) * 1024;
    }
  }
  auto issue1 = [&](int j, uint32_t slot_off) {
    load_to_lds<false>(lds0 + slot_off + (uint32_t)(NW * j + w) * 1024u, lane_off, src[j]);
    src[j] += WSB * 1024;
  };

  const int wf = w % WF, wr = w / WF;   // strips NSW wf ..; row tiles MT wr ..
  f32x16_t acc[NSW][MT];
#pragma unroll
  for (int s = 0; s < NSW; ++s)
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[s][i][v] = 0.f;

  bf16x8_t wop[2][NSW], aop[2][MT];
  const uint4 *wbase = lds + wf * (NSW * WSB * 64) + lane, *abase = lds + (WSTRIPS + wr * MT) * (WSB * 64) + lane;
  // operand i of a k block, in the order the products need them: the first strip, the row tiles, the other strips
  constexpr int NF = NSW + MT, NM = NSW * MT, EVERY = NM / NF;   // operands, products; an operand is read behind every EVERY-th product
  static_assert(EVERY >= 1, "");
  auto fetch1 = [&](int set, int i, uint32_t slot_units, int kb) {
    if (i == 0 || i > MT) {
      const int s = i == 0 ? 0 : i - MT;
      uint4 raw = wbase[slot_units + (s * WSB + kb) * 64];
      wop[set][s] = *reinterpret_cast<bf16x8_t *>(&raw);
    } else {
      uint4 raw = abase[slot_units + ((i - 1) * WSB + kb) * 64];
      aop[set][i - 1] = *reinterpret_cast<bf16x8_t *>(&raw);
    }
  };
  auto mfma1 = [&](int set, int i) {
    const int s = i / MT, t = i % MT;
    if constexpr (F16)
      acc[s][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, wop[set][s]), __builtin_bit_cast(f16x8_t, aop[set][t]), acc[s][t], 0, 0, 0);
    else
      acc[s][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wop[set][s], aop[set][t], acc[s][t], 0, 0, 0);
  };

#pragma unroll
  for (int st = 0; st < NS - 1; ++st) {
    if (st < n) {
#pragma unroll
      for (int j = 0; j < LJ; ++j) issue1(j, (uint32_t)st * STAGE);
    }
  }
  // stage 0 has landed everywhere before its first operands are fetched
  if (n >= NS - 1) wait_loads<LJ *(NS - 2)>();
  else wait_loads<0>();
  FSV_BARRIER();
#pragma unroll
  for (int i = 0; i < NF; ++i) fetch1(0, i, 0u, 0);

  uint32_t rd = 0, wrs = (uint32_t)(NS - 1) * STAGE;   // LDS offsets of the stage in use and of the one to be filled next
  auto stage = [&](auto more) {
    uint32_t nx = rd + STAGE;
    if (nx == (uint32_t)NS * STAGE) nx = 0;
#pragma unroll
    for (int kb = 0; kb < WSB; ++kb) {
      const uint32_t so = (kb + 1 < WSB ? rd : nx) / 16u;
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        mfma1(kb & 1, i);
        if (i % EVERY == 0 && i / EVERY < NF) fetch1((kb + 1) & 1, i / EVERY, so, (kb + 1) % WSB);
        constexpr int LEVERY = WSB * NM / LJ;   // and a load behind every LEVERY-th
        const int slot = kb * NM + i;
        if (decltype(more)::value && slot % LEVERY == LEVERY - 1 && slot / LEVERY < LJ) issue1(slot / LEVERY, wrs);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    rd = nx;
    wrs = (wrs + STAGE == (uint32_t)NS * STAGE) ? 0 : wrs + STAGE;
  };
  // Before stage it: stage it + 1 has landed for this wave; after the barrier for all, and nobody reads stage it - 1 any more.
  int it = 0;
  for (; it < n - (NS - 1); ++it) {
    wait_loads<LJ *(NS - 3)>();
    FSV_BARRIER();
    stage(std::true_type{});
  }
  for (; it < n; ++it) {   // the last stages: nothing is left to load
    wait_loads<0>();
    FSV_BARRIER();
    stage(std::false_type{});
  }
  wait_loads<0>();   // nothing may still be on its way into this block's LDS when the wave ends
#pragma unroll
  for (int s = 0; s < NSW; ++s) {
    const int nt = nblk * WSTRIPS + NSW * wf + s, t0 = mt0 + wr * MT;
    __builtin_amdgcn_sched_barrier(0);   // strip by strip: all sums at once would not fit the architectural registers
    store_strip<MT, EPI, F16>(acc[s], out, nt, t0, min(MT, Mt_total - t0), lane, h, split, M, Mpad, N, KBo, oscale);
  }
}

template <int MT, int EPI>
int launch_wide_t(fsv_ctx *c, int cls, const void *Wp, const void *Ap, void *out, int N, int KB, int Mt, int M, int splits, int nchunks,
                  int KBo, int f16, float oscale, int NT, uint32_t strip_bytes, hipStream_t st) {
  const int NB = fsv_ceil_div(NT, WSTRIPS), NBg = (splits % 8 == 0) ? NB : (NB + 7) / 8 * 8, MB = fsv_ceil_div(Mt, 2 * MT);
  const dim3 grid((unsigned)NBg * splits * MB);
  fsv_prof_scope ps(c, st, cls, (double)N * KB * 32.0, true);
#define FSV_WIDE_GO(F16V, OSC)                                                                                                      \
  hipExtLaunchKernelGGL((k_gemm_wide<MT, EPI, F16V>), grid, dim3(64 * wide_geo<MT>::NW), wide_geo<MT>::LDS, st, ps.start(), ps.stop(), 0, (const char *)Wp, \
                        (const char *)Ap, out, N, KB, Mt, M, Mt * 32, splits, nchunks, KBo, NB, MB, OSC, NT, strip_bytes)
  if (f16) FSV_WIDE_GO(true, oscale);
  else FSV_WIDE_GO(false, 1.0f);
#undef FSV_WIDE_GO
  return FSV_OK;
}

template <int EPI>
int launch_wide(fsv_ctx *c, int cls, const void *Wp, const void *Ap, void *out, int N, int K, int NTpad, int M, int splits, int KBo, int f16,
                float oscale, int mt, hipStream_t st) {
  const int Mt = fsv_ceil_div(M, 32), nchunks = K / 256, KB = K / 16;
  const uint32_t strip_bytes = (uint32_t)KB * 1024u + (uint32_t)c->strip_pad_bytes;
  if (splits < 1 || splits > nchunks) FSV_FAIL(c, FSV_E_INVALID_ARG, "bad split count %d for %d granules", splits, nchunks);
  switch (mt) {
    case 2: return launch_wide_t<2, EPI>(c, cls, Wp, Ap, out, N, KB, Mt, M, splits, nchunks, KBo, f16, oscale, NTpad, strip_bytes, st);
    case 3: return launch_wide_t<3, EPI>(c, cls, Wp, Ap, out, N, KB, Mt, M, splits, nchunks, KBo, f16, oscale, NTpad, strip_bytes, st);
    case 4: return launch_wide_t<4, EPI>(c, cls, Wp, Ap, out, N, KB, Mt, M, splits, nchunks, KBo, f16, oscale, NTpad, strip_bytes, st);
    default: FSV_FAIL(c, FSV_E_INVALID_ARG, "internal: %d row tiles per wave", mt);
  }
}

template <int MT, int EPI>
int init_t(fsv_ctx *c) {
  FSV_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void *>(&k_gemm_wide<MT, EPI, false>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, wide_geo<MT>::LDS));
  FSV_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void *>(&k_gemm_wide<MT, EPI, true>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, wide_geo<MT>::LDS));
  return FSV_OK;
}

template <int EPI>
int init_e(fsv_ctx *c) {
  int rc;
  if ((rc = init_t<2, EPI>(c)) || (rc = init_t<3, EPI>(c)) || (rc = init_t<4, EPI>(c))) return rc;
  return FSV_OK;
}

}  // namespace

int fsv_bf16_gemm_wide_init(fsv_ctx *c) {   // the dynamic LDS limits (140 .. 160 KiB), once per context
  int rc;
  if ((rc = init_e<EPI_PARTIAL>(c)) || (rc = init_e<EPI_SWIGLU>(c)) || (rc = init_e<EPI_F32>(c))) return rc;
  return FSV_OK;
}

int fsv_bf16_gemm_wide(fsv_ctx *c, int cls, int epi, const void *Wp, const void *Ap, void *out, int N, int K, int NTpad, int M, int splits,
                       int KBo, int f16, float oscale, int mt, hipStream_t st) {
  int rc;
  switch (epi) {
    case EPI_PARTIAL: rc = launch_wide<EPI_PARTIAL>(c, cls, Wp, Ap, out, N, K, NTpad, M, splits, KBo, f16, oscale, mt, st); break;
    case EPI_SWIGLU: rc = launch_wide<EPI_SWIGLU>(c, cls, Wp, Ap, out, N, K, NTpad, M, splits, KBo, f16, oscale, mt, st); break;
    default: rc = launch_wide<EPI_F32>(c, cls, Wp, Ap, out, N, K, NTpad, M, splits, KBo, f16, oscale, mt, st); break;
  }
  if (rc) return rc;
  FSV_HIP(c, hipGetLastError());
  return FSV_OK;
}
