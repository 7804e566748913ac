// The projections of a layer for calls of few rows (up to 16: one request, or a few with short drafts), 16-bit path (Alg. 2 step 2).
//
// Such a call reads every weight once and has next to nothing to compute, so what counts is the weight stream and, between two
// projections, the start and end of every launch.  k_gemm cuts the contraction over blocks to fill the chip, and a launch of its
// own adds the split sums up and normalises, or rotates and appends.  Here a block keeps whole sums: it owns FT tiles of 16
// features, its eight waves take an eighth of the contraction each, straight from memory into operand registers (weights and
// rows alike: the rows' 16-bit operand is no larger than the weights of one tile), and the eight shares meet in LDS.  The block
// that has a whole sum can finish: rotate and append (q|k|v), SwiGLU (gate|up), add to the residual stream (o, down); and a
// block that reads the whole residual row can normalise it on the way in.  Five launches a layer instead of eight, and no split
// sums in memory.
//
// One 1B request of five rows (2048 wide), per layer: q|k|v 5.5, o 3.9, gate|up 13.2 (67 MB: 5.1 TB/s), down 8.2 us (33.6 MB) against
// 5.3 + 4.0 (rotation and append), 4.0 + 3.7 (sum and norm), 13.6 and 8.1 + 3.7; the call of 16 layers 914 -> 738 us.  8B, five rows, four
// layers 473 -> 433: down 19.9 us (117 MB: 5.9 TB/s), o 7.0, gate|up 37, q|k|v 12.4.
// Which calls (fsv_bf16_few_rows): every block reads and normalises all rows, and a matrix instruction has 16.  39 shapes of 256 .. 4096 features,
// whole calls of four or eight layers, through the eight launches and through these: up to eight rows 1.01 .. 1.4 x.  From nine rows there is room for 16: twice the loads and LDS (128 KiB beyond 2048 features: one block per compute unit).  That pays
// where a wave's share is whole pieces of 256 elements and the projections are not so long that the launches no longer count: up to 2048 features (16
// rows: 256 wide with ffn 4096 1.03 x, 8192 0.98; 512 / 8192 1.01, 14336 0.95; 1024 / 4096 1.11, 14336 0.95; 1536 / 16384 1.00; 2048 / 8192 1.10,
// 16384 1.04, 28672 0.98) and at 4096 (4096 / 8192 1.04, 14336 1.02, 16384 0.99, 22016 0.94).  In between the last piece is partly empty and the
// normalisation takes as long as at 4096: 2304 .. 3840 features 0.92 .. 1.06 with sixteen rows, 0.98 .. 1.10 with nine.
//
// The matrix instruction is 16 x 16 x 32: lane l holds feature (or row) l % 16 and the eight contraction elements 8 (l / 16) .. of
// a step of 32; a lane's accumulator v is feature 4 (l / 16) + v of row l % 16.
#include <hip/hip_ext.h>

#include "gemm_store.h"

using namespace fsv_bf16;

namespace {

typedef __attribute__((ext_vector_type(4))) int i32x4_t;

constexpr int FW = 8;                      // waves of a block
constexpr uint32_t OOB = 0xFFFF0000u;      // beyond every descriptor: the load returns zeros and moves nothing

// What follows the sums of q|k|v (rotation, query operand, KV append) and of gate|up (SwiGLU).
struct few_out {
  int H, Hkv;
  const int4 *row_place;                   // request, index, position, physical page of every row
  const float *rope_tab;
  uint16_t *qp;
  size_t q_plane;
  uint16_t *kpool, *vpool;                 // of the layer
  uint16_t *act;                           // gate|up: operand of the down projection
  int KBo;
};

__device__ __forceinline__ uint4 load16(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
}
__device__ __forceinline__ uint4 load16_nt(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 2));
}
// The block's LDS writes are done and seen; loads from memory stay on their way (a __syncthreads would not wait for them either).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ float4 add4(float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }

enum { FEW_QKV = 0, FEW_GATE_UP = 1 };

// RMSNorm of the residual rows, projection, and what follows it.  Grid = tiles of 16 features / FT.  NS: steps of 32 a wave's share may
// have (d <= 256 NS); MR: rows there is room for (8 or 16).
// A wave reads the residual rows where its share lies, a row at a time and side by side, leaves their sums of squares, and after the
// one barrier puts the normalised rows in operand order into its own piece of LDS: in operand order they would be 2 NS loads a wave
// whatever the number of rows, and every load of a wave, even one of zeros, holds the unit's 64 bytes a cycle for 16 cycles.
template <int KIND, int FT, int NS, int MR>
__global__ __launch_bounds__(64 * FW, 2) void k_few_norm(const void *__restrict__ Wp, const float *__restrict__ x,
                                                         const uint16_t *__restrict__ gain, uint32_t strip_bytes, uint32_t wbytes, int d,
                                                         int M, int tiles, int hd, float eps, float oscale, few_out e) {
  constexpr int P = (FT == 1) ? NS : (FT == 2) ? 8 : (FT == 4) ? 4 : 2;   // steps of weights in flight: 8 .. 16 KiB a wave
  constexpr int DS = NS / 8;                              // pieces of 256 elements in a wave's share
  constexpr int AREA = NS * 4 * MR > FT * 64 ? NS * 4 * MR : FT * 64;   // 16-byte units of a wave's operand; its sums take the same place later
  __shared__ uint4 s_op[FW][AREA];
  __shared__ float s_ss[FW][16];
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, row = lane & 15, kg = lane >> 4;
  const int n = d >> 8, k0 = w * n * 32, half = hd >> 1, tph = hd >> 4;   // tph: tiles of a head
  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc((void *)Wp, 0, wbytes, 0x00020000);
  float4 xv[MR][DS];
  uint2 gv[DS];
#pragma unroll
  for (int j = 0; j < DS; ++j) {
    const int k = j * 256 + 4 * lane;   // the lane's four elements of the share
    const bool live = k < n * 32;
#pragma unroll
    for (int m = 0; m < MR; ++m) {
      xv[m][j] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (m < M && live) xv[m][j] = *reinterpret_cast<const float4 *>(x + (size_t)m * d + k0 + k);
    }
    gv[j] = make_uint2(0, 0);
    if (live) gv[j] = *reinterpret_cast<const uint2 *>(gain + k0 + k);
  }
  uint32_t wo[FT];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
    const int T = blockIdx.x * FT + ft;
    int f = 16 * T + row;
    if (KIND == FEW_QKV) {   // eight rotation pairs of one head: their first and then their second elements
      const int hh = T / tph, i0 = (T - hh * tph) * 8;
      f = hh * hd + i0 + (row < 8 ? row : half + row - 8);
    }
    wo[ft] = T < tiles ? (uint32_t)(f >> 5) * strip_bytes + (uint32_t)((f & 31) * 16 + (kg >> 1) * 1024 + (kg & 1) * 512) + (uint32_t)k0 * 64u : OOB;
  }
  uint4 wb[P][FT];
  auto issue = [&](int s, uint4(&dst)[FT]) {
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) dst[ft] = load16_nt(wrs, (s < n && wo[ft] != OOB) ? wo[ft] + s * 2048u : OOB);
  };
#pragma unroll
  for (int s = 0; s < P; ++s) issue(s, wb[s]);
  // the thread's place in the epilogue: row em, features 4 eg .. of the first and of the second eight of tile eft, and what it
  // looks up there, behind the loads that everything waits for
  const int eft = tid >> 5, em = tid & 15, eg = (tid >> 4) & 1;
  const bool fin = tid < FT * 32 && em < M;
  const int eT = blockIdx.x * FT + eft, ehh = eT / tph, ei0 = (eT - ehh * tph) * 8 + 4 * eg;   // the thread's head and first pair
  // (Undefined in threads that finish nothing: any value there would have to be merged in behind a wait for all loads, and wave 0 would come to
  // the barrier with its weights only: q|k|v of 1B, five rows, 6.3 -> 5.95 us.)
  i32x4_t place;
  f32x4_t t0, t1;
  if (KIND == FEW_QKV && fin) {
    place = *reinterpret_cast<const i32x4_t *>(e.row_place + em);
    t0 = *reinterpret_cast<const f32x4_t *>(e.rope_tab + ((size_t)em * half + ei0) * 2);      // cos, sin, cos, sin
    t1 = *reinterpret_cast<const f32x4_t *>(e.rope_tab + ((size_t)em * half + ei0) * 2 + 4);
  }

  // ---- the rows' sums of squares ----
#pragma unroll
  for (int m0 = 0; m0 < MR; m0 += 8) {
    if (m0 >= M) continue;   // (uniform)
    float sq[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      sq[m] = 0.f;
#pragma unroll
      for (int j = 0; j < DS; ++j) {
        const float4 v = xv[m0 + m][j];
        sq[m] += v.x * v.x + v.y * v.y + (v.z * v.z + v.w * v.w);
      }
    }
    const float t = wave_sum8(sq, lane);   // lane l: row m0 + 4 l5 + 2 l4 + l3
    if ((lane & 7) == 0) s_ss[w][m0 + ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1)] = t;
  }
  lds_barrier();
  float tot = 0.f;
#pragma unroll
  for (int u = 0; u < FW; ++u) tot += s_ss[u][row & (MR - 1)];   // fixed order
  const float rinv = 1.0f / sqrtf(tot / (float)d + eps);         // of row l % 16

  // ---- the normalised rows, as the operand: unit (8 elements k / 8 of the share, row), the row's place turned by the element so that
  // the lanes of a store fall on different banks.  Places of rows beyond M hold anything: they only feed their own results. ----
#pragma unroll
  for (int j = 0; j < DS; ++j) {
    const int k = j * 256 + 4 * lane, u = k >> 3;
    const float g[4] = {__uint_as_float(gv[j].x << 16), __uint_as_float(gv[j].x & 0xffff0000u), __uint_as_float(gv[j].y << 16),
                        __uint_as_float(gv[j].y & 0xffff0000u)};
#pragma unroll
    for (int m = 0; m < MR; ++m) {
      if (m >= M) continue;   // (uniform)
      const float r = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(rinv), m));
      const float4 v = xv[m][j];
      if (k < n * 32)
        *reinterpret_cast<uint2 *>(reinterpret_cast<char *>(&s_op[w][u * MR + ((m ^ u) & (MR - 1))]) + (k & 4) * 2) =
            make_uint2(f2h2(v.x * r * g[0], v.y * r * g[1]), f2h2(v.z * r * g[2], v.w * r * g[3]));
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (a wave reads only what it wrote itself)

  // ---- the products ----
  f32x4_t acc[FT];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) acc[ft] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    if (s < n) {
      const int u = s * 4 + kg;
      const f16x8_t a = __builtin_bit_cast(f16x8_t, s_op[w][u * MR + ((row ^ u) & (MR - 1))]);
#pragma unroll
      for (int ft = 0; ft < FT; ++ft)
        acc[ft] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, wb[s % P][ft]), a, acc[ft], 0, 0, 0);
    }
    if (s + P < NS) issue(s + P, wb[s % P]);
  }
  auto red = [&](int u, int ft, int l) -> float4 & { return reinterpret_cast<float4 *>(s_op[u])[ft * 64 + l]; };
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) red(w, ft, lane) = make_float4(acc[ft][0], acc[ft][1], acc[ft][2], acc[ft][3]);
  lds_barrier();
  if (!fin || eT >= tiles) return;

  // ---- whole sums, in wave order: features 4 eg .. of the tile's first eight (a) and of its second eight (c) ----
  float4 a = red(0, eft, eg * 16 + em), c = red(0, eft, (eg + 2) * 16 + em);
#pragma unroll
  for (int u = 1; u < FW; ++u) {
    a = add4(a, red(u, eft, eg * 16 + em));
    c = add4(c, red(u, eft, (eg + 2) * 16 + em));
  }
  float av[4] = {a.x * oscale, a.y * oscale, a.z * oscale, a.w * oscale}, cv[4] = {c.x * oscale, c.y * oscale, c.z * oscale, c.w * oscale};
  auto pack4 = [](const uint16_t(&h)[4]) { return make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16)); };
  if (KIND == FEW_GATE_UP) {   // gate and up of features 8 eT + 4 eg ..
    uint16_t o4[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) o4[j] = f2bf(av[j] / (1.0f + __expf(-av[j])) * cv[j]);
    *reinterpret_cast<uint2 *>(e.act + tile_unit(em, 8 * eT, e.KBo) * 8 + 4 * eg) = pack4(o4);
    return;
  }
  if (ehh < e.H + e.Hkv) {
    const float cs[4] = {t0.x, t0.z, t1.x, t1.z}, sn[4] = {t0.y, t0.w, t1.y, t1.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float ra = av[j] * cs[j] - cv[j] * sn[j], rb = av[j] * sn[j] + cv[j] * cs[j];
      av[j] = ra;
      cv[j] = rb;
    }
  }
  uint16_t ab[4], cb[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    ab[j] = f2bf(av[j]);
    cb[j] = f2bf(cv[j]);
  }
  if (ehh < e.H) {   // the query operand keeps 16 significant bits: plane 0 the nearest bf16, plane 1 the nearest bf16 of the rest
    const int group = e.H / e.Hkv, kvh = ehh / group, rr = place.y * group + ehh - kvh * group;
    const size_t o0 = q_elem_off(place.x, kvh, rr, ei0, e.Hkv, hd), o1 = q_elem_off(place.x, kvh, rr, ei0 + half, e.Hkv, hd);
    uint16_t al[4], cl[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      al[j] = f2bf(av[j] - bf2f(ab[j]));
      cl[j] = f2bf(cv[j] - bf2f(cb[j]));
    }
    *reinterpret_cast<uint2 *>(e.qp + o0) = pack4(ab);
    *reinterpret_cast<uint2 *>(e.qp + o1) = pack4(cb);
    *reinterpret_cast<uint2 *>(e.qp + e.q_plane + o0) = pack4(al);
    *reinterpret_cast<uint2 *>(e.qp + e.q_plane + o1) = pack4(cl);
    return;
  }
  const int t = place.z & 15;
  const bool is_v = ehh >= e.H + e.Hkv;
  uint16_t *tile = (is_v ? e.vpool : e.kpool) + ((size_t)place.w * e.Hkv + (ehh - e.H - (is_v ? e.Hkv : 0))) * (16 * hd);
  if (!is_v) {
    *reinterpret_cast<uint2 *>(tile + k_tile_off(t, ei0)) = pack4(ab);
    *reinterpret_cast<uint2 *>(tile + k_tile_off(t, ei0 + half)) = pack4(cb);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      tile[v_tile_off(t, ei0 + j)] = ab[j];
      tile[v_tile_off(t, ei0 + half + j)] = cb[j];
    }
  }
}

// Projection of rows that lie in operand order, added to the residual stream: x[m][f] += sum_k W[f][k] a[m][k].
// P: steps of 32 on their way per wave; RG: groups of rows.  Grid = tiles of 16 features, or (HALF) of eight, with groups of eight rows: a
// matrix instruction then takes the same eight features and rows twice, from both halves of the wave's share of the contraction, and the
// two quarters of its result that pair unlike halves are left.  A compute unit draws about 30 GB/s from memory however much it has on
// its way, so a matrix of 2048 features wants 256 blocks.
template <bool F16, bool HALF, int RG, int P>
__global__ __launch_bounds__(64 * FW, 2) void k_few_add(const void *__restrict__ Wp, const void *__restrict__ Ap, float *x, uint32_t strip_bytes,
                                                        uint32_t wbytes, int K, int M, int d, float oscale) {
  constexpr int ROWS = HALF ? 8 : 16;   // rows of a group
  __shared__ float4 s_red[FW][RG][64];
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, kg = lane >> 4;
  const int row = HALF ? lane & 7 : lane & 15, f = (HALF ? 8 : 16) * blockIdx.x + row;   // the lane's row and feature
  const int n = K >> 8, k0 = w * n * 32, steps = HALF ? (n + 1) >> 1 : n, first = HALF && (lane & 8) ? steps : 0;
  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc((void *)Wp, 0, wbytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t ars = __builtin_amdgcn_make_buffer_rsrc((void *)Ap, 0, (uint32_t)K * 64u, 0x00020000);   // one tile of 32 rows
  const uint32_t at = (uint32_t)((kg >> 1) * 1024 + (kg & 1) * 512) + (uint32_t)(k0 + first * 32) * 64u;
  const uint32_t wo = (uint32_t)(f >> 5) * strip_bytes + (uint32_t)(f & 31) * 16u + at, ao = at + (uint32_t)row * 16u;
  const int last = min(steps, n - first);   // (an odd share: the second half is a step shorter)
  uint4 wb[P], ab[P][RG];
  auto issue = [&](int s, uint4 &wd, uint4(&ad)[RG]) {
    wd = load16_nt(wrs, s < last ? wo + (uint32_t)s * 2048u : OOB);
#pragma unroll
    for (int g = 0; g < RG; ++g) ad[g] = load16(ars, s < last && g * ROWS + row < M ? ao + (uint32_t)(s * 2048 + g * ROWS * 16) : OOB);
  };
#pragma unroll
  for (int j = 0; j < P; ++j) issue(j, wb[j], ab[j]);
  // the thread's place in the epilogue: features 4 eg .. of row em
  constexpr int FEAT = HALF ? 8 : 16, FIN = RG * ROWS * FEAT / 4;
  const int em = tid / (FEAT / 4), eg = tid % (FEAT / 4);
  const bool fin = tid < FIN && em < M;
  float4 *const xp = reinterpret_cast<float4 *>(x + (size_t)em * d + FEAT * blockIdx.x + 4 * eg);
  float4 xv = make_float4(0.f, 0.f, 0.f, 0.f);
  if (fin) xv = *xp;
  f32x4_t acc[RG];
#pragma unroll
  for (int g = 0; g < RG; ++g) acc[g] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
  auto use = [&](int j) {   // (steps beyond the share hold zeros)
#pragma unroll
    for (int g = 0; g < RG; ++g) {
      if constexpr (F16)
        acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, wb[j]), __builtin_bit_cast(f16x8_t, ab[j][g]), acc[g], 0, 0, 0);
      else
        acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wb[j]), __builtin_bit_cast(bf16x8_t, ab[j][g]), acc[g], 0, 0, 0);
    }
  };
  int it = 0;
  for (; it + P < steps; it += P) {
#pragma unroll
    for (int j = 0; j < P; ++j) {
      use(j);
      issue(it + P + j, wb[j], ab[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < P; ++j) use(j);   // (apart: with nothing to follow, loads of zeros would hold the unit up as any others do)
#pragma unroll
  for (int g = 0; g < RG; ++g) s_red[w][g][lane] = make_float4(acc[g][0], acc[g][1], acc[g][2], acc[g][3]);
  lds_barrier();
  if (!fin) return;
  const int g = em / ROWS, r = em % ROWS;
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int u = 0; u < FW; ++u) {   // in wave order
    a = add4(a, s_red[u][g][eg * 16 + r]);
    if (HALF) a = add4(a, s_red[u][g][(eg + 2) * 16 + 8 + r]);
  }
  *xp = make_float4(xv.x + a.x * oscale, xv.y + a.y * oscale, xv.z + a.z * oscale, xv.w + a.w * oscale);
}

// Tiles of 16 features per block (1, 2, 4 or 7): the least work per compute unit, rounds x (tiles + what a block costs besides, about
// one).  Seven are for gate|up of the 8B shape: 256 blocks.  22 shapes with 5, 8 and 16 rows, each projection with all four: the rule's is within
// 3 % of the best at 121 of 124, 9 % off at worst (37888 x 3584, five rows: 49.8 us with seven, 45.7 with two); the wrong one costs up to 2 x (22016 x 4096, 16
// rows: 1, 2, 4, 7 tiles 68, 41, 41, 33 us).  All timings: profiles/few_rows_tiles.txt.
int pick_tiles(const fsv_ctx *c, int tiles) {
  int best = 1, cost = 0;
  for (int ft : {7, 4, 2, 1}) {
    const int v = fsv_ceil_div(fsv_ceil_div(tiles, ft), c->n_cus) * (ft + 1);
    if (!cost || v < cost) { best = ft; cost = v; }
  }
  return best;
}

template <int KIND, int FT>
void launch_norm(fsv_ctx *c, int cls, const void *Wp, const void *gain, uint32_t strip_bytes, uint32_t wbytes, int N, int M, float oscale,
                 const few_out &e, hipStream_t st) {
  const int d = c->d.d_model, tiles = N / 16;
  const dim3 grid(fsv_ceil_div(tiles, FT));
  fsv_prof_scope ps(c, st, cls, (double)N * d * 2.0, true);
#define FSV_FEW_GO(NSV, MRV)                                                                                                             \
  hipExtLaunchKernelGGL((k_few_norm<KIND, FT, NSV, MRV>), grid, dim3(64 * FW), 0, st, ps.start(), ps.stop(), 0, Wp, (const float *)c->x, \
                        (const uint16_t *)gain, strip_bytes, wbytes, d, M, tiles, KIND == FEW_QKV ? c->d.head_dim : 32, c->d.rms_eps, oscale, e)
  if (d <= 2048) { if (M <= 8) FSV_FEW_GO(8, 8); else FSV_FEW_GO(8, 16); }
  else { if (M <= 8) FSV_FEW_GO(16, 8); else FSV_FEW_GO(16, 16); }
#undef FSV_FEW_GO
}

}  // namespace

bool fsv_bf16_few_rows(const fsv_ctx *c, int M) {
  const int d = c->d.d_model, ffn = c->d.d_ffn;
  if (M > 16 || d > 4096 || d % 256) return false;
  if (M <= 8) return true;   // (nine and more: see the head of this file)
  return d <= 2048 ? ffn <= min(16 * d, max(8192, 8 * d)) : d == 4096 && ffn <= 14336;
}

int fsv_bf16_few_qkv(fsv_ctx *c, const fsv_batch *b, const void *Wp, const void *gain, uint32_t strip_bytes, uint32_t wbytes, int N, int M,
                     float oscale, size_t layer_off, hipStream_t st) {
  few_out e{};
  e.H = c->d.n_heads; e.Hkv = c->d.n_kv_heads;
  e.row_place = (const int4 *)c->row_place;
  e.rope_tab = c->rope_tab;
  e.qp = (uint16_t *)c->buf_q; e.q_plane = c->q_plane_units * 8;
  e.kpool = (uint16_t *)b->k_pool + layer_off; e.vpool = (uint16_t *)b->v_pool + layer_off;
  switch (pick_tiles(c, N / 16)) {
    case 1: launch_norm<FEW_QKV, 1>(c, FSV_K_GEMM_QKV, Wp, gain, strip_bytes, wbytes, N, M, oscale, e, st); break;
    case 2: launch_norm<FEW_QKV, 2>(c, FSV_K_GEMM_QKV, Wp, gain, strip_bytes, wbytes, N, M, oscale, e, st); break;
    case 4: launch_norm<FEW_QKV, 4>(c, FSV_K_GEMM_QKV, Wp, gain, strip_bytes, wbytes, N, M, oscale, e, st); break;
    default: launch_norm<FEW_QKV, 7>(c, FSV_K_GEMM_QKV, Wp, gain, strip_bytes, wbytes, N, M, oscale, e, st); break;
  }
  FSV_HIP(c, hipGetLastError());
  return FSV_OK;
}

int fsv_bf16_few_gate_up(fsv_ctx *c, const void *Wp, const void *gain, uint32_t strip_bytes, uint32_t wbytes, int N, int M, float oscale,
                         hipStream_t st) {
  few_out e{};
  e.act = (uint16_t *)c->buf_act;
  e.KBo = c->d.d_ffn / 16;
  switch (pick_tiles(c, N / 16)) {
    case 1: launch_norm<FEW_GATE_UP, 1>(c, FSV_K_GEMM_GATE_UP, Wp, gain, strip_bytes, wbytes, N, M, oscale, e, st); break;
    case 2: launch_norm<FEW_GATE_UP, 2>(c, FSV_K_GEMM_GATE_UP, Wp, gain, strip_bytes, wbytes, N, M, oscale, e, st); break;
    case 4: launch_norm<FEW_GATE_UP, 4>(c, FSV_K_GEMM_GATE_UP, Wp, gain, strip_bytes, wbytes, N, M, oscale, e, st); break;
    default: launch_norm<FEW_GATE_UP, 7>(c, FSV_K_GEMM_GATE_UP, Wp, gain, strip_bytes, wbytes, N, M, oscale, e, st); break;
  }
  FSV_HIP(c, hipGetLastError());
  return FSV_OK;
}

int fsv_bf16_few_add(fsv_ctx *c, int cls, const void *Wp, const void *Ap, uint32_t strip_bytes, uint32_t wbytes, int N, int K, int M, int f16,
                     float oscale, hipStream_t st) {
  fsv_prof_scope ps(c, st, cls, (double)N * K * 2.0, true);
  // Tiles of eight where they still fit the compute units at once: down of 2048 features, ffn 8192, five rows 7.8 us and 9.1 with tiles of 16; of
  // 2304, ffn 6144, eight rows 9.6 and 7.3 (288 blocks are a second round), of 3584, ffn 18944 28.5 and 23.0.  Steps in flight, P 4 or 8: within 3 % of
  // each other at 4096 features; at 2048 four 8 .. 12 % faster with ffn 5632, eight 6 % with 16384.
  const bool half = N / 8 <= c->n_cus;
#define FSV_FEW_GO(F16V, HV, RGV, PV, OSC)                                                                                           \
  hipExtLaunchKernelGGL((k_few_add<F16V, HV, RGV, PV>), dim3(N / (HV ? 8 : 16)), dim3(64 * FW), 0, st, ps.start(), ps.stop(), 0, Wp, Ap, c->x, \
                        strip_bytes, wbytes, K, M, N, OSC)
#define FSV_FEW_P(F16V, OSC)                                                                                                  \
  do {                                                                                                                         \
    if (!half) FSV_FEW_GO(F16V, false, 1, 8, OSC);                                                                             \
    else if (M <= 8) { if (K <= 2048) FSV_FEW_GO(F16V, true, 1, 4, OSC); else FSV_FEW_GO(F16V, true, 1, 8, OSC); }             \
    else { if (K <= 2048) FSV_FEW_GO(F16V, true, 2, 4, OSC); else FSV_FEW_GO(F16V, true, 2, 8, OSC); }                         \
  } while (0)
  if (f16) FSV_FEW_P(true, oscale);
  else FSV_FEW_P(false, 1.0f);
#undef FSV_FEW_P
#undef FSV_FEW_GO
  FSV_HIP(c, hipGetLastError());
  return FSV_OK;
}
