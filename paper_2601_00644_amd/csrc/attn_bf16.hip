// Multi-query paged attention of the FSV_BF16 path (the attention step of the target forward in Alg. 2
// step 2, over the user's restored KV session plus the rows appended in this call, Sec. IV-C).
// Built with -mllvm -amdgpu-mfma-vgpr-form: the MFMA accumulators stay in the architectural registers,
// where the softmax arithmetic reaches them, and the accumulation registers hold the K/V tiles in flight.
#include <hip/hip_ext.h>
#include <limits.h>
#include <math.h>
#include <stdlib.h>
#include <type_traits>

#include "bf16_common.h"

using namespace fsv_bf16;

namespace {

// ---------------------------------------------------------------------------------------------
// Work decomposition.  The keys of request b are cut into tiles of 32 (two pages); a "part" is a run of
// tp_b consecutive tiles, s_b runs per request, chosen so that every part of every request has about the
// same length and parts x kv heads comes to one block per compute unit (attn_schedule.h).  A block owns its part completely: its
// waves (eight, or four) take every eighth (fourth) tile each (each byte of the KV stream is read once; all `group` query heads and all gamma+1
// positions share it, except in small calls, where every tile of 32 query rows has parts of its own).  A wave streams the K and V page tiles of its keys straight from HBM into a ring of its own in LDS, forms
// S^T = K Q^T (rows = keys, so a query row's scores sit in two lanes; the queries lie in LDS, shared by the waves), does the
// online softmax in registers, and feeds the probabilities back as the B operand of O^T += V^T P^T without
// any shuffle: the V tile is stored in the key order the score accumulators produce.  The waves' shares are merged through
// LDS; a request with one part is then done, the others leave (m, l, O) per part and the block that comes last merges them.
//
// Why like this: bound by the KV stream where a request has one row tile, by the softmax arithmetic (about 670 cycles of
// it per 32 x 32 tile, which the exponentials and the split into hi + lo take) where it has two or three.  With two waves on a
// SIMD one's arithmetic runs under the other's matrix products; the loads cost no registers and 64 .. 128 KiB per compute unit are on
// their way.  One wave per SIMD with K and V in registers, one tile ahead, and the merge as a launch of its own (16 requests of
// 512 .. 4096 positions, head size 128: 27.3 + 5.9 us; 128 requests of 256 .. 8192: 230 + 14; 2048 prefill rows 128 + 22; 8 requests
// of 4 .. 16 k, head size 64: 37.9 + 7.8) against this: 31.6 (27.9 where the schedule takes the row tiles of such a call apart, which few of that range do), 207, 118, 39 (33.2, 207, 119, 38 before the partial results were stored in
// whole lines, and when the following were measured).  Measured and dropped: four waves per block with the
// queries in registers (33, 249, 141, 46); two blocks per compute unit whose waves share the tiles, one row tile each, a barrier per
// item (40, 249, 148, 54: a tile is a chain of 1.2 us and too few are in work); one block per compute unit that goes through the
// requests of its share, the next one's keys on their way (39, 235, 177, 51: without the rings' place the merge takes 3.3 us a request).
//
// Precision: K and V are the bf16 bits of the cache.  The two operands the kernel itself produces for the matrix
// cores are carried as a pair of bf16 values (hi + lo, hi = the nearest bf16, lo = the nearest bf16 of the rest: 16
// significant bits together) and take two MFMAs each: the rotated queries (two planes of the query buffer) and the
// probabilities.  The result then differs from exact arithmetic on the stored K / V only by fp32 accumulation.

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;

// part_prefix[b] = parts of requests before b; part_desc[global part] = everything a wave of
// the attention kernel needs to start, in one 112-byte record: request, first tile, tiles, parts of the same rows, cached
// length, drafts, first row, first part of the same rows, the physical pages of the part's first eight tiles, its number (records of a
// schedule of several rounds are not in order), its first query row, its query rows, the step to the next part of the same rows -- a wave fetches it with a few scalar loads and can issue its first K/V loads at once, instead of after a chain of dependent ones
constexpr int kDescInts = 28;
// Everything the forward's kernels look up about a call, in one launch: the attention schedule (block 0), for the stand-alone
// attention the query operand (the last blocks; 6 us as a launch of its own, two bytes per lane), and for every row
// its request, index, position and token and the cos / sin of its rotation angles (the other blocks; the angles depend on the
// row's position only, not on the layer: tab[(row * half + i) * 2 + {0, 1}], formed and reduced in fp64).
// Bound by latency: a load of the lengths, a scan or search in LDS, a load of the page ids, the stores.  One thread walking
// the requests, and a launch each for rows and angles, took 13 + 4.5 + 4.5 us for 16 requests and 82 + 6 + 6 for 128; this
// takes 4.7 and 6.3.
constexpr int kSetupThreads = 1024, kSetupB = 2048;   // requests whose prefix sums are kept in LDS (more are searched in memory)
struct setup_args {
  int B, tpw, nw, sorted, split, group, w2, w3, max_pages, num_pages, grid_parts, tickets, M, half, V;   // grid_parts: records the attention's grid reads
  const int32_t *seq_lens, *off, *page_table, *last_token, *draft;
  const double *inv_freq;
  int32_t *part_prefix, *part_desc, *ticket, *row_req, *row_place, *row_tok;
  float *tab;
  // stand-alone attention: the caller's rotated queries [M][heads][hd] (bf16), to be put into the query operand
  int row_blocks = 0, H = 0, Hkv = 0, hd = 0, q_vec = 0;
  const uint16_t *q = nullptr;
  uint16_t *qp = nullptr;
  size_t q_plane = 0;
};
__global__ __launch_bounds__(kSetupThreads) void k_setup(setup_args p) {
  __shared__ int32_t s_pre[kSetupB + 1];
  __shared__ int32_t s_w[kSetupThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, B = p.B;
  // the last index b with pre[b] + step * b <= x, b in [0, B)
  auto find = [&](const int32_t *pre, int step, int x) {
    int lo = 0, hi = B;   // pre[lo] <= x < pre[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (pre[mid] + step * mid <= x) lo = mid; else hi = mid;
    }
    return lo;
  };
  if ((int)blockIdx.x > p.row_blocks) {   // ---- queries, eight features per thread ----
    const bool in_lds = B <= kSetupB;
    if (in_lds) {
      for (int b = tid; b <= B; b += kSetupThreads) s_pre[b] = p.off[b];
      __syncthreads();
    }
    const int32_t *off = in_lds ? s_pre : p.off;
    const int per = p.H * (p.hd / 8), t = (int)(blockIdx.x - 1 - p.row_blocks) * kSetupThreads + tid, r = t / per;
    if (r >= p.M) return;
    const int hh = (t - r * per) / (p.hd / 8), e = ((t - r * per) % (p.hd / 8)) * 8;
    const int b = find(off, 1, r), rr = (r - off[b] - b) * p.group + hh % p.group;
    const uint16_t *src = p.q + (size_t)r * p.H * p.hd + hh * p.hd + e;
    uint4 v;
    if (p.q_vec) {
      v = *reinterpret_cast<const uint4 *>(src);
    } else {
      uint32_t w4[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) w4[j] = (uint32_t)src[2 * j] | ((uint32_t)src[2 * j + 1] << 16);
      v = make_uint4(w4[0], w4[1], w4[2], w4[3]);
    }
    const size_t o = q_elem_off(b, hh / p.group, rr, e, p.Hkv, p.hd);
    *reinterpret_cast<uint4 *>(p.qp + o) = v;
    *reinterpret_cast<uint4 *>(p.qp + p.q_plane + o) = make_uint4(0, 0, 0, 0);   // the caller's queries are bf16 already
    return;
  }
  if (blockIdx.x > 0) {   // ---- rows ----
    const bool in_lds = B <= kSetupB;
    if (in_lds) {
      for (int b = tid; b <= B; b += kSetupThreads) s_pre[b] = p.off[b];
      __syncthreads();
    }
    const int32_t *off = in_lds ? s_pre : p.off;
    const int t = (int)(blockIdx.x - 1) * kSetupThreads + tid, r = t / p.half, i = t - r * p.half;
    if (r >= p.M) return;
    const int b = find(off, 1, r), idx = r - off[b] - b, pos = p.seq_lens[b] + idx;
    if (i == 0) {
      p.row_req[r] = b;
      const int page = p.page_table[(size_t)b * p.max_pages + min(pos >> 4, p.max_pages - 1)];
      reinterpret_cast<int4 *>(p.row_place)[r] = make_int4(b, idx, pos, min(max(page, 0), p.num_pages - 1));
      const int tok = (idx == 0) ? (p.last_token ? p.last_token[b] : 0) : (p.draft ? p.draft[r - b - 1] : 0);
      p.row_tok[r] = min(max(tok, 0), p.V - 1);
    }
    if (p.tab) {
      double sn, cs;
      sincos((double)pos * p.inv_freq[i], &sn, &cs);
      reinterpret_cast<float2 *>(p.tab)[t] = make_float2((float)cs, (float)sn);
    }
    return;
  }
  // ---- attention schedule ----
  auto parts_of = [&](int b, int &L, int &gamma, int &n, int &tp, int &m) {   // key parts; m: row tiles with parts of their own
    L = p.seq_lens[b];
    gamma = p.off[b + 1] - p.off[b];
    n = (L + gamma + 1 + 31) >> 5;
    const int rtc = (p.group * (gamma + 1) + 31) >> 5;
    m = p.split ? rtc : 1;
    return attn_parts(n, p.tpw, p.split || rtc <= 1 ? 16 : rtc == 2 ? p.w2 : p.w3, p.nw, &tp);
  };
  int run = 0;
  for (int b0 = 0; b0 < B; b0 += kSetupThreads) {
    const int b = b0 + tid;
    int L, gamma, n, tp, m;
    const int s = b < B ? parts_of(b, L, gamma, n, tp, m) * m : 0;
    int incl = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(incl, o, 64);
      if (lane >= o) incl += t;
    }
    __syncthreads();   // (s_w of the round before has been read)
    if (lane == 63) s_w[w] = incl;
    __syncthreads();
    int pre = run, tot = 0;
    for (int i = 0; i < kSetupThreads / 64; ++i) {
      pre += i < w ? s_w[i] : 0;
      tot += s_w[i];
    }
    if (b < B) {
      p.part_prefix[b] = pre + incl - s;
      if (b < kSetupB) s_pre[b] = pre + incl - s;
    }
    run += tot;
  }
  if (tid == 0) {
    p.part_prefix[B] = run;
    if (B <= kSetupB) s_pre[B] = run;
  }
  __syncthreads();   // the prefix sums are read back below by other threads of this block
  const int32_t *pre = B <= kSetupB ? s_pre : p.part_prefix;
  // The grid comes from the host copies of the lengths, the parts from the device's.  Should a caller's two not agree, that call's
  // result is not defined, but it stays within the grid, records without a part are empty, and every call begins with all tickets
  // at zero, whatever the one before has left.
  const int total = min(run, p.grid_parts);
  for (int q = total + tid; q < p.grid_parts; q += kSetupThreads) *reinterpret_cast<int4 *>(p.part_desc + (size_t)q * kDescInts) = make_int4(0, 0, 0, 0);
  for (int i = tid; i < p.tickets; i += kSetupThreads) p.ticket[i] = 0;
  // In several rounds the long parts go first, so that the last round is made of short ones: the place of a part is the count of
  // parts in longer classes (128 of them), then as it comes.  What a part computes does not depend on its place.
  __shared__ int32_t s_class[128];
  auto part = [&](int q, int &b, int &k, int &s, int &t0, int &cnt, int &L, int &gamma, int &m) {   // k: number of the part, row tiles first
    b = find(pre, 0, q);
    int n, tp;
    s = parts_of(b, L, gamma, n, tp, m);
    k = q - pre[b];
    t0 = k / m * tp;
    cnt = min(n, t0 + tp) - t0;
  };
  auto class_of = [&](int cnt) { return 127 - min(127, cnt * 128 / (p.tpw + p.nw)); };
  if (p.sorted) {
    if (tid < 128) s_class[tid] = 0;
    __syncthreads();
    for (int q = tid; q < total; q += kSetupThreads) {
      int b, k, s, t0, cnt, L, gamma, m;
      part(q, b, k, s, t0, cnt, L, gamma, m);
      atomicAdd(&s_class[class_of(cnt)], 1);
    }
    __syncthreads();
    if (tid < 64) {
      const int c0 = s_class[2 * tid], c1 = s_class[2 * tid + 1];
      int incl = c0 + c1;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
      }
      s_class[2 * tid] = incl - c0 - c1;
      s_class[2 * tid + 1] = incl - c1;
    }
    __syncthreads();
  }
  for (int q = tid; q < total; q += kSetupThreads) {
    int b, k, s, t0, cnt, L, gamma, m;
    part(q, b, k, s, t0, cnt, L, gamma, m);
    const int npg = (L + gamma + 1 + 15) >> 4;
    const int32_t *pt = p.page_table + (size_t)b * p.max_pages;
    int pg[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) pg[i] = min(max(pt[min(2 * t0 + i, npg - 1)], 0), p.num_pages - 1);
    const int at = p.sorted ? atomicAdd(&s_class[class_of(cnt)], 1) : q;
    int4 *d = reinterpret_cast<int4 *>(p.part_desc + (size_t)at * kDescInts);
    d[0] = make_int4(b, t0, cnt, s);
    d[1] = make_int4(L, gamma, p.off[b] + b, pre[b] + k % m);
#pragma unroll
    for (int i = 0; i < 4; ++i) d[2 + i] = make_int4(pg[4 * i], pg[4 * i + 1], pg[4 * i + 2], pg[4 * i + 3]);
    const int R = p.group * (gamma + 1), rb = k % m * 32;
    d[6] = make_int4(q, rb, m > 1 ? min(32, R - rb) : R, m);
  }
}

// Four fp16 values as floats, for the stand-alone entry point's row-major result (a 16-byte store at any 4-byte boundary).
__device__ inline void store_row4(float *p, uint32_t lo, uint32_t hi) {
  *reinterpret_cast<f32x4_any *>(p) = (f32x4_any){h2f((uint16_t)(lo & 0xffffu)), h2f((uint16_t)(lo >> 16)), h2f((uint16_t)(hi & 0xffffu)),
                                              h2f((uint16_t)(hi >> 16))};
}

// Waits until at most min(n, N) groups of LPG loads of this wave are on their way (n wave-uniform).
template <int N, int LPG>
__device__ __forceinline__ void wait_groups(int n) {
  if constexpr (N == 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  } else {
    if (n >= N) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N * LPG) : "memory");
    else wait_groups<N - 1, LPG>(n);
  }
}

// Device-scope accesses to the partial results that travel between blocks; sixteen bytes at a time through a descriptor of the
// part's rows (sc1, the bit the atomics carry: past the non-coherent caches).  A store of a wave covers whole lines that way.  With eight-byte
// atomics that each covered every fourth eight bytes, the tail of a part (LDS, stores, ticket, merge) took 2 us longer: whole calls,
// head size 128, one request of 1600 positions and eight rows 17.4 -> 15.7 us, 16 requests of 512 .. 4096 36.0 -> 34.4.
constexpr int kDeviceScope = 16;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_of(const float *p) { return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, 0xFFFFFFFFu, 0x00020000); }
__device__ __forceinline__ void store_dev4(__amdgpu_buffer_rsrc_t rows, uint32_t at, float4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), rows, at * 4, 0, kDeviceScope);
}
__device__ __forceinline__ float4 load_dev4(__amdgpu_buffer_rsrc_t rows, uint32_t at) {
  return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rows, at * 4, 0, kDeviceScope));
}
__device__ __forceinline__ void store_dev(float *p, float x, float y) {
  __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), (unsigned long long)__float_as_uint(x) | ((unsigned long long)__float_as_uint(y) << 32),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 load_dev(const float *p) {
  const unsigned long long v = __hip_atomic_load(reinterpret_cast<const unsigned long long *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}

template <int HD, int RT, int NW>
struct attn_geo {
  static constexpr int KS = HD / 16, VC = HD / 32, TILEB = 16 * HD * 2;   // TILEB: bytes of one (page, kv head) tile
  static constexpr int ITEM = 2 * TILEB, LPI = ITEM / 1024;              // an item: K or V of a key tile (two pages); its loads
  static constexpr int BUDGET = ((RT == 3 && HD == 128) ? 8 : NW) * 20 * 1024;   // eight waves per compute unit
  static constexpr int QBYTES = RT * KS * 2048;                          // hi and lo planes of the query operand
  static constexpr int LOOK = (BUDGET - QBYTES) / (2 * NW * ITEM), SLOTS = 2 * LOOK;   // key tiles a wave's ring holds
  static constexpr int LDS = SLOTS * NW * ITEM + QBYTES;
  static constexpr int OROW = HD + 4;                                    // floats per row of the merge area (no bank conflicts)
  static constexpr int MSTEP_ = LDS / (NW * (32 * OROW + 64) * 4), MSTEP = MSTEP_ < RT ? MSTEP_ : RT;   // row tiles the merge area holds
  static_assert(LOOK >= 1 && SLOTS * LPI <= 63 && MSTEP >= 1, "");   // (63: what the load counter holds)
};

template <int HD, int RT, int NW>
__global__ __launch_bounds__(64 * NW, (RT == 3 && HD == 128) ? 1 : 2) void k_attention(
    const int32_t *__restrict__ part_desc, int Hkv, int group, const char *__restrict__ qp, size_t q_plane_bytes,
    const char *__restrict__ kpool, const char *__restrict__ vpool, int max_pages, int num_pages, const int32_t *__restrict__ page_table,
    int rows_cap, float *part_o, float *part_ml, int32_t *__restrict__ ticket, uint16_t *__restrict__ out, int KBq, float *__restrict__ out32) {
  using G = attn_geo<HD, RT, NW>;
  constexpr int KS = G::KS, VC = G::VC, TILEB = G::TILEB, ITEM = G::ITEM, LPI = G::LPI, SLOTS = G::SLOTS, LOOK = G::LOOK;
  extern __shared__ uint4 lds[];
  char *const ldsc = reinterpret_cast<char *>(lds);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)lds;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, h = lane >> 5, r = lane & 31;
  const int gw = blockIdx.x, pp = gw / Hkv, kvh = gw - pp * Hkv;
  const int32_t *desc = part_desc + (size_t)pp * kDescInts;
  const int4 d0 = *reinterpret_cast<const int4 *>(desc), d1 = *reinterpret_cast<const int4 *>(desc + 4);
  const int2 d2 = *reinterpret_cast<const int2 *>(desc + 8 + 2 * w);
  const int4 d6 = *reinterpret_cast<const int4 *>(desc + 24);
  if (d0.w == 0) return;   // no part
  const int b = d0.x, t0 = d0.y + w, nparts = d0.w, L = d1.x, gamma = d1.y, rs = d1.z;
  const int cnt = max(0, (d0.z - w + NW - 1) / NW), total = 2 * cnt;   // key tiles t0, t0 + NW, ... of this wave; items
  const int own = d6.x, rb = d6.y, R = d6.z, rt0 = rb >> 5;   // the query rows of this part: rb .. rb + R - 1
  const int nk = L + gamma + 1;
  const int rtc = min(RT, (R + 31) >> 5);
  const int32_t *pt = page_table + (size_t)b * max_pages;
  const int npg = (nk + 15) >> 4;
  const uint32_t lane_off = (uint32_t)lane * 16u;
  auto pages_of = [&](int j) {  // physical pages of the wave's j-th tile (indices kept in range)
    const int p = 2 * (t0 + NW * j), p0 = min(p, npg - 1), p1 = min(p + 1, npg - 1);
    return make_int2(min(max(pt[p0], 0), num_pages - 1), min(max(pt[p1], 0), num_pages - 1));
  };
  const uint32_t region = lds0 + (uint32_t)(w * SLOTS * ITEM);
  auto issue = [&](const char *pool, int2 pg, uint32_t slot) {   // one item into the slot at byte offset `slot` of this wave's ring
    const char *s0 = pool + (size_t)(uint32_t)(pg.x * Hkv + kvh) * TILEB, *s1 = pool + (size_t)(uint32_t)(pg.y * Hkv + kvh) * TILEB;
#pragma unroll
    for (int q = 0; q < LPI / 2; ++q) load_to_lds<true>(region + slot + q * 1024, lane_off, s0 + q * 1024);
#pragma unroll
    for (int q = 0; q < LPI / 2; ++q) load_to_lds<true>(region + slot + TILEB + q * 1024, lane_off, s1 + q * 1024);
  };

  // The query operand goes to LDS first, each wave a share of its 1 KiB rows, the first tiles behind it.  Query rows beyond R hold
  // whatever an earlier call left there: they only feed their own output rows, which are never stored.
  char *const qlds = ldsc + SLOTS * NW * ITEM;
#pragma unroll
  for (int i = 0; i < (RT * KS * 2 + NW - 1) / NW; ++i) {
    const int c = i * NW + w, rt = c / (2 * KS), ks = (c / 2) % KS;   // row c = (rt * KS + ks) * 2 + plane
    if (rt >= rtc) break;
    const char *src = qp + (size_t)(c & 1) * q_plane_bytes + ((((size_t)b * RTMAX + rt0 + rt) * Hkv + kvh) * KS + ks) * 1024;
    load_to_lds<false>(lds0 + SLOTS * NW * ITEM + c * 1024, lane_off, src);
  }
  int2 pg = d2;   // pages of the next tile to be loaded
#pragma unroll
  for (int j = 0; j < LOOK; ++j) {
    if (j > 0) pg = pages_of(j);
    if (j < cnt) {
      issue(kpool, pg, 2 * j * ITEM);
      issue(vpool, pg, (2 * j + 1) * ITEM);
    }
  }
  wait_groups<SLOTS, LPI>(min(SLOTS, total));   // the query rows this wave loads have landed
  __syncthreads();
  pg = pages_of(LOOK);

  const float sc = kLog2eF / sqrtf((float)HD);
  f32x16_t o[RT][VC];
  float mrun[RT], lrun[RT];
  int lim[RT];  // last key this lane's query row may see
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
    for (int c = 0; c < VC; ++c)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[rt][c][v] = 0.f;
    mrun[rt] = -INFINITY;
    lrun[rt] = 0.f;
    const int rr = rt * 32 + r;
    lim[rt] = (rr < R) ? L + (rb + rr) / group : -1;
  }
  // K operand row = key r (rows 0-15 first page, 16-31 second page); V operand row = feature
  const char *const kl = ldsc + w * SLOTS * ITEM + (r >> 4) * TILEB + (h * 16 + (r & 15)) * 16;
  const char *const vl = ldsc + w * SLOTS * ITEM + (h * 32 + r) * 16;

  auto run = [&](auto nrt_c) {
    constexpr int NRT = decltype(nrt_c)::value;
    uint32_t slot = 0;
    auto advance = [&]() { slot += ITEM; if (slot == (uint32_t)(SLOTS * ITEM)) slot = 0; };
    for (int j = 0; j < cnt; ++j) {
      const int i = 2 * j, kbase = (t0 + NW * j) * 32;
      wait_groups<SLOTS - 1, LPI>(total - 1 - i);   // K has landed
      bf16x8_t kreg[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kreg[ks] = *reinterpret_cast<const bf16x8_t *>(kl + slot + ks * 512);
      const bool need_mask = kbase + 31 > L;  // every query row sees all keys <= L
      bf16x8_t pb[NRT][2], pl[NRT][2];        // probabilities as hi + lo
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) {
        f32x16_t s;   // accumulator v of this lane: key kbase + 8*(v/4) + 4h + v%4, query row rt*32 + r
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const bf16x8_t qh = *reinterpret_cast<const bf16x8_t *>(qlds + ((rt * KS + ks) * 2) * 1024 + lane_off);
          const bf16x8_t ql = *reinterpret_cast<const bf16x8_t *>(qlds + ((rt * KS + ks) * 2 + 1) * 1024 + lane_off);
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kreg[ks], qh, s, 0, 0, 0);
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kreg[ks], ql, s, 0, 0, 0);
        }
        if (need_mask) {
          const int limit = lim[rt];
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int key = kbase + 8 * (v >> 2) + 4 * h + (v & 3);
            s[v] = (key <= limit) ? s[v] : -INFINITY;
          }
        }
        float tmax = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) tmax = fmaxf(tmax, s[v]);
        tmax = fmaxf(tmax, lane_xor<32>(tmax)) * sc;
        // Lazy reference: the running reference m only moves when the tile maximum exceeds it by more than 2^8
        // (probabilities then stay below 256, exact enough in fp32 / bf16), so the accumulators are almost never
        // rescaled; the first tile of a row needs no rescale either (its accumulators are still zero).
        const float mold = mrun[rt];
        const float mnew = (tmax > mold + 8.0f || mold == -INFINITY) ? fmaxf(mold, tmax) : mold;
        const float muse = (mnew == -INFINITY) ? 0.f : mnew;
        const float alpha = __builtin_amdgcn_exp2f(mold - muse);
        const bool rescale = __any(mnew != mold && mold != -INFINITY);
        mrun[rt] = mnew;
        float psum = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[v], sc, -muse));
          psum += p;
          const __bf16 hi = (__bf16)p;
          pb[rt][v >> 3][v & 7] = hi;
          pl[rt][v >> 3][v & 7] = (__bf16)(p - (float)hi);
        }
        lrun[rt] = lrun[rt] * alpha + psum;
        if (rescale) {  // wave-uniform: once the running maxima have settled the accumulators are left alone
#pragma unroll
          for (int c = 0; c < VC; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[rt][c][v] *= alpha;
        }
        __builtin_amdgcn_sched_barrier(0);   // row tiles one after the other: two waves share a SIMD's registers
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the slot has been read
      if (j + LOOK < cnt) issue(kpool, pg, slot);
      advance();
      wait_groups<SLOTS - 1, LPI>(total - 2 - i);   // V has landed
      bf16x8_t vreg[VC][2];
#pragma unroll
      for (int c = 0; c < VC; ++c)
#pragma unroll
        for (int p = 0; p < 2; ++p) vreg[c][p] = *reinterpret_cast<const bf16x8_t *>(vl + slot + p * TILEB + c * 1024);
      if (kbase + 31 >= nk) {
        // (wave-uniform, the last tile of a request only) Slots beyond the last valid position may never have been written:
        // their probabilities are zero, but 0 * NaN is NaN, so the V values of those keys are cleared before they reach the
        // matrix cores.  Element e of vreg[c][pg] belongs to key kbase + 16 pg + 8 (e / 4) + 4 h + e % 4.
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          uint32_t m4[4];
#pragma unroll
          for (int dw = 0; dw < 4; ++dw) {
            const int key = kbase + 16 * p + 8 * (dw >> 1) + 4 * h + 2 * (dw & 1);
            m4[dw] = (key < nk ? 0x0000FFFFu : 0u) | (key + 1 < nk ? 0xFFFF0000u : 0u);
          }
#pragma unroll
          for (int c = 0; c < VC; ++c) {
            u32x4_t raw = __builtin_bit_cast(u32x4_t, vreg[c][p]);
#pragma unroll
            for (int dw = 0; dw < 4; ++dw) raw[dw] &= m4[dw];
            vreg[c][p] = __builtin_bit_cast(bf16x8_t, raw);
          }
        }
      }
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
        for (int c = 0; c < VC; ++c) {
          o[rt][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vreg[c][0], pb[rt][0], o[rt][c], 0, 0, 0);
          o[rt][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vreg[c][1], pb[rt][1], o[rt][c], 0, 0, 0);
          o[rt][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vreg[c][0], pl[rt][0], o[rt][c], 0, 0, 0);
          o[rt][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vreg[c][1], pl[rt][1], o[rt][c], 0, 0, 0);
        }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (j + LOOK < cnt) issue(vpool, pg, slot);
      advance();
      pg = pages_of(j + 1 + LOOK);
    }
  };
  if (rtc == 1) run(std::integral_constant<int, 1>{});
  else if (RT < 3 || rtc == 2) run(std::integral_constant<int, (RT >= 2 ? 2 : 1)>{});
  else run(std::integral_constant<int, RT>{});

  // ---- the waves' shares, one row tile at a time, through LDS (their rings are empty now) ----
  // lane: query row rt*32 + r, features 32c + 8g + 4h + (0..3)
  constexpr int OROW = G::OROW, TPR = HD / 8, MS = G::MSTEP;   // TPR: threads per row, eight features each
  float *const area = reinterpret_cast<float *>(lds);
  const uint32_t group_inv = (65535u + (uint32_t)group) / (uint32_t)group;
  const __amdgpu_buffer_rsrc_t mine = rows_of(part_o + ((size_t)own * Hkv + kvh) * rows_cap * HD);
  float2 *const s_ml = reinterpret_cast<float2 *>(area + NW * MS * 32 * OROW);
  auto write_out = [&](int rr, int e0, const float(&acc)[8], float inv) {   // the output is a convex combination of cached values: bounded, so it is handed on in fp16
    uint32_t pk[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) pk[j] = f2h2(acc[2 * j] * inv, acc[2 * j + 1] * inv);
    rr += rb;
    const int i = (int)(((uint32_t)rr * group_inv) >> 16);   // rr / group (rr < 96: the product is exact)
    const int m = rs + i, col = (kvh * group + rr - i * group) * HD + e0;
    if (out32) {
      float *dst = out32 + (size_t)m * KBq * 16 + col;
      store_row4(dst, pk[0], pk[1]);
      store_row4(dst + 4, pk[2], pk[3]);
    } else {
      reinterpret_cast<uint4 *>(out)[tile_unit(m, col, KBq)] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
    }
  };
  auto write_out4 = [&](int rr, int e0, float4 v, float inv) {
    rr += rb;
    const uint32_t lo = f2h2(v.x * inv, v.y * inv), hi = f2h2(v.z * inv, v.w * inv);
    const int i = (int)(((uint32_t)rr * group_inv) >> 16), m = rs + i, col = (kvh * group + rr - i * group) * HD + e0;
    if (out32) store_row4(out32 + (size_t)m * KBq * 16 + col, lo, hi);
    else *reinterpret_cast<uint2 *>(out + tile_unit(m, col & ~7, KBq) * 8 + (col & 4)) = make_uint2(lo, hi);
  };
#pragma unroll
  for (int m0 = 0; m0 < RT; m0 += MS) {
    if (m0 >= rtc) continue;
    __syncthreads();   // the rings, or the tiles before, have been read
#pragma unroll
    for (int rt = m0; rt < RT && rt < m0 + MS; ++rt) {
      if (rt >= rtc) continue;
      const float ll = lane_pair_sum<32>(lrun[rt]);
      const int at = (w * MS + rt - m0) * 32 + r;
      float *dst = area + at * OROW + 4 * h;
#pragma unroll
      for (int c = 0; c < VC; ++c)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<float4 *>(dst + 32 * c + 8 * g) =
              make_float4(o[rt][c][4 * g], o[rt][c][4 * g + 1], o[rt][c][4 * g + 2], o[rt][c][4 * g + 3]);
      if (h == 0) s_ml[at] = make_float2(mrun[rt], ll);
    }
    __syncthreads();
    const int rows = min(MS * 32, R - m0 * 32);
    for (int it = tid; it < rows * TPR; it += 64 * NW) {
      // eight features side by side for the result; in two halves, so that the lanes of a store lie side by side, for a partial one
      const int row = it / TPR, x = it % TPR, rr = m0 * 32 + row, e0 = nparts == 1 ? 8 * x : 4 * x, e1 = nparts == 1 ? e0 + 4 : e0 + HD / 2;
      float2 ml[NW];
      float mm = -INFINITY, lsum = 0.f, acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (int u = 0; u < NW; ++u) {
        ml[u] = s_ml[u * (MS * 32) + row];
        mm = fmaxf(mm, ml[u].x);
      }
#pragma unroll
      for (int u = 0; u < NW; ++u) {   // in wave order; a share that saw no key of this row has l = 0
        const float f = (ml[u].y == 0.f) ? 0.f : __builtin_amdgcn_exp2f(ml[u].x - mm);
        const float *p = area + (u * (MS * 32) + row) * OROW;
        const float4 a = *reinterpret_cast<const float4 *>(p + e0), c = *reinterpret_cast<const float4 *>(p + e1);
        lsum += ml[u].y * f;
        acc[0] += a.x * f; acc[1] += a.y * f; acc[2] += a.z * f; acc[3] += a.w * f;
        acc[4] += c.x * f; acc[5] += c.y * f; acc[6] += c.z * f; acc[7] += c.w * f;
      }
      if (nparts == 1) {
        write_out(rr, e0, acc, 1.0f / lsum);
      } else {
        // device-scope stores: written through to where every XCD sees them
        if (x == 0) store_dev(part_ml + ((size_t)own * Hkv + kvh) * rows_cap * 2 + rr * 2, mm, lsum);
        store_dev4(mine, rr * HD + e0, make_float4(acc[0], acc[1], acc[2], acc[3]));
        store_dev4(mine, rr * HD + e1, make_float4(acc[4], acc[5], acc[6], acc[7]));
      }
    }
  }
  if (nparts == 1) return;

  // ---- several parts: the block that draws the last ticket of its (request, kv head, rows) merges them, in part order ----
  wait_own_stores();
  __syncthreads();
  int *const s_last = reinterpret_cast<int *>(lds);
  int32_t *const tk = ticket + ((size_t)b * RTMAX + rt0) * Hkv + kvh;
  if (tid == 0) *s_last = (__hip_atomic_fetch_add(tk, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nparts - 1) ? 1 : 0;
  __syncthreads();
  if (!*s_last) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  if (tid == 0) __hip_atomic_store(tk, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next layer's launch
  const size_t base = ((size_t)d1.w * Hkv + kvh) * rows_cap, pstr = (size_t)d6.w * Hkv * rows_cap;   // d1.w: the first part of these rows
  // U parts of IT rows are fetched together: the time is that of a round trip to memory and back
  constexpr int U = 8, IT = 2, TPM = HD / 4;   // TPM: threads per row, four features each
  for (int i0 = tid; i0 < R * TPM; i0 += IT * 64 * NW) {
    float mm[IT], lsum[IT];
    float4 acc[IT];
#pragma unroll
    for (int x = 0; x < IT; ++x) {
      mm[x] = -INFINITY;
      lsum[x] = 0.f;
      acc[x] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    for (int s0 = 0; s0 < nparts; s0 += U) {
      float2 ml[IT][U];
      float4 va[IT][U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (s0 + u >= nparts) continue;   // (uniform)
#pragma unroll
        for (int x = 0; x < IT; ++x) {
          const int i = i0 + x * 64 * NW;
          if (i >= R * TPM) continue;
          const size_t prow = base + (s0 + u) * pstr;
          ml[x][u] = load_dev(part_ml + (prow + i / TPM) * 2);
          va[x][u] = load_dev4(rows_of(part_o + prow * HD), i * 4);
        }
      }
#pragma unroll
      for (int x = 0; x < IT; ++x) {
        if (i0 + x * 64 * NW >= R * TPM) continue;
        const float mold = mm[x];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (s0 + u < nparts) mm[x] = fmaxf(mm[x], ml[x][u].x);
        const float f0 = (mold == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(mold - mm[x]);
        lsum[x] *= f0;
        acc[x] = make_float4(acc[x].x * f0, acc[x].y * f0, acc[x].z * f0, acc[x].w * f0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (s0 + u >= nparts) continue;
          const float f = (ml[x][u].y == 0.f) ? 0.f : __builtin_amdgcn_exp2f(ml[x][u].x - mm[x]);
          lsum[x] += ml[x][u].y * f;
          acc[x] = make_float4(acc[x].x + va[x][u].x * f, acc[x].y + va[x][u].y * f, acc[x].z + va[x][u].z * f, acc[x].w + va[x][u].w * f);
        }
      }
    }
#pragma unroll
    for (int x = 0; x < IT; ++x) {
      const int i = i0 + x * 64 * NW;
      if (i < R * TPM) write_out4(i / TPM, (i % TPM) * 4, acc[x], 1.0f / lsum[x]);
    }
  }
}

// Size the parts from the host copies of the lengths.
int plan_attention(fsv_ctx *c, const fsv_batch *b, fsv_attn_plan *pl) {
  const fsv_model_desc &d = c->d;
  const attn_shape sh{d.head_dim, d.n_kv_heads, c->group, c->n_cus, c->attn_wave_target, c->attn_min_tpw, c->attn_w2, c->attn_w3};
  *pl = attn_schedule(sh, b->batch, b->seq_lens_host, b->draft_offsets_host);
  if (pl->waves > c->attn_wave_cap) FSV_FAIL(c, FSV_E_CAPACITY, "%d attention parts > %d the workspace holds", pl->waves, c->attn_wave_cap);
  if ((size_t)b->num_pages * d.n_kv_heads * 16 * d.head_dim * 2 > 0xFFFF0000ull)
    FSV_FAIL(c, FSV_E_UNSUPPORTED, "one layer of a KV pool must stay below 4 GiB (%d pages given)", b->num_pages);
  return FSV_OK;
}

int launch_setup(fsv_ctx *c, const fsv_batch *b, const fsv_attn_plan &pl, int M, bool rope, const void *q, hipStream_t st) {
  setup_args a;
  a.B = b->batch; a.tpw = pl.tpw; a.nw = pl.nw; a.sorted = pl.sorted; a.split = pl.split; a.group = c->group; a.w2 = c->attn_w2; a.w3 = c->attn_w3;
  a.max_pages = c->d.max_pages_per_req; a.num_pages = b->num_pages; a.grid_parts = pl.waves / c->d.n_kv_heads;
  a.tickets = b->batch * RTMAX * c->d.n_kv_heads; a.ticket = c->attn_ticket;
  a.M = M; a.half = rope ? c->d.head_dim / 2 : 1; a.V = c->d.vocab;   // without the angles: one thread per row
  a.seq_lens = b->seq_lens; a.off = b->draft_offsets; a.page_table = b->page_table;
  a.last_token = b->last_token; a.draft = b->draft_tokens; a.inv_freq = (const double *)c->inv_freq;
  a.part_prefix = c->attn_part_prefix; a.part_desc = c->attn_part_map;
  a.row_req = c->row_req; a.row_place = c->row_place; a.row_tok = c->row_tok;
  a.tab = rope ? (float *)c->rope_tab : nullptr;
  a.row_blocks = fsv_ceil_div(M * a.half, kSetupThreads);
  int q_blocks = 0;
  if (q) {
    a.H = c->d.n_heads; a.Hkv = c->d.n_kv_heads; a.hd = c->d.head_dim; a.q_vec = ((uintptr_t)q % 16 == 0) ? 1 : 0;
    a.q = (const uint16_t *)q; a.qp = (uint16_t *)c->buf_q; a.q_plane = c->q_plane_units * 8;
    q_blocks = fsv_ceil_div(M * a.H * (a.hd / 8), kSetupThreads);
  }
  hipLaunchKernelGGL(k_setup, dim3(1 + a.row_blocks + q_blocks), dim3(kSetupThreads), 0, st, a);
  FSV_HIP(c, hipGetLastError());
  return FSV_OK;
}

int launch_attention(fsv_ctx *c, const fsv_batch *b, const fsv_attn_plan &pl, size_t layer_off, float *out32, hipStream_t st) {
  const fsv_model_desc &d = c->d;
  const int group = c->group, KBq = d.n_heads * d.head_dim / 16;
  const int rows_cap = group * (d.max_gamma + 1);
  float *po = (float *)c->attn_part;
  float *pml = po + (size_t)c->attn_wave_cap * rows_cap * d.head_dim;
  uint16_t *out = (uint16_t *)c->buf_att;
  const uint16_t *kl = (const uint16_t *)b->k_pool + layer_off, *vl = (const uint16_t *)b->v_pool + layer_off;
  {
    fsv_prof_scope ps(c, st, FSV_K_ATTENTION, pl.kv_tokens * d.n_kv_heads * d.head_dim * 4.0, true);
#define FSV_ATTN_LAUNCH(HDV, RTV, NWV)                                                                                            \
  hipExtLaunchKernelGGL((k_attention<HDV, RTV, NWV>), dim3(pl.waves), dim3(64 * NWV), (attn_geo<HDV, RTV, NWV>::LDS), st, ps.start(), \
                        ps.stop(), 0, c->attn_part_map, d.n_kv_heads, group, (const char *)c->buf_q, c->q_plane_units * 16, (const char *)kl, \
                        (const char *)vl, d.max_pages_per_req, b->num_pages, b->page_table, rows_cap, po, pml, c->attn_ticket, out, KBq, out32)
    if (d.head_dim == 128) {
      if (pl.rt <= 1) { if (pl.nw == 8) FSV_ATTN_LAUNCH(128, 1, 8); else FSV_ATTN_LAUNCH(128, 1, 4); }
      else if (pl.rt == 2) FSV_ATTN_LAUNCH(128, 2, 8);
      else FSV_ATTN_LAUNCH(128, 3, 4);
    } else {
#define FSV_ATTN_NW(RTV) do { if (pl.nw == 8) FSV_ATTN_LAUNCH(64, RTV, 8); else FSV_ATTN_LAUNCH(64, RTV, 4); } while (0)
      if (pl.rt <= 1) FSV_ATTN_NW(1);
      else if (pl.rt == 2) FSV_ATTN_NW(2);
      else FSV_ATTN_NW(3);
#undef FSV_ATTN_NW
    }
#undef FSV_ATTN_LAUNCH
    FSV_HIP(c, hipGetLastError());
  }
  return FSV_OK;
}

}  // namespace

int fsv_bf16_attn_plan_host(fsv_ctx *c, const fsv_batch *b, fsv_attn_plan *pl) { return plan_attention(c, b, pl); }

int fsv_bf16_setup_launch(fsv_ctx *c, const fsv_batch *b, const fsv_attn_plan *pl, int M, bool rope, const void *q, hipStream_t st) {
  return launch_setup(c, b, *pl, M, rope, q, st);
}

int fsv_bf16_attn_launch(fsv_ctx *c, const fsv_batch *b, const fsv_attn_plan *pl, size_t layer_off, float *out32, hipStream_t st) {
  return launch_attention(c, b, *pl, layer_off, out32, st);
}

int fsv_bf16_attn_create(fsv_ctx *c) {
  const fsv_model_desc &d = c->d;
  if (const char *e = getenv("FSV_ATTN_TUNE")) {   // "fewest tiles per part[,w2,w3]": measurement knob
    int mt = 0, w2 = 0, w3 = 0;
    const int n = sscanf(e, "%d,%d,%d", &mt, &w2, &w3);
    if (n >= 1 && mt >= 8 && mt <= 256) c->attn_min_tpw = mt;
    if (n == 3 && w2 >= 16 && w2 <= 64 && w3 >= w2 && w3 <= 96) { c->attn_w2 = w2; c->attn_w3 = w3; }
  }
  c->attn_wave_target = c->n_cus;
  c->attn_wave_cap = 4 * c->attn_wave_target + 2 * d.max_batch * d.n_kv_heads;  // multi-round schedules: see attn_schedule.h
  const int rows_cap = c->group * (d.max_gamma + 1);
  c->attn_part_bytes = (size_t)c->attn_wave_cap * rows_cap * (d.head_dim + 2) * 4;
  auto zalloc = [&](void **p, size_t bytes) -> int {
    FSV_HIP(c, hipMalloc(p, bytes));
    FSV_HIP(c, hipMemset(*p, 0, bytes));
    return FSV_OK;
  };
  int rc;
#define FSV_ATTN_ATTR(HDV, RTV, NWV)                                                                  \
  FSV_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void *>(&k_attention<HDV, RTV, NWV>),         \
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (attn_geo<HDV, RTV, NWV>::LDS)))
  FSV_ATTN_ATTR(128, 1, 8); FSV_ATTN_ATTR(128, 2, 8); FSV_ATTN_ATTR(128, 3, 4);
  FSV_ATTN_ATTR(64, 1, 8); FSV_ATTN_ATTR(64, 2, 8); FSV_ATTN_ATTR(64, 3, 8); FSV_ATTN_ATTR(128, 1, 4);
  FSV_ATTN_ATTR(64, 1, 4); FSV_ATTN_ATTR(64, 2, 4); FSV_ATTN_ATTR(64, 3, 4);
#undef FSV_ATTN_ATTR
  if ((rc = zalloc((void **)&c->attn_ticket, sizeof(int32_t) * (size_t)d.max_batch * RTMAX * d.n_kv_heads))) return rc;
  if ((rc = zalloc(&c->attn_part, c->attn_part_bytes))) return rc;
  if ((rc = zalloc((void **)&c->attn_part_prefix, sizeof(int32_t) * (d.max_batch + 1)))) return rc;
  if ((rc = zalloc((void **)&c->attn_part_map, sizeof(int32_t) * kDescInts * (c->attn_wave_cap / d.n_kv_heads + 1)))) return rc;
  return FSV_OK;
}
