// Vocabulary-wide softmax statistics, acceptance tests, residual / bonus token selection and KV
// rollback: the accept / reject part of Alg. 2 step 2 (greedy form as printed there; for
// temperature > 0 the speculative-sampling rule that keeps the output law equal to the target's,
// Sec. II and Regime B of Sec. V) and the rollback of Sec. IV-C.
//
// Two launches, both streaming logits from HBM:
//   k_row_stats   grid (chunks / 4, row of the request, request)   one pass over every logits row: per chunk
//                 (max, sum e^{(l-max)/T}) or the argmax
//   k_decide      grid (sub-blocks / 4, requests)   every block first repeats the request's acceptance tests (row
//                 statistics combined, two gathered scalars per draft: cheap, and it saves a launch and a round trip
//                 through memory), then the blocks of a request stream the one row its token is drawn from (and the
//                 draft-law row) into the masses of its 2048-id sub-blocks; the block that finishes last (an integer
//                 ticket per request) locates the sub-block and the id by inverse CDF, emits the outputs and rolls back
// plus, when a request asks for a top-k / nucleus (top-p) cut of the target law, between the two: k_cut, one block per row
// that finds the row's cut in one or two passes over it and a short list of candidates; on bf16 logits two launches of
// k_cut_window before it, which settle the rows whose cut lies near their maximum in one pass.
// Rows are addressed as (request, row within the request), so the step needs no row map.  Every floating-point sum is
// taken in a fixed order (the ticket only decides WHICH block adds the sub-block masses up: three consecutive ones per lane, then
// a scan over the lanes); the only other atomics are on integers in the histograms of the cuts, whose result does not depend on
// their order.
#include <limits.h>
#include <math.h>
#include <stdlib.h>
#include <type_traits>
#include <mutex>

#include "fsv_internal.h"

namespace {

constexpr double kLog2e = 1.4426950408889634074;

// e^{d / T} for d <= 0 as 2^{d * k}, k = log2(e) / T carried as a float pair (k_hi + k_lo) so that its rounding does not
// tilt large against small terms; the product is formed in fp32 (the error it leaves is relative to a term's own size,
// 1e-7 for the terms that carry the mass) and 2^z comes from the transcendental unit.  Vocabulary-wide sums are bound by
// this arithmetic, not by HBM, if it is done in fp64.
struct exp_scale {
  float hi, lo;
};
__device__ inline exp_scale make_exp_scale(double k) {
  exp_scale s;
  s.hi = (float)k;
  s.lo = (float)(k - (double)s.hi);
  return s;
}
__device__ inline float exp_scaled(float d, exp_scale k) {
  const float z = fmaf(d, k.lo, d * k.hi);
  return __builtin_amdgcn_exp2f(fmaxf(z, -160.f));  // 0 from there on; -inf and NaN (a chunk that is all -inf) end there too
}

// Sixteen bytes at a time from any row: a vocabulary that is no multiple of four or eight leaves the rows at 4- or 2-byte boundaries,
// and a load of four dwords takes those as they come (one element per load instead: 576 rows x 50257 fp32, top-k 50, 267 us a call;
// 75 like this, bf16 with top-p 0.9 157 and 77).
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));

template <typename LT>
struct loader;

template <>
struct loader<uint16_t> {  // bf16 bit patterns
  // eight ids, all in range: no bounds logic, so that a run of these loads is
  // issued back to back (a branch per load makes the wave wait for each load before the next)
  static __device__ inline void load8_fast(const uint16_t *row, int i0, float (&v)[8]) {
    const u32x4_any w = *reinterpret_cast<const u32x4_any *>(row + i0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[2 * j] = __uint_as_float(w[j] << 16);
      v[2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u);
    }
  }
  static __device__ inline void load8(const uint16_t *row, int i0, int V, float fill, float (&v)[8]) {
    if (i0 + 8 <= V) {
      load8_fast(row, i0, v);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = (i0 + j < V) ? __uint_as_float((uint32_t)row[i0 + j] << 16) : fill;
    }
  }
};

template <>
struct loader<float> {
  static __device__ inline void load8_fast(const float *row, int i0, float (&v)[8]) {
    const f32x4_any a = *reinterpret_cast<const f32x4_any *>(row + i0), b = *reinterpret_cast<const f32x4_any *>(row + i0 + 4);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = a[j];
      v[4 + j] = b[j];
    }
  }
  static __device__ inline void load8(const float *row, int i0, int V, float fill, float (&v)[8]) {
    if (i0 + 8 <= V) {
      load8_fast(row, i0, v);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = (i0 + j < V) ? row[i0 + j] : fill;
    }
  }
};

// Inclusive scan of one double per thread over a 256-thread block, fixed order.  s_w: 4 doubles of LDS.
__device__ inline double block_incl_scan(double v, double *s_w, double *total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    double t = __shfl_up(v, off, 64);
    if (lane >= off) v += t;
  }
  __syncthreads();  // protect s_w from a previous use
  if (lane == 63) s_w[w] = v;
  __syncthreads();
  double pre = 0.0, tot = 0.0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (i < w) pre += s_w[i];
    tot += s_w[i];
  }
  if (total) *total = tot;
  return v + pre;
}

__global__ void k_build_rows(int B, const int32_t *seq_lens, const int32_t *off, int32_t *row_req, int32_t *row_pos) {
  int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  int o = off[b], g = off[b + 1] - o, rs = o + b;
  int L = seq_lens ? seq_lens[b] : 0;
  for (int i = 0; i <= g; ++i) {
    row_req[rs + i] = b;
    row_pos[rs + i] = L + i;
  }
}

// One wave per 8192-id chunk of a row: all of the chunk's loads are issued before the first use (sixteen 16-byte loads
// per lane for bf16), the maximum and the sum are reduced over the wave, and no LDS or barrier is
// involved; waves are independent, so a compute unit keeps a dozen of them streaming.
// grid = (chunks / 4, largest gamma of the batch + 1, requests): row i of request b is logits row off[b] + b + i.
// LAW: the statistics feed k_draft_law: greedy requests need none, and with drafts_only neither does a request's last row.
template <typename LT, bool LAW = false>
__global__ __launch_bounds__(256) void k_row_stats(const int32_t *__restrict__ off, const float *__restrict__ temperature,
                                                   const LT *__restrict__ logits, int V, int nc, float *__restrict__ pmax,
                                                   double *__restrict__ psum, int32_t *__restrict__ parg, int drafts_only = 0) {
  constexpr int P = FSV_CHUNK / 512;  // passes of 64 lanes x 8 ids
  const int tid = threadIdx.x, lane = tid & 63, c = blockIdx.x * 4 + (tid >> 6), bq = blockIdx.z;
  if (c >= nc) return;
  const int o = off[bq];
  if ((int)blockIdx.y > off[bq + 1] - o - (LAW ? drafts_only : 0)) return;   // the request has fewer rows
  if (LAW && !(temperature[bq] > 0.f)) return;
  const int r = o + bq + blockIdx.y;
  const LT *row = logits + (size_t)r * V;
  const float T = temperature[bq];
  float v[P][8];
  const int base = c * FSV_CHUNK + lane * 8;
  if ((c + 1) * FSV_CHUNK <= V) {  // wave-uniform: every chunk but a ragged last one
#pragma unroll
    for (int p = 0; p < P; ++p) loader<LT>::load8_fast(row, base + p * 512, v[p]);
  } else {
    // The ragged last chunk, with its loads issued together like the others': groups of eight beyond the row load its last eight ids
    // instead and become -inf, and the group the row ends in (V no multiple of eight) is then loaded id by id.
    if (V >= 8) {
#pragma unroll
      for (int p = 0; p < P; ++p) loader<LT>::load8_fast(row, min(base + p * 512, V - 8), v[p]);
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int j = 0; j < 8; ++j) v[p][j] = (base + p * 512 + 8 <= V) ? v[p][j] : -INFINITY;
    }
    if (V < 8 || (V & 7)) {
#pragma unroll
      for (int p = 0; p < P; ++p)
        if (base + p * 512 < V && base + p * 512 + 8 > V) loader<LT>::load8(row, base + p * 512, V, -INFINITY, v[p]);
        else if (V < 8) {
#pragma unroll
          for (int j = 0; j < 8; ++j) v[p][j] = -INFINITY;
        }
    }
  }
  // A row needs either the argmax (greedy, T = 0) or the sum of exponentials (T > 0), never both; the vocabulary-wide
  // pass is bound by its arithmetic as soon as it carries more than a handful of operations per id.
  float mx = -INFINITY;
  int ai = INT_MAX;
  double sum = 0.0;
  if (T > 0.f) {
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int j = 0; j < 8; ++j) mx = fmaxf(mx, v[p][j]);
    mx = lanes_max(mx);
    if (mx > -INFINITY) {  // wave-uniform; an all -inf chunk carries no mass
      // 2^{(l - max) k} with k in fp32: its rounding moves a term by 6e-8 of its own exponent, nothing for the terms
      // that carry the sum; ids beyond the vocabulary were loaded as -inf and come out as 0
      const float k = (float)(kLog2e / (double)T);
#pragma unroll
      for (int p = 0; p < P; ++p) {  // eight terms at a time in fp32, the groups in fp64
        float part = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) part += __builtin_amdgcn_exp2f((v[p][j] - mx) * k);
        sum += (double)part;
      }
      sum = lanes_sum(sum);
    } else if (LAW) {   // a NaN makes the whole law NaN, also where nothing else in its chunk carries mass
      bool nan = false;
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int j = 0; j < 8; ++j) nan |= v[p][j] != v[p][j];
      if (__any(nan)) sum = __longlong_as_double(0x7FF8000000000000ll);
    }
  } else {
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (v[p][j] > mx) { mx = v[p][j]; ai = base + p * 512 + j; }   // ids ascend with (p, j): the first maximum stays
    // wave (max, lowest id attaining it)
    lanes_argmax(mx, ai);
  }
  if (lane == 0) {
    pmax[(size_t)r * nc + c] = mx;
    psum[(size_t)r * nc + c] = sum;
    parg[(size_t)r * nc + c] = ai;
  }
}

// The draft model's laws q = softmax(z / T_b), fp32, from its logits z and the chunk statistics k_row_stats left: every
// block combines the row's chunks by itself (a few hundred bytes; chunks in lanes, fixed tree) and writes the law
// of its LAW_IDS ids.  Two streaming passes over z (the second finds most of it in the memory-side cache) and one over q is
// the bound.  Measured for 71 rows x 128256 (8B vocabulary, 55 drafts): 10 us for the statistics and 11 us here, against
// 359 us for one block per row that went over the row three times, one value per load.
// grid = (ceil(V / LAW_IDS), largest gamma + 1 - drafts_only, requests); all_rows 0: the laws the verification call takes
// (draft i+1 of request b from row i < gamma_b, written to q row off[b] + i); 1: every row, to its own index.
constexpr int LAW_IDS = 4096;   // 256 threads x four loads of four ids
__global__ __launch_bounds__(256) void k_draft_law(const float *__restrict__ z, int V, int nc, const int32_t *__restrict__ off,
                                                   const float *__restrict__ temperature, const float *__restrict__ pmax,
                                                   const double *__restrict__ psum, int all_rows, float *__restrict__ q) {
  const int tid = threadIdx.x, lane = tid & 63, b = blockIdx.z, o = off[b], i = blockIdx.y;
  if (i > off[b + 1] - o - (all_rows ? 0 : 1)) return;
  const float T = temperature[b];
  if (!(T > 0.f)) return;   // greedy requests need no law
  const int r = o + b + i, i0 = blockIdx.x * LAW_IDS + tid * 4;
  const float *zr = z + (size_t)r * V;
  float *qr = q + (size_t)(all_rows ? r : o + i) * V;
  float v[4][4];
  const bool fast = (int)(blockIdx.x + 1) * LAW_IDS <= V;   // block-uniform
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if (fast) {
      const f32x4_any a = *reinterpret_cast<const f32x4_any *>(zr + i0 + u * 1024);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[u][j] = a[j];
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[u][j] = (i0 + u * 1024 + j < V) ? zr[i0 + u * 1024 + j] : 0.f;
    }
  }
  float mx = -INFINITY;
  for (int c = lane; c < nc; c += 64) mx = fmaxf(mx, pmax[(size_t)r * nc + c]);
  mx = lanes_max(mx);
  const double invT = 1.0 / (double)T;
  double sum = 0.0;
  for (int c = lane; c < nc; c += 64) {
    const float pm = pmax[(size_t)r * nc + c];
    sum += psum[(size_t)r * nc + c] * ((pm == mx) ? 1.0 : exp(((double)pm - (double)mx) * invT));
  }
  sum = lanes_sum(sum);
  const float k = (float)(kLog2e / (double)T), inv = (float)(1.0 / sum);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[u][j] = __builtin_amdgcn_exp2f((v[u][j] - mx) * k) * inv;
    if (fast) {
      *reinterpret_cast<f32x4_any *>(qr + i0 + u * 1024) = (f32x4_any){v[u][0], v[u][1], v[u][2], v[u][3]};
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (i0 + u * 1024 + j < V) qr[i0 + u * 1024 + j] = v[u][j];
    }
  }
}

// ---- top-k / nucleus (top-p) cut of the target law ----------------------------------------------------------
// The cut keeps every token whose logit is at least the cut value: for top-k the value of the top_k-th most probable
// token, for top-p the largest value for which the kept mass reaches top_p of what the top-k cut left (tokens tied at
// the cut value are all kept, so the set does not depend on an order among ties).  Masses are integers in 2^-40 fixed point
// throughout, so that no sum depends on the order of its terms.
__device__ inline uint32_t okey(float f) {  // monotone: a < b  <=>  okey(a) < okey(b)
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

constexpr int FSV_NUC_BINS = 2048;
constexpr double kNucScale = 1099511627776.0;  // 2^40
constexpr int kCutThreads = 1024;
constexpr int kCutBins = 8192;
constexpr float kCutBinsPerLog2 = 192.0f;   // bins per factor of two of the probability: they span 42.7 factors of two
constexpr int kCutList = 2 * kCutThreads;   // candidates the last step can hold

__device__ inline unsigned long long nuc_mass(float d, exp_scale k) {
  return (unsigned long long)((double)exp_scaled(d, k) * kNucScale + 0.5);
}

// What the passes over a row hand to each other, in LDS.
struct cut_state {
  float m;                                   // row maximum
  float vlow, vtop;                          // smallest candidate, smallest value above them
  int n, found, bad;                         // candidates, selection done, a NaN in the row
  uint32_t bin_lo, bin_hi, before, upto;     // bins the cut can lie in, running sum before the first and up to the last
  uint32_t kkey, cut;
  unsigned long long kmass, kept, acc, total;
  double S;                                  // normaliser from the row statistics, in units of the maximum's probability
  uint32_t lo, hi, cabove;                   // narrowing passes: the interval of keys left, tokens and mass above it
  int last;                                  // it is one key
  unsigned long long above;
  uint32_t w32[kCutThreads / 64];
  unsigned long long w64[kCutThreads / 64], t64[kCutThreads / 64];
};

// f(first id, eight values) over the block's share of a row, ids beyond the vocabulary as -inf.  Rounds of U loads per
// thread are issued back to back, without a branch between them (a branch per load makes the wave wait for each load
// before the next); the U loads of a round lie a U-th of the whole rounds apart, so that the first round is a sample of the
// vocabulary.  after_round(r, values of the round) is met by every thread of the block after each whole round.
__device__ __host__ inline int whole_rounds(int V) { return V / (4 * kCutThreads * 8); }
template <typename LT, typename F, typename G>
__device__ inline void over_row(const LT *row, int V, int tid, F &&f, G &&after_round) {
  constexpr int U = 4, STEP = kCutThreads * 8;
  const int R = whole_rounds(V);
  for (int r = 0; r < R; ++r) {
    const int base = r * STEP + tid * 8;
    float v[U][8];
#pragma unroll
    for (int u = 0; u < U; ++u) loader<LT>::load8_fast(row, base + u * R * STEP, v[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) f(base + u * R * STEP, v[u]);
    after_round(r, v);
  }
  // the rest, less than a round, with its loads issued together too: threads beyond the row load its last eight ids and leave them out
  const int rest = R * U * STEP + tid * 8;
  if (R * U * STEP >= V) return;
  float v[U][8];
  if (V >= 8) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if ((R * U + u) * STEP < V) loader<LT>::load8_fast(row, min(rest + u * STEP, V - 8), v[u]);   // (uniform)
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i0 = rest + u * STEP;
    if (i0 >= V) continue;
    if (i0 + 8 > V) loader<LT>::load8(row, i0, V, -INFINITY, v[u]);
    f(i0, v[u]);
  }
}

// The general way: passes over the row that narrow an interval of keys, 2048 bins of equal width each time, until a bin is a
// single key (16 bits wide for bf16 logits, whose keys have no information below).  A pass builds a histogram of the mass (and,
// for top-k, the count) per bin in LDS, and a scan from the top picks the bin at which the kept mass (count) crosses.  From the
// whole range these are digits of 11, 11 and 10 bits.  `whole` = false (by mass): the cut is expected in [lo, hi], the first pass
// adds up the mass above, st->total is known; false is returned if the cut does not lie there.  These passes also keep the lowest
// and highest key of each bin (in hcnt): tied tokens, and a bin of one token, need no further pass.
// COUNT selects by count and leaves kkey / kmass; by mass, among the keys from lowkey on, leaves cut / kept / acc / total.
template <typename LT, bool COUNT>
__device__ inline bool cut_narrow(const LT *row, int V, float m, exp_scale k, uint32_t lo, uint32_t hi, bool whole, uint32_t lowkey,
                                  int tk, float tp, unsigned long long *hist, uint32_t *hcnt, cut_state *st) {
  constexpr int LAST = (sizeof(LT) == 2) ? 16 : 0;   // widest bin that holds one key
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  for (bool first = true;; first = false) {
    const uint32_t span = hi - lo;
    int shift = span ? 32 - __clz((int)span) - 11 : 0;
    if (shift < 0) shift = 0;
    if ((hi >> shift) - (lo >> shift) >= (uint32_t)FSV_NUC_BINS) ++shift;   // (an interval that does not begin on a bin's edge)
    const uint32_t base = lo >> shift, from = max(lo, lowkey);
    const bool ends = !COUNT && !whole && shift > LAST, sum_above = first && !whole;
    for (int i = tid; i < FSV_NUC_BINS; i += kCutThreads) {
      hist[i] = 0ull;
      if (COUNT) hcnt[i] = 0u;
      if (ends) { hcnt[i] = ~0u; hcnt[FSV_NUC_BINS + i] = 0u; }
    }
    __syncthreads();
    double above = 0.0;   // exact: a whole number below 2^53
    over_row<LT>(row, V, tid, [&](int i0, const float(&v)[8]) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (i0 + j >= V) continue;   // ids beyond the vocabulary are not tokens (they would count for top-k)
        if (COUNT && v[j] != v[j]) continue;   // nor is a NaN one, which carries no mass
        const uint32_t key = okey(v[j]);
        if (key - from > hi - from) {
          if (!COUNT && sum_above && key > hi) above += floor((double)exp_scaled(v[j] - m, k) * kNucScale + 0.5);
          continue;
        }
        const unsigned long long q = nuc_mass(v[j] - m, k);
        const uint32_t bin = (key >> shift) - base;
        if (q) atomicAdd(&hist[bin], q);
        if (COUNT) atomicAdd(&hcnt[bin], 1u);
        if (ends) { atomicMin(&hcnt[bin], key); atomicMax(&hcnt[FSV_NUC_BINS + bin], key); }
      }
    }, [](int, const auto &) {});
    if (sum_above) {
      unsigned long long ta = (unsigned long long)above;
      ta = lanes_sum(ta);
      if (lane == 0) st->w64[w] = ta;
    }
    __syncthreads();
    if (tid < 64) {
      // lane l owns the 32 bins below (64 - l) * 32, the highest keys in lane 0: masses above each lane's group
      constexpr int PER = FSV_NUC_BINS / 64;
      unsigned long long mine = 0ull, above0 = first ? 0ull : st->above;
      uint32_t minec = 0u;
      const int top = (63 - lane) * PER + PER - 1;
#pragma unroll 8
      for (int i = 0; i < PER; ++i) {
        mine += hist[top - i];
        if (COUNT) minec += hcnt[top - i];
      }
      if (sum_above)
        for (int i = 0; i < kCutThreads / 64; ++i) above0 += st->w64[i];
      unsigned long long incl = mine;
      uint32_t inclc = minec;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long t = __shfl_up(incl, o, 64);
        const uint32_t tc = __shfl_up(inclc, o, 64);
        if (lane >= o) { incl += t; inclc += tc; }
      }
      const unsigned long long before = above0 + (incl - mine);   // mass strictly above this lane's group
      const uint32_t beforec = (first ? 0u : st->cabove) + (inclc - minec);
      const unsigned long long total = (first && whole) ? __shfl(incl, 63, 64) : st->total;
      const double target = (double)tp * (double)total;
      const bool crosses = COUNT ? (beforec + minec >= (uint32_t)tk) : ((double)(before + mine) >= target);
      const unsigned long long ballot = __ballot(crosses);
      if (sum_above && (!ballot || (double)above0 >= target)) {
        if (lane == 0) st->found = 0;
      } else {
        // the whole range always has a crossing (tk < V tokens are counted; the last lane holds the total mass), a bin is chosen
        // because it crosses; the guard only keeps the index in range
        const int pick_lane = ballot ? (int)__builtin_ctzll(ballot) : 63;
        if (lane == pick_lane) {
          unsigned long long acc = before;
          uint32_t accc = beforec;
          int bin = top - (PER - 1);
#pragma unroll 1
          for (int i = 0; i < PER; ++i) {
            const unsigned long long hbin = hist[top - i];
            const bool hit = COUNT ? (accc + hcnt[top - i] >= (uint32_t)tk) : ((double)(acc + hbin) >= target);
            if (hit || i == PER - 1) { bin = top - i; break; }
            acc += hbin;
            if (COUNT) accc += hcnt[top - i];
          }
          const uint32_t edge = (base + (uint32_t)bin) << shift;
          st->found = 1;
          st->lo = ends ? hcnt[bin] : edge;
          st->hi = ends ? hcnt[FSV_NUC_BINS + bin] : min(hi, edge + ((1u << shift) - 1u));
          st->above = acc;
          st->cabove = accc;
          st->last = (shift <= LAST || (ends && st->lo == st->hi)) ? 1 : 0;
          if (!COUNT) st->total = total;
          if (st->last) {
            const uint32_t key = ends ? st->lo : edge;
            if (COUNT) { st->kkey = key; st->kmass = acc + hist[bin]; }
            else { st->cut = key; st->kept = acc + hist[bin]; st->acc = acc; }
          }
        }
      }
    }
    __syncthreads();
    if (!st->found || st->last) break;
    lo = st->lo;
    hi = st->hi;
  }
  return st->found != 0;
}

// First bins at which the running sum of the bins reaches x0 and x1, to bin_lo and bin_hi (kCutBins: never).
__device__ inline void cut_find_bins(const uint32_t *hist, uint32_t x0, uint32_t x1, cut_state *st) {
  constexpr int PER = kCutBins / kCutThreads;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid == 0) st->bin_lo = st->bin_hi = kCutBins;
  uint32_t h[PER], incl = 0u;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    h[i] = hist[PER * tid + i];
    incl += h[i];
  }
  uint32_t run = incl;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  run = incl - run;
  if (lane == 63) st->w32[w] = incl;
  __syncthreads();
  for (int i = 0; i < w; ++i) run += st->w32[i];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const uint32_t before = run;
    run += h[i];
    if (before < x0 && x0 <= run) { st->bin_lo = PER * tid + i; st->before = before; }
    if (before < x1 && x1 <= run) { st->bin_hi = PER * tid + i; st->upto = run; }
  }
  __syncthreads();
}

// The value a key stands for.
__device__ inline float okey_value(uint32_t key) { return __uint_as_float((key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key); }

// The cuts on bf16 logits, in ONE pass, whenever they lie near the row maximum: only the W highest values of the key's top 11
// bits, at and below the row maximum's, get histogram bins, 32 each (a bf16 key has five bits below, so a bin is one key and
// needs no list): W = 4 is one binade of the logit, tried first, W = 8 two, for the rows the first leaves (done[r] = 0).  Every
// other token is dismissed by one comparison: no exponential, no LDS add.  top_p is measured against the normaliser of the
// statistics pass, or the mass the top-k cut kept.  Rows neither settles go on to k_cut (done[r] = 2 keeps the second window off
// a row that would most likely fail there: under a normal law of the logits the mass below two binades is about 0.25 .. 0.55 of
// the square of the mass below one; the lower factor, since a vain second window costs 65 us and k_cut for few rows 60).
// Measured for 584 rows x 152064, logits N(0, 3), all launches of a cut: T = 0.7, top-p 0.9 54 us (first window); T = 1.0 128 and
// T = 0.8, top-p 0.95 127 (second; 199 and 188 with the first window and k_cut alone); T = 1.0, top-p 0.99 257 (k_cut after the
// first); top-k 50 58, 1000 99, 5000 130 (k_cut alone: 76, 141, 363); top-k 50 then top-p 0.9 61.
template <int W, bool FIRST>
__global__ __launch_bounds__(1024) void k_cut_window(const uint16_t *__restrict__ logits, int V, int nc,
                                                      const int32_t *__restrict__ off,
                                                      const float *__restrict__ temperature,
                                                      const float *__restrict__ top_p, const int32_t *__restrict__ top_k,
                                                      const float *__restrict__ pmax, const double *__restrict__ psum,
                                                      uint32_t *__restrict__ nuc_key, double *__restrict__ nuc_S,
                                                      int32_t *__restrict__ nuc_near, int32_t *__restrict__ done) {
  constexpr int FB = 32;
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  if ((int)blockIdx.x > off[b + 1] - off[b]) return;
  const int r = off[b] + b + blockIdx.x;
  if (!FIRST && done[r]) return;   // settled by the narrower window, or left to k_cut
  const float T = temperature[b], tp = top_p ? top_p[b] : 1.f;
  const int tk = top_k ? top_k[b] : 0;
  const bool use_k = T > 0.f && tk > 0 && tk < V, use_p = T > 0.f && tp < 1.f;
  if (!use_k && !use_p) {
    if (tid == 0) { nuc_key[r] = 0u; nuc_S[r] = -1.0; nuc_near[r] = 0; done[r] = 1; }
    return;
  }
  __shared__ unsigned long long hist[W * FB];
  __shared__ uint32_t hcnt[W * FB];
  __shared__ float s_m;
  __shared__ double s_total;
  for (int i = tid; i < W * FB; i += 1024) {
    hist[i] = 0ull;
    hcnt[i] = 0u;
  }
  if (tid < 64) {   // the row's maximum and normaliser from the per-chunk statistics (chunks in lanes, 64 at a time)
    float mx = -INFINITY;
    for (int c = lane; c < nc; c += 64) mx = fmaxf(mx, pmax[(size_t)r * nc + c]);
    mx = lanes_max(mx);
    double term = 0.0;
    const double invT = 1.0 / (double)T;
    for (int c = lane; c < nc; c += 64) {
      const float pm = pmax[(size_t)r * nc + c];
      term += psum[(size_t)r * nc + c] * ((pm == mx) ? 1.0 : exp(((double)pm - (double)mx) * invT));
    }
    term = lanes_sum(term);
    if (lane == 0) {
      s_m = mx;
      s_total = term * kNucScale;
    }
  }
  __syncthreads();
  const float m = s_m;
  const exp_scale k = make_exp_scale(kLog2e / (double)T);
  const uint32_t d0 = okey(m) >> 21;                              // the row's highest digit
  const uint16_t *row = logits + (size_t)r * V;
  // the lowest value inside the window: the value whose key is the window's lowest key
  const uint32_t wlow = (d0 >= (uint32_t)(W - 1)) ? ((d0 - (uint32_t)(W - 1)) << 21) : 0u;
  float vlow = okey_value(wlow);
  if (!(vlow == vlow)) vlow = (wlow & 0x80000000u) ? INFINITY : -INFINITY;   // (keys of NaN patterns: only when the row holds them)
  // Eight ids of a thread at a time: a bit per id that falls into the window, then the wave works through the set bits,
  // every lane on its next one, so that the exponential and the atomics are issued about as often as the busiest lane
  // has window tokens among its eight, not once per id.
  auto add8 = [&](int i0, const float (&v)[8], auto in_range) {
    uint32_t mask = 0u;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      bool ok = v[j] >= vlow;   // the key order is the order of the values: one comparison places a token
      if (!decltype(in_range)::value) ok = ok && (i0 + j < V);   // ids beyond the vocabulary are not tokens
      mask |= ok ? (1u << j) : 0u;
    }
    while (__any(mask != 0u)) {
      if (mask) {
        const int j = __builtin_ctz(mask);
        mask &= mask - 1u;
        const float a0 = (j & 1) ? v[1] : v[0], a1 = (j & 1) ? v[3] : v[2], a2 = (j & 1) ? v[5] : v[4], a3 = (j & 1) ? v[7] : v[6];
        const float b0 = (j & 2) ? a1 : a0, b1 = (j & 2) ? a3 : a2;
        const float val = (j & 4) ? b1 : b0;
        const uint32_t key = okey(val);
        const unsigned long long q = (unsigned long long)((double)exp_scaled(val - m, k) * kNucScale + 0.5);
        const uint32_t idx = (d0 - (key >> 21)) * FB + ((key >> 16) & (FB - 1));
        if (q) atomicAdd(&hist[idx], q);
        if (use_k) atomicAdd(&hcnt[idx], 1u);
      }
    }
  };
  constexpr int U = 4, STEP = 1024 * 8;
  // Most of the first round inside the window (logits far from zero, close together): a top-k that k_cut finds in one pass is
  // left to it.
  const bool sample = FIRST && use_k && V >= U * STEP && 6l * tk <= kCutList;
  int base = tid * 8;
  {
    for (; base + (U - 1) * STEP + 8 <= V; base += U * STEP) {
      float v[U][8];
#pragma unroll
      for (int u = 0; u < U; ++u) loader<uint16_t>::load8_fast(row, base + u * STEP, v[u]);
      if (sample && base < STEP) {
        int seen = 0;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int j = 0; j < 8; ++j) seen += v[u][j] >= vlow ? 1 : 0;
        if (__syncthreads_count(seen > 4) > 512) {
          if (tid == 0) done[r] = 2;
          return;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) add8(base + u * STEP, v[u], std::true_type{});
    }
  }
  if (base < V) {   // the rest, at most a round: as in over_row
    float v[U][8];
    if (V >= 8) {
#pragma unroll
      for (int u = 0; u < U; ++u) loader<uint16_t>::load8_fast(row, min(base + u * STEP, V - 8), v[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i0 = base + u * STEP;
      if (i0 >= V) continue;
      if (i0 + 8 > V) loader<uint16_t>::load8(row, i0, V, -INFINITY, v[u]);
      add8(i0, v[u], std::false_type{});
    }
  }
  __syncthreads();
  if (tid >= 64) return;
  // lane l < W owns the window's digit d0 - l: the highest keys in lane 0
  unsigned long long mine = 0ull;
  uint32_t minec = 0u;
  if (lane < W) {
#pragma unroll
    for (int f = 0; f < FB; ++f) {
      mine += hist[lane * FB + f];
      minec += hcnt[lane * FB + f];
    }
  }
  unsigned long long incl = mine;
  uint32_t inclc = minec;
#pragma unroll
  for (int o2 = 1; o2 < W; o2 <<= 1) {
    const unsigned long long t = __shfl_up(incl, o2, 64);
    const uint32_t tc = __shfl_up(inclc, o2, 64);
    if (lane >= o2) { incl += t; inclc += tc; }
  }
  const unsigned long long before = incl - mine;   // mass strictly above this lane's digit
  const uint32_t beforec = inclc - minec;
  const bool digit = lane < W && lane <= (int)d0;   // digits below zero do not exist
  double total = s_total, target = 0.0;
  uint32_t cut = 0u;
  unsigned long long kept = 0ull, acc = 0ull;   // mass down to and with the cut, and above it
  // the key in the chosen lane's digit, from the top, at which the running count or mass crosses; to every lane
  auto select = [&](unsigned long long lanes, bool by_count) {
    const int from = (int)__builtin_ctzll(lanes);
    acc = before;
    uint32_t accc = beforec;
    int fsel = 0;
    if (lane == from) {
      for (int f = FB - 1; f >= 0; --f) {
        const unsigned long long hbin = hist[lane * FB + f];
        const bool hit = by_count ? (accc + hcnt[lane * FB + f] >= (uint32_t)tk) : ((double)(acc + hbin) >= target);
        if (hit || f == 0) { fsel = f; break; }
        acc += hbin;
        accc += hcnt[lane * FB + f];
      }
      kept = acc + hist[lane * FB + fsel];
    }
    cut = ((d0 - (uint32_t)from) << 21) | ((uint32_t)__shfl(fsel, from, 64) << 16);
    kept = __shfl(kept, from, 64);
    acc = __shfl(acc, from, 64);
  };
  bool settled = true;
  if (use_k) {
    const unsigned long long ballot = __ballot(digit && beforec + minec >= (uint32_t)tk);
    settled = ballot != 0ull;
    if (settled) {
      select(ballot, true);
      total = (double)kept;   // top-p works on what the top-k cut kept
    }
  }
  settled = settled && (!use_p || total > 0.0);   // (not top-p with a NaN or an infinite maximum)
  if (settled && use_p) {
    target = (double)tp * total;
    const unsigned long long ballot = __ballot(digit && (double)(before + mine) >= target);
    settled = ballot != 0ull;
    if (settled) select(ballot, false);
  }
  const unsigned long long inside = __shfl(incl, W - 1, 64);
  if (lane != 0) return;
  if (!settled) {   // a cut lies below the window, or the row is out of the ordinary (2: nothing for the wider window either)
    const double outside = 1.0 - (double)inside / total;
    const bool wider = use_k || (total > 0.0 && 0.25 * outside * outside <= 1.0 - (double)tp);
    done[r] = (FIRST && wider) ? 0 : 2;
    return;
  }
  done[r] = 1;
  nuc_key[r] = cut;
  nuc_S[r] = (double)kept / kNucScale;
  nuc_near[r] = (use_p && fmin(target - (double)acc, (double)kept - target) < 1e-6 * total) ? 1 : 0;
}

// What k_row_stats leaves for a row, by the waves of one block: the same chunks, the same sums in the same order, but a quarter of a
// chunk's loads at a time and a second trip (from the cache) for the sums, so that it fits this kernel's registers.  A function of its own:
// inlined it spilled 295 registers; called, k_cut<float, true> saves four registers and has a stack of 384 bytes a lane for it (112, unused,
// are set aside in k_cut<float, false>).
template <typename LT>
__device__ __attribute__((noinline)) void row_stats_by_block(const LT *row, int V, int nc, float T, float *pm, double *ps, int32_t *pa, int w, int lane) {
  constexpr int P = FSV_CHUNK / 512;
  for (int c = w; c < nc; c += kCutThreads / 64) {
    const int base = c * FSV_CHUNK + lane * 8;
    const bool whole = (c + 1) * FSV_CHUNK <= V;   // wave-uniform
    auto quarter = [&](int p0, float(&v)[P / 4][8]) {
      if (whole) {
#pragma unroll
        for (int p = 0; p < P / 4; ++p) loader<LT>::load8_fast(row, base + (p0 + p) * 512, v[p]);
      } else {
#pragma unroll
        for (int p = 0; p < P / 4; ++p) loader<LT>::load8(row, base + (p0 + p) * 512, V, -INFINITY, v[p]);
      }
    };
    float mx = -INFINITY, v[P / 4][8];
    int ai = INT_MAX;
    double sum = 0.0;
    for (int p0 = 0; p0 < P; p0 += P / 4) {
      quarter(p0, v);
#pragma unroll
      for (int p = 0; p < P / 4; ++p)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          if (T > 0.f) mx = fmaxf(mx, v[p][j]);
          else if (v[p][j] > mx) { mx = v[p][j]; ai = base + (p0 + p) * 512 + j; }   // ids ascend: the first maximum stays
        }
    }
    if (T > 0.f) {
      mx = lanes_max(mx);
      if (mx > -INFINITY) {
        const float k = (float)(kLog2e / (double)T);
        for (int p0 = 0; p0 < P; p0 += P / 4) {
          quarter(p0, v);
#pragma unroll
          for (int p = 0; p < P / 4; ++p) {
            float part = 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) part += __builtin_amdgcn_exp2f((v[p][j] - mx) * k);
            sum += (double)part;
          }
        }
        sum = lanes_sum(sum);
      }
    } else {
      lanes_argmax(mx, ai);
    }
    if (lane == 0) { pm[c] = mx; ps[c] = sum; pa[c] = ai; }
  }
}

// A top-k of this size takes one pass, which needs nothing from the row statistics (4 x top_k candidates are expected in the list).
__device__ __host__ inline bool cut_takes_one_pass(int top_k, int V) { return top_k > 0 && top_k < V && 6l * top_k <= kCutList; }

// The cut of every row that asks for one: cut key, kept mass, and whether top_p falls within 1e-6 of the row's mass of it.
// grid = rows, one block each (a block fills its compute unit: blocks that only find they have no row would cost a round).
//
// The first pass files the tokens under 8192 bins of the exponent (log2 of the probability relative to the maximum, 192 bins
// per factor of two): their count for top-k, their mass in 32-bit fixed point for top-p; the bins in which the cut can lie
// follow from the running sum and a bound of its rounding.  The second collects the tokens of those bins (for top-k: of all
// bins down to it) and adds up, exactly, what lies above.  The list is sorted by key, and its running sum of exact 2^-40
// masses decides.  A top-k of a few hundred takes one pass: the first round of loads (32768 ids, sampled across the vocabulary)
// is filed, the bin at which these already hold top_k tokens bounds the cut, and everything from that bin on goes to the list
// at once.  For top-p, tokens so improbable that all of them together do not matter to the sums are not filed.
// When the list cannot hold the candidates (near-flat laws, many ties), top-p goes on with passes that narrow the keys of those
// bins (cut_narrow).  Rows with NaN or an infinite maximum, a top-k beyond the list, a top-p too close to 1 for the sums of the
// first pass, and every row with `digits` (FSV_NUCLEUS_FULL=1, the test of one against the other) narrow from the whole range.
// Bound by HBM with a row for every compute unit (a pass over 204 rows x 128256 fp32 takes 21 us by itself), by the per-token
// arithmetic of a single compute unit with few rows (71 rows of a flat law, top-p 0.9: two passes of about 19 us, 48.2 in all).  204 rows, top-k 50
// and top-p 0.9, 30 us: 16 of them the stream, 4.5 the bound from the first round, 6 the list.  Measured on 166 rows x 128256 fp32,
// N(0, 3), T = 0.8, against passes by digits alone: top-k 50 then top-p 0.9 32 us (195), top-p 0.9 51 (81), top-k 5000 93 (155), top-p 0.9999 91 (84: the same
// passes, without fixed shifts); logits N(0, 0.02), top-p 0.9 91 (85: a pass to find that the list is too short), on 4 rows 86
// (74); logits rounded to whole numbers, top-p 0.99 110 (110).
template <typename LT, bool STATS>
__global__ __launch_bounds__(kCutThreads) void k_cut(const int32_t *__restrict__ off, int B, int V, const int32_t *__restrict__ done,
                                                     const LT *__restrict__ logits, const float *__restrict__ temperature,
                                                     const float *__restrict__ top_p, const int32_t *__restrict__ top_k, int nc, int digits, float *pmax, double *psum, int32_t *parg,
                                                     uint32_t *__restrict__ nuc_key, double *__restrict__ nuc_S,
                                                     int32_t *__restrict__ nuc_near) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r = blockIdx.x;
  if (done && done[r] == 1) return;   // k_cut_window has settled this row
  int b = -1;   // the row's request: the last one whose first row, off[b] + b, is not beyond r (every wave by itself)
  for (int b0 = 0; b0 < B; b0 += 64) b += __popcll(__ballot(b0 + lane < B && off[min(b0 + lane, B)] + b0 + lane <= r));
  const float T = temperature[b], tp = top_p ? top_p[b] : 1.f;
  const int tk = top_k ? top_k[b] : 0;
  const bool use_k = T > 0.f && tk > 0 && tk < V, use_p = T > 0.f && tp < 1.f;
  const LT *row = logits + (size_t)r * V;
  if (!use_k && !use_p) {
    if (STATS) row_stats_by_block(row, V, nc, T, pmax + (size_t)r * nc, psum + (size_t)r * nc, parg + (size_t)r * nc, w, lane);
    if (tid == 0) { nuc_key[r] = 0u; nuc_S[r] = -1.0; nuc_near[r] = 0; }
    return;
  }
  // 32 KiB of bins; later the narrowing passes' masses (16) and counts (8) or lowest and highest keys (16)
  __shared__ unsigned long long s_raw[kCutBins / 2];
  __shared__ __align__(16) uint32_t lkey[kCutList];
  __shared__ uint32_t lrank[256];
  __shared__ cut_state st;
  uint32_t *hist = reinterpret_cast<uint32_t *>(s_raw);
  for (int i = tid; i < kCutBins; i += kCutThreads) hist[i] = 0u;
  if (tid == 0) { st.n = 0; st.found = 0; st.bad = 0; }
  const bool one_pass = use_k && !digits && cut_takes_one_pass(tk, V) && whole_rounds(V) > 0;   // block-uniform
  float m = 0.f;    // the row's maximum; the one-pass form: first that of its sample, then that of its list, which is the row's
  double S = 0.0;
  auto row_max = [&]() __attribute__((always_inline)) {
    if (STATS) {
      row_stats_by_block(row, V, nc, T, pmax + (size_t)r * nc, psum + (size_t)r * nc, parg + (size_t)r * nc, w, lane);
      __syncthreads();
    }
    if (tid < 64) {   // the row's maximum and normaliser from the per-chunk statistics (chunks in lanes, 64 at a time)
      float mx = -INFINITY;
      for (int c = lane; c < nc; c += 64) mx = fmaxf(mx, pmax[(size_t)r * nc + c]);
      mx = lanes_max(mx);
      const double invT = 1.0 / (double)T;
      double term = 0.0;
      for (int c = lane; c < nc; c += 64) {
        const float pm = pmax[(size_t)r * nc + c];
        term += psum[(size_t)r * nc + c] * ((pm == mx) ? 1.0 : exp(((double)pm - (double)mx) * invT));
      }
      term = lanes_sum(term);
      if (lane == 0) { st.m = mx; st.S = term; }
    }
    __syncthreads();
    m = st.m;
    S = st.S;
  };
  if (!one_pass) row_max();
  else __syncthreads();
  const exp_scale k = make_exp_scale(kLog2e / (double)T);
  // The bin of a token is a chain of correctly rounded, monotone steps, so that no token is filed above one with a larger
  // logit; -inf (and NaN, which leaves the fast way) ends in the last bin.
  auto bin_of = [&](float v) { return min((uint32_t)(fmaxf((v - m) * k.hi, -150.0f) * -kCutBinsPerLog2), (uint32_t)(kCutBins - 1)); };
  auto put = [&](float v) {
    const int at = atomicAdd(&st.n, 1);
    if (at < kCutList) lkey[at] = okey(v);
  };
  // The first pass sums in units of 2^-31 of the row's mass.  A running sum is within half a unit per token of the mass it stands
  // for, the normaliser within 1e-6.
  const double slack = 0.5 * V + 2147483648.0 * 2e-6, room = (1.0 - (double)tp) * 2147483648.0 - 2.0 * slack;
  // a top-k beyond the list, or (top-p alone) no room between top_p and the whole for the sums' error: the general way at once
  bool fast = one_pass || (!digits && fabsf(m) < INFINITY && S >= 0.5 && S < 1e9 && (use_k ? tk <= kCutList : room > 6.0 * slack));   // block-uniform

  bool crowded = false;           // top-p alone, too many candidates for the list:
  uint32_t klo = 0u, khi = ~0u;   // the keys of the bins the cut can lie in

  if (fast) {
    double tot = 0.0;     // top-p alone: the row's mass as an integer sum (exact in a double: < 2^53 per thread)
    double above = 0.0;   // likewise the mass above the candidates
    bool bad = false;
    if (one_pass) {
      // The bins are those of the sample's maximum (a token above it goes to the first).  Once the bin that bounds the cut is known, a
      // token is dismissed by comparing it with a value a little below that bin's lower edge (extra candidates do no harm): most
      // groups of eight by one branch.
      float vlim = -INFINITY, mx = -INFINITY;
      bool sampled = false;
      over_row<LT>(row, V, tid, [&](int, const float(&v)[8]) {
        if (!sampled) {   // block-uniform
#pragma unroll
          for (int j = 0; j < 8; ++j) bad |= v[j] != v[j];
          return;
        }
        bool any = false;
#pragma unroll
        for (int j = 0; j < 8; ++j) any |= !(v[j] < vlim);
        if (any) {
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            bad |= v[j] != v[j];
            if (v[j] >= vlim) put(v[j]);
          }
        }
      }, [&](int round, const auto &v) {
        if (round != 0) return;
        float own[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          own[j] = fmaxf(fmaxf(v[0][j], v[1][j]), fmaxf(v[2][j], v[3][j]));
          mx = fmaxf(mx, own[j]);
        }
        mx = lanes_max(mx);
        if (lane == 0) st.w32[w] = __float_as_uint(mx);
        __syncthreads();
        for (int i = 0; i < kCutThreads / 64; ++i) mx = fmaxf(mx, __uint_as_float(st.w32[i]));
        m = mx;
        bad |= !(fabsf(m) < INFINITY);
        // Of every four tokens, a quarter of the row apart, the largest is filed: where these reach top_k, so do the tokens.  Far apart because
        // probable ids may lie side by side: with the largest of every eight neighbours, runs of eight likely ids put up to eight times as many tokens
        // above the bound, and from a top_k of 64 the list overflows (204 rows x 128256, top-k 100, independent ids 48.1 us, runs 190; like this 47.5
        // and 49.6; every token filed 51.7 and 54.5).
        if (fabsf(m) < INFINITY) {
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const uint32_t bin = bin_of(own[j]);
            if (bin < kCutBins - 1) atomicAdd(&hist[bin], 1u);
          }
        }
        __syncthreads();   // (the bins are complete, and w32 has been read)
        cut_find_bins(hist, (uint32_t)tk, (uint32_t)tk, &st);
        const float depth = (float)(min(st.bin_lo, (uint32_t)(kCutBins - 2)) + 1) / (kCutBinsPerLog2 * k.hi);
        vlim = (m - depth * 1.00001f) - 5e-7f * (fabsf(m) + depth);
        sampled = true;
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int j = 0; j < 8; ++j)
            if (v[u][j] >= vlim) put(v[u][j]);
      });
      if (__any(bad) && lane == 0) st.bad = 1;
      __syncthreads();
      fast = !st.bad;
    } else {
      // ---- pass 1: bins ----
      const float scale = (float)(2147483648.0 / S), drop = (float)(0.9 * room / 2147483648.0 * S / V);
      if (use_k) {
        over_row<LT>(row, V, tid, [&](int, const float(&v)[8]) {
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            bad |= !(v[j] <= m);
            const uint32_t bin = bin_of(v[j]);
            if (bin < kCutBins - 1) atomicAdd(&hist[bin], 1u);
          }
        }, [](int, const auto &) {});
      } else {   // (a NaN has made the normaliser one, or carries no mass)
        over_row<LT>(row, V, tid, [&](int, const float(&v)[8]) {
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const float e = exp_scaled(v[j] - m, k);
            tot += floor((double)e * kNucScale + 0.5);
            if (e >= drop) atomicAdd(&hist[bin_of(v[j])], (uint32_t)fmaf(e, scale, 0.5f));
          }
        }, [](int, const auto &) {});
      }
      if (__any(bad) && lane == 0) st.bad = 1;
      __syncthreads();
      const double target32 = (double)tp * 2147483648.0;
      const uint32_t x0 = use_k ? (uint32_t)tk : (uint32_t)fmax(1.0, target32 - slack), x1 = use_k ? (uint32_t)tk : (uint32_t)(target32 + slack);
      cut_find_bins(hist, x0, x1, &st);
      const uint32_t lo = use_k ? 0u : st.bin_lo, hi = st.bin_hi;
      fast = !st.bad && hi < kCutBins - 1;
      if (fast && !use_k) {
        // the values at the bins' edges, a little outside, as in the one-pass form
        const float d_lo = (float)lo / (kCutBinsPerLog2 * k.hi), d_hi = (float)(hi + 1) / (kCutBinsPerLog2 * k.hi);
        khi = okey((m - d_lo * 0.99999f) + 5e-7f * (fabsf(m) + d_lo));
        klo = okey((m - d_hi * 1.00001f) - 5e-7f * (fabsf(m) + d_hi));
        // a token of these bins has at most the mass of the first one's upper edge: at least this many of them
        crowded = (float)(st.upto - st.before) * __builtin_amdgcn_exp2f((float)lo / kCutBinsPerLog2) > scale * (float)kCutList;
      }
      // ---- pass 2: candidates, and the mass above them ----
      if (fast && !crowded) {
        // The values at the bins' edges, exactly: the smallest whose bin is at most `bin`, found by a wave among the keys around the rounded
        // one (64 a step; should it not lie there, from -inf to the maximum), so that two comparisons place a token.  The pass is bound by the instructions a single compute unit
        // issues for its row: a flat law has most of its mass above the cut, so the mass is summed without a branch per token;
        // a peaked one leaves nothing to do for most groups of eight, which are left at once (800 rows x 50257, T = 0.6, the whole call
        // 191.7 -> 187.0 us; 71 rows x 128256, peaked or flat, are 1.4 us longer for it, 204 rows up to 1.5).
        auto edge = [&](uint32_t bin) {
          const float depth = (float)(bin + 1) / (kCutBinsPerLog2 * k.hi), off = 5e-7f * (fabsf(m) + depth);
          uint32_t below = okey((m - depth * 1.00001f) - off), at = okey(fminf((m - depth * 0.99999f) + off, m));
          if (!(bin_of(okey_value(below)) > bin && bin_of(okey_value(at)) <= bin)) {   // (uniform)
            below = okey(-INFINITY);
            at = okey(m);
          }
          while (at - below > 1u) {
            const uint64_t d = at - below;
            const uint32_t key = below + (uint32_t)((d * (uint32_t)(lane + 1)) >> 6);
            const int f = (int)__builtin_ctzll(__ballot(bin_of(okey_value(key)) <= bin));   // (lane 63 holds `at`)
            at = below + (uint32_t)((d * (uint32_t)(f + 1)) >> 6);
            below += (uint32_t)((d * (uint32_t)f) >> 6);
          }
          return okey_value(at);
        };
        if (w == 0) st.vlow = edge(hi);
        if (w == 1) st.vtop = lo ? edge(lo - 1) : INFINITY;
        __syncthreads();
        const float vlow = st.vlow, vtop = st.vtop;
        over_row<LT>(row, V, tid, [&](int, const float(&v)[8]) {
          float most = v[0];
#pragma unroll
          for (int j = 1; j < 8; ++j) most = fmaxf(most, v[j]);
          if (!(most >= vlow)) return;
          uint32_t mask = 0u;   // candidates are few: noted, and put afterwards
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const float d = v[j] - m, e = __builtin_amdgcn_exp2f(fmaf(d, k.lo, d * k.hi));   // (of a token above the candidates: not small)
            above += floor((double)(v[j] >= vtop ? e : 0.f) * kNucScale + 0.5);
            mask |= v[j] >= vlow && !(v[j] >= vtop) ? 1u << j : 0u;
          }
          while (mask) {
            const int j = __builtin_ctz(mask);
            mask &= mask - 1u;
            const float a0 = (j & 1) ? v[1] : v[0], a1 = (j & 1) ? v[3] : v[2], a2 = (j & 1) ? v[5] : v[4], a3 = (j & 1) ? v[7] : v[6];
            const float b0 = (j & 2) ? a1 : a0, b1 = (j & 2) ? a3 : a2;
            put((j & 4) ? b1 : b0);
          }
        }, [](int, const auto &) {});
      }
    }
    // sums over the block: the mass above, and the total
    unsigned long long A = 0ull, all = 0ull;   // (the one-pass form has neither)
    if (!one_pass) {
      unsigned long long ta = (unsigned long long)above, tt = (unsigned long long)tot;
      ta = lanes_sum(ta);
      tt = lanes_sum(tt);
      if (lane == 0) { st.w64[w] = ta; st.t64[w] = tt; }
      __syncthreads();
      for (int i = 0; i < kCutThreads / 64; ++i) { A += st.w64[i]; all += st.t64[i]; }
    }
    double total = (double)all;
    const int n = st.n;
    crowded |= n > kCutList && fast && !use_k;   // block-uniform
    if (crowded && tid == 0) st.total = all;
    fast = fast && !crowded && n <= kCutList && n > 0;

    // ---- the list, in descending order of the keys ----
    if (fast) {
      if (n <= 256) {
        // by rank: four threads per candidate, each against a quarter of the list (a short sort by exchanges takes 36 barriers, 6 us)
        const int i = tid & 255, part = tid >> 8;
        for (int x = n + tid; x < 256; x += kCutThreads) lkey[x] = 0u;
        if (tid < 256) lrank[tid] = 0u;
        __syncthreads();
        const uint32_t mine = lkey[i];
        uint32_t rank = 0u;
#pragma unroll
        for (int y = 0; y < 64; y += 4) {
          const int x = part * 64 + y;
          const uint4 kx = *reinterpret_cast<const uint4 *>(lkey + x);
          rank += (kx.x > mine || (kx.x == mine && x < i)) + (kx.y > mine || (kx.y == mine && x + 1 < i)) +
                  (kx.z > mine || (kx.z == mine && x + 2 < i)) + (kx.w > mine || (kx.w == mine && x + 3 < i));
        }
        atomicAdd(&lrank[i], rank);
        __syncthreads();
        if (tid < 256) lkey[lrank[tid]] = mine;
        __syncthreads();
      } else {
        int P2 = 512;
        while (P2 < n) P2 <<= 1;
        for (int i = n + tid; i < P2; i += kCutThreads) lkey[i] = 0u;
        for (int size = 2; size <= P2; size <<= 1)
          for (int gap = size >> 1; gap > 0; gap >>= 1) {
            __syncthreads();
            if (tid < P2 / 2) {
              const int i = 2 * tid - (tid & (gap - 1)), j = i + gap;
              const uint32_t x = lkey[i], y = lkey[j];
              if ((x < y) == ((i & size) == 0)) { lkey[i] = y; lkey[j] = x; }
            }
          }
        __syncthreads();
      }
      if (one_pass) {   // the list begins with the row's maximum
        m = okey_value(lkey[0]);
        if (!(fabsf(m) < INFINITY)) fast = false;   // block-uniform
      }
      // running mass up to and with each candidate, two consecutive ones per thread
      unsigned long long q[2], mle[2];
      uint32_t key[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int i = 2 * tid + u;
        key[u] = i < n ? lkey[i] : 0u;
        q[u] = i < n ? nuc_mass(okey_value(key[u]) - m, k) : 0ull;
      }
      unsigned long long incl = q[0] + q[1];
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
      }
      if (lane == 63) st.t64[w] = incl;   // (read by everyone before the sort)
      __syncthreads();
      unsigned long long pre = A;
      for (int i = 0; i < w; ++i) pre += st.t64[i];
      mle[1] = pre + incl;
      mle[0] = mle[1] - q[1];
      const uint32_t prev = tid > 0 && 2 * tid - 1 < n ? lkey[2 * tid - 1] : 0u, next = 2 * tid + 2 < n ? lkey[2 * tid + 2] : 0u;
      // first / last of its key, u = 0, 1
      const bool is0 = 2 * tid < n, is1 = 2 * tid + 1 < n;
      const bool first0 = is0 && (tid == 0 || prev != key[0]), last0 = is0 && (!is1 || key[1] != key[0]);
      const bool first1 = is1 && key[1] != key[0], last1 = is1 && (2 * tid + 2 >= n || next != key[1]);
      if (use_k) {
        const uint32_t kk = lkey[min(tk, n) - 1];
        if (last0 && key[0] == kk) { st.kkey = kk; st.kmass = mle[0]; }
        if (last1 && key[1] == kk) { st.kkey = kk; st.kmass = mle[1]; }
        if (tid == 0) st.found = n >= tk ? 1 : 0;
        __syncthreads();
      }
      if (use_p) {
        if (use_k) total = (double)st.kmass;
        const double target = (double)tp * total;
        const bool ok = !use_k || st.found;
        __syncthreads();   // found has been read
        if (tid == 0) st.found = 0;
        __syncthreads();
        // the first candidate with which the running mass reaches the target, and the group of equal keys around it
        if (ok && is0 && (double)mle[0] >= target && !((double)(mle[0] - q[0]) >= target)) { st.cut = key[0]; st.found = 1; }
        if (ok && is1 && (double)mle[1] >= target && !((double)mle[0] >= target)) { st.cut = key[1]; st.found = 1; }
        __syncthreads();
        const uint32_t cut = st.cut;
        if (first0 && key[0] == cut) st.acc = mle[0] - q[0];
        if (first1 && key[1] == cut) st.acc = mle[1] - q[1];
        if (last0 && key[0] == cut) st.kept = mle[0];
        if (last1 && key[1] == cut) st.kept = mle[1];
        __syncthreads();
      }
      fast = fast && st.found != 0;
      if (STATS && fast && one_pass && tid < nc) {   // what k_decide takes from the statistics of a row that is cut: its maximum
        pmax[(size_t)r * nc + tid] = tid == 0 ? m : -INFINITY;
        psum[(size_t)r * nc + tid] = 0.0;
        parg[(size_t)r * nc + tid] = INT_MAX;
      }
      if (fast && tid == 0) {
        const double target = (double)tp * total;
        nuc_key[r] = use_p ? st.cut : st.kkey;
        nuc_S[r] = (double)(use_p ? st.kept : st.kmass) / kNucScale;
        nuc_near[r] = (use_p && fmin(target - (double)st.acc, (double)st.kept - target) < 1e-6 * total) ? 1 : 0;
      }
    }
    if (fast) return;
    __syncthreads();   // the bins and the list make room for the passes below
    if (one_pass) row_max();
  }
  uint32_t *hcnt = reinterpret_cast<uint32_t *>(s_raw + FSV_NUC_BINS);
  if (use_k) cut_narrow<LT, true>(row, V, m, k, 0u, ~0u, true, 0u, tk, tp, s_raw, hcnt, &st);
  const uint32_t kkey = use_k ? st.kkey : 0u;
  if (use_p) {
    // (a second trip over the whole range if the interval the bins left does not hold the cut)
    while (!cut_narrow<LT, false>(row, V, m, k, crowded ? klo : 0u, crowded ? khi : ~0u, !crowded, kkey, tk, tp, s_raw, hcnt, &st) &&
           crowded)
      crowded = false;
  }
  if (tid == 0) {
    if (use_p) {
      const double total = (double)st.total, target = (double)tp * total;
      nuc_key[r] = st.cut;
      nuc_S[r] = (double)st.kept / kNucScale;
      nuc_near[r] = (fmin(target - (double)st.acc, (double)st.kept - target) < 1e-6 * total) ? 1 : 0;
    } else {
      nuc_key[r] = kkey;
      nuc_S[r] = kkey ? (double)st.kmass / kNucScale : -1.0;
      nuc_near[r] = 0;
    }
  }
}

#define FSV_MAX_GAMMA 16

// The tokens a cut key keeps: those whose logit is not below the value the key stands for.  Only where that value is a zero (the keys tell
// -0 from +0) or no number are the keys themselves compared.
struct cut_test {
  float value;
  uint32_t key;   // 0: `value` decides
};
__device__ inline cut_test make_cut_test(uint32_t key) {   // 0: nothing is cut
  const float v = okey_value(key);
  if (key && !(v < 0.f) && !(v > 0.f)) return cut_test{-INFINITY, key};
  return cut_test{key ? v : -INFINITY, 0u};
}

// Eight ids' masses from their logits and draft probabilities: p, or (RES) max(0, p - q); their sum in id order.  This is what the
// vocabulary-wide part of k_decide consists of besides its loads: 12 instructions an id.
template <bool RES>
__device__ inline double masses_of(float (&lv)[8], const float (&qv)[8], float m, exp_scale k, double invS, cut_test cut, double (&mass)[8]) {
  if (cut.key) {   // (uniform)
#pragma unroll
    for (int j = 0; j < 8; ++j) lv[j] = okey(lv[j]) >= cut.key ? lv[j] : -INFINITY;
  }
  double t = 0.0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float d = lv[j] - m, z = fmaxf(fmaf(d, k.lo, d * k.hi), -160.f);   // exp_scaled; a NaN and -inf end as 0 here, too
    const double e = (double)(lv[j] >= cut.value ? __builtin_amdgcn_exp2f(z) : 0.f);
    const double p = RES ? fma(e, invS, -(double)qv[j]) : e * invS;
    mass[j] = RES ? fmax(p, 0.0) : p;
    t += mass[j];
  }
  return t;
}

template <typename LT>
__device__ inline double thread_masses(const LT *lrow, const float *qrow, int i0, int V, float m, exp_scale k, double invS, bool residual, cut_test cut,
                                       double (&mass)[8]) {
  float lv[8], qv[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  loader<LT>::load8(lrow, i0, V, -INFINITY, lv);
  if (!residual) return masses_of<false>(lv, qv, m, k, invS, cut, mass);
  loader<float>::load8(qrow, i0, V, 0.f, qv);
  return masses_of<true>(lv, qv, m, k, invS, cut, mass);
}

#define FSV_MAX_NSB 160

// Acceptance tests, masses and token selection of one request.  grid = (ceil(sub-blocks / 4), requests).
//
// Phase 1, every block: the acceptance tests.  Sixteen lanes combine the per-chunk statistics of a row (up to three chunks per
//   lane: row max with the lowest id attaining it, then the sum of the rescaled chunk sums over a fixed tree), all rows
//   of the request side by side (four rows per wave one after the other took 3 us longer at 16 drafts); then thread i tests
//   draft i+1 from two gathered scalars, and
//   thread 0 takes the accepted prefix.  Every block of the request repeats this (a few KB from L2) instead of waiting
//   for a launch of its own.
// Phase 2: wave w of block x takes sub-block 4x + w of the row the emitted token is drawn from (the residual
//   max(0, p - q) after a rejection, p itself when every draft passed): four passes of 512 ids, mass to bsum.
// Phase 3: the blocks of a request take a ticket; the one that draws the last ticket adds the sub-block masses up (lane sums
//   and their scan), finds the sub-block and the id by inverse CDF, writes every output of the request (accepted length,
//   token, flags, rollback) and clears the ticket for the next call.
// Bound by its chain of round trips (3.5 us to the accepted prefix, 6 from the last mass to the token) around a stream of two rows.  Five waves on
// a SIMD (96 registers), so that a call of 64 requests x 152064 ids (1216 blocks) is resident at once; with 113 registers four were, 1024 blocks, and a
// sixth of them began when others had ended.  That and the shorter arithmetic of masses_of: 23.9 -> 20 us.
template <typename LT>
__global__ __launch_bounds__(256, 5) void k_decide(
    const int32_t *__restrict__ off, const float *__restrict__ temperature, const float *__restrict__ pmax,
    const double *__restrict__ psum, const int32_t *__restrict__ parg, const int32_t *__restrict__ draft, int V, int nc, int nsb,
    const LT *__restrict__ logits, const float *__restrict__ q, const float *__restrict__ u_acc,
    const float *__restrict__ u_smp, const uint32_t *__restrict__ nuc_key, const double *__restrict__ nuc_S, const int32_t *__restrict__ nuc_near, double *__restrict__ bsum,
    int32_t *__restrict__ ticket, int32_t *__restrict__ accepted_len, int32_t *__restrict__ next_token,
    uint32_t *__restrict__ flags, const int32_t *__restrict__ seq_lens, int32_t *__restrict__ new_seq_lens,
    int32_t *__restrict__ pages_released, int page_size) {
  const int b = blockIdx.y, tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int o = off[b], gamma_all = off[b + 1] - o, gamma = min(gamma_all, FSV_MAX_GAMMA), rs = o + b;
  const float T = temperature[b];
  const double invT = (T > 0.f) ? 1.0 / (double)T : 0.0;
  __shared__ double s_m[FSV_MAX_GAMMA + 1], s_S[FSV_MAX_GAMMA + 1];
  __shared__ int s_arg[FSV_MAX_GAMMA + 1], s_acc[FSV_MAX_GAMMA], s_near[FSV_MAX_GAMMA];
  __shared__ int s_tau, s_last;
  __shared__ uint32_t s_flags;
  auto rollback = [&](int tau) {  // KV rollback: keep [0, L+1+tau)
    if (seq_lens && new_seq_lens) {
      const int L = seq_lens[b], keep = L + 1 + tau, written = L + 1 + gamma_all;
      new_seq_lens[b] = keep;
      if (pages_released) pages_released[b] = (written + page_size - 1) / page_size - (keep + page_size - 1) / page_size;
    }
  };

  // ---- phase 1: acceptance ----
  LT lv_raw{};
  float qd_in = 0.f, u_in = 0.f;
  uint32_t cut_in = 0u;
  {
    constexpr int CPL = (FSV_MAX_NSB / FSV_SPC + 15) / 16;   // chunks per lane
    const int l16 = tid & 15;
    float pm[CPL];
    double ps[CPL];
    int pa[CPL];
    auto load_row = [&](int i) {
#pragma unroll
      for (int j = 0; j < CPL; ++j) {
        const int c = l16 + 16 * j;
        const bool live = i <= gamma && c < nc;
        const size_t at = (size_t)(rs + min(i, gamma)) * nc + min(c, nc - 1);
        pm[j] = live ? pmax[at] : -INFINITY;
        ps[j] = live ? psum[at] : 0.0;
        pa[j] = live ? parg[at] : INT_MAX;
      }
    };
    load_row(tid >> 4);
    // What draft tid + 1 is tested on: its logit, its draft probability, its uniform.  Issued here, so that the two dependent
    // round trips (token, then the values it points at) pass while the statistics are combined.
    if (T > 0.f && tid < gamma) {
      const int d = min(max(draft[o + tid], 0), V - 1);
      lv_raw = logits[(size_t)(rs + tid) * V + d];
      qd_in = q[(size_t)(o + tid) * V + d];
      u_in = u_acc[o + tid];
      if (nuc_key) cut_in = nuc_key[rs + tid];
    }
    for (int i = tid >> 4; i <= gamma; i += 16) {   // (a second trip for the first sixteen threads only when gamma is 16)
      if (i >= 16) load_row(i);
      float mx = pm[0];
      int ai = pa[0];
#pragma unroll
      for (int j = 1; j < CPL; ++j)
        if (pm[j] > mx || (pm[j] == mx && pa[j] < ai)) { mx = pm[j]; ai = pa[j]; }
      lanes_argmax<8>(mx, ai);
      double term = 0.0;
      if (T > 0.f) {
#pragma unroll
        for (int j = 0; j < CPL; ++j)
          if (l16 + 16 * j < nc) term += ps[j] * ((pm[j] == mx) ? 1.0 : exp(((double)pm[j] - (double)mx) * invT));
      }
      term = lanes_sum<8>(term);
      if (l16 == 0) {
        s_m[i] = (double)mx;
        // a row cut to its most probable tokens is normalised by the kept mass; its cut key masks the tokens outside
        s_S[i] = (nuc_S && nuc_S[rs + i] >= 0.0) ? nuc_S[rs + i] : term;
        s_arg[i] = ai;
      }
    }
  }
  __syncthreads();
  if (T <= 0.f) {  // greedy (Alg. 2): accept while the draft equals the argmax, emit the argmax
    if (blockIdx.x == 0 && tid == 0) {
      int tau = 0;
      while (tau < gamma && draft[o + tau] == s_arg[tau]) ++tau;
      accepted_len[b] = tau;
      next_token[b] = s_arg[tau];
      flags[b] = 0u;
      rollback(tau);
    }
    return;
  }
  if (tid < gamma) {  // row rs + tid scores draft tid + 1
    float lv;
    if constexpr (sizeof(LT) == 2) lv = __uint_as_float((uint32_t)lv_raw << 16);
    else lv = lv_raw;
    const bool kept = !nuc_key || okey(lv) >= cut_in;
    const double p = kept ? exp(((double)lv - s_m[tid]) * invT) / s_S[tid] : 0.0;
    const double qd = (double)qd_in;
    const double ratio = p / qd;
    double a = (ratio >= 1.0) ? 1.0 : ratio;
    if (!(a == a)) a = 0.0;
    const double u = (double)u_in;
    s_acc[tid] = (u < a) ? 1 : 0;
    s_near[tid] = (fabs(u - a) < 1e-4) ? 1 : 0;
  }
  __syncthreads();
  if (tid == 0) {
    int tau = 0;
    while (tau < gamma && s_acc[tau]) ++tau;
    uint32_t f = (tau < gamma) ? 4u : 0u;
    for (int i = 0; i < gamma && i <= tau; ++i) f |= s_near[i] ? 1u : 0u;
    if (nuc_near)
      for (int i = 0; i <= tau; ++i) f |= nuc_near[rs + i] ? 8u : 0u;   // rows 0..tau are the ones the outcome rests on
    s_tau = tau;
    s_flags = f;
  }
  __syncthreads();
  const int tau = s_tau;
  bool residual = tau < gamma;
  const double m = s_m[tau], invS = 1.0 / s_S[tau];
  const cut_test cut = make_cut_test(nuc_key ? nuc_key[rs + tau] : 0u);
  const exp_scale k = make_exp_scale(kLog2e / (double)T);
  const LT *lrow = logits + (size_t)(rs + tau) * V;
  const float *qrow = residual ? q + (size_t)(o + tau) * V : nullptr;

  // ---- phase 2: mass of this wave's sub-block ----
  {
    const int sb = blockIdx.x * 4 + w;
    if (sb < nsb) {
      constexpr int PARTS = FSV_SBK / 512;
      double tot = 0.0, mass[8];
      if ((sb + 1) * FSV_SBK <= V) {   // wave-uniform; all loads of the sub-block before the first use
        float lv[PARTS][8], qv[PARTS][8];
#pragma unroll
        for (int part = 0; part < PARTS; ++part) loader<LT>::load8_fast(lrow, sb * FSV_SBK + part * 512 + lane * 8, lv[part]);
        if (residual) {
#pragma unroll
          for (int part = 0; part < PARTS; ++part) loader<float>::load8_fast(qrow, sb * FSV_SBK + part * 512 + lane * 8, qv[part]);
#pragma unroll
          for (int part = 0; part < PARTS; ++part) tot += masses_of<true>(lv[part], qv[part], (float)m, k, invS, cut, mass);
        } else {
#pragma unroll
          for (int part = 0; part < PARTS; ++part) tot += masses_of<false>(lv[part], qv[part], (float)m, k, invS, cut, mass);
        }
      } else {
#pragma unroll 1
        for (int part = 0; part < PARTS; ++part)
          tot += thread_masses<LT>(lrow, qrow, sb * FSV_SBK + part * 512 + lane * 8, V, (float)m, k, invS,
                                   residual, cut, mass);
      }
      tot = lanes_sum(tot);
      // a device-scope atomic store: written through to where every XCD sees it (a plain store would stay in this XCD's L2)
      if (lane == 0)
        __hip_atomic_store(reinterpret_cast<unsigned long long *>(bsum) + (size_t)b * nsb + sb,
                           (unsigned long long)__double_as_longlong(tot), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }

  // ---- phase 3: the last block of the request selects the token ----
  // The masses travel between blocks as device-scope atomics (stores above, loads below); no device-wide fence, which would write back
  // and invalidate the whole L2 of the XCD for every block (measured: 40 us on top of a 30 us kernel).
  wait_own_stores();
  __syncthreads();
  if (tid == 0)
    s_last = (__hip_atomic_fetch_add(&ticket[b], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1) ? 1 : 0;
  __syncthreads();
  if (!s_last) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  __shared__ double s_sb[FSV_MAX_NSB];
  __shared__ double s_w[4];
  __shared__ double s_Z, s_lo;
  __shared__ int s_pick, s_wfirst[4], s_wlast[4];
  if (tid == 0) {
    __hip_atomic_store(&ticket[b], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
    accepted_len[b] = tau;
    rollback(tau);
  }
  // Wave 0 takes the sub-block masses, PER consecutive ones per lane, and finds the first sub-block whose running mass exceeds
  // u times the total (lane sums and their scan: a fixed order).  One thread adding and comparing them one after the
  // other cost 3 us of this kernel's serial tail.
  auto pick_sb = [&](auto mass_of) {
    constexpr int PER = (FSV_MAX_NSB + 63) / 64;
    double m_[PER], t = 0.0;
#pragma unroll
    for (int j = 0; j < PER; ++j) m_[j] = (lane * PER + j < nsb) ? mass_of(lane * PER + j) : 0.0;
#pragma unroll
    for (int j = 0; j < PER; ++j) t += m_[j];
    double incl = t;
#pragma unroll
    for (int sh = 1; sh < 64; sh <<= 1) {
      const double up = __shfl_up(incl, sh, 64);
      if (lane >= sh) incl += up;
    }
    const double Z = __shfl(incl, 63, 64), target = (double)u_smp[b] * Z;
    double pre = __shfl_up(incl, 1, 64), run = (lane == 0) ? 0.0 : pre, lo = 0.0;
    int pick = -1, last = -1;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const double prev = run;
      run += m_[j];
      if (m_[j] > 0.0) last = lane * PER + j;
      if (pick < 0 && m_[j] > 0.0 && run > target) { pick = lane * PER + j; lo = prev; }
    }
    const unsigned long long hit = __ballot(pick >= 0), any = __ballot(last >= 0);
    if (hit) {
      const int from = (int)__builtin_ctzll(hit);
      pick = __shfl(pick, from, 64);
      lo = __shfl(lo, from, 64);
    } else {   // rounding left no crossing: last sub-block with mass
      pick = any ? __shfl(last, 63 - (int)__builtin_clzll(any), 64) : 0;
      lo = INFINITY;
    }
    if (lane == 0) { s_Z = Z; s_pick = pick; s_lo = lo; }
  };
  if (w == 0)
    pick_sb([&](int sb) {
      return __longlong_as_double((long long)__hip_atomic_load(reinterpret_cast<const unsigned long long *>(bsum) + (size_t)b * nsb + sb,
                                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    });
  __syncthreads();
  if (residual && !(s_Z > 0.0)) {
    // p <= q everywhere after rounding: the residual carries no mass, draw from p itself
    residual = false;
    qrow = nullptr;
    for (int sb = 0; sb < nsb; ++sb) {
      double mass[8], tot;
      double t = thread_masses<LT>(lrow, qrow, sb * FSV_SBK + tid * 8, V, (float)m, k, invS,
                                   false, cut, mass);
      block_incl_scan(t, s_w, &tot);
      if (tid == 0) s_sb[sb] = tot;
    }
    __syncthreads();   // (also: every thread has read s_Z above)
    if (w == 0) pick_sb([&](int sb) { return s_sb[sb]; });
    __syncthreads();
  }
  const double Z = s_Z, target = (double)u_smp[b] * Z;
  const int sb = s_pick;
  const double lo = s_lo;
  double mass[8];
  const int i0 = sb * FSV_SBK + tid * 8;
  double t = thread_masses<LT>(lrow, qrow, i0, V, (float)m, k, invS, residual, cut, mass);
  double incl = block_incl_scan(t, s_w, nullptr);
  // the first thread whose running mass crosses, and the last id with mass: a ballot per wave (LDS atomics of all 256 threads
  // on one address cost 3 us here).  Only a thread and an id that hold mass can be taken: lane sums, their scan and the sums
  // id by id are rounded differently, so lo may already lie a rounding above the target.
  const bool crosses = t > 0.0 && (lo + incl) > target;  // false for every thread when lo == inf
  int lp = -1;
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (mass[j] > 0.0) lp = i0 + j;
  const unsigned long long cb = __ballot(crosses), pb = __ballot(lp >= 0);
  const int wave_lp = __shfl(lp, pb ? 63 - (int)__builtin_clzll(pb) : 0, 64);
  if (lane == 0) {
    s_wfirst[w] = cb ? w * 64 + (int)__builtin_ctzll(cb) : INT_MAX;
    s_wlast[w] = pb ? wave_lp : -1;
  }
  __syncthreads();
  const int first = min(min(s_wfirst[0], s_wfirst[1]), min(s_wfirst[2], s_wfirst[3]));
  if (first == INT_MAX) {
    if (tid == 0) {
      next_token[b] = max(max(max(s_wlast[0], s_wlast[1]), max(s_wlast[2], s_wlast[3])), 0);
      flags[b] = (s_flags & (residual ? ~0u : ~4u)) | 2u;
    }
    return;
  }
  if (tid == first) {
    double run = lo + (incl - t), margin = 0.0;
    int pick = -1;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      double prev = run;
      run += mass[j];
      if (pick < 0 && mass[j] > 0.0 && run > target) {
        pick = i0 + j;
        margin = fmin(target - prev, run - target) / Z;
      }
    }
    if (pick < 0) { pick = lp; margin = 0.0; }
    next_token[b] = pick;
    uint32_t f = s_flags;
    if (!residual) f &= ~4u;
    if (margin < 1e-6) f |= 2u;
    flags[b] = f;
  }
}

__global__ void k_rollback(int B, const int32_t *seq_lens, const int32_t *off, const int32_t *accepted,
                           int32_t *new_seq_lens, int32_t *pages_released, int page_size) {
  int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  int g = off[b + 1] - off[b], tau = min(max(accepted[b], 0), g);
  int L = seq_lens[b], keep = L + 1 + tau, written = L + 1 + g;
  new_seq_lens[b] = keep;
  if (pages_released) pages_released[b] = (written + page_size - 1) / page_size - (keep + page_size - 1) / page_size;
}

template <typename LT>
int launch_sampler_t(fsv_ctx *c, const LT *logits, const fsv_batch *b, const fsv_result *r, int M, bool with_rollback,
                     hipStream_t s) {
  const int V = c->d.vocab, B = b->batch, nc = c->nc, nsb = c->nsb;
  int32_t *acc = r->accepted_len ? r->accepted_len : c->acc_scratch;
  int gmax = 0;
  for (int i = 0; i < B; ++i) gmax = max(gmax, b->draft_offsets_host[i + 1] - b->draft_offsets_host[i]);
  // Top-k / top-p cut: only when some request asks for it.
  bool any_k = false, any_p = false;
  int one_pass_rows = 0, other_rows = 0;   // of the sampled requests: rows that k_cut settles without statistics, and others
  for (int i = 0; i < B; ++i) {
    const bool sampled = !b->temperature_host || b->temperature_host[i] > 0.f;
    any_p |= sampled && b->top_p && b->top_p_host && b->top_p_host[i] < 1.f;
    const int tk = sampled && b->top_k && b->top_k_host ? b->top_k_host[i] : 0;
    any_k |= tk > 0 && tk < V;
    const int rows = b->draft_offsets_host[i + 1] - b->draft_offsets_host[i] + 1;
    if (cut_takes_one_pass(tk, V)) one_pass_rows += rows; else if (sampled) other_rows += rows;
  }
  const bool nucleus = any_k || any_p;
  // (FSV_NUCLEUS_FULL=1 in the environment narrows every row from the whole key range: a test compares the two)
  const char *full_env = nucleus ? getenv("FSV_NUCLEUS_FULL") : nullptr;
  const int digits = (full_env && full_env[0] == '1') ? 1 : 0;
  // fp32 logits, every sampled request with a top-k that takes k_cut one pass: the statistics are not needed and the rows are read
  // once; k_cut makes those of the greedy rows among them.  Half of the rows may be greedy while there is a compute unit for every
  // row, a third otherwise (a block per row streams at 3.3 TB/s, k_row_stats at 5.5).  Whole calls, V = 128256, top-k 50 and top-p 0.9: 204 rows
  // 69.6 -> 51.2 us, 5 rows 39.5 -> 33.5, 576 rows 156 -> 116; every second request greedy: 192 rows 57.8 -> 45.1, 576 rows 115 (122 without
  // the statistics); logits rounded to whole numbers, whose lists overflow: 192 rows 68 -> 53.
  const bool skip_stats = sizeof(LT) == 4 && !digits && other_rows == 0 && one_pass_rows > 0 && (M <= 256 ? 2 * one_pass_rows >= M : 3 * one_pass_rows >= 2 * M) &&
                          whole_rounds(V) > 0 && nc <= kCutThreads;
  if (!skip_stats) {
    fsv_prof_scope ps(c, s, FSV_K_SAMPLE_STATS, (double)M * V * sizeof(LT));
    hipLaunchKernelGGL((k_row_stats<LT>), dim3(fsv_ceil_div(nc, 4), gmax + 1, B), dim3(256), 0, s, b->draft_offsets,
                       b->temperature, logits, V, nc, c->pmax, c->psum, c->parg, 0);
  }
  if (nucleus) {
    // bytes: every row once, what no form can do without; how many passes a row takes is decided on the device
    fsv_prof_scope ps(c, s, FSV_K_SAMPLE_NUCLEUS, (double)M * V * sizeof(LT));
    // bf16 logits: the cuts lie within one or two binades of the maximum more often than not, which is one pass
    const bool window = sizeof(LT) == 2 && !digits;
#define FSV_WINDOW(W, FIRST)                                                                                                           \
  hipLaunchKernelGGL((k_cut_window<W, FIRST>), dim3(gmax + 1, B), dim3(1024), 0, s, (const uint16_t *)logits, V, nc, b->draft_offsets, \
                     b->temperature, b->top_p, b->top_k, c->pmax, c->psum, c->nuc_key, c->nuc_S, c->nuc_near, c->nuc_done)
    if (window) {
      FSV_WINDOW(4, true);
      FSV_WINDOW(8, false);
    }
#undef FSV_WINDOW
#define FSV_CUT(ST)                                                                                                                      \
  hipLaunchKernelGGL((k_cut<LT, ST>), dim3(M), dim3(kCutThreads), 0, s, b->draft_offsets, B, V, window ? c->nuc_done : nullptr, logits, \
                     b->temperature, b->top_p, b->top_k, nc, digits, c->pmax, c->psum, c->parg, c->nuc_key, c->nuc_S, c->nuc_near)
    if constexpr (sizeof(LT) == 4) {
      if (skip_stats) FSV_CUT(true);
      else FSV_CUT(false);
    } else {
      FSV_CUT(false);
    }
#undef FSV_CUT
  }
  {
    fsv_prof_scope ps(c, s, FSV_K_SAMPLE_DECIDE, (double)B * V * (sizeof(LT) + 4));
    hipLaunchKernelGGL(k_decide<LT>, dim3(fsv_ceil_div(nsb, 4), B), dim3(256), 0, s, b->draft_offsets, b->temperature, c->pmax,
                       c->psum, c->parg, b->draft_tokens, V, nc, nsb, logits, b->draft_probs, b->u_accept, b->u_sample, nucleus ? c->nuc_key : nullptr, nucleus ? c->nuc_S : nullptr, nucleus ? c->nuc_near : nullptr, c->bsum,
                       c->sel_ticket, acc, r->next_token, r->flags, with_rollback ? b->seq_lens : nullptr,
                       with_rollback ? r->new_seq_lens : nullptr, with_rollback ? r->pages_released : nullptr,
                       c->d.page_size);
  }
  FSV_HIP(c, hipGetLastError());
  return FSV_OK;
}

}  // namespace

int fsv_launch_build_rows(fsv_ctx *c, const fsv_batch *b, hipStream_t s) {
  hipLaunchKernelGGL(k_build_rows, dim3(fsv_ceil_div(b->batch, 256)), dim3(256), 0, s, b->batch, b->seq_lens, b->draft_offsets, c->row_req,
                     c->row_pos);
  FSV_HIP(c, hipGetLastError());
  return FSV_OK;
}

int fsv_launch_sampler(fsv_ctx *c, const void *logits, int logits_dtype, const fsv_batch *b, const fsv_result *r,
                       int M, bool with_rollback, hipStream_t s) {
  if (logits_dtype == FSV_BF16)
    return launch_sampler_t<uint16_t>(c, (const uint16_t *)logits, b, r, M, with_rollback, s);
  return launch_sampler_t<float>(c, (const float *)logits, b, r, M, with_rollback, s);
}

int fsv_launch_draft_law(fsv_ctx *c, const float *z, const fsv_batch *b, int all_rows, float *q, hipStream_t s) {
  const int V = c->d.vocab, B = b->batch, last = all_rows ? 0 : 1;   // a verification call takes no law of a request's last row
  int gmax = 0;
  for (int i = 0; i < B; ++i) gmax = max(gmax, b->draft_offsets_host[i + 1] - b->draft_offsets_host[i]);
  const int rows = gmax + 1 - last;   // widest request
  if (rows < 1) return FSV_OK;
  hipLaunchKernelGGL((k_row_stats<float, true>), dim3(fsv_ceil_div(c->nc, 4), rows, B), dim3(256), 0, s, b->draft_offsets, b->temperature,
                     z, V, c->nc, c->pmax, c->psum, c->parg, last);
  hipLaunchKernelGGL(k_draft_law, dim3(fsv_ceil_div(V, LAW_IDS), rows, B), dim3(256), 0, s, z, V, c->nc, b->draft_offsets,
                     b->temperature, c->pmax, c->psum, all_rows, q);
  FSV_HIP(c, hipGetLastError());
  return FSV_OK;
}

int fsv_launch_rollback(fsv_ctx *c, const fsv_batch *b, const int32_t *accepted, const fsv_result *r, hipStream_t s) {
  hipLaunchKernelGGL(k_rollback, dim3(fsv_ceil_div(b->batch, 256)), dim3(256), 0, s, b->batch, b->seq_lens,
                     b->draft_offsets, accepted, r->new_seq_lens, r->pages_released, c->d.page_size);
  FSV_HIP(c, hipGetLastError());
  return FSV_OK;
}

// ---------------------------------------------------------------------------------------------
// fsv_sample_static: the accept / resample step for callers that cannot allocate device memory.
// ---------------------------------------------------------------------------------------------
// The sampler's workspace (row map, per-chunk statistics, per-sub-block masses, nucleus state) lives in a device array
// of fixed size that is part of the library's code object: every GPU the library runs on holds its own copy at its own
// address for the life of the process.  The array's name is only a host-side handle; the address kernels can use is
// asked for once per device (hipGetSymbolAddress, with that device current) and kept.
#define FSV_STATIC_MAX_BATCH 128
#define FSV_STATIC_MAX_ROWS 1024
#define FSV_STATIC_MAX_NSB 160                                            /* vocabulary <= 160 * 2048 = 327680 */
#define FSV_STATIC_MAX_NC ((FSV_STATIC_MAX_NSB + FSV_SPC - 1) / FSV_SPC)
#define FSV_STATIC_BYTES (1u << 20)

static __device__ __align__(256) unsigned char scratch[FSV_STATIC_BYTES];

namespace {

struct static_slot {
  bool ready = false;
  fsv_ctx ctx;   // a context whose workspace pointers point into this device's copy of `scratch`; owns nothing
};
constexpr int kMaxDevices = 64;
static_slot *g_slots[kMaxDevices] = {};
std::mutex g_static_mu;

// Carve the workspace out of the array (256-byte aligned pieces, sized for the maxima above).  Returns false if it
// does not fit, which would be a mistake in the constants above.
bool carve_static(fsv_ctx &c, unsigned char *base) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    void *p = base + off;
    off += (bytes + 255) & ~(size_t)255;
    return p;
  };
  const size_t R = FSV_STATIC_MAX_ROWS, B = FSV_STATIC_MAX_BATCH, NC = FSV_STATIC_MAX_NC, NSB = FSV_STATIC_MAX_NSB;
  c.pmax = (float *)take(4 * R * NC); c.psum = (double *)take(8 * R * NC); c.parg = (int32_t *)take(4 * R * NC);
  c.bsum = (double *)take(8 * B * NSB);
  c.acc_scratch = (int32_t *)take(4 * B);
  c.nuc_key = (uint32_t *)take(4 * R); c.nuc_S = (double *)take(8 * R); c.nuc_near = (int32_t *)take(4 * R);
  c.nuc_done = (int32_t *)take(4 * R);
  c.sel_ticket = (int32_t *)take(4 * B);   // starts at zero with the array and is left at zero by every call
  return off <= FSV_STATIC_BYTES;
}

}  // namespace

extern "C" int fsv_sample_static(int32_t vocab, const void *logits, int32_t logits_dtype, const fsv_batch *b,
                                 const fsv_result *r, void *stream) {
  if (!logits || !b || !r || !r->next_token || !r->flags) return FSV_E_INVALID_ARG;
  if (logits_dtype != FSV_F32 && logits_dtype != FSV_BF16) return FSV_E_INVALID_ARG;
  if (vocab <= 0) return FSV_E_INVALID_ARG;
  if (fsv_ceil_div(vocab, FSV_SBK) > FSV_STATIC_MAX_NSB) return FSV_E_CAPACITY;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return FSV_E_HIP;
  if (dev < 0 || dev >= kMaxDevices) return FSV_E_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_static_mu);   // the per-device context below is shared by every call on that device
  if (!g_slots[dev]) g_slots[dev] = new (std::nothrow) static_slot();   // host memory, once per device
  static_slot *slot = g_slots[dev];
  if (!slot) return FSV_E_HIP;
  if (!slot->ready) {
    void *ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return FSV_E_HIP;
    if (!carve_static(slot->ctx, (unsigned char *)ptr)) return FSV_E_UNSUPPORTED;
    slot->ctx.d.max_batch = FSV_STATIC_MAX_BATCH;
    slot->ctx.d.max_gamma = FSV_MAX_GAMMA;
    slot->ctx.d.page_size = 16;
    slot->ctx.max_rows = FSV_STATIC_MAX_ROWS;
    slot->ready = true;
  }
  fsv_ctx *c = &slot->ctx;
  c->d.vocab = vocab;
  c->nsb = fsv_ceil_div(vocab, FSV_SBK);
  c->nc = fsv_ceil_div(vocab, FSV_CHUNK);
  const int M = fsv_check_batch(c, b, false, true);   // batch <= 128, gamma <= 16, rows <= 1024, pointers, temperatures
  if (M <= 0) return M;
  return fsv_launch_sampler(c, logits, logits_dtype, b, r, M, false, (hipStream_t)stream);
}
