// FSV_F32 instantiation of the target forward (Alg. 2 step 2: the target model scores the pending
// token and the draft block on top of the restored KV session, Sec. IV-C).  This is the
// correctness configuration (a tiny fp32 decoder): plain fp32 kernels, no matrix cores; norms, rotation,
// KV append and SwiGLU are part of the projections' launches.  The bf16 path in path_bf16.hip is the one built for throughput.
#include <math.h>

#include "fsv_internal.h"

namespace {

// The rows of a call, their embeddings and the cos, sin of their rotation angles (fp64 angles; the same in every layer), a block per
// row: its request is the last one whose first row, off[b] + b, is not beyond it (every wave by itself, 64 requests at a time).  One launch instead of two: 2.2 + 2.4 -> 3.5 us for 5 rows, the angles included.
__global__ void k_embed_rows(int B, int V, int d, const int32_t *__restrict__ seq_lens, const int32_t *__restrict__ last_token,
                             const int32_t *__restrict__ off, const int32_t *__restrict__ draft, const float *__restrict__ E,
                             int32_t *__restrict__ row_req, int32_t *__restrict__ row_pos, float *__restrict__ x, int hd, double theta,
                             float2 *__restrict__ tab) {
  const int r = blockIdx.x, lane = threadIdx.x & 63;
  int b = -1;
  for (int b0 = 0; b0 < B; b0 += 64) b += __popcll(__ballot(b0 + lane < B && off[min(b0 + lane, B)] + b0 + lane <= r));
  const int i = r - off[b] - b;
  const int t = (i == 0) ? (last_token ? last_token[b] : 0) : (draft ? draft[r - b - 1] : 0);
  const int pos = (seq_lens ? seq_lens[b] : 0) + i;
  if (threadIdx.x == 0) {
    row_req[r] = b;
    row_pos[r] = pos;
  }
  const float *src = E + (size_t)min(max(t, 0), V - 1) * d;
  for (int k = threadIdx.x; k < d; k += blockDim.x) x[(size_t)r * d + k] = src[k];
  const int half = hd / 2;
  for (int f = threadIdx.x; f < half; f += blockDim.x) {
    const double ang = (double)pos * pow(theta, -2.0 * (double)f / (double)hd);
    tab[(size_t)r * half + f] = make_float2((float)cos(ang), (float)sin(ang));
  }
}

// y[m][n] (+)= sum_k a[m][k] w[n][k]; one wave per output column and eight rows, lanes stride over k.
// NORM: the rows are RMS-normalised on the way, y = (sum a g w) / sqrt(mean(a^2) + eps): a wave reads whole rows anyway, so
// the sum of squares costs an operation per element and saves a launch and a pass.  SWIGLU: columns n and n + N of w are gate
// and up, y = silu(gate) up, for the same reason.  ROWS = 1 for a call of one row: seven repeated rows cost nothing on a small
// matrix, but 131 MB of head take 34 us with them and 19 without (26 before rows were taken by eight).
// Bound by latency at the sizes this path is for (5 rows, 256 .. 4096 columns): one round of loads and ten exchanges per eight
// rows.  Measured there: 3.4 .. 5.0 us per projection against 7.6 .. 15.3 us row by row plus 4.2 us per norm and 3.4 for SwiGLU.
template <bool NORM, bool SWIGLU, int ROWS>
__global__ __launch_bounds__(256) void k_linear(int M, int N, int K, float eps, const float *__restrict__ a, const float *__restrict__ g,
                                                const float *__restrict__ w, float *__restrict__ y, int accumulate, int vec) {
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (n >= N) return;
  // the same sums in the same order for one row as for eight: a row's result does not depend on its batch
  auto sums_of = [lane](float(&v)[ROWS]) {
    if constexpr (ROWS == 1) return wave_sum(v[0]);
    else return wave_sum8(v, lane);
  };
  const float *wr = w + (size_t)n * K, *wu = wr + (SWIGLU ? (size_t)N * K : 0);
  for (int m0 = blockIdx.y * ROWS; m0 < M; m0 += gridDim.y * ROWS) {
    const float *ar[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) ar[i] = a + (size_t)min(m0 + i, M - 1) * K;   // (rows beyond M repeat the last; not stored)
    float acc[ROWS], up[ROWS], ss[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) acc[i] = up[i] = ss[i] = 0.f;
    auto add = [&](int i, float av, float wv, float uv, float gv) {
      const float x = NORM ? av * gv : av;
      acc[i] = fmaf(x, wv, acc[i]);
      if (SWIGLU) up[i] = fmaf(x, uv, up[i]);
      if (NORM) ss[i] = fmaf(av, av, ss[i]);
    };
    const int m = m0 + (ROWS == 1 ? 0 : ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1));
    const bool mine = !(lane & (ROWS == 1 ? 63 : 7)) && m < M;
    const size_t o = (size_t)min(m, M - 1) * N + n;
    const float before = (accumulate && mine) ? y[o] : 0.f;   // fetched with the first operands
    if (vec) {
      for (int k = lane * 4; k < K; k += 256) {
        const float4 w4 = *reinterpret_cast<const float4 *>(wr + k);
        const float4 u4 = SWIGLU ? *reinterpret_cast<const float4 *>(wu + k) : w4;
        const float4 g4 = NORM ? *reinterpret_cast<const float4 *>(g + k) : w4;
        float4 a4[ROWS];
#pragma unroll
        for (int i = 0; i < ROWS; ++i) a4[i] = *reinterpret_cast<const float4 *>(ar[i] + k);
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
          add(i, a4[i].x, w4.x, u4.x, g4.x);
          add(i, a4[i].y, w4.y, u4.y, g4.y);
          add(i, a4[i].z, w4.z, u4.z, g4.z);
          add(i, a4[i].w, w4.w, u4.w, g4.w);
        }
      }
    } else {
      for (int k = lane; k < K; k += 64) {
        const float w1 = wr[k], u1 = SWIGLU ? wu[k] : 0.f, g1 = NORM ? g[k] : 0.f;
#pragma unroll
        for (int i = 0; i < ROWS; ++i) add(i, ar[i][k], w1, u1, g1);
      }
    }
    float r = sums_of(acc);
    const float u = SWIGLU ? sums_of(up) : 0.f;
    const float rinv = NORM ? 1.0f / sqrtf(sums_of(ss) / (float)K + eps) : 1.0f;
    if (!mine) continue;
    r *= rinv;
    if (SWIGLU) r = r / (1.0f + expf(-r)) * (u * rinv);
    y[o] = accumulate ? before + r : r;
  }
}

// q|k|v = norm(a) w^T, q and k rotated by their position (half-split pairing), q to qbuf and k, v into the paged pools: k_linear's
// sums in k_linear's order, a wave per pair of features (i, i + hd / 2) and eight rows, so that the lane that ends up with both turns
// and stores them.  A launch for the rotation took 4.1 us beside the projection's 3.7 (5 rows, with the angles in fp64 every time); this takes 4.9.
template <int ROWS>
__global__ __launch_bounds__(256) void k_qkv_rope(int M, int H, int Hkv, int hd, int K, float eps, const float2 *__restrict__ tab, int num_pages, int max_pages,
                                                  const float *__restrict__ a, const float *__restrict__ g, const float *__restrict__ w,
                                                  const int32_t *__restrict__ row_req, const int32_t *__restrict__ row_pos,
                                                  const int32_t *__restrict__ page_table, float *__restrict__ qbuf, float *__restrict__ kpool,
                                                  float *__restrict__ vpool, size_t layer_off, int page_size, int vec) {
  const int pair = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, half = hd / 2;
  if (pair >= (H + 2 * Hkv) * half) return;
  const int h = pair / half, f = pair - h * half;
  auto sums_of = [lane](float(&v)[ROWS]) {
    if constexpr (ROWS == 1) return wave_sum(v[0]);
    else return wave_sum8(v, lane);
  };
  const float *w0 = w + (size_t)(h * hd + f) * K, *w1 = w0 + (size_t)half * K;
  for (int m0 = blockIdx.y * ROWS; m0 < M; m0 += gridDim.y * ROWS) {
    const float *ar[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) ar[i] = a + (size_t)min(m0 + i, M - 1) * K;   // (rows beyond M repeat the last; not stored)
    const int m = m0 + (ROWS == 1 ? 0 : ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1)), mc = min(m, M - 1);
    const bool mine = !(lane & (ROWS == 1 ? 63 : 7)) && m < M;
    const int pos = row_pos[mc], b = row_req[mc];
    const float2 cs_sn = tab[(size_t)mc * half + f];
    float lo[ROWS], hi[ROWS], ss[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) lo[i] = hi[i] = ss[i] = 0.f;
    auto add = [&](int i, float av, float v0, float v1, float gv) {
      const float x = av * gv;
      lo[i] = fmaf(x, v0, lo[i]);
      hi[i] = fmaf(x, v1, hi[i]);
      ss[i] = fmaf(av, av, ss[i]);
    };
    if (vec) {
      for (int k = lane * 4; k < K; k += 256) {
        const float4 p4 = *reinterpret_cast<const float4 *>(w0 + k), q4 = *reinterpret_cast<const float4 *>(w1 + k);
        const float4 g4 = *reinterpret_cast<const float4 *>(g + k);
        float4 a4[ROWS];
#pragma unroll
        for (int i = 0; i < ROWS; ++i) a4[i] = *reinterpret_cast<const float4 *>(ar[i] + k);
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
          add(i, a4[i].x, p4.x, q4.x, g4.x);
          add(i, a4[i].y, p4.y, q4.y, g4.y);
          add(i, a4[i].z, p4.z, q4.z, g4.z);
          add(i, a4[i].w, p4.w, q4.w, g4.w);
        }
      }
    } else {
      for (int k = lane; k < K; k += 64) {
        const float v0 = w0[k], v1 = w1[k], g1 = g[k];
#pragma unroll
        for (int i = 0; i < ROWS; ++i) add(i, ar[i][k], v0, v1, g1);
      }
    }
    // page ids live on the device: an id outside the pool is clamped into it (wrong data, never a wild write)
    const int page = min(max(page_table[(size_t)b * max_pages + pos / page_size], 0), num_pages - 1), slot = pos % page_size;
    const float cs = cs_sn.x, sn = cs_sn.y;
    const float s0 = sums_of(lo), s1 = sums_of(hi), rinv = 1.0f / sqrtf(sums_of(ss) / (float)K + eps);
    if (!mine) continue;
    const float x0 = s0 * rinv, x1 = s1 * rinv;
    float *dst;
    if (h < H) dst = qbuf + ((size_t)m * H + h) * hd;
    else if (h < H + Hkv) dst = kpool + layer_off + (((size_t)page * Hkv + (h - H)) * page_size + slot) * hd;
    else dst = vpool + layer_off + (((size_t)page * Hkv + (h - H - Hkv)) * page_size + slot) * hd;
    dst[f] = h < H + Hkv ? x0 * cs - x1 * sn : x0;
    dst[f + half] = h < H + Hkv ? x0 * sn + x1 * cs : x1;
  }
}

// One block per (row, query head): scores into LDS (sixteen lanes per key, two pages of keys per step of the block), softmax, then
// the weighted sum of values with the keys dealt to groups of threads, added up in group order.  The page ids are in LDS before
// the loops, so that every loop's loads are independent.
// Bound by latency; 133 keys of 64: 8.7 us, against 38 us for one wave that went from key to key.  Eight waves per block
// and no integer division per key: 12 -> 8.7 us, 162 -> 112 us for a two-layer call of 16 rows at 1000 positions, 1030 -> 907 us
// for a prefill of 1024 rows (sixteen waves: the single call 9.8 against 10 us before the division went, the prefill 12 % slower).
constexpr int ATT_SUMS = 512;   // (feature, group of keys) pairs, whatever the block: a row's result does not depend on its batch
template <int ATT>
__global__ __launch_bounds__(ATT) void k_attention(int H, int Hkv, int hd, int max_pages, int num_pages, int page_size, int key_cap,
                                                  const float *__restrict__ qbuf, const int32_t *__restrict__ row_req,
                                                  const int32_t *__restrict__ row_pos, const int32_t *__restrict__ page_table,
                                                  const float *__restrict__ kpool, const float *__restrict__ vpool,
                                                  size_t layer_off, float *__restrict__ out) {
  extern __shared__ float sc[];   // [key_cap] scores, then [key_cap / page_size + 1] page ids, then [ATT_SUMS] partial sums
  __shared__ float s_red[ATT / 64];
  const int r = blockIdx.x, h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int b = row_req[r], nkeys = min(row_pos[r] + 1, key_cap), kvh = h / (H / Hkv), npg = (nkeys + page_size - 1) / page_size;
  int32_t *s_pg = reinterpret_cast<int32_t *>(sc + key_cap);
  float *s_part = reinterpret_cast<float *>(s_pg + key_cap / page_size + 1);
  for (int p = tid; p < npg; p += ATT) s_pg[p] = min(max(page_table[(size_t)b * max_pages + p], 0), num_pages - 1);
  __syncthreads();
  const float inv_page = 1.0f / (float)page_size;
  auto row_of = [&](const float *pool, int j) {
    const int p = (int)(((float)j + 0.5f) * inv_page);   // exact: j + 1/2 is 1/2 of a key away from a page's edge, keys stay below 2^15
    return pool + layer_off + (((size_t)s_pg[p] * Hkv + kvh) * page_size + (j - p * page_size)) * hd;
  };
  const float *q = qbuf + ((size_t)r * H + h) * hd;
  const float scale = 1.0f / sqrtf((float)hd);
  const int l16 = tid & 15;
  float mx = -INFINITY;
  auto score = [&](int j, float s) {   // all sixteen lanes of a key
    s = lanes_sum<8>(s);
    s *= scale;
    if (j < nkeys) {
      if (l16 == 0) sc[j] = s;
      mx = fmaxf(mx, s);
    }
  };
  constexpr int KPS = ATT / 16, U = 4, EP = 4;   // keys per step, steps in flight, feature pairs per lane (head_dim up to 128)
  if (hd <= 32 * EP) {
    float qv[EP][2];
#pragma unroll
    for (int i = 0; i < EP; ++i) {
      const int e = 2 * l16 + 32 * i;   // (head_dim is even)
      qv[i][0] = e < hd ? q[e] : 0.f;
      qv[i][1] = e < hd ? q[e + 1] : 0.f;
    }
    for (int j0 = tid >> 4; j0 < nkeys; j0 += KPS * U) {   // (the same trips for the four keys of a wave's step, and beyond: clamped)
      float kv[U][EP][2];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float *kr = row_of(kpool, min(j0 + u * KPS, nkeys - 1));
#pragma unroll
        for (int i = 0; i < EP; ++i) {
          const int e = min(2 * l16 + 32 * i, hd - 2);
          kv[u][i][0] = kr[e];
          kv[u][i][1] = kr[e + 1];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < EP; ++i) {
          if (2 * l16 + 32 * i >= hd) continue;   // (a clamped pair: not a feature of this lane)
          s = fmaf(qv[i][0], kv[u][i][0], s);
          s = fmaf(qv[i][1], kv[u][i][1], s);
        }
        score(j0 + u * KPS, s);
      }
    }
  } else {
    for (int j = tid >> 4; j < nkeys; j += KPS) {
      const float *kr = row_of(kpool, j);
      float s = 0.f;
      for (int e = 2 * l16; e < hd; e += 32) {
        s = fmaf(q[e], kr[e], s);
        s = fmaf(q[e + 1], kr[e + 1], s);
      }
      score(j, s);
    }
  }
  mx = lanes_max(mx);
  if (lane == 0) s_red[w] = mx;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < ATT / 64; ++i) mx = fmaxf(mx, s_red[i]);
  float den = 0.f;
  for (int j = tid; j < nkeys; j += ATT) {
    const float p = expf(sc[j] - mx);
    sc[j] = p;
    den += p;
  }
  den = wave_sum(den);
  __syncthreads();   // (s_red has been read, the scores are probabilities)
  if (lane == 0) s_red[w] = den;
  auto total = [&]() {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < ATT / 64; ++i) t += s_red[i];
    return t;
  };
  float *dst = out + ((size_t)r * H + h) * hd;
  if (hd > ATT) {   // block-uniform; a thread has several features
    __syncthreads();
    den = total();
    for (int e = tid; e < hd; e += ATT) {
      float acc = 0.f;
#pragma unroll 4
      for (int j = 0; j < nkeys; ++j) acc = fmaf(sc[j], row_of(vpool, j)[e], acc);
      dst[e] = acc / den;
    }
    return;
  }
  const int groups = ATT_SUMS / hd;
  for (int i = tid; i < groups * hd; i += ATT) {
    const int g = i / hd, e = i - g * hd;
    float acc = 0.f;
#pragma unroll 8
    for (int j = g; j < nkeys; j += groups) acc = fmaf(sc[j], row_of(vpool, j)[e], acc);
    s_part[i] = acc;
  }
  __syncthreads();
  den = total();
  if (tid < hd) {
    float acc = 0.f;
    for (int i = 0; i < groups; ++i) acc += s_part[i * hd + tid];
    dst[tid] = acc / den;
  }
}

__global__ void k_kv_copy(int Hkv, int hd, int page_size, int n_layers, int num_pages, const int32_t *__restrict__ pt,
                          int pos0, int n, float *__restrict__ kpool, float *__restrict__ vpool, float *__restrict__ klin,
                          float *__restrict__ vlin, int import) {
  // one block per (position, layer)
  const int p = blockIdx.x, l = blockIdx.y, pos = pos0 + p;
  const size_t layer_off = (size_t)l * num_pages * Hkv * page_size * hd;
  const int page = min(max(pt[pos / page_size], 0), num_pages - 1), slot = pos % page_size;
  for (int t = threadIdx.x; t < Hkv * hd; t += blockDim.x) {
    const int h = t / hd, e = t % hd;
    const size_t pi = layer_off + (((size_t)page * Hkv + h) * page_size + slot) * hd + e;
    const size_t li = (((size_t)l * n + p) * Hkv + h) * hd + e;
    if (import) { kpool[pi] = klin[li]; vpool[pi] = vlin[li]; }
    else { klin[li] = kpool[pi]; vlin[li] = vpool[pi]; }
  }
}

int dev_copy(fsv_ctx *c, void **dst, const void *src, size_t bytes) {
  FSV_HIP(c, hipMalloc(dst, bytes));
  FSV_HIP(c, hipMemcpy(*dst, src, bytes, hipMemcpyDeviceToDevice));
  return FSV_OK;
}

size_t layer_stride(const fsv_ctx *c, int num_pages) {
  return (size_t)num_pages * c->d.n_kv_heads * c->d.page_size * c->d.head_dim;
}

// y (+)= a w^T; with gains: of the RMS-normalised rows; swiglu: w holds gate then up, N = columns of each
void launch_linear(int M, int N, int K, const float *a, const float *w, float *y, int acc, hipStream_t s, const float *gain = nullptr,
                   float eps = 0.f, bool swiglu = false) {
  const int vec = (K % 4 == 0 && (((uintptr_t)a | (uintptr_t)w | (uintptr_t)gain) % 16) == 0) ? 1 : 0;
  // row blocks side by side only as far as the columns alone leave the chip idle; the rest in turn, the weight row still in L1
  const int nb = fsv_ceil_div(N, 4);
  const dim3 grid(nb, max(1, min(fsv_ceil_div(M, 8), 2048 / nb)));
#define FSV_F32_LIN(NORM, SWIGLU)                                                                                                    \
  do {                                                                                                                              \
    if (M == 1) hipLaunchKernelGGL((k_linear<NORM, SWIGLU, 1>), grid, dim3(256), 0, s, M, N, K, eps, a, gain, w, y, acc, vec);       \
    else hipLaunchKernelGGL((k_linear<NORM, SWIGLU, 8>), grid, dim3(256), 0, s, M, N, K, eps, a, gain, w, y, acc, vec);              \
  } while (0)
  if (swiglu) FSV_F32_LIN(true, true);
  else if (gain) FSV_F32_LIN(true, false);
  else FSV_F32_LIN(false, false);
#undef FSV_F32_LIN
}

// LDS of k_attention for key_cap keys: 70.0 KiB at the 16384 that fsv_f32_check admits
constexpr int ATT_WIDE = 512, ATT_NARROW = 128;   // threads per block
size_t attention_lds(const fsv_model_desc &d, int key_cap) {
  return sizeof(float) * ((size_t)key_cap + key_cap / d.page_size + 1 + ATT_SUMS);
}

void launch_attention(const fsv_model_desc &d, const fsv_ctx *c, const fsv_batch *b, int M, int keys, const float *q, size_t lo, float *out,
                      hipStream_t s) {
#define FSV_F32_ATT(T)                                                                                                              \
  hipLaunchKernelGGL(k_attention<T>, dim3(M, d.n_heads), dim3(T), attention_lds(d, keys), s, d.n_heads, d.n_kv_heads, d.head_dim, \
                     d.max_pages_per_req, b->num_pages, d.page_size, keys, q, c->row_req, c->row_pos, b->page_table,                \
                     (const float *)b->k_pool, (const float *)b->v_pool, lo, out)
  // Many blocks of few keys run in rounds, and eight waves of a block then have less to do than it takes to start them: 4096 blocks
  // of 24 keys 34 us with 512 threads, 20 with 128, of 40 keys 38 and 27.  Up to 1024 blocks both take the same up to 64 keys, and
  // 128 threads fall behind beyond (1024 blocks of 254 keys 27 us and 32), as they do where a thread has several features.
  if (keys <= 64 && d.head_dim <= ATT_NARROW && (long)M * d.n_heads >= 2048) FSV_F32_ATT(ATT_NARROW);
  else FSV_F32_ATT(ATT_WIDE);
#undef FSV_F32_ATT
}

}  // namespace

int fsv_f32_create(fsv_ctx *c, const fsv_weights *w) {
  const fsv_model_desc &d = c->d;
  const size_t f = sizeof(float);
  const int qd = d.n_heads * d.head_dim, qkvd = (d.n_heads + 2 * d.n_kv_heads) * d.head_dim;
  int rc;
  if ((rc = dev_copy(c, &c->embed, w->embed, f * d.vocab * d.d_model))) return rc;
  if ((rc = dev_copy(c, &c->final_norm, w->final_norm, f * d.d_model))) return rc;
  if ((rc = dev_copy(c, &c->lm_head, w->lm_head, f * d.vocab * d.d_model))) return rc;
  c->layers.resize(d.n_layers);
  for (int l = 0; l < d.n_layers; ++l) {
    fsv_layer_w &L = c->layers[l];
    if ((rc = dev_copy(c, &L.attn_norm, w->attn_norm[l], f * d.d_model))) return rc;
    if ((rc = dev_copy(c, &L.w_qkv, w->w_qkv[l], f * qkvd * d.d_model))) return rc;
    if ((rc = dev_copy(c, &L.w_o, w->w_o[l], f * d.d_model * qd))) return rc;
    if ((rc = dev_copy(c, &L.mlp_norm, w->mlp_norm[l], f * d.d_model))) return rc;
    if ((rc = dev_copy(c, &L.w_gate_up, w->w_gate_up[l], f * 2 * d.d_ffn * d.d_model))) return rc;
    if ((rc = dev_copy(c, &L.w_down, w->w_down[l], f * d.d_model * d.d_ffn))) return rc;
  }
  if (attention_lds(d, min(16384, d.max_pages_per_req * d.page_size)) > 64 * 1024)   // beyond what a launch may take unasked
    FSV_HIP(c, hipFuncSetAttribute(reinterpret_cast<const void *>(&k_attention<ATT_WIDE>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)attention_lds(d, 16384)));
  const size_t R = c->max_rows;
  FSV_HIP(c, hipMalloc(&c->buf_q, f * R * qd));
  FSV_HIP(c, hipMalloc((void **)&c->rope_tab, f * R * d.head_dim));
  FSV_HIP(c, hipMalloc(&c->buf_att, f * R * qd));
  FSV_HIP(c, hipMalloc(&c->buf_act, f * R * d.d_ffn));
  return FSV_OK;
}

static int max_keys_of(const fsv_batch *b) {
  int max_keys = 0;
  for (int i = 0; i < b->batch; ++i) {
    int g = b->draft_offsets_host[i + 1] - b->draft_offsets_host[i];
    max_keys = max(max_keys, b->seq_lens_host[i] + g + 1);
  }
  return max_keys;
}

int fsv_f32_check(fsv_ctx *c, const fsv_batch *b) {
  const int max_keys = max_keys_of(b);
  if (sizeof(float) * (size_t)max_keys > 64 * 1024)
    FSV_FAIL(c, FSV_E_UNSUPPORTED, "fp32 path: %d keys exceed the 16384 it keeps in LDS", max_keys);
  return FSV_OK;
}

int fsv_f32_forward(fsv_ctx *c, const fsv_batch *b, int M, float *logits, hipStream_t s) {
  const fsv_model_desc &d = c->d;
  const int qd = d.n_heads * d.head_dim, qkvd = (d.n_heads + 2 * d.n_kv_heads) * d.head_dim;
  float *x = c->x, *qb = (float *)c->buf_q;
  float *att = (float *)c->buf_att, *act = (float *)c->buf_act;
  const int keys = max_keys_of(b);   // fsv_f32_check has bounded it
  hipLaunchKernelGGL(k_embed_rows, dim3(M), dim3(256), 0, s, b->batch, d.vocab, d.d_model, b->seq_lens, b->last_token, b->draft_offsets,
                     b->draft_tokens, (const float *)c->embed, c->row_req, c->row_pos, x, d.head_dim, (double)d.rope_theta, (float2 *)c->rope_tab);
  for (int l = 0; l < d.n_layers; ++l) {
    const fsv_layer_w &L = c->layers[l];
    const size_t lo = (size_t)l * layer_stride(c, b->num_pages);
    {
      const int nb = fsv_ceil_div(qkvd / 2, 4), vec = (d.d_model % 4 == 0 && (((uintptr_t)x | (uintptr_t)L.w_qkv | (uintptr_t)L.attn_norm) % 16) == 0) ? 1 : 0;
      const dim3 grid(nb, max(1, min(fsv_ceil_div(M, 8), 2048 / nb)));
#define FSV_F32_QKV(R)                                                                                                               \
  hipLaunchKernelGGL((k_qkv_rope<R>), grid, dim3(256), 0, s, M, d.n_heads, d.n_kv_heads, d.head_dim, d.d_model, d.rms_eps,              \
                     (const float2 *)c->rope_tab, b->num_pages, d.max_pages_per_req, x, (const float *)L.attn_norm, (const float *)L.w_qkv,     \
                     c->row_req, c->row_pos, b->page_table, qb, (float *)b->k_pool, (float *)b->v_pool, lo, d.page_size, vec)
      if (M == 1) FSV_F32_QKV(1);
      else FSV_F32_QKV(8);
#undef FSV_F32_QKV
    }
    launch_attention(d, c, b, M, keys, qb, lo, att, s);
    launch_linear(M, d.d_model, qd, att, (const float *)L.w_o, x, 1, s);
    launch_linear(M, d.d_ffn, d.d_model, x, (const float *)L.w_gate_up, act, 0, s, (const float *)L.mlp_norm, d.rms_eps, true);
    launch_linear(M, d.d_model, d.d_ffn, act, (const float *)L.w_down, x, 1, s);
  }
  launch_linear(M, d.vocab, d.d_model, x, (const float *)c->lm_head, logits, 0, s, (const float *)c->final_norm, d.rms_eps);
  FSV_HIP(c, hipGetLastError());
  return FSV_OK;
}

int fsv_f32_linear(fsv_ctx *c, int which, int layer, const void *x, int M, float *y, hipStream_t s) {
  const fsv_model_desc &d = c->d;
  const int qd = d.n_heads * d.head_dim, qkvd = (d.n_heads + 2 * d.n_kv_heads) * d.head_dim;
  const float *w;
  int N, K;
  switch (which) {
    case FSV_W_QKV: w = (const float *)c->layers[layer].w_qkv; N = qkvd; K = d.d_model; break;
    case FSV_W_O: w = (const float *)c->layers[layer].w_o; N = d.d_model; K = qd; break;
    case FSV_W_GATE_UP: w = (const float *)c->layers[layer].w_gate_up; N = 2 * d.d_ffn; K = d.d_model; break;
    case FSV_W_DOWN: w = (const float *)c->layers[layer].w_down; N = d.d_model; K = d.d_ffn; break;
    default: w = (const float *)c->lm_head; N = d.vocab; K = d.d_model; break;
  }
  launch_linear(M, N, K, (const float *)x, w, y, 0, s);
  FSV_HIP(c, hipGetLastError());
  return FSV_OK;
}

int fsv_f32_attention(fsv_ctx *c, int layer, const void *q, const fsv_batch *b, int M, float *out, hipStream_t s) {
  const fsv_model_desc &d = c->d;
  const int keys = max_keys_of(b);   // fsv_f32_check has bounded it
  const size_t lo = (size_t)layer * layer_stride(c, b->num_pages);
  launch_attention(d, c, b, M, keys, (const float *)q, lo, out, s);
  FSV_HIP(c, hipGetLastError());
  return FSV_OK;
}

int fsv_f32_kv_copy(fsv_ctx *c, void *k_pool, void *v_pool, int num_pages, const int32_t *pt_row, int pos0, int n,
                    void *k_lin, void *v_lin, bool import, hipStream_t s) {
  const fsv_model_desc &d = c->d;
  hipLaunchKernelGGL(k_kv_copy, dim3(n, d.n_layers), dim3(256), 0, s, d.n_kv_heads, d.head_dim, d.page_size,
                     d.n_layers, num_pages, pt_row, pos0, n, (float *)k_pool, (float *)v_pool, (float *)k_lin,
                     (float *)v_lin, import ? 1 : 0);
  FSV_HIP(c, hipGetLastError());
  return FSV_OK;
}
