// Internal declarations shared by the translation units of libflexverify (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include <stdint.h>
#include <stdio.h>
#include <string>
#include <vector>

#include "attn_schedule.h"
#include "flexverify.h"
#include "wave_ops.h"

#define FSV_WAVE 64

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;   // one MFMA A/B operand (8 bf16 per lane)
typedef __attribute__((ext_vector_type(16))) float f32x16_t;   // one 32x32 MFMA accumulator
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // rows of any length: sixteen bytes at any 4-byte boundary

// ---- sampler geometry -------------------------------------------------------------------------
// A vocabulary row is cut into sub-blocks of SBK ids and chunks of SPC sub-blocks; the statistics
// kernel keeps one (max, sum, argmax) triple per chunk (one wave per chunk), the mass kernel one sum
// per sub-block (one wave per sub-block); the selection kernel scans one sub-block with 256 threads
// x 8 consecutive ids.
#define FSV_SBK 2048
#define FSV_SPC 4
#define FSV_CHUNK (FSV_SBK * FSV_SPC)

// Sum of eight values over the wave, all eight at once: every exchange halves the values a lane still carries, so it takes
// ten exchanges instead of forty-eight.  Lane l ends with the sum of value 4 l5 + 2 l4 + l3 (l5 .. l3: bits of l).
__device__ inline float wave_sum8(float (&v)[8], int lane) {
  const float a0 = lane_fold<32>(v[0], v[4], lane), a1 = lane_fold<32>(v[1], v[5], lane);
  const float a2 = lane_fold<32>(v[2], v[6], lane), a3 = lane_fold<32>(v[3], v[7], lane);
  float r = lane_fold<8>(lane_fold<16>(a0, a2, lane), lane_fold<16>(a1, a3, lane), lane);
  r = lanes_sum<4>(r);
  return r;
}

// Waits until every store this wave has issued is complete (stores count in vmcnt here).  Between blocks of one launch results travel as
// device-scope atomic stores and loads, which bypass the non-coherent caches by themselves; what is left to order is completion.
// Every wave waits here, a barrier collects the waves of the block, and only then is the ticket drawn that tells the other blocks.
// Neither the barrier nor a workgroup-scope release does this wait: outside threadgroup-split mode that release is a wait for lgkmcnt
// alone.  (A device-scope release would also write back the XCD's whole L2 for every block.)
__device__ __forceinline__ void wait_own_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

struct fsv_prof_rec {
  int cls;
  double bytes;
  hipEvent_t e0, e1;
};

struct fsv_layer_w {
  // fp32 path: plain copies [out][in]; bf16 path: re-tiled matrices, plain gains
  void *attn_norm = nullptr, *w_qkv = nullptr, *w_o = nullptr, *mlp_norm = nullptr, *w_gate_up = nullptr,
       *w_down = nullptr;
  // bf16 path: the matrices stored in fp16 carry a power of two; the projection's sums are multiplied by its inverse
  float os_qkv = 1.0f, os_o = 1.0f, os_gate_up = 1.0f;
};

struct fsv_ctx {
  fsv_model_desc d{};
  int max_rows = 0;
  int group = 1;          // query heads per KV head
  int nc = 0;             // vocabulary chunks per row
  int nsb = 0;            // vocabulary sub-blocks per row
  std::string err;

  // weights (library-owned)
  void *embed = nullptr, *final_norm = nullptr, *lm_head = nullptr;
  std::vector<fsv_layer_w> layers;
  float *inv_freq = nullptr;        // [head_dim/2] rotary frequencies (bf16 path; fp64 values)
  float *rope_tab = nullptr;        // [max_rows][head_dim/2][2] cos, sin of the rows of the current call

  // row map, built per call on the device
  int32_t *row_req = nullptr;       // request
  int32_t *row_pos = nullptr;       // fp32 path: position
  int32_t *row_tok = nullptr;       // bf16 path: token
  int32_t *row_place = nullptr;     // bf16 path: [max_rows][4] request, index, position, physical page of the position

  // sampler workspace
  float *pmax = nullptr;    // [max_rows][nc]
  double *psum = nullptr;   // [max_rows][nc]
  int32_t *parg = nullptr;  // [max_rows][nc]
  double *bsum = nullptr;   // [max_batch][nsb]
  int32_t *sel_ticket = nullptr;   // [max_batch] blocks of a request that have left their masses; zero between calls
  int32_t *acc_scratch = nullptr;  // [max_batch] accepted_len when the caller passes none
  // top-k / top-p cut, per logits row: cut key, kept mass (-1: nothing is cut), whether top_p falls near it
  uint32_t *nuc_key = nullptr;
  double *nuc_S = nullptr;
  int32_t *nuc_near = nullptr, *nuc_done = nullptr;   // nuc_done: the one-pass form has settled the row

  // model workspace (both paths)
  float *x = nullptr;       // [rows_pad][d_model] residual stream, fp32
  float *logits = nullptr;  // [max_rows][vocab] fp32 when the caller passes no logits_out
  int strip_pad_bytes = 8192;   // bf16 path: padding between the weight strips of a re-tiled matrix (FSV_STRIP_PAD_KIB overrides)
  int gemm_ncw_force = 0;       // bf16 path: 2..4 = weight strips per GEMM block fixed (FSV_GEMM_NCW, a measurement and test knob)
  int gemm_wide_force = -1;     // bf16 path: FSV_GEMM_WIDE, a measurement and test knob: 0 = never the many-row kernel, 2..4 = always, with that many row tiles per wave
  float os_lm_head = 1.0f;      // bf16 path: inverse of the power of two the fp16 LM-head matrix carries
  uint32_t *absmax = nullptr;   // bf16 path: one word for the largest weight magnitude of the matrix being converted
  void *buf_a = nullptr, *buf_q = nullptr, *buf_att = nullptr,
       *buf_act = nullptr, *buf_part = nullptr;
  size_t part_bytes = 0;
  size_t q_plane_units = 0;     // 16-byte units of one plane of buf_q (bf16 path: plane 0 = hi, plane 1 = lo of the queries)
  void *attn_part = nullptr;    // per-part attention results (O, then (m, l)) of requests with several parts
  size_t attn_part_bytes = 0;
  int n_cus = 0;                // compute units of the device the context was created on
  int attn_wave_target = 0;     // compute units: blocks of eight waves the attention schedule aims at
  int attn_wave_cap = 0;        // blocks the partial buffers hold
  int32_t *attn_ticket = nullptr;  // [max_batch][row tiles][kv heads] parts of the same rows that have left their results; zero between the launches of a call
  int attn_min_tpw = 16, attn_w2 = 20, attn_w3 = 26;   // see attn_shape
  int32_t *attn_part_prefix = nullptr, *attn_part_map = nullptr;   // parts before each request; 28-int record per part

  // LoRA adapters of the evolved target (bf16 path): tables [layer < n_layers - 1][adapter][...], library-owned
  int lora_n = 0, lora_rank = 0;
  uint16_t *lora_aq = nullptr, *lora_bq = nullptr, *lora_ao = nullptr, *lora_bo = nullptr;
  float *lora_scale = nullptr;   // [lora_n]
  float *lora_t = nullptr;       // [max_rows][64] A_qkv x of the rows of the current call

  // head of the edge draft model (bf16 path): re-tiled W_1, W_2, W_v and the operands between them
  int draft_dh = 0, draft_dp = 0;
  void *draft_w1 = nullptr, *draft_w2 = nullptr, *draft_wv = nullptr, *draft_h1 = nullptr, *draft_h2 = nullptr;

  // profiling
  uint32_t prof_mask = 0;
  int prof_every = 1;                     // record every n-th launch of an enabled class (fsv_profile_sample)
  int prof_seen[16] = {0};                // launches of each class seen since profiling was enabled
  std::vector<fsv_prof_rec> prof;
  std::vector<hipEvent_t> prof_pool;      // events of records already read, reused by later records
};

#define FSV_FAIL(ctx, code, ...)                                   \
  do {                                                             \
    char _b[512];                                                  \
    snprintf(_b, sizeof _b, __VA_ARGS__);                          \
    if (ctx) (ctx)->err = _b;                                      \
    return (code);                                                 \
  } while (0)

#define FSV_HIP(ctx, call)                                                                  \
  do {                                                                                      \
    hipError_t _e = (call);                                                                 \
    if (_e != hipSuccess) FSV_FAIL(ctx, FSV_E_HIP, "%s: %s", #call, hipGetErrorString(_e)); \
  } while (0)

// scoped event pair around one kernel class (no-op unless profiling is on).  By default the pair is recorded on the
// stream before and after whatever is launched inside the scope; a launch that can carry its own start / stop events
// (hipExtLaunchKernelGGL) takes them with ext() instead, which times the kernel itself without the dispatch gaps.
struct fsv_prof_scope {
  fsv_ctx *c;
  hipStream_t s;
  fsv_prof_rec r{};
  bool on, external;
  fsv_prof_scope(fsv_ctx *ctx, hipStream_t st, int cls, double bytes, bool ext_mode = false)
      : c(ctx), s(st), on(ctx && ((ctx->prof_mask >> cls) & 1u)), external(ext_mode) {
    if (!on) return;
    if (c->prof_every > 1 && (c->prof_seen[cls]++ % c->prof_every) != 0) { on = false; return; }
    if (c->prof.size() >= 8192) { on = false; return; }
    r.cls = cls;
    r.bytes = bytes;
    auto get = [&](hipEvent_t *e) {
      if (!c->prof_pool.empty()) { *e = c->prof_pool.back(); c->prof_pool.pop_back(); return true; }
      return hipEventCreate(e) == hipSuccess;
    };
    if (!get(&r.e0)) { on = false; return; }
    if (!get(&r.e1)) { c->prof_pool.push_back(r.e0); on = false; return; }
    if (!external) (void)hipEventRecord(r.e0, s);
  }
  hipEvent_t start() const { return (on && external) ? r.e0 : nullptr; }
  hipEvent_t stop() const { return (on && external) ? r.e1 : nullptr; }
  ~fsv_prof_scope() {
    if (!on) return;
    if (!external) (void)hipEventRecord(r.e1, s);
    c->prof.push_back(r);
  }
};

// ---- entry points of the other translation units ----------------------------------------------
// api.hip: CSR shape, capacity and pointer checks shared by the entry points.  Returns the number of rows or a status < 0.
int fsv_check_batch(fsv_ctx *c, const fsv_batch *b, bool need_kv, bool need_sampling);
// sampler.hip
int fsv_launch_build_rows(fsv_ctx *c, const fsv_batch *b, hipStream_t s);
int fsv_launch_sampler(fsv_ctx *c, const void *logits, int logits_dtype, const fsv_batch *b, const fsv_result *r,
                       int M, bool with_rollback, hipStream_t s);
int fsv_launch_draft_law(fsv_ctx *c, const float *z, const fsv_batch *b, int all_rows, float *q, hipStream_t s);
int fsv_launch_rollback(fsv_ctx *c, const fsv_batch *b, const int32_t *accepted, const fsv_result *r, hipStream_t s);
// path_f32.hip
int fsv_f32_create(fsv_ctx *c, const fsv_weights *w);
int fsv_f32_check(fsv_ctx *c, const fsv_batch *b);   // host only: what the launches of a forward / attention need
int fsv_f32_forward(fsv_ctx *c, const fsv_batch *b, int M, float *logits, hipStream_t s);
int fsv_f32_linear(fsv_ctx *c, int which, int layer, const void *x, int M, float *y, hipStream_t s);
int fsv_f32_attention(fsv_ctx *c, int layer, const void *q, const fsv_batch *b, int M, float *out, hipStream_t s);
int fsv_f32_kv_copy(fsv_ctx *c, void *k_pool, void *v_pool, int num_pages, const int32_t *pt_row, int pos0, int n,
                    void *k_lin, void *v_lin, bool import, hipStream_t s);
// attn_bf16.hip
int fsv_bf16_attn_create(fsv_ctx *c);
int fsv_bf16_attn_plan_host(fsv_ctx *c, const fsv_batch *b, fsv_attn_plan *pl);          // host only; may fail
// row map, attention schedule and (rope) rotation angles of a call, on the device; q: rotated queries to put into the query
// operand (the stand-alone attention), or NULL
int fsv_bf16_setup_launch(fsv_ctx *c, const fsv_batch *b, const fsv_attn_plan *pl, int M, bool rope, const void *q, hipStream_t s);
// out32: row-major fp32 result [M][heads * hd], or NULL = the operand of the output projection (buf_att)
int fsv_bf16_attn_launch(fsv_ctx *c, const fsv_batch *b, const fsv_attn_plan *pl, size_t layer_off, float *out32, hipStream_t s);
// gemm_bf16.hip: y = x W^T, through the many-row kernel with `wide` row tiles per wave or (wide 0) the weight-streaming one; epi 0 = fp32 split partials [splits][Mpad][N],
// 1 = SwiGLU to the bf16 operand order, 2 = fp32 rows [M][N]
int fsv_bf16_gemm_init(fsv_ctx *c);
int fsv_bf16_gemm(fsv_ctx *c, int cls, int epi, const void *Wp, const void *Ap, void *out, int N, int K, int NTpad, int M,
                  int splits, int KBo, int f16, float oscale, int ncw, int wide, hipStream_t st);
// gemm_wide.hip: the many-row kernel, mt row tiles per wave
int fsv_bf16_gemm_wide_init(fsv_ctx *c);
int fsv_bf16_gemm_wide(fsv_ctx *c, int cls, int epi, const void *Wp, const void *Ap, void *out, int N, int K, int NTpad, int M, int splits,
                       int KBo, int f16, float oscale, int mt, hipStream_t st);
// few_rows.hip: the projections of a layer for calls of up to 16 rows, with what precedes and follows them.  strip_bytes, wbytes: distance
// between the weight strips, size of the re-tiled matrix
bool fsv_bf16_few_rows(const fsv_ctx *c, int M);
int fsv_bf16_few_qkv(fsv_ctx *c, const fsv_batch *b, const void *Wp, const void *gain, uint32_t strip_bytes, uint32_t wbytes, int N, int M,
                     float oscale, size_t layer_off, hipStream_t st);   // norm of x, q|k|v, rotation, query operand, KV append
int fsv_bf16_few_gate_up(fsv_ctx *c, const void *Wp, const void *gain, uint32_t strip_bytes, uint32_t wbytes, int N, int M, float oscale,
                         hipStream_t st);                                // norm of x, gate|up, SwiGLU
int fsv_bf16_few_add(fsv_ctx *c, int cls, const void *Wp, const void *Ap, uint32_t strip_bytes, uint32_t wbytes, int N, int K, int M, int f16,
                     float oscale, hipStream_t st);                      // x += W a
// path_bf16.hip
int fsv_bf16_create(fsv_ctx *c, const fsv_weights *w);
int fsv_bf16_forward(fsv_ctx *c, const fsv_batch *b, const fsv_attn_plan *pl, int M, float *logits, int draft, hipStream_t s);
int fsv_bf16_draft_attach(fsv_ctx *c, const fsv_draft_head *h);
int fsv_bf16_draft_probs(fsv_ctx *c, const fsv_batch *b, const fsv_attn_plan *pl, int M, int all_rows, float *q_out, float *logits,
                         hipStream_t s);
int fsv_bf16_linear(fsv_ctx *c, int which, int layer, const void *x, int M, float *y, hipStream_t s);
int fsv_bf16_lora_load(fsv_ctx *c, const fsv_lora *lo);
int fsv_bf16_attention(fsv_ctx *c, int layer, const void *q, const fsv_batch *b, const fsv_attn_plan *pl, int M, float *out,
                       hipStream_t s);
int fsv_bf16_kv_copy(fsv_ctx *c, void *k_pool, void *v_pool, int num_pages, const int32_t *pt_row, int pos0, int n,
                     void *k_lin, void *v_lin, bool import, int layers, hipStream_t s);
void fsv_free_weights(fsv_ctx *c);
