// The attention schedule of a call, from the host copies of its lengths: plain C++, so that it can be looked at without a GPU.
#pragma once
#include <algorithm>
#include <climits>
#include <cstdint>

static inline int fsv_ceil_div(int a, int b) { return (a + b - 1) / b; }

// parts of a request with n key tiles when a part of a request with ONE query-row tile should hold about tpw tiles; *tp = tiles per
// part.  A key tile costs more when the request has more query rows (the score and value
// products and the softmax arithmetic on the same K and V), so such a request is cut into shorter parts, by the
// cost ratio w16 / 16: 16 requests, 512 .. 4096 positions, 1 .. 9 rows: 35 us with all tiles alike, 30.7 with 20 / 16 for two row tiles
// and 26 / 16 for three, 31.5 with 26 / 16 and 36 / 16.  As many parts as parts of whole rounds of the waves would be, but alike: 1909 ..
// 2674 positions, 12 requests, 28.8 us a layer with parts of whole rounds, 27.3 like this.  Up to two tiles a wave are one part: two of half
// of it take 2.0 us longer with one row tile (10 key tiles 11.3 and 9.3 us), 2.4 with two.
__host__ __device__ inline int attn_parts(int n, int tpw, int w16, int nw, int *tp) {
  tpw = n <= 2 * nw ? n : tpw * 16 / w16 > 1 ? tpw * 16 / w16 : 1;
  const int s0 = (n + tpw - 1) / tpw, whole = ((n + s0 - 1) / s0 + nw - 1) / nw * nw, parts = (n + whole - 1) / whole;
  *tp = (n + parts - 1) / parts;
  return parts;
}

struct fsv_attn_plan {
  int tpw = 0;          // target key tiles per part
  int waves = 0;        // parts x kv heads: blocks
  int rt = 1;           // query-row tiles of the widest part
  int nw = 8;           // waves per block
  bool split = false;   // the row tiles of a request are parts of their own
  bool sorted = false;  // the parts run in several rounds, long ones first
  double kv_tokens = 0;
};

// What the schedule depends on besides the lengths.  target: blocks of eight waves it aims at; min_tpw: fewest key tiles a part is given, two
// per wave: one 2048-position request 11.2 us, with 24 tiles 11.7 (half of it in short requests, see below); w2, w3: cost of a key tile for a request
// with two / three query-row tiles, in 1/16 of one with one
struct attn_shape {
  int head_dim, n_kv_heads, group, n_cus, target, min_tpw, w2, w3;
};

// A call's lengths and what follows from them alone.
struct attn_call {
  const attn_shape &sh;
  int batch;
  const int32_t *seq_lens, *offsets;
  int max_rows = 0, longest = 0;    // query rows of the widest request, key tiles of the longest
  long row_tiles = 0, items = 0;    // query-row tiles, (row tile, key tile) pairs
  double kv_tokens = 0;

  attn_call(const attn_shape &shape, int batch_, const int32_t *lens, const int32_t *offs) : sh(shape), batch(batch_), seq_lens(lens), offsets(offs) {
    for (int i = 0; i < batch; ++i) {
      max_rows = std::max(max_rows, sh.group * (gamma(i) + 1));
      longest = std::max(longest, tiles(i));
      row_tiles += rtc(i);
      items += (long)tiles(i) * rtc(i);
      kv_tokens += keys(i);
    }
  }
  int gamma(int i) const { return offsets[i + 1] - offsets[i]; }
  int keys(int i) const { return seq_lens[i] + gamma(i) + 1; }
  int tiles(int i) const { return fsv_ceil_div(keys(i), 32); }
  int rtc(int i) const { return fsv_ceil_div(sh.group * (gamma(i) + 1), 32); }
};

// The schedule with the row tiles of a request together or (split) as parts of their own.
struct attn_cut {
  int rt, nw, tpw, blocks;
  int cost16;    // of its longest part, in 1/16 of a tile of a request with one row tile
  bool sorted;   // several rounds
};
inline attn_cut attn_cut_for(const attn_call &call, bool split) {
  const attn_shape &sh = call.sh;
  attn_cut k{};
  auto w16_of = [&](int i) { return split || call.rtc(i) <= 1 ? 16 : call.rtc(i) == 2 ? sh.w2 : sh.w3; };
  k.rt = split ? 1 : fsv_ceil_div(call.max_rows, 32);
  // Waves per block.  Eight, one block per compute unit, while requests are few: a part then takes an eighth of its tiles' time.  Four, two blocks per
  // compute unit, from 192 (request, kv head) pairs on, so that a request need not be cut, and one block computes while the other
  // starts or merges; where the queries leave room for it (not with head size 128 and more than one row tile).  Head size 64, whole call
  // of the stand-alone entry: 8 requests of 2000 .. 6000 positions 24.8 us with eight, 28.6 with four; 24 of 200 .. 1000 16.6 and 16.6; 54 of 1000
  // 36.8 and 28.5.  Three row tiles of head size 128: four waves, one block (eight waves' rings and the queries exceed the LDS).
  const bool two_blocks = sh.head_dim == 64 || k.rt == 1, wide_q = sh.head_dim == 128 && k.rt > 2;
  k.nw = wide_q || (two_blocks && call.batch * sh.n_kv_heads >= 192) ? 4 : 8;
  // One round if it can be had: the smallest part length, up to twice the even share, for which parts x kv heads fit the
  // compute units.  Otherwise parts of up to five quarters of the even share in several rounds, the long ones first (a block costs 6 us besides
  // its tiles, so few and long is right as long as the last round is short).  In the order of the requests, and in parts of half the share:
  // 128 requests of 256 .. 8192 positions 240 us instead of 207, 2048 prefill rows 127 and 119.
  const int target = sh.target * (k.nw == 4 && !wide_q ? 2 : 1);
  auto count = [&](int tpw, int most) {   // parts x kv heads; counted no further than `most`
    int parts = 0;
    k.cost16 = 0;
    for (int i = 0; i < call.batch && parts * sh.n_kv_heads <= most; ++i) {
      int tp;
      parts += attn_parts(call.tiles(i), tpw, w16_of(i), k.nw, &tp) * (split ? call.rtc(i) : 1);
      k.cost16 = std::max(k.cost16, tp * w16_of(i));
    }
    return parts * sh.n_kv_heads;
  };
  long total_tiles = 0;   // in units of the cost of a tile of a request with one query-row tile
  for (int i = 0; i < call.batch; ++i) total_tiles += ((long)call.tiles(i) * w16_of(i) + 15) / 16;
  if (split) total_tiles = call.items;
  // Fewest key tiles a part is given: two for each of eight waves, or one while that makes no more parts than the merge fetches at once
  // (1600 positions, head size 128, one row tile 13.9 and 12.5 us; 3200 positions 16.2 and 18.3).
  const int fewest = k.nw == 8 && call.longest <= 64 ? sh.min_tpw / 2 : sh.min_tpw;
  const int even = (int)std::max((long)fewest, (total_tiles * sh.n_kv_heads + target - 1) / target);
  // Every request has a part, so with more pairs than blocks there is nothing to look for; otherwise at most 129 lengths are tried.
  // (Host time of all lengths one by one, before the first launch: 128 requests of 256 .. 8192 positions 0.33 ms, of 8 .. 32 k 2.6 ms.)
  for (int t = even; call.batch * sh.n_kv_heads <= target && t <= 2 * even; t += std::max(1, even / 128)) {
    if (count(t, target) <= target) { k.tpw = t; break; }
  }
  k.sorted = k.tpw == 0;
  if (!k.tpw) k.tpw = std::max(8, even * 5 / 4);
  k.blocks = count(k.tpw, INT_MAX);
  return k;
}

inline fsv_attn_plan attn_schedule(const attn_shape &sh, int batch, const int32_t *seq_lens, const int32_t *offsets) {
  fsv_attn_plan pl;
  const attn_call call(sh, batch, seq_lens, offsets);
  pl.kv_tokens = call.kv_tokens;
  // Row tiles as parts of their own, which read the same keys (neighbouring blocks, on one XCD with eight kv heads), while all fit the compute units
  // at once and leave a wave at most four (row tile, key tile) pairs: every block then has the short chain of one row tile, and a request's merge
  // is spread over as many blocks.  Beyond, the row tiles of a request share the keys they read.  Calls of the stand-alone entry in a graph, head
  // size 128, eight kv heads, shared and split: one request of 1600 positions, two row tiles 23.5 and 18.2 us, three 32.4 and 18.3; 16 of 800 .. 1600, two
  // 34.2 and 28.4; past the line 16 of 1600 .. 3200 43.4 and 45.9, 48 of 800 .. 1600 55.1 and 57.9.
  // Past it the longest parts of both schedules decide, while they are short enough for the merge to show: split if the shared one's is at
  // least 0.625 (head size 64) or 0.7 (128) of the split one's.  180 calls past it, drawn, timed both ways (every call and both costs:
  // profiles/attention_row_tiles_sweep.txt): head size 64, 60 that the rule takes 0.96 .. 1.36 x as fast split, mean 1.07, four of them slower; 30 that it leaves 0.83 .. 1.15, mean
  // 0.99.  Head size 128, 11 that it takes 1.00 .. 1.17, mean 1.08; 79 that it leaves 0.77 .. 1.13, mean 0.99.  The limits of 66 and 42 tiles are where
  // the gain ends: head size 128, ratio met, up to 42 tiles no call is slower, 42 .. 48 mean 1.00 and down to 0.90, beyond 1.00 and 0.94.  So 16 requests of
  // 512 .. 4096 positions, 1 .. 8 drafts, take it always at head size 64 and seldom at 128 (3 of 48 draws; one with costs of 41 and 52 tiles 34.7 and 32.8 us).
  const bool may = call.max_rows > 32 && call.row_tiles * sh.n_kv_heads <= sh.n_cus;
  pl.split = may && call.items * sh.n_kv_heads <= 32l * sh.n_cus;
  attn_cut k = attn_cut_for(call, pl.split);
  if (may && !pl.split && !k.sorted && k.nw == 8 && k.cost16 <= 16 * (sh.head_dim == 64 ? 66 : 42)) {
    const attn_cut s = attn_cut_for(call, true);
    if (!s.sorted && s.nw == 8 && (sh.head_dim == 64 ? 8 * k.cost16 >= 5 * s.cost16 : 10 * k.cost16 >= 7 * s.cost16)) {
      pl.split = true;
      k = s;
    }
  }
  pl.rt = k.rt;
  pl.nw = k.nw;
  pl.tpw = k.tpw;
  pl.sorted = k.sorted;
  pl.waves = k.blocks;
  return pl;
}
