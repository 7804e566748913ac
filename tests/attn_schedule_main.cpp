// Driver of tests/test_attention_schedule.py (CPU only): reads calls from stdin, one a line,
//   head_dim n_kv_heads group compute_units batch L_0 gamma_0 L_1 gamma_1 ..
// and prints for each the schedule's query-row tiles, waves per block, tiles per part, blocks, split, sorted, and the cost of the longest part
// (1/16 of a tile), blocks and rounds of the two schedules it chooses from: row tiles together, and apart.
#include <stdio.h>
#include <vector>
#define __host__
#define __device__

#include "../paper_2601_00644_amd/csrc/attn_schedule.h"

int main() {
  attn_shape sh{};
  int batch;
  while (scanf("%d %d %d %d %d", &sh.head_dim, &sh.n_kv_heads, &sh.group, &sh.n_cus, &batch) == 5) {
    sh.target = sh.n_cus;
    sh.min_tpw = 16;
    sh.w2 = 20;
    sh.w3 = 26;
    std::vector<int32_t> lens(batch), offsets(batch + 1, 0);
    for (int i = 0; i < batch; ++i) {
      int gamma;
      if (scanf("%d %d", &lens[i], &gamma) != 2) return 1;
      offsets[i + 1] = offsets[i] + gamma;
    }
    const fsv_attn_plan p = attn_schedule(sh, batch, lens.data(), offsets.data());
    const attn_call call(sh, batch, lens.data(), offsets.data());
    const attn_cut together = attn_cut_for(call, false), apart = attn_cut_for(call, true);
    printf("%d %d %d %d %d %d %d %d %d %d %d %d\n", p.rt, p.nw, p.tpw, p.waves, p.split, p.sorted, together.cost16, together.blocks, together.sorted,
           apart.cost16, apart.blocks, apart.sorted);
  }
  return 0;
}
