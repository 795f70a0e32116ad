// Reads "dtype hidden experts inter batch_tokens flags batches" lines and prints, for groups of 1 batch, 2 batches, ... up
// to the largest that a call with so many batches takes: "total items item_rows tile_gate_up tile_down ksplit gram_splits
// gram_staged item_bytes part_bytes wide_gate_up y_bytes h_bytes cka_parts cka_blocks gram_steps few_steps", item_bytes,
// part_bytes, y_bytes and h_bytes the room for an array of the work list, for the partial Gram matrices, for y and for h,
// gram_steps the 16-wide steps of a slice and few_steps those that pair_gram_few_kernel takes a turn of its loop; groups separated
// by ';'.  Host code only.
#include <cstdio>

#include "../paper_2602_07616_amd/csrc/similarity_plan.hpp"

int main() {
  sere_config c{};
  int n = 0, batches = 0;
  while (std::scanf("%d %d %d %d %d %d %d", &c.dtype, &c.hidden, &c.num_experts, &c.inter, &n, &c.flags,
                    &batches) == 7) {
    const int most = sere::sim_group(c, n), whole = batches < most ? batches : most;
    for (int g = 1; g <= whole; ++g) {
      const sere::SimLayout l = sere::make_sim_layout(c, n, g, whole);
      std::printf("%zu %d %d %d %d %d %d %d %zu %zu %d %zu %zu %d %d %lld %d;", l.total, l.items, l.plan.item_rows,
                  l.plan.tile_gate_up, l.plan.tile_down, l.plan.ksplit, l.gram_splits, l.gram_staged, l.work_off - l.work_expert,
                  l.gram_splits > 0 ? l.gram - l.gram_part : 0, l.plan.wide_gate_up, l.h - l.y,
                  c.flags & SERE_FLAG_SIM_CKA_LINEAR ? l.gram - l.block_sums : 0, l.cka_parts, sere::cka_blocks(n), l.gram_chunk / 16,
                  8 * sere::gram_few_steps((c.num_experts + 15) / 16, (c.flags & SERE_FLAG_SIM_COSINE) != 0));
    }
    std::printf("\n");
  }
  return 0;
}
