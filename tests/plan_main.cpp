// Reads "hidden inter shared tokens experts rows spread slots split max_ksplit" lines and prints the plan of each:
// "item_rows tile_gate_up tile_down ksplit"; with an argument the plan of an fp32 layer.  Host code only.
#include <cstdio>

#include "../paper_2602_07616_amd/csrc/ffn_plan.hpp"

int main(int argc, char**) {
  sere::FfnShape s{};
  int split = 0;
  while (std::scanf("%d %d %d %d %lf %lf %lf %lf %d %d", &s.hidden, &s.inter, &s.num_shared, &s.tokens, &s.experts, &s.rows,
                    &s.spread, &s.slots_per_expert, &split, &s.max_ksplit) == 10) {
    s.split_h = split != 0;
    const sere::FfnPlan p = argc > 1 ? sere::plan_ffn_f32(s) : sere::plan_ffn(s);
    std::printf("%d %d %d %d\n", p.item_rows, p.tile_gate_up, p.tile_down, p.ksplit);
  }
  return 0;
}
