// Prints the plan of every input line, "item_rows tile_gate_up tile_down ksplit wide_gate_up".  Lines without an argument, or
// with "f32" (an fp32 layer): "hidden inter shared tokens experts rows spread slots split max_ksplit"; with "call":
// "dtype tokens hidden experts top_k inter shared S rho reroute", a call of the library; with "small": the same lines, printed is
// "fits pays split units" of the launches for few slots.  Host code only.
#include <cstdio>
#include <cstring>

#include "../paper_2602_07616_amd/csrc/ffn_plan.hpp"

static void print(const sere::FfnPlan& p) {
  std::printf("%d %d %d %d %d\n", p.item_rows, p.tile_gate_up, p.tile_down, p.ksplit, p.wide_gate_up);
}

int main(int argc, char** argv) {
  if (argc > 1 && std::strcmp(argv[1], "call") == 0) {
    sere_config c{};
    int reroute = 0;
    while (std::scanf("%d %d %d %d %d %d %d %d %f %d", &c.dtype, &c.num_tokens, &c.hidden, &c.num_experts, &c.top_k, &c.inter,
                      &c.num_shared, &c.select_top_k, &c.threshold, &reroute) == 10)
      print(sere::plan_decode(c, reroute != 0));
    return 0;
  }
  if (argc > 1 && std::strcmp(argv[1], "small") == 0) {
    sere_config c{};
    int reroute = 0;
    while (std::scanf("%d %d %d %d %d %d %d %d %f %d", &c.dtype, &c.num_tokens, &c.hidden, &c.num_experts, &c.top_k, &c.inter,
                      &c.num_shared, &c.select_top_k, &c.threshold, &reroute) == 10) {
      const int split = sere::small_split(c.hidden * (c.dtype == SERE_F32 ? 4 : 2) / sere::kSmallBlock, c.inter);
      std::printf("%d %d %d %d\n", sere::small_call_fits(c), sere::small_call_pays(c, reroute != 0), split, sere::small_units(c.inter, split));
    }
    return 0;
  }
  sere::FfnShape s{};
  int split = 0;
  while (std::scanf("%d %d %d %d %lf %lf %lf %lf %d %d", &s.hidden, &s.inter, &s.num_shared, &s.tokens, &s.experts, &s.rows,
                    &s.spread, &s.slots_per_expert, &split, &s.max_ksplit) == 10) {
    s.split_h = split != 0;
    print(argc > 1 ? sere::plan_ffn_f32(s) : sere::plan_ffn(s));
  }
  return 0;
}
