// Which workgroup of the persistent FFN kernels has which units, walked as ffn_tile.hpp walks them.  Reads "f32 gate_up items longs
// parts_out ksplit steps tail" lines: work items, of which `longs` come first (fp32), blocks of output columns of an item (whole
// units), slices, k steps of a unit, and whether an item's last unit has columns in its second half; prints "wrong whole halves most both": half
// units (of a unit's columns) that are not owned exactly once, whole units and halves in all, the most halves of a workgroup, and the
// workgroups that have a long unit and another one.  Host code only.
#include <cstdio>
#include <vector>

#include "../paper_2602_07616_amd/csrc/ffn_plan.hpp"
#include "../paper_2602_07616_amd/csrc/rules.hpp"

int main() {
  using namespace sere;
  int f32 = 0, gate_up = 0, items = 0, long_items = 0, out_blocks = 0, ksplit = 0, steps = 0, tail = 0;
  while (std::scanf("%d %d %d %d %d %d %d %d", &f32, &gate_up, &items, &long_items, &out_blocks, &ksplit, &steps, &tail) == 8) {
    const int out = 128, outs = out_blocks * out - (tail ? 0 : out / 2);   // columns of a unit, of an item
    const unsigned parts = out_blocks * ksplit, total = items * parts;
    std::vector<int> owned(2 * total, 0);
    int whole_units = 0, halves = 0, most = 0, both = 0;
    for (unsigned b = 0; b < kTileGroups; ++b) {
      const unsigned xcd = b % kXcds, turn = b / kXcds;
      int mine = 0, own = 0, longs = 0;
      const auto whole_unit = [&](unsigned u) {
        if (u < total) ++owned[2 * u], ++owned[2 * u + 1]; else owned[0] += 2;
        ++own;
      };
      if (f32) {
        const LongFirst f = long_first(total, long_items * parts, xcd);
        for (unsigned u = turn; u < f.count; u = next_place_long_first(u, turn, f.longs))
          longs += u < f.longs, whole_unit(unit_at_long_first(u, f.longs, f.to_long, f.to_other));
      } else {
        const unsigned lo = xcd_share(total, xcd), hi = xcd_share(total, xcd + 1), whole = whole_units_end(lo, hi, halves_pay(gate_up, steps));
        for (unsigned u = lo + turn; u < whole; u += kXcdGroups) whole_unit(u);
        for (unsigned u = 2 * whole + turn; whole < hi && u < 2 * hi; u += kXcdGroups) {
          if (unit_first_out(u, 2, parts, ksplit, out / 2) >= outs) break;   // no columns: the workgroup ends
          if (u < 2 * total) ++owned[u]; else owned[0] += 2;
          ++mine;
        }
      }
      whole_units += own, halves += mine, most = mine > most ? mine : most;
      both += longs > 0 && own > 1;
    }
    int wrong = 0;
    for (unsigned u = 0; u < total; ++u)
      for (int h = 0; h < 2; ++h) {
        const bool exists = unit_first_out(2 * u + h, 2, parts, ksplit, out / 2) < outs;
        wrong += exists ? owned[2 * u + h] != 1 : owned[2 * u + h] > 1;
      }
    std::printf("%d %d %d %d %d\n", wrong, whole_units, halves, most, both);
  }
  return 0;
}
