// Host side: which FFN kernels serve a call (bf16: plan_ffn, fp32: plan_ffn_f32), with which work item size and how
// many slices of the down projection's contraction.  A function of the sizes alone.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>

#include "../../include/sere.h"

namespace sere {

inline size_t align_up(size_t v) { return (v + 255) & ~static_cast<size_t>(255); }   // of a buffer in the workspace

// bf16 down projection: d_m is cut into slices of at most 2048 so that one
// wavefront streams at most 64 KB of weights whatever the expert width
inline int down_ksplit(const sere_config& c) { return c.dtype == SERE_BF16 ? (c.inter + 2047) / 2048 : 1; }

// wide experts: h keeps its bf16 rounding residual in a second plane (see decode())
inline int wants_split_h(const sere_config& c) { return (c.dtype == SERE_BF16 && c.inter >= 4096) ? 1 : 0; }

constexpr int kSmallSlots = 64;   // slots of a call that the kernels of ffn_small.hpp serve: one to a lane

constexpr int kItemRows = 32;     // rows of the sorted slot list per FFN work item (FfnPlan::item_rows may be larger)
constexpr int kTileGroups = 256;  // persistent workgroups of the kernels of ffn_tile.hpp: one per compute unit

struct FfnShape {
  int hidden, inter, num_shared, tokens;
  double experts;      // routed experts that own rows
  double rows;         // rows of each of them, on average
  double spread;       // standard deviation of that
  double slots_per_expert;  // rows per expert, all experts counted
  bool split_h;        // h carried as two bf16 planes
  int max_ksplit;      // slices of d_m that the workspace has room for
};

struct FfnPlan {
  int item_rows = kItemRows;
  bool tile_gate_up = false, tile_down = false;   // the persistent kernels of ffn_tile.hpp
  bool wide_gate_up = false;                      // items of 256 rows: gate/up units of 256 weight rows instead of 128
  int ksplit = 1;                                 // slices of d_m in the down projection
};

struct TileVariant {
  int rows;            // of a work item, at most
  int gate_up_out;     // intermediate indices per gate/up unit
  int down_out;        // output rows per down unit
  double gate_up_step, down_step;  // us per 64-wide k step of a unit
};

// The constants of this file are fitted to measured launches of 300 layers (those of workloads.py at 4 to 4096
// tokens and random ones: d_h 256 to 4096, d_m 128 to 14336, 2 to 160 experts, 1 to 4000 tokens), every item size
// and both kinds of kernels timed on each.  Over these layers what plan_ffn picks, with all its rules, takes 2.6 %
// longer than the best choice on average, 17 % less than the decode kernels alone, and 15 % less than one rule for
// all (items of 32 to 256 rows by rows per expert) with the workgroup-staged kernels of earlier.  (Timed and fitted before last rounds
// of units were cut into halves, rules.hpp: the costs charge a part-filled round as a whole one, where halves make it two thirds.)
inline const TileVariant* tile_variants(bool split_h, int* count) {
  // a step of a unit of 256 weight rows: 0.74 us and 2.6 ns for every token row; of 128 rows measured on its own
  static const TileVariant plain[] = {{32, 128, 256, 0.82, 0.82},  {64, 128, 256, 0.91, 0.91}, {96, 128, 256, 0.99, 0.99},
                                      {128, 128, 256, 1.07, 1.07}, {160, 128, 256, 1.16, 1.16}, {192, 64, 128, 0.74, 0.74},
                                      {256, 64, 128, 0.84, 0.84}};
  // both planes of h count in the down projection
  static const TileVariant split[] = {{32, 128, 256, 0.82, 0.91}, {64, 128, 256, 0.91, 1.07}, {128, 128, 128, 1.07, 0.84}};
  *count = split_h ? 3 : 7;
  return split_h ? split : plain;
}

// expected work items of an expert whose row count is about normal: sum over k of P(rows > k * item_rows)
inline double items_per_expert(const FfnShape& s, int item_rows) {
  double n = 1.0;
  for (int k = 1; k <= 4096 && k * item_rows < s.rows + 6.0 * s.spread + 1.0; ++k)
    n += s.spread > 0.0 ? 0.5 * std::erfc((k * item_rows + 0.5 - s.rows) / (s.spread * 1.4142135623730951))
                        : (s.rows > k * item_rows ? 1.0 : 0.0);
  return n;
}
inline double total_items(const FfnShape& s, int item_rows) {
  return s.experts * items_per_expert(s, item_rows) + static_cast<double>(s.num_shared) * ((s.tokens + item_rows - 1) / item_rows);
}

// us to stream the weights: the first 130 MB of a launch come partly from the last-level cache
inline double stream_us(double bytes, double near_rate, double far_rate) {
  constexpr double kNear = 1.3e8;
  return std::min(bytes, kNear) / near_rate + std::max(0.0, bytes - kNear) / far_rate;
}
inline double unit_rounds(double units) { return std::max(1.0, std::ceil(units / kTileGroups - 0.02)); }
// us of a launch of the persistent kernels: rounds of 256 units, each its k steps and `change` us to change units
// (down stores y, four times the bytes of h), but no less than the weights take, and 2.8 us to fill the ring.
// With few units a step is bound by latency alone and a little shorter.
inline double tile_cost(double units, double steps, double step_us, double change, double weight_bytes) {
  const double rounds = unit_rounds(units);
  const double busy = std::min(1.0, std::max(0.8, units / rounds / kTileGroups));
  return std::max(rounds * (steps * step_us * busy + change), stream_us(weight_bytes, 9.8e6, 5.8e6)) + 2.8;
}
// us of a launch of the kernels of ffn_mfma.hpp (items of kItemRows): the weights, an expert's further items
// from cache, and launch, first loads and drain
inline double row_cost(const FfnShape& s, double weight_bytes, double near_rate, double far_rate, double again_rate, double fixed) {
  const double again = total_items(s, kItemRows) / (s.experts + s.num_shared) - 1.0;
  return stream_us(weight_bytes, near_rate, far_rate) + again * weight_bytes / again_rate + fixed;
}

// Smallest number of slices up to max_ksplit that wastes the fewest rounds; no slice may be empty.  `ksplit`: that
// many and no other.
inline int tile_ksplit(const FfnShape& s, double units, double step_us, double weight_bytes, int ksplit, double* cost) {
  const int blocks = s.inter / 64;
  int best = 1;
  *cost = 1e30;
  for (int k = ksplit > 0 ? ksplit : 1; k <= (ksplit > 0 ? ksplit : s.max_ksplit); ++k) {
    const int per = (blocks + k - 1) / k;
    if ((k - 1) * per >= blocks) continue;
    const double c = tile_cost(units * k, per, step_us, 4.4, weight_bytes) + 0.55 * (k - 1);
    if (c < *cost) {
      *cost = c;
      best = k;
    }
  }
  return best;
}

constexpr double kGateUpChange = 0.9;   // us to change gate/up units
// us of the two launches of the persistent kernels with items of v.rows, and the slices of the second
struct TileCost {
  double gate_up, down;
  int ksplit;
};
inline TileCost tile_costs(const FfnShape& s, const TileVariant& v, double gu_bytes, int ksplit = 0) {
  TileCost t;
  const double items = total_items(s, v.rows);
  t.gate_up = tile_cost(items * std::ceil(static_cast<double>(s.inter) / v.gate_up_out), s.hidden / 64, v.gate_up_step, kGateUpChange,
                        gu_bytes);
  t.ksplit = tile_ksplit(s, items * std::ceil(static_cast<double>(s.hidden) / v.down_out), v.down_step, 0.5 * gu_bytes, ksplit, &t.down);
  return t;
}
inline double gate_up_bytes(const FfnShape& s) { return (s.experts + s.num_shared) * 4.0 * s.hidden * s.inter; }

// Items of 256 rows: a gate/up unit of 256 weight rows takes less of a compute unit's intake per product than two of 128, but
// half as many units fill a round less evenly (us a launch, 256 rows an expert: 128 experts of the Qwen3 shape 210 -> 199,
// three rounds of 32 steps for six, 60 experts of d_m 1408 206 -> 190, 40 of d_h 1024, d_m 768 86 -> 77; 60 experts of d_m 768,
// 1.4 rounds for 2.8, 213 -> 241).  The steps are those of weights that come from cache, like the ones of tile_variants.  A
// part-filled round of these units is no shorter than a full one, as tile_cost takes it to be for the narrower ones, so their
// rounds have to be the shorter ones without that, too.  us a call of 59 layers whose tokens select all 1 to 16 experts, by the
// rounds' time against that of the units of 128: below 0.9 times 3 to 9 % less (157.6 -> 150.2; one layer the same), 0.9 to 1.0
// times 1 % more to 6 % less, 1.0 to 1.04 times 2 % less to 2 % more, beyond 1 to 8 % more (127.8 -> 134.1).  Where they are taken
// they still pay now that last rounds of the narrower units are cut into halves: ten layers by these units / by those, 1 to 8 % less
// (141 / 152, 158 / 165, 75.5 / 76.0).
// For items that are known, or all but known (spread 0): similarity calls, where every expert has every token, and
// layers whose tokens select every expert (K = M; re-routing that takes an expert out gives its rows to another, and the
// number of items stays about the same: 12 layers with S = 1 gained as much as without re-routing).  Where the rows per
// expert are only expected it lost as often as it gained (130 decode layers).  Down units of that size gained nothing
// (157 -> 156, 128 experts; 155 -> 158).
inline bool wide_gate_up_pays(const FfnShape& s, const FfnPlan& p) {
  if (s.split_h || s.spread > 0.0 || p.item_rows != 256 || !p.tile_gate_up) return false;
  const TileVariant wide{256, 128, 256, 1.5, 1.5}, narrow{256, 64, 128, 0.84, 0.84};
  const auto rounds_us = [&](const TileVariant& v) {
    return unit_rounds(total_items(s, v.rows) * std::ceil(static_cast<double>(s.inter) / v.gate_up_out)) *
           (s.hidden / 64 * v.gate_up_step + kGateUpChange);
  };
  const double bytes = gate_up_bytes(s);
  return rounds_us(wide) < rounds_us(narrow) && tile_costs(s, wide, bytes).gate_up < 0.95 * tile_costs(s, narrow, bytes).gate_up;
}

inline FfnPlan plan_ffn(const FfnShape& s) {
  const double gu_bytes = gate_up_bytes(s), dn_bytes = 0.5 * gu_bytes;
  FfnPlan best;
  best.ksplit = s.max_ksplit;
  // from 8 rows per expert on the token rows that the gate/up kernel stages slow the weights down
  const double row_gu = row_cost(s, gu_bytes, 9.2e6, s.split_h || s.slots_per_expert < 8 ? 6.0e6 : 5.2e6, 5.0e6, 6.8);
  const double row_dn = row_cost(s, dn_bytes, 6.3e6, s.split_h ? 3.9e6 : 5.7e6, 7.1e6, 6.2);
  constexpr double kMargin = 0.9;    // what the persistent kernels have to promise to be taken
  double best_cost = row_gu + row_dn;
  int n = 0;
  const TileVariant* v = tile_variants(s.split_h, &n);
  for (int i = 0; i < n; ++i) {
    const TileCost t = tile_costs(s, v[i], gu_bytes);
    FfnPlan p;
    p.item_rows = v[i].rows;
    p.tile_gate_up = v[i].rows != kItemRows || t.gate_up < kMargin * row_gu;   // the other kernels take items of kItemRows
    p.tile_down = v[i].rows != kItemRows || t.down < kMargin * row_dn;
    p.ksplit = p.tile_down ? t.ksplit : s.max_ksplit;
    const double cost = (p.tile_gate_up ? t.gate_up : row_gu) + (p.tile_down ? t.down : row_dn);
    // larger items leave no choice for either kernel: gate/up, two thirds of the bytes, has to promise it by itself
    // (64 experts, d_m 1408, 46 active of 56 expected: promised 0.94 + 0.80, measured 104 + 52 us against 96 + 52; of
    // the 300 layers above four get another plan by this, 9 % slower to 3 % faster: 0.03 % on average)
    if (v[i].rows != kItemRows && t.gate_up >= kMargin * row_gu) continue;
    if (cost < best_cost * (best.tile_gate_up || best.tile_down ? 1.0 : kMargin)) {
      best_cost = cost;
      best = p;
    }
  }
  best.wide_gate_up = wide_gate_up_pays(s, best);
  return best;
}

// The persistent kernels whatever the others cost, with `ksplit` slices (0: the best number), for callers whose sums must
// not depend on the number of rows: with equal slices these kernels add up an output in the same order for every
// item size.
inline FfnPlan plan_ffn_tile(const FfnShape& s, int ksplit) {
  FfnPlan best;
  best.tile_gate_up = best.tile_down = true;
  double best_cost = 1e30;
  int n = 0;
  const TileVariant* v = tile_variants(s.split_h, &n);
  for (int i = 0; i < n; ++i) {
    const TileCost t = tile_costs(s, v[i], gate_up_bytes(s), ksplit);
    if (t.gate_up + t.down < best_cost) {
      best_cost = t.gate_up + t.down;
      best.item_rows = v[i].rows;
      best.ksplit = t.ksplit;
    }
  }
  best.wide_gate_up = wide_gate_up_pays(s, best);
  return best;
}

// fp32 layers: the persistent kernels take 128 weight rows a unit (20 KB a stage, eight stages), 32-wide k steps
// and items of 32 rows; the matrix cores' fp32 rate bounds them from some 20 rows per expert on, so longer items
// would gain nothing (measured with 256 x 64 units: 54 + 38 -> 93 + 65 us at 96 tokens of a 1024-wide layer).  The
// vector-ALU kernels serve 8 rows in one pass and start faster: they keep batches of at most 8 tokens whose
// contractions are long and whose experts are few (one token, d_h 1472: 27 against 37 us; 8 tokens, d_h 256: 24
// against 14 us; 96 tokens, d_h 1024: 260 against 103 us).  Both sides fitted to 45 measured layers.
constexpr int kTileF32Rows = 128;
inline FfnPlan plan_ffn_f32(const FfnShape& s) {
  const double experts = s.experts + s.num_shared;
  const double gu_units = total_items(s, kItemRows) * std::ceil(s.inter / (0.5 * kTileF32Rows));
  const double dn_units = total_items(s, kItemRows) * std::ceil(s.hidden / (1.0 * kTileF32Rows));
  const double tile = std::ceil(gu_units / kTileGroups) * (s.hidden / 32 * 0.62 + 2.5) +
                      std::ceil(dn_units / kTileGroups) * (s.inter / 32 * 0.62 + 2.5);
  const double rows = 22.0 + experts * 12.0 * s.hidden * s.inter / 3.5e6;
  FfnPlan p;
  p.tile_gate_up = p.tile_down = s.tokens > 8 || tile < rows;
  return p;
}

// Work item size and kernels of a call whose experts own the slots of T tokens.  Which experts those are is
// known on the device only; here it is what independent tokens give: an expert stays if some token has it among
// its top S (its top K without re-routing or with a threshold).
inline FfnPlan plan_decode(const sere_config& c, bool reroute) {
  const double T = c.num_tokens, M = c.num_experts, K = c.top_k;
  const double kept = reroute && !(c.threshold > 0.0f) ? c.select_top_k : K;
  FfnShape s{};
  s.hidden = c.hidden;
  s.inter = c.inter;
  s.num_shared = c.num_shared;
  s.tokens = c.num_tokens;
  s.experts = std::max(1.0, M * (1.0 - std::pow(1.0 - kept / M, T)));
  s.rows = T * K / s.experts;
  s.slots_per_expert = T * K / M;
  s.spread = K < M ? 1.5 * std::sqrt(s.rows) : 0.0;  // tokens of a batch resemble each other: wider than by chance
  s.split_h = wants_split_h(c) != 0;
  s.max_ksplit = down_ksplit(c);
  return c.dtype == SERE_F32 ? plan_ffn_f32(s) : plan_ffn(s);
}

// ---- calls of at most kSmallSlots slots: the two launches of ffn_small.hpp behind the router logits
constexpr int kSmallOut = 8;             // intermediate indices of a wavefront (gate/up), output rows of a workgroup (down)
constexpr int kSmallBlock = 128;         // bytes of every row that a step takes: 64 bf16 or 32 fp32
constexpr int kSmallAhead = 4;           // blocks whose loads are issued together
constexpr int kSmallWaves = 8;           // wavefronts of a workgroup
constexpr int kSmallGroups = 511;        // gate/up workgroups that run side by side, without the one that writes
constexpr int kSmallTile = 16;           // rows that an item's weights are read for at a time

// A wavefront ranks the upper halves of a token's lists and holds all slots, and a workgroup of the down launch holds the
// rows of y for its columns.  bf16: up to a tile of tokens (238 layers of 17 to 64 tokens: the median 0.81 times as fast by these
// launches, 9 more than 1.1 times).
inline bool small_call_fits(const sere_config& c) {
  const long long T = c.num_tokens, slots = T * c.top_k;
  return c.top_k <= 8 && (T <= kSmallTile || c.dtype == SERE_F32) && slots + c.num_shared <= kSmallSlots && slots + T * c.num_shared <= 2 * kSmallSlots && !wants_split_h(c);
}

// Gate/up: wavefronts that share a contraction (1, 2, 4 or 8): as many as have kSmallAhead blocks each, more while all `rows`
// rows of h still fit one round of units.  A unit costs some 3 us of latencies whatever it holds, so that a contraction of few
// blocks leaves room for more weight rows in it.
inline int small_units(int rows, int split) { return rows / (kSmallOut * kSmallWaves / split); }
inline int small_split(int blocks, int rows) {
  int split = 1;
  while (split < kSmallWaves && (split * kSmallAhead < blocks || small_units(rows, 2 * split) <= kSmallGroups)) split *= 2;
  return split;
}

// Whether these launches are the faster ones: us of a call by either way, both fitted to 885 bf16 and 495 fp32 layers that
// small_call_fits, timed with both (d_h 256 to 4096, d_m 128 to 4032, 2 to 160 experts, 1 to 16 tokens, 1 to 740 MB of weights).
// What costs most here is rounds of units and, in a long contraction, of loads; then the top-K, a wavefront's tokens one after the
// other, the exchange between wavefronts that more than eight primary slots need, and the rows of h and y.  The other launches start at 23 us
// (fp32 29 and more) and take the weights as they come.  The fits are within 5 to 15 % of a layer, hence the margin.  On these layers and
// 650 others: bf16 675 of 1280 taken, 0.95 to 1.7 times as fast there, 1.2 on average, four of them less than 0.97 times (without
// the top-K, the exchange and the rows 44 were, down to 0.68); fp32 711 of 750, 0.95 to 2.6 times, three less than 0.97.  fp32 calls of more than 16
// tokens: with up to a dozen items, 154 of 182 layers, 0.96 to 2.0 times as fast, 1.45 on average; with more items 0.7 to 1.6 times, and what
// the rule reads of a layer does not tell which.
inline bool small_call_pays(const sere_config& c, bool reroute) {
  if (!small_call_fits(c)) return false;
  const auto ceil_div = [](int a, int b) { return (a + b - 1) / b; };
  const double T = c.num_tokens, M = c.num_experts, slots = T * c.top_k, bytes = c.dtype == SERE_F32 ? 4.0 : 2.0;
  const double kept = reroute && !(c.threshold > 0.0f) ? c.select_top_k : c.top_k;
  const double routed = std::max(1.0, M * (1.0 - std::pow(1.0 - kept / M, T))), items = routed + c.num_shared;
  const double mb = items * 3e-6 * c.hidden * c.inter * bytes;
  const int gu_blocks = static_cast<int>(c.hidden * bytes) / kSmallBlock, dn_blocks = static_cast<int>(c.inter * bytes) / kSmallBlock;
  const int most = static_cast<int>(std::min(T * kept, M)) + c.num_shared;
  const int split = small_split(gu_blocks, most * c.inter), slices = std::max(1, std::min(static_cast<int>(kSmallWaves / items), dn_blocks));
  if (c.num_tokens > kSmallTile && items > 12.0) return false;
  // the weights of an item with more rows than a tile are read for every tile
  double passes = slots > 10.0 * routed ? 2.0 : 1.0;
  if (c.num_tokens > kSmallTile) passes = std::max({passes, std::ceil((slots / routed + 6.0) / kSmallTile), c.num_shared > 0 ? std::ceil(T / kSmallTile) : 1.0});
  const double gu = std::max(1.0, std::ceil(items * c.inter * split / (kSmallOut * kSmallWaves) / kSmallGroups - 0.02)) *
                    ceil_div(ceil_div(gu_blocks, split), kSmallAhead);
  const double dn = std::ceil(items * slices / kSmallWaves) * ceil_div(ceil_div(dn_blocks, slices), kSmallAhead) *
                    std::max(1.0, c.hidden / (256.0 * kSmallOut));
  const double topk = std::ceil(T / kSmallWaves) * (M <= 128 ? std::ceil(M / 16.0) / 8.0 : 2.0);
  const double exchange = reroute && c.select_top_k < c.top_k && T * c.select_top_k > 8 ? 1.0 : 0.0, rows = slots + T * c.num_shared;
  const double small = c.dtype == SERE_F32
                           ? 16.1 + passes * (0.55 * gu + 0.84 * dn) + 0.014 * slots + 0.175 * mb + 1.44 * topk + 0.94 * exchange + 0.027 * rows
                           : 13.3 + passes * (3.18 * gu + 0.45 * dn) + 0.06 * slots + 0.098 * mb + 1.15 * topk + 0.82 * exchange + 0.019 * rows;
  const double other = c.dtype == SERE_F32 ? 27.2 + 0.167 * mb + 0.0089 * c.hidden
                                           : 22.7 + 0.156 * mb + 0.25 * std::ceil(M / 16.0) - 0.129 * items;
  return small < 0.93 * other;
}

}  // namespace sere
