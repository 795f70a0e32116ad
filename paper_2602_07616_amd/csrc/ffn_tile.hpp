// Grouped expert FFN for batches that give the experts a dozen rows and more (bf16), and for most fp32
// layers: persistent workgroups fed by loads that go straight to LDS.
//
// What bounds these launches is how many bytes a compute unit keeps in flight.  The weights come
// from HBM at about 3 us of latency under load, so 27 GB/s per compute unit (7 TB/s for the chip)
// needs some 80 KB on their way at all times, next to the token rows, which come from L2.  Loads
// into registers cannot hold that; the 160 KB of LDS can: global_load_lds writes a stage of weight
// and token rows straight into a ring of two to four stages (36 to 64 KB each; fp32: eight of
// 20 KB), nothing passes through registers until the matrix cores read it.
//
//  - A unit of work is BM weight rows x all token rows of a work item (at most BN) over the whole
//    contraction, 128 bytes of every row a step.  256 workgroups, one per compute unit, walk their units
//    without a gap: the ring is a single sequence of (unit, 64-wide k step), so the next unit's loads are in
//    flight while the last one is finished and stored.
//  - A row of a stage is 128 bytes, eight 16-byte pieces; piece c of row r lies at position
//    c ^ (r & 7).  The loads put it there by having each lane fetch the piece that belongs at its
//    place, still eight whole 128-byte lines per instruction, and a matrix operand (16 rows x 16
//    bytes, rows in the wavefront's lane order) then reads every LDS bank once.
//  - Eight wavefronts share a stage as 8 / WN x WN: 32, 64 or 128 weight rows and every WN-th token
//    tile each.  While the second half of a stage is multiplied the first half of the next one is read
//    from LDS, so that reads and products overlap inside a wavefront (gate/up at 2048 tokens of
//    the Qwen3 shape, one launch over and over: 165 -> 151 us).
//  - A compute unit takes in 64 bytes a cycle at best and its queue is short: eight wavefronts that issue a
//    stage's 36 to 64 loads (fp32: 20) at once stand still until they are accepted.  So the loads go out one by one among the
//    products (us, gate/up + down: 777 tokens of d_h 2880, d_m 1472 170 + 97 -> 161 + 93, 2048 tokens of the Qwen3
//    shape 156 + 112 -> 150 + 109, 256 rows an expert 231 + 166 -> 231 + 158; fp32 below 63 + 39 -> 57 + 37).
//  - Workgroups are handed to the 8 XCDs round-robin; each XCD walks a contiguous range of units,
//    so the parts of one item run side by side and share its token rows in one L2.  Every part of
//    256 weight rows starts at another k step (not the same offset of every row at once, that is, not
//    the same memory channels: 115 -> 107 us at 128 tokens).
//
//  - Where at most half of an XCD's workgroups would get one more unit, these units are cut into halves of their weight rows, one for
//    every workgroup: half the weights and the same token rows are some two thirds of the time, less 2 us to start again (us, gate/up +
//    down: 777 tokens of d_h 2880, d_m 1472, 2.3 rounds each, 156 + 92 -> 149 + 88, a call 279 -> 263; 2048 tokens of the Qwen3
//    shape, items in excess of three and four rounds, 175 + 121 -> 166 + 117; 128 tokens, down 59.6 -> 57.7).  The sums are the same ones.
//    (Not for gate/up units of fewer than five k steps behind whole ones, halves_pay in rules.hpp, nor for those of 256 weight rows x 256
//    token rows, whose wavefronts have no registers to spare.)
//  - fp32: an item of more than 16 rows takes half as long again as a shorter one (31 against 23 us a gate/up unit in a first
//    round, 25 against 17 in a second; d_h 1024), and few layers have more than two rounds of units.  The work list then has
//    the long items first, every XCD gets an eighth of their units, and a workgroup that starts with one is the
//    last to get a second unit (96 tokens of 32 experts and a shared one, d_h 1024, d_m 704: the XCD with the shared expert's rows ended
//    after 56 us, the others after 41; now all after 44.  Down 34 -> 30.  All calls of that size 111 -> 91).
//  - fp32: matrix cores and vector ALU take turns (16x16x4 products and seven additions in one wavefront: 65 cycles, 32 + 28 alone), so
//    that the additions of a step are kept behind its products, where the compiler otherwise starts the first ones between products and
//    waits for these, and one of the two wavefronts of a SIMD goes first: 1 to 3 % of a call, 91 -> 88 us of the one above.
//
// Measured on the Qwen3 shape (d_h 2048, d_m 768, 128 experts), us per launch, gate/up + down, within steps on four
// copies of the weights in turn, against the kernels with eight wavefronts that staged token rows through registers,
// both on one card that has been busy for some 20 ms (from idle the first steps take a tenth longer):
//   tokens   128: 111 + 60 -> 104 + 58     512: 140 + 81 -> 127 + 75    1024: 153 + 94 -> 137 + 89
//           2048: 212 + 119 -> 143 + 109   3072: 242 + 145 -> 208 + 140   4096: 371 + 198 -> 261 + 179
// (2048 tokens, items of 160 rows: while no expert has more.  Where one does, its second item makes the launch start a
// fourth round of units on every compute unit: 173 + 124.)
// fp32 layers against the vector-ALU kernels: 150 + 111 -> 42 + 31 us at 96 tokens (d_h 1024, d_m 704, 32 experts);
// relative error of the layer 1.8e-7 -> 1.4e-7.
// Not faster, one launch over and over: 32-wide steps with more stages (64-byte rows: 165 -> 236 us at 2048 tokens);
// the same first step for all parts of an item; plain instead of non-temporal weight loads (151 -> 162 us).
#pragma once

#include <algorithm>
#include <utility>

#include "common.hpp"
#include "ffn_generic.hpp"
#include "ffn_mfma.hpp"
#include "rules.hpp"

namespace sere {

// uniform load through the scalar cache (of arrays that earlier kernels wrote)
__device__ __forceinline__ int scalar_load(const int32_t* p, int i) {
  return reinterpret_cast<const __attribute__((address_space(4))) int32_t*>(reinterpret_cast<uintptr_t>(p))[i];
}

// the value of the first lane, for operands that have to be in scalar registers wherever the compiler kept them
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ const char* uniform(const char* p) {
  const uint64_t a = reinterpret_cast<uintptr_t>(p);
  return reinterpret_cast<const char*>(static_cast<uintptr_t>(static_cast<uint64_t>(uniform(static_cast<uint32_t>(a >> 32))) << 32 |
                                                             uniform(static_cast<uint32_t>(a))));
}

// 64 lanes x 16 bytes from memory to 1 KB of LDS at byte `lds` (lane l's bytes land at lds + 16 l).
// They are asm so that the compiler does not wait for them on its own; nothing else of these kernels'
// main loop counts in vmcnt but them and the result stores.
__device__ __forceinline__ void lds_load_weights(uint32_t lds, uint32_t lane_off, const char* base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(lane_off), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void lds_load_tokens(uint32_t lds, const char* addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(addr) : "memory", "m0");
}
// all but the youngest N vector memory operations, and this wavefront's LDS reads
template <int N>
__device__ __forceinline__ void wait_loads() {
  static_assert(N >= 0 && N <= 63, "vmcnt has six bits");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

constexpr int kTileThreads = 512;
constexpr int kTileWaves = kTileThreads / kWave;
constexpr int kTileLds = 160 * 1024;
constexpr int kRowBytes = 128;       // of a stage: one k step, 64 wide in bf16, 32 in fp32
constexpr int kLoadRows = 8;         // rows one load instruction fills

// BM weight rows x BN token rows per unit, WN wavefronts along the tokens.  LO: the token operand has a
// second plane (the rounding residual of h); BN then counts the rows of both planes.
template <int BM, int BN, int WN, bool LO>
struct TileShape {
  static constexpr int kStageBytes = (BM + BN) * kRowBytes;
  static constexpr int kStages = kTileLds / kStageBytes >= 8 ? 8 : kTileLds / kStageBytes;
  static constexpr int kRealRows = LO ? BN / 2 : BN;
  static constexpr int kWeightLoads = BM / kLoadRows / kTileWaves;  // per wavefront and step
  static constexpr int kTokenInstr = BN / kLoadRows;                // per workgroup and step
  static constexpr int kTokenLoads = (kTokenInstr + kTileWaves - 1) / kTileWaves;  // of the first kFullWaves wavefronts; the others one less
  static constexpr int kFullWaves = kTokenInstr % kTileWaves == 0 ? kTileWaves : kTokenInstr % kTileWaves;
  static constexpr int kTilesPerWave = kRealRows / kTile / WN;
  static constexpr int kWaveRows = BM * WN / kTileWaves;            // weight rows of a wavefront
  static constexpr int kWeightTiles = kWaveRows / kTile;
  static_assert(kWeightTiles % 2 == 0 && BM % (kLoadRows * kTileWaves) == 0, "gate and up rows pair up inside a wavefront");
  static_assert(kRealRows % (kTile * WN) == 0 && kStages >= 2, "the ring holds a stage in use and one on its way");
};

template <int... I, typename F>
__device__ __forceinline__ void unrolled(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}

static_assert(kXcds * kXcdGroups == kTileGroups, "every workgroup has its turn on an XCD");

// units of an item
template <bool GATEUP, int BM>
__device__ __forceinline__ int tile_parts(const FfnArgs& p) {
  constexpr int kOut = GATEUP ? BM / 2 : BM;
  return ((GATEUP ? p.dm : p.dh) + kOut - 1) / kOut * (GATEUP ? 1 : p.ksplit);
}

// h[row, j] = silu(gate) * up, or y[slice][row][r] = partial down projection, of the units of an XCD from place `lo` up to `hi`, of which
// this workgroup takes one of every kXcdGroups.  Items have at most TileShape::kRealRows rows; p.ksplit slices of d_m (down), none
// of them empty.  SPLIT = 2: halves of units of 2 BM weight rows, and at most one for a workgroup.
template <int DT, bool GATEUP, int BM, int BN, int WN, bool LO, int SPLIT>
__device__ __forceinline__ void tile_units(const FfnArgs& p, unsigned char* lds, unsigned lo, unsigned hi, unsigned longs, unsigned to_long,
                                           unsigned to_other) {
  using Sh = TileShape<BM, BN, WN, LO>;
  constexpr int EB = Store<DT>::bytes;
  constexpr int S = Sh::kStages, NQ = Sh::kWeightLoads, NI = Sh::kTokenLoads, NT = Sh::kTilesPerWave;
  const uint32_t lds0 = static_cast<uint32_t>(
      reinterpret_cast<uintptr_t>(reinterpret_cast<__attribute__((address_space(3))) unsigned char*>(
          reinterpret_cast<uintptr_t>(lds))));
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int i = lane & 15, g = lane >> 4;
  // the wavefronts of one SIMD (w and w + 4) differ in wn: an item of few rows keeps all four SIMDs busy
  constexpr int WM = kTileWaves / WN, RW = Sh::kWaveRows, NA = Sh::kWeightTiles;
  const int wm = wave % WM, wn = wave / WM;
  const int dh = p.dh, dm = p.dm;
  const int ld = GATEUP ? dh : dm;                       // row length of both operands
  const int outs = GATEUP ? dm : dh;
  constexpr int kOut = GATEUP ? BM / 2 : BM;             // output columns of a unit
  const int ksplit = GATEUP ? 1 : p.ksplit;
  const int parts = tile_parts<GATEUP, BM * SPLIT>(p);
  const int blocks = ld * EB / kRowBytes, per = (blocks + ksplit - 1) / ksplit;
  constexpr bool kLongFirst = DT == SERE_F32;
  const unsigned turn = blockIdx.x / kXcds;
  const auto next_unit = [&](unsigned u) __attribute__((always_inline)) {
    return kLongFirst ? next_place_long_first(u, turn, longs) : u + kXcdGroups;
  };
  const auto unit_at = [&](unsigned u) __attribute__((always_inline)) { return kLongFirst ? unit_at_long_first(u, longs, to_long, to_other) : u; };
  unsigned pu = lo + turn;                               // unit being loaded
  unsigned cu = pu;                                      // unit being multiplied
  if (pu >= hi) return;
  if (SPLIT > 1 && unit_first_out(pu, SPLIT, parts, ksplit, kOut) >= outs) return;

  // ---- loading side
  constexpr int CH = kRowBytes / 16;                     // pieces of a row
  const uint32_t piece = ((lane & (CH - 1)) ^ (lane / CH)) << 4;   // of a lane's row, see the layout above
  const uint32_t lane_off = static_cast<uint32_t>(lane / CH) * ld * EB + piece;
  const char* wbase[NQ];
  const char* tptr[NI];
  int pk = 0, pbeg = 0, pnk = 0, pleft = 0;
  auto open_load_unit = [&](unsigned u) __attribute__((always_inline)) {
    const int item = u / SPLIT / parts, part = u / SPLIT % parts;
    const int e = scalar_load(p.work_expert, item), off = scalar_load(p.work_off, item), cnt = scalar_load(p.work_cnt, item);
    const int slab = part / ksplit, slice = part % ksplit;
    const char* W = static_cast<const char*>(expert_base<DT>(GATEUP ? p.w_gate_up : p.w_down,
                                                             GATEUP ? p.shared_gate_up : p.shared_down, e, p.M,
                                                             static_cast<size_t>(GATEUP ? 2 : 1) * dm * dh));
    const int o0 = (slab * SPLIT + u % SPLIT) * kOut;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int r = kLoadRows * (wave * NQ + q);                // first of the LDS rows of this load
      int row;
      if (GATEUP) {
        // of a wavefront's RW rows the first half are gate rows, the second half the matching up rows
        int j = o0 + r / RW * (RW / 2) + r % (RW / 2);
        if (j >= dm) j = o0 + r % (RW / 2);
        row = r % RW >= RW / 2 ? dm + j : j;
      } else {
        row = o0 + r < dh ? o0 + r : o0;
      }
      wbase[q] = W + static_cast<size_t>(row) * ld * EB;
    }
#pragma unroll
    for (int n = 0; n < NI; ++n) {
      const int v0 = kLoadRows * (wave + kTileWaves * n);       // first of the token rows
      size_t row = 0;
      if (GATEUP) {
        int tok = 0;
#pragma unroll
        for (int s = 0; s < kLoadRows; ++s) {
          const int t = scalar_load(p.sorted_token, off + min(v0 + s, cnt - 1));
          tok = lane / CH == s ? t : tok;
        }
        row = tok;
      } else {
        const int v = v0 + lane / CH;
        const int plane = LO && v >= Sh::kRealRows ? 1 : 0;
        row = static_cast<size_t>(plane) * p.rows + off + min(v - plane * Sh::kRealRows, cnt - 1);
      }
      const char* base = GATEUP ? static_cast<const char*>(p.hidden) : reinterpret_cast<const char*>(p.h);
      tptr[n] = base + row * ld * EB + piece;
    }
    pbeg = min(slice * per, blocks);
    pnk = min((slice + 1) * per, blocks) - pbeg;
    // Units of 128 bf16 weight rows start where the unit of 256 that covers them would: with the same slices of d_m
    // the sums then have the same order whatever the item size, which calibration batches in groups rely on.
    constexpr int kShared = DT == SERE_BF16 ? 256 / (BM * SPLIT) : 1;
    pk = (slab / kShared * ksplit + slice) * 5 % pnk;
    pleft = pnk;
  };
  constexpr int P = NQ + NI;                             // loads of a stage
  auto issue_some = [&](int slot, auto from, auto to) __attribute__((always_inline)) {  // loads from .. to - 1 of the next stage, into `slot`
    const size_t koff = static_cast<size_t>(pbeg + pk) * kRowBytes;
    const uint32_t at = lds0 + slot * Sh::kStageBytes;
#pragma unroll
    for (int n = decltype(from)::value; n < decltype(to)::value; ++n) {
      if (n < NQ) {
        lds_load_weights(uniform(at + (wave * NQ + n) * 1024), lane_off, uniform(wbase[n < NQ ? n : 0] + koff));
      } else if (n + 1 < P || wave < Sh::kFullWaves) {
        lds_load_tokens(uniform(at + BM * kRowBytes + (wave + kTileWaves * (n - NQ)) * 1024), tptr[n - NQ < 0 ? 0 : n - NQ] + koff);
      }
    }
  };
  auto next_load_step = [&]() __attribute__((always_inline)) {
    if (++pk == pnk) pk = 0;
    if (--pleft == 0) {
      pu = next_unit(pu);
      if (pu < hi) open_load_unit(unit_at(pu));
    }
  };

  // ---- multiplying side
  const uint32_t frag = i * kRowBytes + ((g ^ (i & 7)) << 4);
  f32x4 acc[NA][NT];
  f32x4 low[DT == SERE_F32 ? NA : 1][DT == SERE_F32 ? NT : 1];   // what acc has lost (fp32)
  int cnt = 0, off = 0, part = 0, half = 0, left = 0;
  auto open_unit = [&](unsigned u) __attribute__((always_inline)) {
    const int item = u / SPLIT / parts;
    part = u / SPLIT % parts;
    half = u % SPLIT;
    off = scalar_load(p.work_off, item);
    cnt = scalar_load(p.work_cnt, item);
    const int slice = part % ksplit;
    left = min((slice + 1) * per, blocks) - min(slice * per, blocks);
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        acc[a][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (DT == SERE_F32) low[a][t] = acc[a][t];
      }
  };
  struct Frags {
    u32x4 w[NA], x[NT], y[LO ? NT : 1];
  };
  auto fetch = [&](Frags& f, int slot, int h) __attribute__((always_inline)) {          // operands of one 32-wide half of a stage
    const unsigned char* st = lds + slot * Sh::kStageBytes + (frag ^ (h << 6));
#pragma unroll
    for (int a = 0; a < NA; ++a) f.w[a] = *reinterpret_cast<const u32x4*>(st + (wm * RW + a * 16) * kRowBytes);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int tile = wn + WN * t;
      f.x[t] = *reinterpret_cast<const u32x4*>(st + (BM + tile * kTile) * kRowBytes);
      if (LO) f.y[t] = *reinterpret_cast<const u32x4*>(st + (BM + Sh::kRealRows + tile * kTile) * kRowBytes);
    }
  };
  f32x4 sums[4][DT == SERE_F32 ? NA : 1][DT == SERE_F32 ? NT : 1];
  auto multiply = [&](const Frags& f, auto which, auto&& between) __attribute__((always_inline)) {
    auto tile_of = [&](int t) __attribute__((always_inline)) {
      if constexpr (DT == SERE_F32) {
        // 16 of the step's 32 k: lane (g, i) has four consecutive k of its rows, one product each.  The matrix
        // cores add one after the other; a chain over the whole contraction would round more than a sum over
        // 64 lanes does (2.6e-7 against 1.8e-7 relative error at d_h = 1024).  So every 8 products are summed
        // on their own, a step's four sums pairwise, and what each addition of a step's sum to the unit's
        // rounds away is kept in a sum of its own, which is added at the end.  It never enters the running
        // sum: once that is infinite the rounded-away part is a NaN.
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int a = 0; a < NA; ++a) {
            f32x4& sum = sums[2 * decltype(which)::value + j / 2][a][t];
            sum = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(f.w[a][j]), __uint_as_float(f.x[t][j]),
                                                       j % 2 == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sum, 0, 0, 0);
          }
        __builtin_amdgcn_sched_barrier(0);   // the additions behind all products
        if constexpr (decltype(which)::value == 1) {
#pragma unroll
          for (int a = 0; a < NA; ++a) {
            const f32x4 add = (sums[0][a][t] + sums[1][a][t]) + (sums[2][a][t] + sums[3][a][t]);
            const f32x4 next = acc[a][t] + add;
            low[a][t] += add - (next - acc[a][t]);
            acc[a][t] = next;
          }
        }
        return;
      }
#pragma unroll
      for (int a = 0; a < NA; ++a) acc[a][t] = mfma_bf16(f.w[a], f.x[t], acc[a][t]);
      if (LO) {
#pragma unroll
        for (int a = 0; a < NA; ++a) acc[a][t] = mfma_bf16(f.w[a], f.y[t], acc[a][t]);
      }
    };
    unrolled(std::make_integer_sequence<int, NT>{}, [&](auto t) __attribute__((always_inline)) {
      if ((wn + WN * decltype(t)::value) * kTile < cnt) tile_of(decltype(t)::value);
      between(t);
    });
  };
  auto store = [&]() __attribute__((always_inline)) {
    if constexpr (DT == SERE_F32) {
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float sum = acc[a][t][r] + low[a][t][r];
            acc[a][t][r] = __builtin_amdgcn_fmed3f(sum, sum, acc[a][t][r]);   // acc where the sum is a NaN
          }
    }
    const int slab = part / ksplit, slice = part % ksplit;
    if (GATEUP) {
      const int j0 = (slab * SPLIT + half) * kOut + wm * (RW / 2);
      if (j0 >= dm) return;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int n = (wn + WN * t) * kTile + i;
        if (n < cnt) {
#pragma unroll
          for (int a = 0; a < NA / 2; ++a)               // gate tiles, then the matching up tiles
            store_h4<DT>(p, static_cast<size_t>(off + n) * dm + j0 + 16 * a + 4 * g, acc[a][t], acc[a + NA / 2][t]);
        }
      }
    } else {
      const int r0 = (slab * SPLIT + half) * kOut + wm * RW;
      if (r0 >= dh) return;
      float* y = p.y + static_cast<size_t>(slice) * p.rows * dh;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int n = (wn + WN * t) * kTile + i;
        if (n < cnt) {
          float* dst = y + static_cast<size_t>(off + n) * dh + r0 + 4 * g;
#pragma unroll
          for (int a = 0; a < NA; ++a) *reinterpret_cast<f32x4*>(dst + 16 * a) = acc[a][t];
        }
      }
    }
  };

  // Steps run half a step out of phase with the stages: while a stage's second half is multiplied, the first
  // half of the next one is read from LDS, so that reads and products overlap within a wavefront.
  if (DT == SERE_F32 && wn == 0) __builtin_amdgcn_s_setprio(1);   // of the two wavefronts of a SIMD
  open_load_unit(unit_at(pu));
  int ahead = 0, slot = 0;                               // stages issued and not yet waited for; slot in use
  for (; ahead < S && pu < hi; ++ahead) {
    issue_some(ahead, std::integral_constant<int, 0>{}, std::integral_constant<int, P>{});
    next_load_step();
  }
  open_unit(unit_at(cu));
  auto wait_stage = [&](auto issued) {                   // the oldest of the stages issued, by all wavefronts
    constexpr int D = decltype(issued)::value;           // how many there are while units are left to load
    if (ahead == D) {
      // everything but the youngest D - 1 stages (stores among them make the wait longer, never shorter)
      if (wave < Sh::kFullWaves) wait_loads<(D - 1) * (NQ + NI)>(); else wait_loads<(D - 1) * (NQ + NI - 1)>();
    } else {
      wait_loads<0>();
    }
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    --ahead;
  };
  Frags f0, f1;
  // One stage: the second half of the products of the stage before it, then the first half of its own.
  auto step = [&](bool more) __attribute__((always_inline)) { // more: a stage is left to load
    const int used = slot;
    slot = slot + 1 == S ? 0 : slot + 1;
    fetch(f0, slot, 0);
    // the loads of a stage, spread over the first three quarters of the products, each after a token tile's (one token tile:
    // all of them after the first half; two stages: over the first quarter, they are waited for at the end of the same
    // products)
    auto loads = [&](auto half) __attribute__((always_inline)) {
      return [&](auto t) __attribute__((always_inline)) {
        constexpr int h = decltype(half)::value * NT + decltype(t)::value, groups = NT == 1 ? 1 : S == 2 ? NT / 2 : (3 * NT + 1) / 2;
        constexpr int n0 = std::min(P, h * P / groups), n1 = std::min(P, (h + 1) * P / groups);
        if (n0 < n1 && more) issue_some(used, std::integral_constant<int, n0>{}, std::integral_constant<int, n1>{});
      };
    };
    multiply(f1, std::integral_constant<int, 1>{}, loads(std::integral_constant<int, 0>{}));
    if (--left == 0) {
      store();
      cu = next_unit(cu);
      open_unit(unit_at(cu));
    }
    fetch(f1, slot, 1);
    multiply(f0, std::integral_constant<int, 0>{}, loads(std::integral_constant<int, 1>{}));
    if (more) {
      next_load_step();
      ++ahead;
    }
  };
  const auto nothing = [](auto) __attribute__((always_inline)) {};
  wait_stage(std::integral_constant<int, S>{});
  fetch(f0, 0, 0);
  fetch(f1, 0, 1);
  multiply(f0, std::integral_constant<int, 0>{}, nothing);
  while (ahead > 0) {
    // the wait also covers this wavefront's reads of the stage in use, whose slot is then free
    wait_stage(std::integral_constant<int, S - 1>{});
    step(pu < hi);
  }
  multiply(f1, std::integral_constant<int, 1>{}, nothing);
  store();
}

// grid kTileGroups, 512 threads
template <int DT, bool GATEUP, int BM, int BN, int WN, bool LO>
__global__ __launch_bounds__(kTileThreads, 1) void ffn_tile(FfnArgs p) {
  using Sh = TileShape<BM, BN, WN, LO>;
  static_assert(DT == SERE_BF16 || !LO, "fp32 keeps h as it is");
  constexpr bool kHalves = DT == SERE_BF16 && !(BM == 256 && BN == 256);
  using Half = TileShape<kHalves ? BM / 2 : BM, BN, WN, LO>;
  constexpr int kRing = Sh::kStages * Sh::kStageBytes, kHalfRing = Half::kStages * Half::kStageBytes;
  __shared__ __attribute__((aligned(16))) unsigned char lds[kRing > kHalfRing ? kRing : kHalfRing];
  const unsigned parts = tile_parts<GATEUP, BM>(p), total = static_cast<unsigned>(scalar_load(p.n_work, 0)) * parts;
  const unsigned xcd = blockIdx.x % kXcds;
  // This workgroup's units: one of every round of its XCD's contiguous range.
  if constexpr (kHalves) {
    const unsigned lo = xcd_share(total, xcd), hi = xcd_share(total, xcd + 1);
    const unsigned whole = whole_units_end(lo, hi, halves_pay(GATEUP, p.dh / 64));   // (p.dh: of gate/up)
    tile_units<DT, GATEUP, BM, BN, WN, LO, 1>(p, lds, lo, whole, 0, 0, 0);
    if (whole < hi) {
      __builtin_amdgcn_s_barrier();                      // every wavefront has read its last stage
      asm volatile("" ::: "memory");
      tile_units<DT, GATEUP, BM / 2, BN, WN, LO, 2>(p, lds, 2 * whole, 2 * hi, 0, 0, 0);
    }
  } else if constexpr (DT == SERE_BF16) {
    tile_units<DT, GATEUP, BM, BN, WN, LO, 1>(p, lds, xcd_share(total, xcd), xcd_share(total, xcd + 1), 0, 0, 0);
  } else {
    const LongFirst f = long_first(total, static_cast<unsigned>(scalar_load(p.n_work, 2)) * parts, xcd);
    tile_units<DT, GATEUP, BM, BN, WN, LO, 1>(p, lds, 0, f.count, f.longs, f.to_long, f.to_other);
  }
}

}  // namespace sere
