// Host side of the similarity estimation: how many calibration batches a group takes, which kernels serve it and
// where its buffers lie in the workspace.  A function of the sizes alone.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "../../include/sere.h"
#include "ffn_plan.hpp"

namespace sere {

constexpr int kGramBlock = 64;     // experts per side of a block of pair_gram_kernel: 2 x 2 wavefronts, each 2 x 2 tiles of 16 x 16; up to
                                   // that many experts pair_gram_few_kernel
constexpr int kGramGroups = 8;     // group sums that gram_reduce_kernel leaves
// 16-wide k steps of a load group of pair_gram_few_kernel (16 `tiles` experts): enough bytes in flight; with the cosine metric a
// group, 64 k at most, lies in one token
constexpr int gram_few_steps(int tiles, bool cosine) { return tiles == 1 ? (cosine ? 4 : 8) : tiles == 2 ? 4 : 2; }
// partial Gram matrices lie M * M + kGramPad doubles apart: a power-of-two distance would put the
// same entry of every split on the same memory channel
constexpr int kGramPad = 96;
constexpr size_t gram_part_stride(int M) { return static_cast<size_t>(M) * M + kGramPad; }
// pair_gram_staged_kernel: triangles of 128 experts, and squares, which are pairs of 64-row groups that lie in
// different triangles
constexpr int gram_squares(int M) {
  const int n64 = (M + 63) / 64;
  int count = 0;
  for (int p = 0; p < n64; ++p) count += n64 > 2 * (p / 2 + 1) ? n64 - 2 * (p / 2 + 1) : 0;
  return count;
}
constexpr int gram_triangles(int M) { return (M + 127) / 128; }

// Calibration batches are served in groups within kSimGroupBytes of workspace, so that an expert's weights are streamed once per group and
// a stage is one launch: 32 tokens of the Qwen3 shape 200 us alone, 110 / 66 / 50 us a batch in groups of 2 / 4 / 8.  A call with
// less workspace, or with fewer batches, runs smaller groups.  Groups are of kSimGroupMin batches, whatever
// their length, up to kSimGroupRows tokens; short batches of kSimGroupShortRows tokens together.  us a call, groups of 256 tokens / of 512 /
// of 1024 (the longest ones that the batches allow): Qwen3 shape, four batches of 128 1094 / 988, of 78 tokens, 94 experts, d_h 1664, d_m
// 1088 758 / 632; 11 experts, d_h 2048, four of 83 258 / 212; eight of 114, 41 experts, d_h 832 395 / 308 / 262; twelve of 83, 5
// experts, d_h 1920 450 / 288 / 249.  41 calls with more than 256 tokens: 1.45 / 1.47 times as fast on average, none slower.
// Measured on 14 layers of 0.8 to 288 MB, three metrics, 2 to 16 batches of 4 to 100 tokens: a group takes 0.1 to 0.9
// times what its batches take one by one, the less the smaller layer and batch (12 MB, 8 batches of 32 tokens: 249 / 58
// us, 288 MB: 667 / 225).  us a call of layers of at most 8 MiB, one batch at a time / in a group: 3 batches of 66 tokens, 2
// experts, d_h 576 109 / 47, 4 of 13, 4 experts of d_h 384 in fp32 116 / 38, 2 of 31, 19 experts of d_h 256 54 / 34; 13 calls 2.1
// times as fast on average, none less than 1.35 times.
constexpr int kSimGroupRows = 1024, kSimGroupShortRows = 256, kSimGroupMin = 8, kSimGroupMax = 16;
constexpr size_t kSimGroupBytes = size_t{1} << 30;

struct SimLayout {
  size_t sorted_token, work_expert, work_off, work_cnt, n_work, h, y, dist, acc, gram, rowsum, diag, gram_part, inv_norm, max_bits,
      total;
  size_t block_sums;    // linear CKA: the Gram matrices' row sums block by block, in the place of h
  int cka_parts;        // summands of a pair's estimate (CKA); several lie in the place of y
  int rows, ksplit;
  FfnPlan plan;
  int items;            // work items of an expert
  bool gram_staged;     // Frobenius: the Gram kernel that stages through LDS
  int gram_splits;      // slices of the flattened outputs in the Gram kernel
  long long gram_chunk; // ... and their length
};

inline FfnShape sim_ffn_shape(const sere_config& c, int rows) {
  FfnShape s{};
  s.hidden = c.hidden;
  s.inter = c.inter;
  s.tokens = rows;
  s.experts = c.num_experts;
  s.rows = rows;
  s.slots_per_expert = rows;
  s.split_h = wants_split_h(c) != 0;
  s.max_ksplit = down_ksplit(c);
  return s;
}

// The kernels of a group of g batches, of a call whose groups would hold `whole` batches if the workspace had room for
// them.  What decides the order of a sum follows from `whole`, so that neither the size of the workspace nor a shorter
// last group changes a batch's outputs: for bf16 layers the persistent kernels and their slices of d_m, for fp32 layers one
// kernel or the other.  The item size follows the group's own rows.
// (Not from the layer and the batch size alone, which would free them from the number of batches, too: single batches of
// layers with few, wide experts want other kernels than large groups.  4 experts, d_h and d_m 4096, one batch of 20 tokens:
// 113 -> 123 us; 12 experts, d_h and d_m 3072, 8 batches of 16: 257 -> 290.  As it is, two batches of 8 tokens of 8
// experts, d_h 4096, d_m 14336, lose 468 -> 480 and four gain 531 -> 512 against a choice for every group by itself.)
inline FfnPlan sim_ffn_plan(const sere_config& c, int n, int g, int whole) {
  const FfnShape all = sim_ffn_shape(c, n * whole);
  if (c.dtype == SERE_F32) return plan_ffn_f32(all);
  if (whole == 1) return plan_ffn(all);
  return plan_ffn_tile(sim_ffn_shape(c, n * g), plan_ffn_tile(all, 0).ksplit);
}

// Where pair_gram_staged_kernel is the faster one; it needs y in one slice.  `length`: numbers in the outputs of an expert,
// all batches of a group.  us of the pair stage, kernel of 64 x 64 blocks against staged:
//  - One triangle, 65 to 128 experts: a workgroup takes a whole compute unit, so short groups lose (length 8192:
//    25 / 36, 32768: 1.05 times), longer ones gain (49152: 0.88 times, 128 experts: 65536 55 / 48, 262144 0.79 times,
//    524288 300 / 180).  Up to 64 experts pair_gram_few_kernel computes no tile that is not needed.
//  - Beyond, two triangles and two squares take as long as four triangles (129 to 192 experts: 1.4 times), and two with
//    all four squares 1.08 times.  But a row every multiple of 2 MiB puts the rows that the other kernel reads
//    together on the same memory channels: 256 experts of length 524288 970 / 790, of 1048576 1890 / 1520 (of 518400
//    724 / 782, of 557056 770 / 825); 193 experts 826 / 774, 192 still 605 / 637.
constexpr long long kGramStagedLength = 40960;
inline bool gram_staged_pays(int experts, long long length) {
  if (experts <= 128) return experts > kGramBlock && length >= kGramStagedLength;
  return experts > 192 && length * 4 % (2 << 20) == 0;
}

// Centered kernel alignment: the estimator's lower limit; M * n * n doubles of workspace
constexpr int kCkaMinTokens = 4, kCkaMaxTokens = 512;
// side of cka_gram_kernel's blocks (why 48 stands at the kernel), and blocks of a row of a batch's n tokens
constexpr int kCkaSmallTokens = 48;
constexpr int cka_block(int n) { return n <= kCkaSmallTokens ? 16 : 32; }
constexpr int cka_blocks(int n) { return (n + cka_block(n) - 1) / cka_block(n); }

// Parts of a batch's n * n products in cka_pair_kernel, 512 products and more each, and one more for its row sums: a
// wavefront's products wait for their operands one after the other (60 experts, 64 tokens: one part 23 us, eight 8), while
// similarity_accumulate_kernel adds up an entry's parts (32 of them: 7 -> 25 us).  The parts lie where y was: there
// has to be room.
inline int cka_parts(int n, int hidden, int experts) {
  return std::max(1, std::min(1 + std::min(8, (n * n + 511) / 512), static_cast<int>(static_cast<long long>(n) * hidden / (2 * experts))));
}

// Layout of groups of g batches of n tokens.  A call checks its workspace against its largest group and launches
// smaller ones in it (the last of a call), so no buffer's room may shrink as g grows, whatever is chosen by g; and what is
// chosen by `whole` changes nothing about the room, which a caller asks for without naming the number of batches.
inline SimLayout make_sim_layout(const sere_config& c, int n, int g, int whole) {
  SimLayout l{};
  const size_t M = c.num_experts, R = M * static_cast<size_t>(n) * g;
  l.rows = static_cast<int>(R);
  l.ksplit = down_ksplit(c);
  l.plan = sim_ffn_plan(c, n, g, whole);
  l.items = (n * g + l.plan.item_rows - 1) / l.plan.item_rows;
  const size_t W = M * ((static_cast<size_t>(n) * g + kItemRows - 1) / kItemRows);  // room: the shortest items
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o = align_up(o + bytes);
    return at;
  };
  l.acc = take(M * M * sizeof(double));  // first: the same place for groups of every size
  l.sorted_token = take(R * 4);
  l.work_expert = take(W * 4);
  l.work_off = take(W * 4);
  l.work_cnt = take(W * 4);
  l.n_work = take(12);
  l.dist = take(g * M * M * sizeof(double));
  l.max_bits = take(g * 8);
  l.y = take(static_cast<size_t>(l.ksplit) * R * c.hidden * sizeof(float));
  const bool cka = (c.flags & SERE_FLAG_SIM_CKA_LINEAR) != 0;
  const size_t sums = cka ? R * cka_blocks(n) * sizeof(double) : 0;   // no more than h at today's limits (d_m of 64 and more)
  l.h = take(std::max(R * c.inter * sizeof(float), sums));
  if (cka) {  // Gram matrix per expert; its row sums and diagonal for the kernels with parameters
    l.block_sums = l.h;
    l.cka_parts = cka_parts(n, c.hidden, c.num_experts);
    l.gram = take(R * n * sizeof(double));
    l.rowsum = take(R * sizeof(double));
    l.diag = take(R * sizeof(double));
  } else {                                   // partial Gram matrices of the experts' flattened outputs
    // the cosine metric keeps them in the place of h, which is no longer needed when they are written
    const bool in_h = (c.flags & SERE_FLAG_SIM_COSINE) != 0;
    const size_t end = o;
    if (in_h) {
      o = l.h;
      l.inv_norm = take(R * sizeof(double));
    }
    const long long L = static_cast<long long>(n) * c.hidden;
    // about three workgroups for every compute unit, 16 .. 256 splits, each a multiple of the Gram kernel's
    // 64-wide load group (staged kernel: one workgroup to a compute unit at a time; a single triangle: one even
    // wave of them)
    const auto splits = [&](bool staged) {   // of a group of one batch
      const int m = static_cast<int>(M), nb = (m + kGramBlock - 1) / kGramBlock;
      const int blocks = staged ? gram_triangles(m) + gram_squares(m) : nb * (nb + 1) / 2;
      return (staged && blocks == 1 ? 256 : 768) / blocks;
    };
    l.gram_staged = !in_h && l.plan.ksplit == 1 && gram_staged_pays(static_cast<int>(M), g * L);
    const int want = std::min(256, std::max(16, splits(l.gram_staged) / g));
    long long chunk = (L + want - 1) / want;
    chunk = std::max<long long>(256, (chunk + 63) / 64 * 64);
    l.gram_chunk = chunk;
    l.gram_splits = static_cast<int>((L + chunk - 1) / chunk);
    // Room for g * gram_splits partial matrices of this group and of every smaller one, by either kernel: these are at
    // most g * want and at most g * L / 256, but rounding the chunk may give a group of g - 1 batches more of them than
    // one of g.
    const int most = std::min(256 * g, std::max(splits(false), splits(true)));
    const long long room = std::min(g * ((L + 255) / 256), std::max<long long>(16 * g, most));
    l.gram_part = take(static_cast<size_t>(room) * gram_part_stride(static_cast<int>(M)) * sizeof(double));
    l.gram = take(static_cast<size_t>(g) * kGramGroups * M * M * sizeof(double));
    if (in_h) o = std::max(end, o);
  }
  l.total = o;
  return l;
}

// Largest group of a call; a workspace is sized for it.
inline int sim_group(const sere_config& c, int n) {
  const int batches = std::max(std::min(kSimGroupMin, kSimGroupRows / n), std::min(kSimGroupMax, kSimGroupShortRows / n));
  int g = std::max(1, batches);
  while (g > 1 && make_sim_layout(c, n, g, g).total > kSimGroupBytes) --g;
  return g;
}

}  // namespace sere
