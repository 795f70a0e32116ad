// Expert-similarity estimation (Sec. 3.1.1, the appendix on similarity metrics
// and the appendix algorithm "Expert Similarity Estimation"): every expert
// runs on every calibration token through the same grouped FFN kernels the
// decode path uses (a work list in which each expert owns all tokens of the
// batch); then, with the Frobenius metric, x_pq = ||A_p - A_q||_F for all
// pairs and Sim = 1 - x / max(x) per batch, or, with the cosine metric, the
// mean over tokens of the cosine between the two experts' outputs, or linear
// CKA of the experts' Gram matrices; Sim is accumulated over batches and
// averaged.
//
// Calibration batches are taken in groups of g: an expert's weights are streamed once for the g * n
// tokens of a group (a batch of 32 tokens of the Qwen3 shape: forward pass 200 us alone, 66 us in a
// group of four), and every kernel of the pair stage serves the whole group in one
// launch.  Rows of y: expert-major, then batch, then token; V_e of a batch is n * d_h consecutive
// numbers, and the same batch of the next expert lies g * n * d_h further.
#pragma once

#include "common.hpp"
#include "ffn_tile.hpp"
#include "similarity_plan.hpp"

namespace sere {

// work list "every expert, all n tokens" (n: of a group) in items of at most item_rows rows (about equal ones, of whole
// 16-row tiles): grid ceil(M*n/256), 256 threads
__global__ __launch_bounds__(256) void similarity_worklist_kernel(int M, int n, int item_rows, int32_t* sorted_token,
                                                                  int32_t* work_expert, int32_t* work_off,
                                                                  int32_t* work_cnt, int32_t* n_work) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < M * n) sorted_token[i] = i % n;
  const int items = (n + item_rows - 1) / item_rows;
  if (i < M * items) {
    const int e = i / items, j = i % items;
    const int per = items > 1 ? min(item_rows, ((n + items - 1) / items + 15) & ~15) : n;
    const int first = min(j * per, n);
    work_expert[i] = e;
    work_off[i] = e * n + first;
    work_cnt[i] = min(per, n - first);
  }
  if (i == 0) {
    n_work[0] = M * items;
    n_work[1] = 0;  // many long items: coarse cut
    n_work[2] = 0;
  }
}

// Frobenius distances of all pairs (appendix "Frobenius Similarity"), x_pq = ||A_p - A_q||_F, from
// the Gram matrix of the experts' outputs: with V_e the output of expert e on the batch, flattened
// to one vector of L = n * d_h numbers (A_e = sum over slices of y[slice][e*n .. e*n+n) rows),
//   x_pq^2 = <V_p, V_p> + <V_q, V_q> - 2 <V_p, V_q>.
// The Gram matrix is a dense contraction over L and runs on the matrix cores in fp64
// (v_mfma_f64_16x16x4: products of fp32 numbers are exact in fp64, sums carry ~1e-16 relative
// rounding each), so the cancellation in the formula above costs at most ~1e-15 of an output's
// squared norm: harmless for every pair but near-identical twins, which are recomputed as a
// direct difference by the wavefront that finds them.
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kGramSteps = 2;      // 16-wide k steps per load group (two groups are in flight)
constexpr double kGramTwinThreshold = 1e-9;  // x_pq^2 below this fraction of <V_p,V_p> + <V_q,V_q>: recompute directly

// upper-triangular blocks (bp <= bq) numbered row by row
__device__ __forceinline__ void gram_block_of(int index, int nb, int& bp, int& bq) {
  bp = 0;
  while (index >= nb - bp) {
    index -= nb - bp;
    ++bp;
  }
  bq = bp + index;
}

// part[split][p][q] = sum over the split's range of L of V_p[k] * V_q[k], for every (p, q) of the
// upper-triangular 64 x 64 blocks.  grid (nb (nb + 1) / 2, nsplit), 256 threads; lane l of a
// wavefront holds row l % 16 of each of its tiles, and of every 16 consecutive k the four
// 4 (l / 16) ... + 3 (the order of k inside the sum is free as long as both operands agree).
// `chunk` (the split's length) is a multiple of 2 * 16 * kGramSteps (= 64, as L is).  blockIdx.z: batch of
// the group.
// More than 64 experts: the cosine metric, y in slices, and the groups for which the staged kernel below is the slower one
// (gram_staged_pays).  43 TFLOP/s at 128 experts, 128 tokens, d_h 2048 (147 us a batch; the fp64 matrix cores reach
// 69 in a large product).  Neither more workgroups (three for every compute unit instead of one and a half) nor
// four independent sums between two products of one changed that: it waits for its operands.
// COSINE: every row of A is divided by its length first (inv_norm[row]; see row_norm_kernel), so the entries
// are sums over tokens of cosines.
template <bool COSINE>
__global__ __launch_bounds__(256) void pair_gram_kernel(const float* __restrict__ y, int ksplit, int rows, int n,
                                                        int dh, int M, long long chunk, double* __restrict__ part,
                                                        const double* __restrict__ inv_norm,
                                                        unsigned long long* __restrict__ max_bits) {
  if (!COSINE && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) max_bits[blockIdx.z] = 0ull;   // for frobenius_distance_kernel
  const int nb = (M + kGramBlock - 1) / kGramBlock;
  int bp, bq;
  gram_block_of(blockIdx.x, nb, bp, bq);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r16 = lane & 15, kq = lane >> 4;
  const int p0 = bp * kGramBlock + (wave >> 1) * 32, q0 = bq * kGramBlock + (wave & 1) * 32;
  const long long L = static_cast<long long>(n) * dh;             // multiple of 64
  const size_t slice = static_cast<size_t>(rows) * dh;
  const int g = gridDim.z, batch = blockIdx.z;
  const float* ap[2];
  const float* aq[2];
  const double* ip[2];
  const double* iq[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {   // rows beyond M repeat the last one (their results are not stored)
    const size_t rp = static_cast<size_t>(min(p0 + 16 * t + r16, M - 1)) * g + batch;
    const size_t rq = static_cast<size_t>(min(q0 + 16 * t + r16, M - 1)) * g + batch;
    ap[t] = y + rp * L + 4 * kq;
    aq[t] = y + rq * L + 4 * kq;
    ip[t] = inv_norm + rp * n;
    iq[t] = inv_norm + rq * n;
  }
  const long long kbeg = blockIdx.y * chunk, kend = min(kbeg + chunk, L);
  auto fetch = [&](const float* row, long long k) {
    float4 v = *reinterpret_cast<const float4*>(row + k);
    for (int s = 1; s < ksplit; ++s) {
      const float4 v2 = *reinterpret_cast<const float4*>(row + s * slice + k);
      v.x += v2.x; v.y += v2.y; v.z += v2.z; v.w += v2.w;
    }
    return v;
  };
  f64x4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  // groups of kGramSteps steps, double buffered: the loads of the next group are in flight while
  // the current one is multiplied (the split's length is a multiple of 2 * 16 * kGramSteps)
  float4 va[2][kGramSteps][2], vb[2][kGramSteps][2];
  double sa[2][2], sb[2][2];   // COSINE: the group's row factors (a group of 32 consecutive k lies in one token: d_h % 64 == 0)
  auto fetch_group = [&](int buf, long long k) {
    if constexpr (COSINE) {
      const int token = static_cast<int>(k) / dh;   // L is below 2^29
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        sa[buf][t] = ip[t][token];
        sb[buf][t] = iq[t][token];
      }
    }
#pragma unroll
    for (int st = 0; st < kGramSteps; ++st)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        va[buf][st][t] = fetch(ap[t], k + 16 * st);
        vb[buf][st][t] = fetch(aq[t], k + 16 * st);
      }
  };
  auto multiply_group = [&](int buf) {
#pragma unroll
    for (int st = 0; st < kGramSteps; ++st)
#pragma unroll
      for (int j = 0; j < 4; ++j) {   // four independent sums between two products of one
        double x[2], w[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          x[t] = static_cast<double>(reinterpret_cast<const float*>(&va[buf][st][t])[j]);
          w[t] = static_cast<double>(reinterpret_cast<const float*>(&vb[buf][st][t])[j]);
          if constexpr (COSINE) {
            x[t] *= sa[buf][t];
            w[t] *= sb[buf][t];
          }
        }
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[a], w[b], acc[a][b], 0, 0, 0);
      }
  };
  constexpr int kGroup = 16 * kGramSteps;
  fetch_group(0, kbeg);
  for (long long k = kbeg; k < kend; k += 2 * kGroup) {
    fetch_group(1, k + kGroup);                               // in range: the split holds whole pairs of groups
    multiply_group(0);
    fetch_group(0, k + 2 * kGroup < kend ? k + 2 * kGroup : kbeg);   // after the last pair: a harmless re-read
    multiply_group(1);
  }
  // lane l holds D[l / 16 + 4 r][l % 16], r = 0..3 (the fp64 tile interleaves its row blocks)
  double* out = part + (static_cast<size_t>(batch) * gridDim.y + blockIdx.y) * gram_part_stride(M);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int pp = p0 + 16 * a + kq + 4 * r, qq = q0 + 16 * b + r16;
        if (pp < M && qq < M) out[static_cast<size_t>(pp) * M + qq] = acc[a][b][r];
      }
}

// The same for up to 64 experts, 16 TILES of them: a wavefront holds all tiles of the upper triangle (10 at most, where the
// kernel above computes 16 whatever M is) and reads every row once for them; the four wavefronts of a workgroup take every
// fourth group of k and add up through LDS in a fixed order.  Bound by the fp64 matrix cores at 64 experts and by reading y at
// 16.  us of the pair stage, 64 x 64 blocks against this (with the unrolled reduction below), four batches of 128 tokens, d_h
// 2048: 60 experts 206 -> 131, 16 experts 184 -> 44, 8 experts with the cosine metric 198 -> 50; 40 experts, d_h 1024 116 -> 61;
// 64 experts, four batches of 16 tokens 39 -> 32.
// grid (1, nsplit, g), 256 threads.
template <int TILES, bool COSINE>
__global__ __launch_bounds__(256) void pair_gram_few_kernel(const float* __restrict__ y, int ksplit, int rows, int n, int dh, int M,
                                                            long long chunk, double* __restrict__ part,
                                                            const double* __restrict__ inv_norm,
                                                            unsigned long long* __restrict__ max_bits) {
  constexpr int kPairs = TILES * (TILES + 1) / 2;
  constexpr int kSteps = gram_few_steps(TILES, COSINE);
  __shared__ double s_part[4][kPairs * 4][kWave];
  if (!COSINE && blockIdx.y == 0 && threadIdx.x == 0) max_bits[blockIdx.z] = 0ull;   // for frobenius_distance_kernel
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r16 = lane & 15, kq = lane >> 4;
  const long long L = static_cast<long long>(n) * dh;             // multiple of 64
  const size_t slice = static_cast<size_t>(rows) * dh;
  const int g = gridDim.z, batch = blockIdx.z;
  const long long kbeg = blockIdx.y * chunk, kend = min(kbeg + chunk, L);   // multiples of 64
  const int steps = static_cast<int>((kend - kbeg) / 16);
  const float* row[TILES];
  const double* inv[TILES];
#pragma unroll
  for (int t = 0; t < TILES; ++t) {   // rows beyond M repeat the last one (their results are not stored)
    const size_t r = static_cast<size_t>(min(16 * t + r16, M - 1)) * g + batch;
    row[t] = y + r * L + kbeg + 4 * kq;
    inv[t] = inv_norm + r * n;
  }
  f64x4 acc[kPairs];
#pragma unroll
  for (int c = 0; c < kPairs; ++c) acc[c] = f64x4{0.0, 0.0, 0.0, 0.0};
  float4 v[2][kSteps][TILES];
  double scale[2][TILES];
  auto fetch = [&](int buf, int first) {   // a step beyond the last re-reads that one and is not used
    if constexpr (COSINE) {
      const int token = static_cast<int>(kbeg + 16 * min(first, steps - 1)) / dh;   // L is below 2^29
#pragma unroll
      for (int t = 0; t < TILES; ++t) scale[buf][t] = inv[t][token];
    }
#pragma unroll
    for (int st = 0; st < kSteps; ++st)
#pragma unroll
      for (int t = 0; t < TILES; ++t) {
        const float* at = row[t] + 16 * min(first + st, steps - 1);
        float4 x = *reinterpret_cast<const float4*>(at);
        for (int s = 1; s < ksplit; ++s) {
          const float4 x2 = *reinterpret_cast<const float4*>(at + s * slice);
          x.x += x2.x; x.y += x2.y; x.z += x2.z; x.w += x2.w;
        }
        v[buf][st][t] = x;
      }
  };
  auto multiply = [&](int buf, int first) {
#pragma unroll
    for (int st = 0; st < kSteps; ++st)
      if (first + st < steps) {   // wave-uniform
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          double x[TILES];
#pragma unroll
          for (int t = 0; t < TILES; ++t) {
            x[t] = static_cast<double>(reinterpret_cast<const float*>(&v[buf][st][t])[j]);
            if constexpr (COSINE) x[t] *= scale[buf][t];
          }
          int c = 0;
#pragma unroll
          for (int a = 0; a < TILES; ++a)
#pragma unroll
            for (int b = a; b < TILES; ++b, ++c) acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[a], x[b], acc[c], 0, 0, 0);
        }
      }
  };
  int at = wave * kSteps;
  fetch(0, at);
  for (; at < steps; at += 8 * kSteps) {
    fetch(1, at + 4 * kSteps);
    multiply(0, at);
    fetch(0, at + 8 * kSteps);
    multiply(1, at + 4 * kSteps);
  }
#pragma unroll
  for (int c = 0; c < kPairs; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) s_part[wave][4 * c + r][lane] = acc[c][r];
  __syncthreads();
  // wavefront w finishes register w of every tile: lane l holds D[l / 16 + 4 r][l % 16]
  double* out = part + (static_cast<size_t>(batch) * gridDim.y + blockIdx.y) * gram_part_stride(M);
  int c = 0;
#pragma unroll
  for (int a = 0; a < TILES; ++a)
#pragma unroll
    for (int b = a; b < TILES; ++b, ++c) {
      const int reg = 4 * c + wave, pp = 16 * a + kq + 4 * wave, qq = 16 * b + r16;
      const double sum = ((s_part[0][reg][lane] + s_part[1][reg][lane]) + s_part[2][reg][lane]) + s_part[3][reg][lane];
      if (pp < M && qq < M) out[static_cast<size_t>(pp) * M + qq] = sum;
    }
}

// The same partial Gram matrices (Frobenius metric, y in one slice, where gram_staged_pays) with the operands
// staged through LDS: a workgroup takes a triangle of 128 experts, or a square of 64 x 64 between two such
// triangles, and a range of L, and reads each of its 128 rows once, in whole 128-byte lines that go straight to a
// ring of kGramRing stages (128 rows x 32 k; 16-byte piece c of a row lies at c ^ (row & 7), so that the reads are
// free of bank conflicts).  In the kernel above every row is read by two blocks and by two wavefronts of each, 64
// bytes at a time, and a diagonal block computes its lower half as well.
// 8 wavefronts: wavefront w takes the 16 k of half w / 4 of each stage and, of the triangle's 8 x 8 tiles, the
// cyclic share b = 2 (w & 3): (b, b + d) and (b + 1, b + 1 + d) for d = 0..3 and one of the four tiles at
// d = 4 (rows modulo 8), nine tiles each; of a square's 4 x 4 tiles row w & 3.  The two halves are added at the end.
// Bound by the fp64 matrix cores and the conversions between their products: 128 experts, 128 tokens, d_h 2048 take
// 91 us a batch (4.8 GFLOP of fp64: 53 TFLOP/s; the kernel above: 147 us for 6.4 GFLOP); reading a stage from LDS
// while the one before it is multiplied changed nothing.  With the cosine metric or y in slices the loads need
// arithmetic.
constexpr int kGramRing = 8;
constexpr int kGramRowsLds = 128;
constexpr int kGramStageBytes = kGramRowsLds * kRowBytes;
constexpr int kGramStagedThreads = 512;

// grid (gram_triangles + gram_squares, nsplit, g), 512 threads
__global__ __launch_bounds__(kGramStagedThreads) void pair_gram_staged_kernel(const float* __restrict__ y, int n, int dh,
                                                                              int M, long long chunk,
                                                                              double* __restrict__ part,
                                                                              unsigned long long* __restrict__ max_bits) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[kGramRing * kGramStageBytes];
  const uint32_t lds0 = static_cast<uint32_t>(
      reinterpret_cast<uintptr_t>(reinterpret_cast<__attribute__((address_space(3))) unsigned char*>(
          reinterpret_cast<uintptr_t>(lds))));
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) max_bits[blockIdx.z] = 0ull;   // for frobenius_distance_kernel
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r16 = lane & 15, kq = lane >> 4, half = wave >> 2;
  const int g = gridDim.z, batch = blockIdx.z;
  const long long L = static_cast<long long>(n) * dh;             // multiple of 64
  const bool triangle = static_cast<int>(blockIdx.x) < gram_triangles(M);
  int p0, q0;   // first expert of the stage's rows 0..63 and 64..127
  if (triangle) {
    p0 = blockIdx.x * 128;
    q0 = p0 + 64;
  } else {
    const int n64 = (M + 63) / 64;
    int index = blockIdx.x - gram_triangles(M), p = 0;
    while (index >= max(n64 - 2 * (p / 2 + 1), 0)) {
      index -= max(n64 - 2 * (p / 2 + 1), 0);
      ++p;
    }
    p0 = p * 64;
    q0 = (2 * (p / 2 + 1) + index) * 64;
  }
  const long long kbeg = blockIdx.y * chunk, kend = min(kbeg + chunk, L);
  const int steps = static_cast<int>((kend - kbeg) / 32);         // >= 2: chunks are multiples of 64, as L is
  const char* src[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {   // rows beyond M repeat the last one (their results are not stored)
    const int row = 16 * wave + 8 * i + (lane >> 3);
    const int e = min((row < 64 ? p0 : q0 - 64) + row, M - 1);
    src[i] = reinterpret_cast<const char*>(y + (static_cast<size_t>(e) * g + batch) * L + kbeg) + 16 * ((lane & 7) ^ (row & 7));
  }
  auto issue = [&](int step) {
    const uint32_t at = lds0 + (step % kGramRing) * kGramStageBytes + wave * 16 * kRowBytes;
#pragma unroll
    for (int i = 0; i < 2; ++i) lds_load_tokens(at + i * kLoadRows * kRowBytes, src[i] + static_cast<size_t>(step) * kRowBytes);
  };
  auto fetch = [&](int step, int tile) {   // 4 consecutive k of row r16 of a 16-row tile
    const int row = 16 * tile + r16;
    return *reinterpret_cast<const float4*>(lds + (step % kGramRing) * kGramStageBytes + row * kRowBytes +
                                            16 * ((4 * half + kq) ^ (row & 7)));
  };
  auto next_stage = [&](int step) {   // stage `step` is there; the stage before it is free and is filled again
    if (step + kGramRing - 1 <= steps) wait_loads<2 * (kGramRing - 2)>(); else wait_loads<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (step + kGramRing - 1 < steps) issue(step + kGramRing - 1);
  };
  for (int s = 0; s < min(kGramRing - 1, steps); ++s) issue(s);
  // lane l holds D[l / 16 + 4 r][l % 16], r = 0..3 (the fp64 tile interleaves its row blocks).  The second half's
  // sums pass through the ring, which is free by then.
  double* out = part + (static_cast<size_t>(batch) * gridDim.y + blockIdx.y) * gram_part_stride(M);
  auto finish = [&](auto& acc, auto count, auto tile_of) {
    constexpr int N = decltype(count)::value;
    double* sums = reinterpret_cast<double*>(lds) + (wave & 3) * N * 4 * kWave;
    __syncthreads();
    if (half == 1) {
#pragma unroll
      for (int t = 0; t < N; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) sums[(4 * t + r) * kWave + lane] = acc[t][r];
    }
    __syncthreads();
    if (half == 1) return;
#pragma unroll
    for (int t = 0; t < N; ++t) {
      int ti, tj;
      tile_of(t, ti, tj);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double v = acc[t][r] + sums[(4 * t + r) * kWave + lane];
        const int row = 16 * ti + kq + 4 * r, col = 16 * tj + r16;
        int pp = (row < 64 ? p0 : q0 - 64) + row, qq = (col < 64 ? p0 : q0 - 64) + col;
        if (ti > tj) {   // only tiles of the upper triangle are kept
          const int swap = pp;
          pp = qq;
          qq = swap;
        }
        if (pp < M && qq < M) out[static_cast<size_t>(pp) * M + qq] = v;
      }
    }
  };
  auto element = [](const float4& v, int j) { return static_cast<double>(j == 0 ? v.x : j == 1 ? v.y : j == 2 ? v.z : v.w); };
  if (triangle) {
    const int b = 2 * (wave & 3), last = (wave & 3) < 2 ? 0 : 1;   // row b + last has the tile at d = 4
    f64x4 acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    for (int s = 0; s < steps; ++s) {
      next_stage(s);
      float4 v[7];
#pragma unroll
      for (int t = 0; t < 5; ++t) v[t] = fetch(s, (b + t) & 7);
      v[5] = fetch(s, (b + last) & 7);
      v[6] = fetch(s, (b + last + 4) & 7);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        double x[7];
#pragma unroll
        for (int t = 0; t < 7; ++t) x[t] = element(v[t], j);
#pragma unroll
        for (int t = 0; t < 8; ++t)
          acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[t >> 2], x[(t >> 2) + (t & 3)], acc[t], 0, 0, 0);
        acc[8] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[5], x[6], acc[8], 0, 0, 0);
      }
    }
    finish(acc, std::integral_constant<int, 9>{}, [&](int t, int& ti, int& tj) {
      ti = (t < 8 ? b + (t >> 2) : b + last) & 7;
      tj = (t < 8 ? b + (t >> 2) + (t & 3) : b + last + 4) & 7;
    });
  } else {
    f64x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    for (int s = 0; s < steps; ++s) {
      next_stage(s);
      float4 v[5];
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] = fetch(s, 4 + t);
      v[4] = fetch(s, wave & 3);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(element(v[4], j), element(v[t], j), acc[t], 0, 0, 0);
    }
    finish(acc, std::integral_constant<int, 4>{}, [&](int t, int& ti, int& tj) {
      ti = wave & 3;
      tj = 4 + t;
    });
  }
}

// The partial Gram matrices are added in two fixed-order levels: group r of kGramGroups takes the
// splits r, r + kGramGroups, ... (this kernel; entries below the diagonal of 16 x 16 tiles are
// copies of their mirror image), and the distance kernel adds the kGramGroups group sums.
// Only the upper entries are summed, in rows, and written twice: 8 us for 128 experts and 256 splits, against 28 with
// the lower entries read down the columns of their mirror image.  Eight splits are requested together: with one after the other
// 40 experts took 10 us, 16 experts as long, now 5.
// grid (ceil(M * M / 256), kGramGroups, g), 256 threads.
__global__ __launch_bounds__(256) void gram_reduce_kernel(const double* __restrict__ part, int nsplit, int M,
                                                          double* __restrict__ gram) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= M * M) return;
  const int a = idx / M, b = idx % M;
  if (a / 16 > b / 16) return;   // written by its mirror entry: read in rows, the partial sums come in whole lines
  const size_t mm = gram_part_stride(M);
  const double* src = part + static_cast<size_t>(blockIdx.z) * nsplit * mm + idx;
  double g = 0.0;
#pragma unroll 8
  for (int s = blockIdx.y; s < nsplit; s += kGramGroups) g += src[s * mm];
  double* out = gram + (static_cast<size_t>(blockIdx.z) * kGramGroups + blockIdx.y) * M * M;
  out[idx] = g;
  if (a / 16 < b / 16) out[b * M + a] = g;
}

// dist[p][q] = sqrt(G_pp + G_qq - 2 G_pq), G = the sum of the group sums `gram`.  A pair whose squared distance is below
// kGramTwinThreshold of G_pp + G_qq (near-identical outputs: the subtraction has cancelled most
// digits) is recomputed as a direct difference sqrt(sum_i (A_p[i] - A_q[i])^2) by the whole
// wavefront, one such pair after the other.  The largest distance of the batch is gathered in
// *max_bits (the bits of a non-negative double order like the number; cleared by the Gram kernel).
// grid (ceil(M * M / 256), g), 256 threads.
__global__ __launch_bounds__(256) void frobenius_distance_kernel(const double* __restrict__ gram,
                                                                 const float* __restrict__ y, int ksplit, int rows,
                                                                 int n, int dh, int M, double* __restrict__ dist,
                                                                 unsigned long long* __restrict__ max_bits) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  const int lane = threadIdx.x & 63;
  const int g = gridDim.y, batch = blockIdx.y;
  const bool valid = idx < M * M;
  gram += static_cast<size_t>(batch) * kGramGroups * M * M;
  dist += static_cast<size_t>(batch) * M * M;
  const int p = valid ? idx / M : 0, q = valid ? idx % M : 0;
  double d = 0.0;
  bool twin = false;
  auto entry = [&](int at) {   // the group sums of one entry, in fixed order
    double g = 0.0;
#pragma unroll
    for (int r = 0; r < kGramGroups; ++r) g += gram[static_cast<size_t>(r) * M * M + at];
    return g;
  };
  if (valid && p != q) {
    const double gpp = entry(p * M + p), gqq = entry(q * M + q);
    const double d2 = (gpp + gqq) - 2.0 * entry(idx);
    twin = d2 < kGramTwinThreshold * (gpp + gqq);
    if (!twin) d = sqrt(d2);
  }
  unsigned long long todo = __ballot(twin);
  const size_t len = static_cast<size_t>(n) * dh;          // multiple of 64
  const size_t slice = static_cast<size_t>(rows) * dh;
  while (todo != 0ull) {                                   // wave-uniform
    const int src = __ffsll(static_cast<long long>(todo)) - 1;
    todo &= todo - 1ull;
    const int tp = __shfl(p, src, kWave), tq = __shfl(q, src, kWave);
    const float* ap = y + (static_cast<size_t>(tp) * g + batch) * len;
    const float* aq = y + (static_cast<size_t>(tq) * g + batch) * len;
    double acc = 0.0;
    for (size_t i = static_cast<size_t>(lane) * 4; i < len; i += 256) {
      float4 a = *reinterpret_cast<const float4*>(ap + i), b = *reinterpret_cast<const float4*>(aq + i);
      for (int s = 1; s < ksplit; ++s) {
        const float4 a2 = *reinterpret_cast<const float4*>(ap + s * slice + i);
        const float4 b2 = *reinterpret_cast<const float4*>(aq + s * slice + i);
        a.x += a2.x; a.y += a2.y; a.z += a2.z; a.w += a2.w;
        b.x += b2.x; b.y += b2.y; b.z += b2.z; b.w += b2.w;
      }
      const double dx = static_cast<double>(a.x) - b.x, dy = static_cast<double>(a.y) - b.y;
      const double dz = static_cast<double>(a.z) - b.z, dw = static_cast<double>(a.w) - b.w;
      acc += dx * dx + dy * dy + dz * dz + dw * dw;
    }
    acc = wave_sum(acc);
    if (lane == src) d = sqrt(acc);
  }
  if (valid) dist[idx] = d;
  double m = d;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, kWave));
  if (lane == 0 && m > 0.0) atomicMax(max_bits + batch, static_cast<unsigned long long>(__double_as_longlong(m)));
}

// Cosine metric (appendix "Cosine Similarity"): Sim(p, q) = (1/n) sum over tokens i of <A_p[i], A_q[i]> /
// (|A_p[i]| |A_q[i]|); a token where the product of the two lengths is not positive (either output is the
// zero vector, or has a NaN) contributes 0.  With every row divided by its length that sum is an entry of the Gram
// matrix of the flattened outputs, so it takes the Frobenius metric's kernels: M * M / 2 products on the fp64
// matrix cores instead of a workgroup per ordered pair that reads both experts' outputs from cache (two batches of
// 32 tokens, 128 experts, d_h 2048, forward pass included: 1278 -> 329 us).
// A sum over tokens cannot leave one out after the fact (NaN * 0 is NaN), so rows without a finite positive
// length are set to zero here, before the Gram kernel reads them:
// inv_norm[row] = 1 / |y[row]|, 0 for a zero row and one with a NaN, -1 for an infinite one.
// grid ceil(rows / 4), 256 threads: a wavefront per row.
__global__ __launch_bounds__(256) void row_norm_kernel(float* __restrict__ y, int ksplit, int rows, int dh,
                                                       double* __restrict__ inv_norm) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= rows) return;
  const size_t slice = static_cast<size_t>(rows) * dh;
  float* a = y + static_cast<size_t>(row) * dh;
  double sum = 0.0;
  for (int c = lane * 4; c < dh; c += 256) {
    float4 v = *reinterpret_cast<const float4*>(a + c);
    for (int s = 1; s < ksplit; ++s) {
      const float4 w = *reinterpret_cast<const float4*>(a + s * slice + c);
      v.x += w.x; v.y += w.y; v.z += w.z; v.w += w.w;
    }
    const double x = v.x, yy = v.y, z = v.z, w = v.w;
    sum += x * x + yy * yy + z * z + w * w;
  }
  sum = wave_sum(sum);
  const bool normal = sum > 0.0 && sum < INFINITY;
  if (!normal)   // wave-uniform
    for (int s = 0; s < ksplit; ++s)
      for (int c = lane * 4; c < dh; c += 256) *reinterpret_cast<float4*>(a + s * slice + c) = float4{0.0f, 0.0f, 0.0f, 0.0f};
  if (lane == 0) inv_norm[row] = normal ? 1.0 / sqrt(sum) : sum > 0.0 ? -1.0 : 0.0;
}

// dist[batch][p][q] = (1/n) sum of the group sums; grid (ceil(M * M / 256), g), 256 threads.  A token whose output
// is infinite makes the quotient NaN, unless the other expert's is zero or has a NaN there.  Such tokens
// are missing from an expert's sum with itself, which otherwise is n, so few pairs look for them.
__global__ __launch_bounds__(256) void cosine_mean_kernel(const double* __restrict__ gram,
                                                          const double* __restrict__ inv_norm, int n, int M,
                                                          double* __restrict__ dist) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= M * M) return;
  const int g = gridDim.y, batch = blockIdx.y, p = idx / M, q = idx % M;
  auto entry = [&](int at) {   // the group sums of one entry, in fixed order
    double sum = 0.0;
#pragma unroll
    for (int r = 0; r < kGramGroups; ++r) sum += gram[(static_cast<size_t>(batch) * kGramGroups + r) * M * M + at];
    return sum;
  };
  double sum = entry(idx);
  const double pp = entry(p * M + p), qq = entry(q * M + q);   // (all three requested together)
  if (fmin(pp, qq) < n - 0.5) {
    const double* a = inv_norm + (static_cast<size_t>(p) * g + batch) * n;
    const double* b = inv_norm + (static_cast<size_t>(q) * g + batch) * n;
    for (int i = 0; i < n; ++i)
      if ((a[i] < 0.0 && b[i] != 0.0) || (b[i] < 0.0 && a[i] != 0.0)) sum = NAN;
  }
  dist[static_cast<size_t>(batch) * M * M + idx] = sum / n;
}

// Linear CKA (appendix "Centered Kernel Alignment"), step 1: the Gram matrix of every expert's
// outputs with its diagonal set to zero, gram[e][i][j] = <A_e[i], A_e[j]> (i != j), and the sums of its
// rows, block by block: rowsum[e][bj][i] = sum of row i over the columns of block bj.  (e: expert and batch.)
// A workgroup takes a block of 16 B x 16 B entries of the upper triangle over the whole d_h on the fp64 matrix cores
// (operands as in pair_gram_kernel: 16 rows x 64 bytes an instruction, the next group of loads in flight while one is
// multiplied); its four wavefronts take every fourth group of k and their sums are added in a fixed order through LDS.
// Entries below the diagonal are copies, so the matrix is symmetric to the bit.  Bound by the rows' way from cache, which
// B = 2 halves; B = 1 gives batches of up to kCkaSmallTokens tokens three times as many workgroups (us, launch: 60
// experts, d_h 2048, two batches of 32 tokens B = 1 20, of 64 tokens B = 1 55, B = 2 49, of 128 B = 2 115, 70 TFLOP/s;
// 128 experts, d_h 512, 60 tokens B = 1 54, B = 2 23).  With a wavefront per entry on the vector ALU: 77 us at 32 tokens.
// More groups in flight or eight wavefronts changed nothing at 32 tokens and lost on short rows (d_h 512: 19 -> 32 us).
// With `diag` (RBF and polynomial kernels) the diagonal <A_e[i], A_e[i]> goes there and the row
// sums are left to gram_transform_kernel.  grid (nb (nb + 1) / 2, M * g), nb = ceil(n / (16 B)), 256 threads.
template <int B>
__global__ __launch_bounds__(256) void cka_gram_kernel(const float* __restrict__ y, int ksplit, int rows, int n, int dh,
                                                       double* __restrict__ gram, double* __restrict__ rowsum,
                                                       double* __restrict__ diag) {
  constexpr int W = 4, kSide = 16 * B, kAhead = 2, kSteps = B == 1 ? 4 : 2, kGroup = 16 * kSteps;   // d_h is a multiple of 64
  __shared__ double s_part[W][B * B * 4][kWave];
  __shared__ double s_tile[kSide][kSide + 1];
  const int nb = (n + kSide - 1) / kSide, e = blockIdx.y;
  int bi, bj;
  gram_block_of(blockIdx.x, nb, bi, bj);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r16 = lane & 15, kq = lane >> 4;
  const size_t slice = static_cast<size_t>(rows) * dh;
  const float* ai[B];
  const float* aj[B];
#pragma unroll
  for (int t = 0; t < B; ++t) {   // rows beyond n repeat the last one (their results are not stored)
    ai[t] = y + (static_cast<size_t>(e) * n + min(bi * kSide + 16 * t + r16, n - 1)) * dh + 4 * kq;
    aj[t] = y + (static_cast<size_t>(e) * n + min(bj * kSide + 16 * t + r16, n - 1)) * dh + 4 * kq;
  }
  auto fetch = [&](const float* row, int k) {
    float4 v = *reinterpret_cast<const float4*>(row + k);
    for (int s = 1; s < ksplit; ++s) {
      const float4 v2 = *reinterpret_cast<const float4*>(row + s * slice + k);
      v.x += v2.x; v.y += v2.y; v.z += v2.z; v.w += v2.w;
    }
    return v;
  };
  f64x4 acc[B][B];
#pragma unroll
  for (int a = 0; a < B; ++a)
#pragma unroll
    for (int b = 0; b < B; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  float4 va[kAhead][kSteps][B], vb[kAhead][kSteps][B];   // groups whose loads are in flight
  auto fetch_group = [&](int buf, int group) {
#pragma unroll
    for (int st = 0; st < kSteps; ++st)
#pragma unroll
      for (int t = 0; t < B; ++t) {
        va[buf][st][t] = fetch(ai[t], group * kGroup + 16 * st);
        vb[buf][st][t] = fetch(aj[t], group * kGroup + 16 * st);
      }
  };
  auto multiply_group = [&](int buf) {
#pragma unroll
    for (int st = 0; st < kSteps; ++st)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int a = 0; a < B; ++a)
#pragma unroll
          for (int b = 0; b < B; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(reinterpret_cast<const float*>(&va[buf][st][a])[j]),
                                                             static_cast<double>(reinterpret_cast<const float*>(&vb[buf][st][b])[j]),
                                                             acc[a][b], 0, 0, 0);
  };
  const int groups = dh / kGroup;
#pragma unroll
  for (int d = 0; d < kAhead; ++d)
    if (wave + d * W < groups) fetch_group(d, wave + d * W);
  for (int i = wave; i < groups; i += kAhead * W) {
#pragma unroll
    for (int d = 0; d < kAhead; ++d) {
      if (i + d * W < groups) multiply_group(d);
      if (i + (d + kAhead) * W < groups) fetch_group(d, i + (d + kAhead) * W);
    }
  }
#pragma unroll
  for (int a = 0; a < B; ++a)
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) s_part[wave][(a * B + b) * 4 + r][lane] = acc[a][b][r];
  __syncthreads();
  // a wavefront finishes one register of a tile at a time: lane l holds D[l / 16 + 4 r][l % 16]
  gram += static_cast<size_t>(e) * n * n;
  for (int at = wave; at < 4 * B * B; at += W) {
    const int t = at / 4;
    double v = s_part[0][at][lane];
#pragma unroll
    for (int w = 1; w < W; ++w) v += s_part[w][at][lane];
    const int li = 16 * (t / B) + kq + 4 * (at % 4), lj = 16 * (t % B) + r16;
    const int i = bi * kSide + li, j = bj * kSide + lj;
    const bool inside = i < n && j < n;
    if (bi == bj && li > lj) continue;        // written by its mirror entry
    if (i == j) {
      if (diag != nullptr && inside) diag[static_cast<size_t>(e) * n + i] = v;
      v = 0.0;
    }
    if (!inside) v = 0.0;
    s_tile[li][lj] = v;
    if (bi == bj) s_tile[lj][li] = v;
    if (inside) {
      gram[static_cast<size_t>(i) * n + j] = v;
      gram[static_cast<size_t>(j) * n + i] = v;
    }
  }
  if (diag != nullptr) return;
  __syncthreads();
  rowsum += static_cast<size_t>(e) * nb * n;
  if (threadIdx.x < kSide) {
    const int i = bi * kSide + threadIdx.x;
    double sum = 0.0;
#pragma unroll
    for (int j = 0; j < kSide; ++j) sum += s_tile[threadIdx.x][j];
    if (i < n) rowsum[static_cast<size_t>(bj) * n + i] = sum;
  } else if (threadIdx.x >= kWave && threadIdx.x < kWave + kSide && bi != bj) {   // the mirror block's rows
    const int c = threadIdx.x - kWave, j = bj * kSide + c;
    double sum = 0.0;
#pragma unroll
    for (int i = 0; i < kSide; ++i) sum += s_tile[i][c];
    if (j < n) rowsum[static_cast<size_t>(bi) * n + j] = sum;
  }
}

constexpr int kCkaLinear = 0, kCkaRbf = 1, kCkaPoly = 2;  // SERE_CKA_* of the header

// The other two kernels of that appendix, from the linear Gram matrix G (off-diagonal entries in
// `gram`, diagonal in `diag`), in place, with the row sums of the result:
//   RBF:        K_ij = exp(-(G_ii + G_jj - 2 G_ij) / (2 sigma^2)),  sigma = p0
//   polynomial: K_ij = (G_ij + c)^d,  c = p0, d = degree (repeated multiplication)
// The diagonal stays 0 (the HSIC estimator ignores it); (i, j) and (j, i) take the same operations
// on the same values, so the matrix stays symmetric to the bit.  grid (n, M * g), 256 threads.
__global__ __launch_bounds__(256) void gram_transform_kernel(double* __restrict__ gram,
                                                             const double* __restrict__ diag, int n, int kernel,
                                                             double p0, int degree,
                                                             double* __restrict__ rowsum) {
  __shared__ double part[4];
  const int i = blockIdx.x, e = blockIdx.y;
  double* row = gram + (static_cast<size_t>(e) * n + i) * n;
  const double* d = diag + static_cast<size_t>(e) * n;
  const double di = d[i];
  double sum = 0.0;
  for (int j = threadIdx.x; j < n; j += 256) {
    double v = 0.0;
    if (j != i) {
      const double g = row[j];
      if (kernel == kCkaRbf) {
        v = exp(-((di + d[j]) - 2.0 * g) / (2.0 * p0 * p0));
      } else {
        const double base = g + p0;
        v = base;
        for (int k = 1; k < degree; ++k) v *= base;
      }
    }
    row[j] = v;
    sum += v;
  }
  sum = wave_sum(sum);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x == 0) rowsum[static_cast<size_t>(e) * n + i] = (part[0] + part[1]) + (part[2] + part[3]);
}

// CKA, step 2: the unbiased estimator of HSIC for every pair of experts (Song et al. 2012,
// the O(n^2) estimator the appendix refers to), from the zero-diagonal Gram matrices Kt_p, Kt_q:
//   hsic[p][q] = [ tr(Kt_p Kt_q) + (1'Kt_p 1)(1'Kt_q 1) / ((n-1)(n-2)) - 2 (1'Kt_p Kt_q 1) / (n-2) ] / (n (n-3))
// with tr(Kt_p Kt_q) = sum_ij Kt_p[i][j] Kt_q[i][j] (symmetric matrices) and 1'Kt_p Kt_q 1 = the
// dot product of the two row-sum vectors.  Traces and dot products are Gram matrices again, of the M flattened
// matrices and the M row-sum vectors: 16 x 16 pairs a workgroup on the fp64 matrix cores, the upper triangle of the
// pairs only (60 experts, two batches of 32 tokens: 7 us; a workgroup for every ordered pair that reads both
// matrices from cache: 20).  n * n is cut into gridDim.y parts, hsic[batch][part][p][q]; the last one has
// the terms of the row sums (in `nb` blocks a row), alone if there are several.  grid (mb (mb + 1) / 2, parts, g), mb = ceil(M / 16), 256 threads; n >= 4.
typedef double f64x2_unaligned __attribute__((ext_vector_type(2), aligned(8)));
__global__ __launch_bounds__(256) void cka_pair_kernel(const double* __restrict__ gram, const double* __restrict__ rowsum,
                                                       int nb, int n, int M, double* __restrict__ hsic) {
  __shared__ double s_part[4][4][4][kWave];   // [wavefront][trace, cross, sum of p, sum of q][register][lane]
  int bp, bq;
  gram_block_of(blockIdx.x, (M + 15) / 16, bp, bq);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r16 = lane & 15, kq = lane >> 4;
  const int g = gridDim.z, batch = blockIdx.z, part = blockIdx.y;
  // rows beyond M repeat the last one (their results are not stored)
  const size_t p = static_cast<size_t>(min(16 * bp + r16, M - 1)) * g + batch, q = static_cast<size_t>(min(16 * bq + r16, M - 1)) * g + batch;
  const int parts = max(static_cast<int>(gridDim.y) - 1, 1);          // of the products
  const int K = n * n, groups = (K + 15) / 16, per = (groups + parts - 1) / parts;
  const int gend = min((part + 1) * per, groups);
  const double* kp = gram + p * K;
  const double* kv = gram + q * K;
  f64x4 trace = {0.0, 0.0, 0.0, 0.0}, cross = trace, sp = trace, sq = trace;
  constexpr int kAhead = 2;    // groups of 16 k whose loads are issued together
  struct Operands {
    double a[kAhead][4], b[kAhead][4];
  };
  auto fetch = [&](Operands& o, int group) {   // lane (r16, kq): k = 16 group + 4 kq .. + 3 of its rows
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int k0 = 16 * min(group + 4 * u, groups - 1), k = k0 + 4 * kq;
      if (k0 + 16 <= K) {   // wave-uniform; all but the last group of an n that is no multiple of 4
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f64x2_unaligned x = *reinterpret_cast<const f64x2_unaligned*>(kp + k + 2 * h);
          const f64x2_unaligned w = *reinterpret_cast<const f64x2_unaligned*>(kv + k + 2 * h);
          o.a[u][2 * h] = x[0];
          o.a[u][2 * h + 1] = x[1];
          o.b[u][2 * h] = w[0];
          o.b[u][2 * h + 1] = w[1];
        }
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          o.a[u][j] = k + j < K ? kp[k + j] : 0.0;
          o.b[u][j] = k + j < K ? kv[k + j] : 0.0;
        }
      }
    }
  };
  auto multiply = [&](const Operands& o, int group) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      if (group + 4 * u < gend) {   // wave-uniform
#pragma unroll
        for (int j = 0; j < 4; ++j) trace = __builtin_amdgcn_mfma_f64_16x16x4f64(o.a[u][j], o.b[u][j], trace, 0, 0, 0);
      }
  };
  Operands o0, o1;
  int at = part * per + wave;
  if (at < gend) fetch(o0, at);
  for (; at < gend; at += 8 * kAhead) {
    fetch(o1, at + 4 * kAhead);
    multiply(o0, at);
    fetch(o0, at + 8 * kAhead);
    multiply(o1, at + 4 * kAhead);
  }
  if (part == static_cast<int>(gridDim.y) - 1) {
    const double* rp = rowsum + p * nb * n;
    const double* rq = rowsum + q * nb * n;
    for (int st = wave; st * 4 < n; st += 4) {
      const int i = 4 * st + kq;
      double x = 0.0, w = 0.0;
      if (i < n)
#pragma unroll 4
        for (int b = 0; b < nb; ++b) {
          x += rp[static_cast<size_t>(b) * n + i];
          w += rq[static_cast<size_t>(b) * n + i];
        }
      cross = __builtin_amdgcn_mfma_f64_16x16x4f64(x, w, cross, 0, 0, 0);
      sp = __builtin_amdgcn_mfma_f64_16x16x4f64(x, 1.0, sp, 0, 0, 0);
      sq = __builtin_amdgcn_mfma_f64_16x16x4f64(1.0, w, sq, 0, 0, 0);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    s_part[wave][0][r][lane] = trace[r];
    s_part[wave][1][r][lane] = cross[r];
    s_part[wave][2][r][lane] = sp[r];
    s_part[wave][3][r][lane] = sq[r];
  }
  __syncthreads();
  double v[4];   // wavefront w finishes register w
#pragma unroll
  for (int c = 0; c < 4; ++c)
    v[c] = ((s_part[0][c][wave][lane] + s_part[1][c][wave][lane]) + s_part[2][c][wave][lane]) + s_part[3][c][wave][lane];
  const int pp = 16 * bp + kq + 4 * wave, qq = 16 * bq + r16;
  if (pp > qq || qq >= M) return;   // below the diagonal: written by the mirror entry
  const double dn = n;
  const double h = (v[0] + v[2] * v[3] / ((dn - 1.0) * (dn - 2.0)) - 2.0 * v[1] / (dn - 2.0)) / (dn * (dn - 3.0));
  hsic += (static_cast<size_t>(batch) * gridDim.y + part) * M * M;
  hsic[static_cast<size_t>(pp) * M + qq] = h;
  hsic[static_cast<size_t>(qq) * M + pp] = h;
}

constexpr int kMetricFrobenius = 0, kMetricCosine = 1, kMetricCkaLinear = 2;

// Frobenius: acc[p][q] (+)= 1 - dist/max(dist), the maximum of the batch given as the bits of a
// double in *max_bits; cosine: acc[p][q] (+)= dist[p][q] (the pair kernel's value as it is); linear
// CKA: acc[p][q] (+)= dist[p][q] / sqrt(dist[p][p] dist[q][q]), dist holding the HSIC estimates in `parts` summands (0
// where a self-term is not positive: the quotient is undefined there).  The g batches of the group are added
// in order.  With the last batch sim = acc / N.  grid ceil(M * M / 256), 256 threads.
__global__ __launch_bounds__(256) void similarity_accumulate_kernel(const double* __restrict__ dist, int parts, int M,
                                                                    int batch0, int g, int num_batches, int metric,
                                                                    const unsigned long long* __restrict__ max_bits,
                                                                    double* __restrict__ acc,
                                                                    float* __restrict__ sim) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= M * M) return;
  double a = batch0 == 0 ? 0.0 : acc[i];
  for (int b = 0; b < g; ++b, dist += static_cast<size_t>(parts) * M * M) {
    double sv;
    if (metric == kMetricCosine) {
      sv = dist[i];
    } else if (metric == kMetricCkaLinear) {
      double h = 0.0, hp = 0.0, hq = 0.0;
#pragma unroll 4
      for (int s = 0; s < parts; ++s) {
        const double* d = dist + static_cast<size_t>(s) * M * M;
        h += d[i];
        hp += d[static_cast<size_t>(i / M) * M + i / M];
        hq += d[static_cast<size_t>(i % M) * M + i % M];
      }
      sv = (hp > 0.0 && hq > 0.0) ? h / sqrt(hp * hq) : 0.0;
    } else {
      const double mx = __longlong_as_double(static_cast<long long>(max_bits[b]));
      sv = mx > 0.0 ? 1.0 - dist[i] / mx : 1.0;  // all pairs identical: Sim = 1
    }
    a += sv;
  }
  acc[i] = a;
  if (batch0 + g == num_batches) sim[i] = static_cast<float>(a / num_batches);
}

}  // namespace sere
