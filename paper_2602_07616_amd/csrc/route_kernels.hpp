// Routing kernels: router logits, ordered top-K + gate, and the batch-wide
// re-routing / compaction step.
//
// Paper anchors: router logits R(x) and the top-k gate of the appendix
// "Preliminaries on MoEs"; primary set, most-similar primary, re-routing
// condition and final set of Sec. 3.2.2 (Steps 1-3).  The appendix algorithm
// "CUDA-accelerated SERE" gives one thread to every (token, secondary slot)
// and lets each scan all M experts; here the scan is done once per secondary
// EXPERT (its result depends only on the expert and the primary mask), and the
// rewritten map is counted, prefix-summed and regrouped per expert by the
// same workgroup, in LDS.
//
// Two launches: (1) router logits, delivered per token as sorted lists of 16;
// (2) top-K per token as a merge of the list heads; the workgroup that finishes
// last (a ticket in global memory, cleared by launch 1) then runs the
// batch-wide step, so no third launch is needed.  From kChunkedSlots slots on
// the batch-wide step is a launch of its own, shared by many workgroups.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace sere {

// ------------------------------------------------------------ wave helpers ---
// Value of lane (l ^ 1), (l ^ 2), mirrored inside 8, mirrored inside 16: four
// DPP exchanges that together reach every lane of a 16-lane row.
template <int STEP>
__device__ __forceinline__ uint32_t row_xchg(uint32_t v) {
  constexpr int ctrl = STEP == 0 ? 0xB1 : STEP == 1 ? 0x4E : STEP == 2 ? 0x141 : 0x140;
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), ctrl, 0xF, 0xF, true));
}
template <int STEP>
__device__ __forceinline__ double row_xchg(double v) {
  const uint64_t b = static_cast<uint64_t>(__double_as_longlong(v));
  const uint64_t r = (static_cast<uint64_t>(row_xchg<STEP>(static_cast<uint32_t>(b >> 32))) << 32) |
                     row_xchg<STEP>(static_cast<uint32_t>(b));
  return __longlong_as_double(static_cast<long long>(r));
}

// sum over the 16 lanes of a row; every lane of the row gets it
__device__ __forceinline__ double row_sum(double v) {
  v += row_xchg<0>(v);
  v += row_xchg<1>(v);
  v += row_xchg<2>(v);
  v += row_xchg<3>(v);
  return v;
}

// sum over the wavefront (rows through scalar registers); wave-uniform result.
// The association order is fixed, so equal inputs give bit-equal sums.
__device__ __forceinline__ double wave_sum_dpp(double v) {
  v = row_sum(v);
  const uint64_t b = static_cast<uint64_t>(__double_as_longlong(v));
  const int lo = static_cast<int>(b), hi = static_cast<int>(b >> 32);
  double r[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint64_t x = (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(hi, 16 * q))) << 32) |
                       static_cast<uint32_t>(__builtin_amdgcn_readlane(lo, 16 * q));
    r[q] = __longlong_as_double(static_cast<long long>(x));
  }
  return (r[0] + r[1]) + (r[2] + r[3]);
}

// Barrier that orders LDS traffic only: global stores issued earlier (results
// that nobody in this workgroup reads back) need not have completed.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// f(std::integral_constant<int, 0>{}), ..., f(... N - 1)
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// order-preserving map double -> uint64 (larger double <=> larger key; -0 == +0)
__device__ __forceinline__ uint64_t sortable_key(double v) {
  uint64_t b = static_cast<uint64_t>(__double_as_longlong(v));
  if (b == 0x8000000000000000ull) b = 0;
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ __forceinline__ double key_to_double(uint64_t k) {
  const uint64_t b = (k >> 63) ? (k & 0x7fffffffffffffffull) : ~k;
  return __longlong_as_double(static_cast<long long>(b));
}

// value of the lane D places further round in the 16-lane row (DPP row rotate)
template <int D>
__device__ __forceinline__ uint32_t row_rot(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x120 + D, 0xF, 0xF, true));
}
template <int D>
__device__ __forceinline__ void rank_step(uint64_t key, uint32_t id, uint32_t& rank) {
  const uint64_t okey = (static_cast<uint64_t>(row_rot<D>(static_cast<uint32_t>(key >> 32))) << 32) |
                        row_rot<D>(static_cast<uint32_t>(key));
  const uint32_t oid = row_rot<D>(id);
  rank += (okey > key || (okey == key && oid < id)) ? 1u : 0u;
  if constexpr (D < 15) rank_step<D + 1>(key, id, rank);
}

// ---------------------------------------------------------------------------
// Router logits in fp64, delivered as SORTED LISTS.  grid (ceil(M/16), T),
// 256 threads; wave w of block (bx, t) computes experts bx*16 + 4w .. +3 for
// token t, the four dot products interleaved.  Every logit is reduced in the
// same lane pattern, so bit-identical router rows give bit-identical logits
// (ties then resolve by index, as in exact arithmetic).  The block then ranks
// its 16 logits (larger first, equal: lower expert first) and writes them as
// order-preserving keys with their expert ids:
//   list_key[(t*L + bx)*16 + rank], list_id[(t*L + bx)*16 + rank],  L = gridDim.x;
// places of experts >= M hold key 0 (below every real key).
// Block (0,0) clears the int32 at clear_word.
// ---------------------------------------------------------------------------
template <int DT>
__global__ __launch_bounds__(256) void router_logits_kernel(
    const void* __restrict__ hidden, const void* __restrict__ router_w, uint64_t* __restrict__ list_key,
    uint8_t* __restrict__ list_id, int /*T: one workgroup row per token, see grid*/, int M, int dh,
    int32_t* clear_word) {
  __shared__ double s_logit[16];
  const int t = blockIdx.y;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (clear_word != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *clear_word = 0;
  const int e0 = blockIdx.x * 16 + wave * 4;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  // four 512-wide chunks per pass, all loads of a pass issued before any arithmetic
  // (the router weights come cold from HBM on every step; one round trip instead of four)
  for (int i0 = lane * 8; i0 < dh; i0 += 2048) {
    Raw8<DT> xr[4], wr[4][4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = i0 + 512 * c;
      if (i < dh) {
        xr[c].load(hidden, static_cast<size_t>(t) * dh + i);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (e0 + q < M) wr[c][q].load(router_w, static_cast<size_t>(e0 + q) * dh + i);  // wave-uniform
      }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (i0 + 512 * c < dh) {
        float xv[8];
        xr[c].widen(xv);
        double xd[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) xd[j] = static_cast<double>(xv[j]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (e0 + q < M) {
            float wv[8];
            wr[c][q].widen(wv);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[q] = fma(xd[j], static_cast<double>(wv[j]), acc[q]);
          }
        }
      }
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double sum = wave_sum_dpp(acc[q]);
    if (lane == 0) s_logit[wave * 4 + q] = sum;
  }
  __syncthreads();
  if (threadIdx.x < 16) {  // one 16-lane row; the other rows of the wavefront idle
    const int e = blockIdx.x * 16 + threadIdx.x;
    const uint64_t key = e < M ? sortable_key(s_logit[threadIdx.x]) : 0ull;
    uint32_t rank = 0;
    rank_step<1>(key, static_cast<uint32_t>(e), rank);
    const size_t at = (static_cast<size_t>(t) * gridDim.x + blockIdx.x) * 16 + rank;
    list_key[at] = key;
    list_id[at] = static_cast<uint8_t>(e);
  }
}

// The same for batches of many tokens: a workgroup serves TB tokens with its 16 experts, so a
// router row is fetched once per TB tokens (at 2048 tokens the one-token kernel reads the
// router weights 2048 times from cache).  Wave w: experts bx*16 + 4w .. +3 x tokens
// by*TB .. +TB-1, one 512-wide chunk of the rows at a time.  Same lane pattern per logit as
// above.  grid (ceil(M/16), ceil(T/TB)), 256 threads.
template <int DT, int TB>
__global__ __launch_bounds__(256) void router_logits_tokens_kernel(
    const void* __restrict__ hidden, const void* __restrict__ router_w, uint64_t* __restrict__ list_key,
    uint8_t* __restrict__ list_id, int T, int M, int dh, int32_t* clear_word) {
  __shared__ double s_logit[TB][16];
  const int t0 = blockIdx.y * TB;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (clear_word != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *clear_word = 0;
  const int e0 = blockIdx.x * 16 + wave * 4;
  double acc[4][TB];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int b = 0; b < TB; ++b) acc[q][b] = 0.0;
  // passes of up to four 512-wide chunks, all loads of a pass issued before any arithmetic (the
  // router weights come cold from HBM on every step: one round trip per pass instead of one per chunk)
  constexpr int kChunks = TB <= 2 ? 4 : 2;
  for (int i0 = lane * 8; i0 < dh; i0 += 512 * kChunks) {
    Raw8<DT> xr[kChunks][TB], wr[kChunks][4];
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const int i = min(i0 + 512 * c, dh - 8);   // a chunk beyond d_h re-reads the row's end and is not used
#pragma unroll
      for (int b = 0; b < TB; ++b) xr[c][b].load(hidden, static_cast<size_t>(min(t0 + b, T - 1)) * dh + i);
#pragma unroll
      for (int q = 0; q < 4; ++q) wr[c][q].load(router_w, static_cast<size_t>(min(e0 + q, M - 1)) * dh + i);
    }
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      if (i0 + 512 * c < dh) {
        double wd[4][8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float wv[8];
          wr[c][q].widen(wv);
#pragma unroll
          for (int j = 0; j < 8; ++j) wd[q][j] = static_cast<double>(wv[j]);
        }
#pragma unroll
        for (int b = 0; b < TB; ++b) {
          float xv[8];
          xr[c][b].widen(xv);
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const double xd = static_cast<double>(xv[j]);
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q][b] = fma(xd, wd[q][j], acc[q][b]);
          }
        }
      }
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int b = 0; b < TB; ++b) {
      const double sum = wave_sum_dpp(acc[q][b]);
      if (lane == 0) s_logit[b][wave * 4 + q] = sum;
    }
  __syncthreads();
  if (threadIdx.x < 16 * TB) {  // one 16-lane row per token
    const int b = threadIdx.x >> 4, t = t0 + b;
    const int e = blockIdx.x * 16 + (threadIdx.x & 15);
    const uint64_t key = e < M ? sortable_key(s_logit[b][threadIdx.x & 15]) : 0ull;
    uint32_t rank = 0;
    rank_step<1>(key, static_cast<uint32_t>(e), rank);
    if (t < T) {
      const size_t at = (static_cast<size_t>(t) * gridDim.x + blockIdx.x) * 16 + rank;
      list_key[at] = key;
      list_id[at] = static_cast<uint8_t>(e);
    }
  }
}

// The same for batches of hundreds of tokens and more, where the logits are a dense contraction
// ([T x d_h] x [d_h x M]) and the vector ALU (fp64 FMAs plus the conversions around them) bounds
// the kernels above: the fp64 matrix cores (v_mfma_f64_16x16x4) multiply a tile of 16 tokens x 16
// experts, fed from registers.  A workgroup owns one tile; its four wavefronts take every fourth
// 32-wide chunk of d_h each, and their partial tiles are added in a fixed order through LDS.
// Lane l of a wavefront holds row l % 16 of both operands (a token, an expert) and, of every 32
// consecutive k, the eight from 8 (l / 16) on: one 128-bit load per operand and chunk feeds eight
// MFMAs (the order of k inside a sum is free as long as both operands agree).  Every logit is the
// same sequence of operations on its two rows, so bit-identical router rows still give
// bit-identical logits.  The result tile has lane l hold D[l / 16 + 4 r][l % 16], r = 0..3: with
// the tokens as rows, a 16-lane row of register r holds one token's 16 logits, which is what the
// ranking wants.  Two chunks are multiplied while the loads of the next two are in flight (us, against four whose loads
// are all waited for: 600 tokens x 64 experts 11.6 -> 9.7, 1000 x 128 16.3 -> 14.2, 777 x 32 of d_h 2880 13.9 -> 12.0, 2048
// x 128 25.5 -> 24.0, where the matrix cores alone take 15; four ahead cost the wavefronts in flight that hide the
// conversions, 26.1; eight or sixteen wavefronts a tile 24.6 and 26.7).  grid (ceil(M/16), ceil(T/16)), 256 threads.
typedef double route_f64x4 __attribute__((ext_vector_type(4)));
template <int DT>
__global__ __launch_bounds__(256) void router_logits_mfma_kernel(
    const void* __restrict__ hidden, const void* __restrict__ router_w, uint64_t* __restrict__ list_key,
    uint8_t* __restrict__ list_id, int T, int M, int dh, int32_t* clear_word) {
  constexpr int W = 4;
  __shared__ double s_part[W][4][kWave];  // [wavefront][register r][lane]
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r16 = lane & 15, kq = lane >> 4;
  if (clear_word != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *clear_word = 0;
  const int t0 = blockIdx.y * 16, e0 = blockIdx.x * 16;
  // rows beyond T or M repeat the last one; their results are not stored
  const size_t xrow = static_cast<size_t>(min(t0 + r16, T - 1)) * dh + 8 * kq;
  const size_t wrow = static_cast<size_t>(min(e0 + r16, M - 1)) * dh + 8 * kq;
  route_f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  const int nch = dh >> 5;  // 32-wide chunks; this wavefront takes chunks wave, wave + W, ...
  // two sets of chunks: the loads of one are in flight while the other is multiplied
  constexpr int kAhead = 2;
  Raw8<DT> xr[2][kAhead], wr[2][kAhead];
  auto fetch = [&](int set, int c0) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int c = min(c0 + W * u, nch - 1);  // a chunk beyond the row re-reads its end and is not used
      xr[set][u].load(hidden, xrow + 32 * static_cast<size_t>(c));
      wr[set][u].load(router_w, wrow + 32 * static_cast<size_t>(c));
    }
  };
  auto multiply = [&](int set, int c0) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if (c0 + W * u < nch) {  // wave-uniform
        float xv[8], wv[8];
        xr[set][u].widen(xv);
        wr[set][u].widen(wv);
#pragma unroll
        for (int j = 0; j < 8; ++j)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(xv[j]), static_cast<double>(wv[j]), acc, 0, 0, 0);
      }
    }
  };
  int c = wave;
  fetch(0, c);
  for (; c + 2 * W * kAhead < nch; c += 2 * W * kAhead) {   // no load under a condition: it would be waited for on its own
    fetch(1, c + W * kAhead);
    multiply(0, c);
    fetch(0, c + 2 * W * kAhead);
    multiply(1, c + W * kAhead);
  }
  fetch(1, c + W * kAhead);
  multiply(0, c);
  multiply(1, c + W * kAhead);
#pragma unroll
  for (int r = 0; r < 4; ++r) s_part[wave][r][lane] = acc[r];
  __syncthreads();
  // wavefront w finishes register w: tokens t0 + kq + 4 w, one per 16-lane row
  const double logit = ((s_part[0][wave][lane] + s_part[1][wave][lane]) + s_part[2][wave][lane]) + s_part[3][wave][lane];
  const int t = t0 + kq + 4 * wave, e = e0 + r16;
  const uint64_t key = e < M ? sortable_key(logit) : 0ull;
  uint32_t rank = 0;
  rank_step<1>(key, static_cast<uint32_t>(e), rank);
  if (t < T) {
    const size_t at = (static_cast<size_t>(t) * gridDim.x + blockIdx.x) * 16 + rank;
    list_key[at] = key;
    list_id[at] = static_cast<uint8_t>(e);
  }
}

// ---------------------------------------------------------------------------
// Ordered top-K and gate by merging the sorted lists.  LP (4, 8 or 16) adjacent
// lanes own one token, lane l of the group holds list l (all 16 entries, in
// registers).  K rounds: the group's arg-max over the list heads (log2 LP DPP
// exchanges; larger key wins, equal keys go to the lower expert id), the
// winning lane pops its head.  Gate = softmax over the K selected logits (fp64
// internally, stored fp32); lane l keeps the selected logits of ranks
// l, l + LP, ... (KS of them, K <= KS*LP).  `active` is false for a group
// without a token.  ids8 (may be NULL) receives the ids as bytes for the
// workgroup's own use.
// ---------------------------------------------------------------------------
template <int STEP>
__device__ __forceinline__ uint64_t max_step(uint64_t key) {
  const uint64_t other = (static_cast<uint64_t>(row_xchg<STEP>(static_cast<uint32_t>(key >> 32))) << 32) | row_xchg<STEP>(static_cast<uint32_t>(key));
  return other > key ? other : key;
}

template <int LP>
__device__ __forceinline__ double group_sum(double v) {
  v += row_xchg<0>(v);
  v += row_xchg<1>(v);
  if constexpr (LP >= 8) v += row_xchg<2>(v);
  if constexpr (LP >= 16) v += row_xchg<3>(v);
  return v;
}

// KEEP (8 or 16, >= min(K, 16)): list entries held per lane; a sorted list cannot
// contribute more than K entries to the top K, so for K <= 8 half a list is enough.
template <int KEEP>
struct ListHead {
  uint64_t key[KEEP];
  uint32_t idw[4];  // expert ids, one byte each (the upper two words stay 0 for KEEP == 8)
};
// lane l's list of a token's (without a condition: a lane without a list reads the first one and drops it in topk_merge)
template <int LP, int KEEP>
__device__ __forceinline__ void load_lists(const uint64_t* __restrict__ list_key, const uint8_t* __restrict__ list_id,
                                           int nlists, ListHead<KEEP>& h) {
  static_assert(KEEP == 8 || KEEP == 16, "half a list or a whole one");
  const int l = threadIdx.x & (LP - 1), at = l < nlists ? l : 0;
  const ulonglong2* kp = reinterpret_cast<const ulonglong2*>(list_key + static_cast<size_t>(at) * 16);
#pragma unroll
  for (int j = 0; j < KEEP / 2; ++j) {
    const ulonglong2 v = kp[j];
    h.key[2 * j] = v.x;
    h.key[2 * j + 1] = v.y;
  }
  if (KEEP == 16) {
    const uint4 iv = *reinterpret_cast<const uint4*>(list_id + static_cast<size_t>(at) * 16);
    h.idw[0] = iv.x; h.idw[1] = iv.y; h.idw[2] = iv.z; h.idw[3] = iv.w;
  } else {
    const uint2 iv = *reinterpret_cast<const uint2*>(list_id + static_cast<size_t>(at) * 16);
    h.idw[0] = iv.x; h.idw[1] = iv.y; h.idw[2] = 0; h.idw[3] = 0;
  }
}

// `chosen(k, id)` is called by one lane of the group for the expert of rank k.  Only the keys go round the group: the winner is the
// first lane that holds the largest one (lists are in the order of the experts, so that is the lower expert among equals), and
// after round k no list needs more than K - 1 - k entries (us a launch,
// against keys and ids going round and whole lists moving up: 32 tokens of 128 experts, K = 8, 8.5 -> 7.7, 128 10.6 -> 9.8, 64 of 64
// experts, K = 6, 6.6 -> 6.3).
template <int LP, int KS, int KEEP, typename Chosen>
__device__ __forceinline__ void topk_merge(ListHead<KEEP>& h, bool active, int nlists, float* __restrict__ w, int K, Chosen&& chosen) {
  const int lane = threadIdx.x & 63, l = lane & (LP - 1);
  uint64_t (&key)[KEEP] = h.key;
  uint32_t (&idw)[4] = h.idw;
  if (!active || l >= nlists) {
#pragma unroll
    for (int j = 0; j < KEEP; ++j) key[j] = 0;
  }
  const uint64_t before = (1ull << lane) - (1ull << (lane - l));   // lanes of the group before this one
  uint64_t mysel[KS];
#pragma unroll
  for (int c = 0; c < KS; ++c) mysel[c] = 0;
  uint64_t top = 0;
  auto round = [&](int k, auto needed) __attribute__((always_inline)) {   // needed: entries of a list that may still be wanted, this round's too
    uint64_t most = key[0];
    most = max_step<0>(most);
    most = max_step<1>(most);
    if constexpr (LP >= 8) most = max_step<2>(most);
    if constexpr (LP >= 16) most = max_step<3>(most);
    const bool equal = key[0] == most;
    const bool mine = equal && (__ballot(equal) & before) == 0 && most != 0;
    const int id = static_cast<int>(idw[0] & 0xffu);
    if (mine) {
      chosen(k, id);
#pragma unroll
      for (int j = 0; j + 1 < decltype(needed)::value; ++j) key[j] = key[j + 1];
      if (KEEP == 16) key[KEEP - 1] = 0;   // a list may be used up
      idw[0] = (idw[0] >> 8) | (idw[1] << 24);
      idw[1] = (idw[1] >> 8) | (idw[2] << 24);
      if (KEEP == 16) {
        idw[2] = (idw[2] >> 8) | (idw[3] << 24);
        idw[3] >>= 8;
      }
    }
    if (k == 0) top = most;
#pragma unroll
    for (int c = 0; c < KS; ++c)
      if (k == l + LP * c) mysel[c] = most;
  };
  if constexpr (KEEP == 8) {   // K <= 8
    static_for<8>([&](auto k) __attribute__((always_inline)) {
      if (decltype(k)::value < K) round(decltype(k)::value, std::integral_constant<int, 8 - decltype(k)::value>{});
    });
  } else {
    for (int k = 0; k < K; ++k) {
      round(k, std::integral_constant<int, KEEP>{});
    }
  }
  double ex[KS];
  double part = 0.0;
#pragma unroll
  for (int c = 0; c < KS; ++c) {
    ex[c] = 0.0;
    if (LP * c < K) {  // uniform
      ex[c] = (l + LP * c < K) ? exp(key_to_double(mysel[c]) - key_to_double(top)) : 0.0;
      part += ex[c];
    }
  }
  const double denom = group_sum<LP>(part);
#pragma unroll
  for (int c = 0; c < KS; ++c)
    if (l + LP * c < K && active) w[l + LP * c] = static_cast<float>(ex[c] / denom);
}

// ---------------------------------------------------------------------------
// Batch-wide re-routing and compaction by ONE workgroup of 1024 threads (smaller batches), and the
// parts of it that the shared form uses too.  A chain of short steps between barriers: counting by expert instead of
// by slot, sums over lanes by DPP and clearing LDS before the top-K took the launch from 9.0 to 8.5 us at 32 tokens, 11.1 to
// 10.6 at 128 (128 experts), 7.2 to 6.6 at 64 tokens of 64 experts.
// ---------------------------------------------------------------------------
struct RouteArgs {
  const int32_t* topk_ids;  // [A]  I
  const float* sim;         // [M,M] (unused when reroute == 0)
  int T, K, M, S, n_sh;
  float rho;
  int reroute;              // 0: identity map (standard top-K MoE)
  int32_t* rerouted_ids;    // [A]  I'
  int32_t* count_before;    // [M]
  int32_t* count_after;     // [M]
  int32_t* primary_mask;    // [M]
  int32_t* num_active;      // [2]
  int32_t* expert_offsets;  // [M+1]
  int32_t* sorted_token;    // [A + n_sh*T]
  int32_t* sorted_slot;     // [A]
  int32_t* sorted_token_out; // [A]  the caller's copy of the routed part of sorted_token, or NULL
  int32_t* slot_pos;        // [A]  position of slot a = t*K+k in the sorted list
  int32_t* work_expert;     // [max items] expert of each work item (M+s for shared expert s); experts
                            //             ascending, an expert's rows cut into items of <= item_rows; the ones of
                            //             more than long_rows before the others
  int32_t* work_off;        // [max items] first row of the item in the sorted list
  int32_t* work_cnt;        // [max items] rows of the item (1 .. item_rows)
  int32_t* n_work;          // [3]: number of items; 1 if the FFN kernels are to cut them fine; items that come first
  int fine_items;           // ... which they do while there are at most this many items
  int topk_threads;         // threads of a workgroup that take part in the top-K merge (256 or 1024)
  int32_t* chunk_hist;      // [chunks][2][M] slots per expert of every chunk of tokens, primary / secondary slots
                            //             (NULL: the batch-wide step runs in the last workgroup of the top-K)
  int chunk_tokens;         // tokens of a chunk
  int item_rows;            // rows per work item, at most: kItemRows and more, the host's choice
  int long_rows;            // items of more rows than this come first in the work list (0: all in order)
  int long_parts;           // gate/up units of an item
};

constexpr int kRouteThreads = 1024;
constexpr int kTopkThreadsMulti = 256;   // threads of a workgroup that merge lists when several workgroups share the batch
constexpr int kTopkLoneThreads = 512;    // one workgroup serves the whole batch up to this many merging threads
                                         // (measured: 1024 threads on one compute unit take 14.5 us, four
                                         // workgroups of 256 take 11.6 us)
constexpr int kTopkMaxSmallGroups = 64;  // groups of 256 threads up to this many workgroups, of 1024 beyond
constexpr int kSimPrefetchMaxGroups = 8;  // workgroups of a top-K launch that all prefetch their similarity rows
constexpr int kRouteWaves = kRouteThreads / kWave;
constexpr int kIdsInLds = 4096;                   // slots whose ids a workgroup keeps in LDS
// Batches from this many slots on: the batch-wide step as a launch of many workgroups.  sere_route / sere_reroute,
// us per call with one workgroup against many: 128 experts, K = 8: 1024 slots 19.0 / 8.0 against 19.5 / 8.2, 1536
// slots 22.4 / 9.1 against 21.2 / 8.9, 4096 slots 35.7 / 14.3 against 25.5 / 8.7, 8000 slots 50.5 / 24.5 against
// 31.1 / 9.3; 64 experts, K = 6: 1536 slots 20.8 / 7.5 against 19.8 / 7.5.
constexpr int kChunkedSlots = 1536;

struct RouteShared {
  int cnt_b[SERE_MAX_EXPERTS];
  int cnt_a[SERE_MAX_EXPERTS];
  int prim[SERE_MAX_EXPERTS];
  int remap[SERE_MAX_EXPERTS];
  int scan_cnt[SERE_MAX_EXPERTS / kWave];
  int scan_act[SERE_MAX_EXPERTS / kWave];
  int scan_before[SERE_MAX_EXPERTS / kWave];
  int scan_items[SERE_MAX_EXPERTS / kWave];
  int scan_long[SERE_MAX_EXPERTS / kWave];
  int cursor[SERE_MAX_EXPERTS];
  __attribute__((aligned(16))) int round_cnt[kRouteWaves][SERE_MAX_EXPERTS];
  uint8_t ids8[kIdsInLds];
  int flag;
};

// Rows of sim are scanned by 16-lane rows of a wavefront: row group q = lane/16
// of wavefront w owns experts u = 4*w + q + 64*r (r = 0, 1, ...); lane i of the
// group reads sim[u][i], sim[u][i + 16], ...: a load instruction touches four
// 64-byte segments, and the arg-max of a row needs only the four in-row DPP
// exchanges.  NC (4, 8 or 16) bounds M <= 16*NC.  The first values of a lane
// are loaded up front, before it is known which experts are secondary at all,
// so that their latency hides behind the top-K.
template <int NC>
struct SimPrefetch {
  static constexpr int NR = NC / 4;              // rounds of 64 experts
  static constexpr int PR = NC == 16 ? 1 : NR;   // rounds fetched ahead (at most 16 values per lane)
  float v[PR * NC];
};
// No load under a condition, or its wait would cover every load before it: values that remap_secondary does not ask for are
// another place of the matrix, or of `any` (readable) where there is nothing to prefetch.
template <int NC>
__device__ __forceinline__ void prefetch_sim(const RouteArgs& p, SimPrefetch<NC>& pf, const void* any, bool enabled = true) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int q = lane >> 4, i = lane & 15;
  const bool on = enabled && p.reroute;
  const float* base = on ? p.sim : static_cast<const float*>(any);
#pragma unroll
  for (int r = 0; r < SimPrefetch<NC>::PR; ++r) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int u = min(4 * wave + q + 64 * r, p.M - 1), v = min(i + 16 * c, p.M - 1);
      pf.v[r * NC + c] = base[on ? u * p.M + v : 0];
    }
  }
}

// arg-max step over (similarity, index): larger similarity wins, equal goes to the lower index
template <int STEP>
__device__ __forceinline__ void simmax_step(float& sv, int& iv) {
  const float os = __uint_as_float(row_xchg<STEP>(__float_as_uint(sv)));
  const int oi = static_cast<int>(row_xchg<STEP>(static_cast<uint32_t>(iv)));
  if (os > sv || (os == sv && oi < iv)) {
    sv = os;
    iv = oi;
  }
}

// Step 2: per secondary expert u (activated, not primary): most similar
// primary v*.  Each lane keeps the first maximum of its own columns in
// ascending order with strict '>' (start value (-inf, expert 0)); lanes are
// merged preferring the larger similarity, then the lower index: together
// the first maximum of an ascending scan, as the paper's algorithm finds it.
// The expert is kept as critical iff rho > 0 and sim* < rho.
// target(u, v) is called by one thread for every expert u < M, v being where its secondary slots go.
template <int NC, typename Target>
__device__ __forceinline__ void remap_secondary(const RouteArgs& p, RouteShared& s, const SimPrefetch<NC>& pf, bool prefetched,
                                                Target&& target) {
  if (!p.reroute) {
    if (static_cast<int>(threadIdx.x) < p.M) target(static_cast<int>(threadIdx.x), static_cast<int>(threadIdx.x));
    return;
  }
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, M = p.M;
  const int q = lane >> 4, i = lane & 15;
#pragma unroll
  for (int r = 0; r < SimPrefetch<NC>::NR; ++r) {
    const int u = 4 * wave + q + 64 * r;
    const bool sec = u < M && s.cnt_b[u] > 0 && !s.prim[u];
    int to = u;
    if (__ballot(sec) != 0) {  // wave-uniform
      float bs = -INFINITY;
      int bv = 0;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int v = i + 16 * c;
        if (v < M) {
          float sv;
          if (r < SimPrefetch<NC>::PR && prefetched)   // prefetched: uniform over the workgroup
            sv = pf.v[(r < SimPrefetch<NC>::PR ? r : 0) * NC + c];
          else
            sv = sec ? p.sim[static_cast<size_t>(u) * M + v] : 0.0f;
          if (s.prim[v] && sv > bs) {
            bs = sv;
            bv = v;
          }
        }
      }
      simmax_step<0>(bs, bv);
      simmax_step<1>(bs, bv);
      simmax_step<2>(bs, bv);
      simmax_step<3>(bs, bv);
      if (sec) {
        to = (p.rho > 0.0f && bs < p.rho) ? u : bv;
        if (i == 0) s.remap[u] = to;
      }
    }
    if (i == 0 && u < M) target(u, to);
  }
}

// inclusive sum over the wavefront's lanes (DPP row shifts, then the row totals into the rows behind)
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111 /*row_shr:1*/, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142 /*row_bcast:15*/, 0xA, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x143 /*row_bcast:31*/, 0xC, 0xF, false);
  return v;
}

// Per-expert results from the counts in s.cnt_b, s.cnt_a and the mask in s.prim: s.cursor[e] = offset of expert e
// in the sorted list and, if `write`, the output arrays and the FFN work list.
// inclusive scans over experts: slots (-> offsets), activity (-> active
// count) and work items (an expert's rows are cut into items of at most
// item_rows rows, so that one long expert cannot hold up the FFN kernels);
// inside each of the first four wavefronts by DPP, across them through
// four totals in LDS
__device__ __forceinline__ void scan_experts(const RouteArgs& p, RouteShared& s, bool write) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int M = p.M, A = p.T * p.K;
  const bool is_e = tid < SERE_MAX_EXPERTS;
  const int my_cnt = (is_e && tid < M) ? s.cnt_a[tid] : 0;
  const int my_act = my_cnt > 0 ? 1 : 0;
  const int item_rows = p.item_rows;
  const int my_items = (my_cnt + item_rows - 1) / item_rows;
  // all items but the last one have item_rows rows
  int my_long = p.long_rows > 0 && my_items > 0 ? my_items - (my_cnt - (my_items - 1) * item_rows <= p.long_rows ? 1 : 0) : 0;
  int inc_cnt = my_cnt, inc_act = my_act, inc_items = my_items, inc_long = 0;
  if (is_e) {  // wave-uniform (waves 0-3)
    inc_cnt = wave_scan(inc_cnt);
    inc_act = wave_scan(inc_act);
    inc_items = wave_scan(inc_items);
    if (p.long_rows > 0) inc_long = wave_scan(my_long);
    if (lane == kWave - 1) {
      s.scan_long[wave] = inc_long;
      s.scan_cnt[wave] = inc_cnt;
      s.scan_act[wave] = inc_act;
      s.scan_items[wave] = inc_items;
    }
    const int nb = __popcll(__ballot(tid < M && s.cnt_b[tid] > 0));
    if (lane == 0) s.scan_before[wave] = nb;
  }
  lds_barrier();
  int n_after = 0, n_before = 0, n_items = 0, n_long = 0;
#pragma unroll
  for (int w = 0; w < SERE_MAX_EXPERTS / kWave; ++w) {
    if (is_e && w < wave) {
      inc_cnt += s.scan_cnt[w];
      inc_items += s.scan_items[w];
      inc_long += s.scan_long[w];
    }
    n_after += s.scan_act[w];
    n_before += s.scan_before[w];
    n_items += s.scan_items[w];
    n_long += s.scan_long[w];
  }
  const int sh_items = (p.T + item_rows - 1) / item_rows;  // per shared expert
  // long items first where there is more than one round of units; in one round all start together, and an expert's
  // items next to each other share its weights in one L2
  const bool long_first = p.long_rows > 0 && (n_items + p.n_sh * sh_items) * p.long_parts > kTileGroups;
  const int sh_long = long_first ? sh_items - (p.T - (sh_items - 1) * item_rows <= p.long_rows ? 1 : 0) : 0;
  if (!long_first) my_long = inc_long = n_long = 0;
  const int routed_long = n_long;
  n_long += p.n_sh * sh_long;
  if (is_e && tid < M) {
    const int off = inc_cnt - my_cnt;
    s.cursor[tid] = off;
    if (write) {
      p.expert_offsets[tid] = off;
      p.count_before[tid] = s.cnt_b[tid];
      p.count_after[tid] = my_cnt;
      p.primary_mask[tid] = s.prim[tid];
      const int first = inc_long - my_long, then = n_long + (inc_items - inc_long) - my_items;   // of the long ones, of the others (from my_long on)
      // Items of 128 rows and more (prefill-sized batches): an expert with a few rows more than one item
      // holds is cut into items of about equal size (multiples of a 16-row tile) instead of a full
      // one and a remnant: its items then take about equally long, and as they are numbered next
      // to each other they stream the expert's weights side by side, the later one from cache.
      int per = item_rows;
      if (item_rows >= 4 * kItemRows && my_items >= 2 && my_items <= 4)
        per = ((my_cnt + my_items - 1) / my_items + 15) & ~15;
      for (int j = 0; j < my_items; ++j) {
        const int at = (j < my_long ? first : then) + j;
        p.work_expert[at] = tid;
        p.work_off[at] = off + j * per;
        p.work_cnt[at] = min(per, my_cnt - j * per);
      }
    }
  }
  if (!write) return;
  if (tid == 0) {
    p.expert_offsets[M] = A;
    p.num_active[0] = n_before;
    p.num_active[1] = n_after;
    p.n_work[0] = n_items + p.n_sh * sh_items;
    p.n_work[1] = (item_rows == kItemRows && n_items + p.n_sh * sh_items <= p.fine_items) ? 1 : 0;
    p.n_work[2] = n_long;
  }
  for (int i = tid; i < p.n_sh * sh_items; i += kRouteThreads) {
    const int sh = i / sh_items, j = i % sh_items;
    const int at = j < sh_long ? routed_long + sh * sh_long + j : n_items + p.n_sh * sh_long + sh * (sh_items - sh_long) + j - sh_long;
    p.work_expert[at] = M + sh;
    p.work_off[at] = A + sh * p.T + j * item_rows;
    p.work_cnt[at] = min(item_rows, p.T - j * item_rows);
  }
}

// Stable regrouping by expert of slots [begin, end): slots keep ascending (token, slot) order
// inside each expert, from position s.cursor[e] on.  A round covers 1024 consecutive slots, one wavefront
// per 64; rank inside the wavefront from ballots, rank across wavefronts
// through the per-round table.  s.round_cnt must be zero at the start.
template <typename IdAt>
__device__ __forceinline__ void regroup_slots(const RouteArgs& p, RouteShared& s, int begin, int end, IdAt&& id_at, bool write_ids) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int M = p.M, K = p.K, S = p.S;
  const bool is_e = tid < SERE_MAX_EXPERTS;
  for (int base = begin; base < end; base += kRouteThreads) {
    const int a = base + tid;
    const bool valid = a < end;
    int e = 0;
    if (valid) {
      const int e0 = id_at(a);
      e = (a % K >= S) ? s.remap[e0] : e0;
      if (write_ids) p.rerouted_ids[a] = e;
    }
    // lanes of this wavefront holding the same expert: intersect, over the 8
    // bits of e, the ballot of lanes that agree with this lane on that bit
    int rank = 0, same = 0;
    if (base + wave * kWave < end) {  // wave-uniform: this wavefront has slots
      uint64_t peers = __ballot(valid);
#pragma unroll
      for (int bit = 0; bit < 8; ++bit) {
        const bool set = (e >> bit) & 1;
        const uint64_t with = __ballot(set);
        peers &= set ? with : ~with;
      }
      same = __popcll(peers);
      rank = __popcll(peers & ((1ull << lane) - 1ull));
    }
    if (valid && rank == 0) s.round_cnt[wave][e] = same;
    lds_barrier();
    if (valid) {
      int pos = s.cursor[e] + rank;
      for (int w = 0; w < wave; ++w) pos += s.round_cnt[w][e];
      p.sorted_token[pos] = a / K;
      p.sorted_slot[pos] = a % K;
      p.slot_pos[a] = pos;
      if (p.sorted_token_out != nullptr) p.sorted_token_out[pos] = a / K;
    }
    if (base + kRouteThreads < end) {  // another round follows: advance the cursors
      lds_barrier();
      if (is_e && tid < M) {
        int add = 0;
        for (int w = 0; w < kRouteWaves; ++w) {
          add += s.round_cnt[w][tid];
          s.round_cnt[w][tid] = 0;
        }
        s.cursor[tid] += add;
      }
      lds_barrier();
    }
  }
}

// what route_phase finds cleared: all threads, before a barrier
__device__ __forceinline__ void clear_counts(RouteShared& s) {
  const int tid = threadIdx.x;
  if (tid < SERE_MAX_EXPERTS) {
    s.cnt_b[tid] = 0;
    s.cnt_a[tid] = 0;
    s.cursor[tid] = 0;
    s.prim[tid] = 0;
    s.remap[tid] = tid;
  }
  static_assert(kRouteWaves * SERE_MAX_EXPERTS == 4 * kRouteThreads, "four counters a thread");
  *reinterpret_cast<int4*>(&s.round_cnt[0][0] + 4 * tid) = int4{0, 0, 0, 0};
}
// (s.cursor: secondary slots of an expert, until scan_experts puts the offsets there; counting them while the lists are
// merged was slower, 8.7 -> 10.5 us at 32 tokens: the atomics lengthen the one chain that everything waits for)
template <bool IDS_IN_LDS, int NC>
__device__ __forceinline__ void route_phase(const RouteArgs& p, RouteShared& s, const SimPrefetch<NC>& pf,
                                            bool prefetched = true) {
  const int tid = threadIdx.x;
  const int M = p.M, K = p.K, S = p.S;
  const int A = p.T * K;
  // ids read from memory may be a caller's (sere_reroute): clamped into [0, M) so that an id outside
  // that range, a broken precondition, cannot send any access out of bounds
  // (device-scope loads: the ids may have been written by other workgroups of this launch)
  auto id_at = [&](int a) -> int {
    return IDS_IN_LDS ? static_cast<int>(s.ids8[a])
                      : min(max(__hip_atomic_load(p.topk_ids + a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), 0), M - 1);
  };

  // Step 1: activation histogram and primary mask (union of every token's top-S)
  for (int a = tid; a < A; a += kRouteThreads) {
    const int e = id_at(a);
    atomicAdd(&s.cnt_b[e], 1);
    if (a % K < S)
      s.prim[e] = 1;
    else
      atomicAdd(&s.cursor[e], 1);
  }
  lds_barrier();
  // Step 2, and the new map's counts: an expert's primary slots stay, its secondary ones all go to one expert
  remap_secondary(p, s, pf, prefetched, [&](int u, int v) {
    const int secondary = s.cursor[u], primary = s.cnt_b[u] - secondary;
    if (primary > 0) atomicAdd(&s.cnt_a[u], primary);
    if (secondary > 0) atomicAdd(&s.cnt_a[v], secondary);
  });
  lds_barrier();

  // Step 3: offsets, then the slots regrouped and rewritten
  scan_experts(p, s, true);
  for (int i = tid; i < p.n_sh * p.T; i += kRouteThreads) p.sorted_token[A + i] = i % p.T;
  lds_barrier();
  regroup_slots(p, s, 0, A, id_at, true);
}

// ---------------------------------------------------------------------------
// The batch-wide step shared by many workgroups (batches of thousands of slots; top-K and re-routing of the
// Qwen3 shape, us a step: 1024 tokens 27 -> 11, 2048 47 -> 11, 4096 89 -> 18).  Where a slot goes depends on its
// expert and on whether it is a primary slot (k < S) only, so two counts per expert and chunk of tokens are
// all that workgroups have to tell each other: the launch before this one writes them (chunk_hist), and every
// workgroup here derives the mask, the map, the new counts, the offsets and its own chunk's starting positions
// from them, then regroups its own slots.
// ---------------------------------------------------------------------------

// counts of the slots whose ids are in s.ids8: hist[0][e] primary slots, hist[1][e] secondary ones; all threads of the workgroup,
// after clear_chunk_counts and a barrier.  (Barriers that order LDS only: the ids and gate weights are still on their way to
// memory.)
__device__ __forceinline__ void clear_chunk_counts(RouteShared& s) {
  for (int i = threadIdx.x; i < SERE_MAX_EXPERTS; i += blockDim.x) s.cnt_a[i] = s.cnt_b[i] = 0;
}
__device__ __forceinline__ void write_chunk_hist(const RouteArgs& p, RouteShared& s, int slots, int32_t* hist) {
  for (int a = threadIdx.x; a < slots; a += blockDim.x) atomicAdd((a % p.K < p.S) ? &s.cnt_a[s.ids8[a]] : &s.cnt_b[s.ids8[a]], 1);
  lds_barrier();
  for (int i = threadIdx.x; i < p.M; i += blockDim.x) {
    hist[i] = s.cnt_a[i];
    hist[p.M + i] = s.cnt_b[i];
  }
}

// chunk counts of given ids (sere_reroute); grid chunks, 1024 threads
__global__ __launch_bounds__(kRouteThreads) void route_hist_kernel(RouteArgs p) {
  __shared__ RouteShared s;
  const int begin = blockIdx.x * p.chunk_tokens * p.K, slots = min(p.chunk_tokens * p.K, p.T * p.K - begin);
  for (int a = threadIdx.x; a < slots; a += kRouteThreads)
    s.ids8[a] = static_cast<uint8_t>(min(max(p.topk_ids[begin + a], 0), p.M - 1));
  clear_chunk_counts(s);
  lds_barrier();
  write_chunk_hist(p, s, slots, p.chunk_hist + static_cast<size_t>(blockIdx.x) * 2 * p.M);
}

// grid chunks (ceil(T / chunk_tokens)), 1024 threads
template <int NC>
__global__ __launch_bounds__(kRouteThreads) void route_chunks_kernel(RouteArgs p) {
  __shared__ RouteShared s;
  __shared__ int s_total[2 * SERE_MAX_EXPERTS], s_before[2 * SERE_MAX_EXPERTS];  // of all chunks / of the chunks before this one
  const int tid = threadIdx.x, M = p.M, chunks = gridDim.x, chunk = blockIdx.x;
  const int A = p.T * p.K, begin = chunk * p.chunk_tokens * p.K, end = min(begin + p.chunk_tokens * p.K, A);
  // The 2 M counts of the chunks, kRouteThreads / (2 M) chunks at a time: kAhead passes are requested together, before the
  // similarity rows, and so are the ids of the chunk's first slots (one pass after the other: both launches 13.4 us instead of 11.7 at
  // 1000 tokens, 13.8 instead of 10.7 at 2048).
  constexpr int kAhead = 8;
  const int per_pass = kRouteThreads / (2 * M);  // >= 2
  const int c = tid % (2 * M), first = tid / (2 * M);
  int n[kAhead];
  auto fetch = [&](int g) __attribute__((always_inline)) {   // a chunk beyond the last: that one again, not used
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      if (u * per_pass < chunks) n[u] = p.chunk_hist[static_cast<size_t>(min(g + u * per_pass, chunks - 1)) * 2 * M + c];   // uniform
  };
  fetch(first);
  const int first_id = p.topk_ids[min(begin + tid, end - 1)];
  SimPrefetch<NC> pf;
  prefetch_sim(p, pf, p.topk_ids);
  for (int i = tid; i < 2 * SERE_MAX_EXPERTS; i += kRouteThreads) s_total[i] = s_before[i] = 0;
  *reinterpret_cast<int4*>(&s.round_cnt[0][0] + 4 * tid) = int4{0, 0, 0, 0};
  lds_barrier();
  if (tid < per_pass * 2 * M) {
    int total = 0, before = 0;
    for (int g = first; g < chunks; g += kAhead * per_pass) {
      if (g != first) fetch(g);
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int at = g + u * per_pass, add = at < chunks ? n[u] : 0;
        total += add;
        before += at < chunk ? add : 0;
      }
    }
    atomicAdd(&s_total[c], total);
    atomicAdd(&s_before[c], before);
  }
  lds_barrier();
  if (tid < SERE_MAX_EXPERTS) {
    const bool is_e = tid < M;
    s.cnt_b[tid] = is_e ? s_total[tid] + s_total[M + tid] : 0;
    s.prim[tid] = is_e && s_total[tid] > 0 ? 1 : 0;
    s.remap[tid] = tid;
    s.cnt_a[tid] = is_e ? s_total[tid] : 0;   // primary slots stay; the secondary ones are added below
  }
  lds_barrier();
  remap_secondary(p, s, pf, true, [&](int u, int v) {  // an expert's secondary slots all go to v
    const int n = s_total[M + u], b = s_before[M + u];
    if (n > 0) atomicAdd(&s.cnt_a[v], n);
    if (b > 0) atomicAdd(&s_before[v], b);
  });
  lds_barrier();
  scan_experts(p, s, chunk == 0);
  lds_barrier();
  if (tid < M) s.cursor[tid] += s_before[tid];
  lds_barrier();
  regroup_slots(p, s, begin, end, [&](int a) { return min(max(a == begin + tid ? first_id : p.topk_ids[a], 0), M - 1); }, true);
  for (int i = chunk * kRouteThreads + tid; i < p.n_sh * p.T; i += chunks * kRouteThreads) p.sorted_token[A + i] = i % p.T;
}

// Re-routing alone (indices in, indices out): grid 1, 1024 threads.
__global__ __launch_bounds__(kRouteThreads) void route_kernel(RouteArgs p) {
  __shared__ RouteShared s;
  SimPrefetch<16> pf;  // any M up to 256
  prefetch_sim(p, pf, p.topk_ids);
  clear_counts(s);
  lds_barrier();
  route_phase<false>(p, s, pf);
}

// Top-K + gate (1024 / LP tokens per workgroup), then the batch-wide step by
// the workgroup that takes the last ticket.  With a single workgroup there is
// no ticket and the ids go from the top-K to the batch-wide step through LDS.
// grid ceil(T*LP/1024), 1024 threads; *ticket must be 0 at launch.
// LP = lanes per token >= number of lists (4, 8, 16); K <= KS*LP; KEEP >= min(K, 16).
template <int LP, int KS, int KEEP>
__global__ __launch_bounds__(kRouteThreads) void topk_route_kernel(const uint64_t* __restrict__ list_key,
                                                                   const uint8_t* __restrict__ list_id,
                                                                   int32_t* __restrict__ topk_ids,
                                                                   float* __restrict__ topk_w, int32_t* ticket,
                                                                   RouteArgs p) {
  __shared__ RouteShared s;
  constexpr int NC = LP;  // the similarity scan uses the same bound M <= 16*LP
  // tokens per workgroup: the first p.topk_threads threads merge lists (the host's choice: all 1024,
  // or 256 -- one wavefront per SIMD, the merge being bound by the vector ALU -- so that a batch
  // shared by several workgroups spreads over more compute units)
  const int group_tokens = p.topk_threads / LP;
  const int nlists = (p.M + 15) >> 4;
  const int t = blockIdx.x * group_tokens + threadIdx.x / LP;
  const bool lone = gridDim.x == 1 && p.T * p.K <= kIdsInLds;
  const bool in_group = static_cast<int>(threadIdx.x) < group_tokens * LP;
  const bool has = in_group && t < p.T;
  const int first_of_wave = blockIdx.x * group_tokens + (threadIdx.x >> 6) * (kWave / LP);
  const bool merges = static_cast<int>(threadIdx.x & ~63u) < group_tokens * LP && first_of_wave < p.T;  // wave-uniform: the wavefront has a token
  const size_t tt = has ? t : 0;
  ListHead<KEEP> head;
  load_lists<LP, KEEP>(list_key + tt * nlists * 16, list_id + tt * nlists * 16, nlists, head);
  // The similarity rows are requested before the top-K so that their latency hides behind it, and after its lists, which the
  // merge waits for (the other way round the launch takes 9.5 us instead of 9.0 at 32 tokens, 128 experts).  Only the workgroup that runs the batch-wide step uses
  // them, and which one that is is not known yet: with a handful of workgroups every one of them asks (the lines come
  // from L2), with many the step is long anyway and the rows are loaded where they are needed instead.
  SimPrefetch<NC> pf;
  prefetch_sim(p, pf, list_key, gridDim.x <= kSimPrefetchMaxGroups && p.chunk_hist == nullptr);
  if (p.chunk_hist == nullptr) clear_counts(s); else clear_chunk_counts(s);   // while the loads are on their way
  if (merges) {
    uint8_t* ids8 = lone ? s.ids8 + tt * p.K : (p.chunk_hist != nullptr ? s.ids8 + (threadIdx.x / LP) * p.K : nullptr);
    topk_merge<LP, KS, KEEP>(head, has, nlists, topk_w + tt * p.K, p.K, [&](int k, int id) {
      // a device-scope store: with several workgroups the ids are read by another one of this launch
      __hip_atomic_store(topk_ids + tt * p.K + k, id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (ids8 != nullptr) ids8[k] = static_cast<uint8_t>(id);
    });
  }
  if (p.chunk_hist != nullptr) {  // the batch-wide step is a launch of its own: leave this chunk's counts
    lds_barrier();
    const int tokens = min(group_tokens, p.T - static_cast<int>(blockIdx.x) * group_tokens);
    write_chunk_hist(p, s, tokens * p.K, p.chunk_hist + static_cast<size_t>(blockIdx.x) * 2 * p.M);
    return;
  }
  if (lone) {
    lds_barrier();   // the ids go on through LDS; what was stored and requested need not have arrived
    route_phase<true>(p, s, pf);
    return;
  }
  if (gridDim.x > 1) {
#if SERE_FORMAL_HANDOFF
    // Ordered by the memory model: the barrier orders every thread's id stores before thread 0's
    // ticket, the ticket is a device-scope release (this workgroup's stores become visible) and
    // acquire (the last taker sees every earlier taker's), the second barrier hands that on to
    // the other threads.  On this multi-die part the release writes the L2 back and the acquire
    // invalidates it, which is what the default path avoids.
    __syncthreads();
    if (threadIdx.x == 0)
      s.flag = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == static_cast<int>(gridDim.x) - 1;
    __syncthreads();
    if (!s.flag) return;
#else
    // Fence-free hand-off.  What it rests on (gfx950, not the HIP memory model):
    //  - the ids were written with device-scope atomic stores, which the compiler emits as
    //    global stores with the sc1 bit: they write through this die's L2 to memory instead of
    //    staying dirty in it, and no compiler transformation may drop or merge them;
    //  - s_waitcnt vmcnt(0) (s_waitcnt(0) below waits on every counter) returns only after those
    //    stores have been acknowledged, i.e. have reached the point of coherence; gfx950 counts
    //    stores in vmcnt like loads (there is no separate store counter), and the builtin is a
    //    scheduling barrier for memory operations;
    //  - the ticket is a device-scope atomic add, performed at the point of coherence, so the
    //    workgroup that reads gridDim.x - 1 runs after every other workgroup's acknowledgement;
    //  - that workgroup reads the ids with device-scope atomic loads (sc1: they bypass its own
    //    die's L2, which may hold stale lines), and ONLY the ids: route_phase<false> must not
    //    read any other data written by this launch's other workgroups (it does not: the gate
    //    weights, for one, are never read back).
    // Two device-scope fences here cost this kernel several microseconds (an L2 write-back and
    // an invalidate on a part with one L2 per die).
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0)
      s.flag = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == static_cast<int>(gridDim.x) - 1;
    __syncthreads();
    if (!s.flag) return;
#endif
  } else {
    __syncthreads();
  }
  route_phase<false>(p, s, pf, gridDim.x <= kSimPrefetchMaxGroups);
}

}  // namespace sere
