// The whole layer behind the router logits in two launches, for calls of at most 64 slots (T * K) where that is faster
// (small_call_pays in ffn_plan.hpp): a decode step of one or a few sequences.
//
// Such a call is bound by its launches and by dependent memory round trips, not by bytes: a launch that depends on the one
// before it takes some 4 us whatever it does, and top-K + re-routing, gate/up, down and combine were four of them.  Here
//  - every workgroup of the gate/up launch works out the routing for itself: 64 slots are one to a lane, so that ranking,
//    re-mapping and regrouping are 3 to 5 us of short steps in registers, of which the weights' way from memory hides
//    nothing, but a launch of its own took 7; one more workgroup writes it down for the next launch and the caller;
//  - a workgroup of the down launch takes eight columns of the output for every expert, keeps the rows of y that the combine
//    step adds up in LDS, and adds them in the same order.
// A wavefront issues the loads of four blocks of 128 bytes of its rows together, and a gate/up contraction is split so that it
// has four blocks or fewer where that still leaves one round of units: a unit is then one memory round trip.
//
// us a call, against four launches behind the router logits (one card, in turn): one token of the Qwen3 shape 28.4 -> 20.2 (kernels: router
// 4.7, gate/up 9.2, of that 3.8 the routing, down 6.8), two tokens 29.3 -> 24.1, one without re-routing 32.7 -> 28.2; 8 tokens of an fp32
// layer of 256 x 128 24.7 -> 16.4; one token of d_h 1024, d_m 704 in fp32 39.7 -> 24.4, four 52 -> 40; one token of d_h 2048,
// d_m 1408 with two shared experts 43 -> 34.
#pragma once

#include "common.hpp"
#include "ffn_generic.hpp"
#include "ffn_mfma.hpp"
#include "route_kernels.hpp"
#include "rules.hpp"

namespace sere {

constexpr int kSmallThreads = kSmallWaves * kWave;
static_assert(kSmallTile == kTile, "a tile of the matrix cores");
constexpr int kSmallSums = kSmallWaves * kSmallSlots;   // rows of partial sums that a down workgroup holds

__device__ __forceinline__ int read_lane(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
// this wavefront's LDS writes before its reads behind it
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// The routing of the whole batch, in every wavefront: lane a holds slot a = t * K + k.
struct SmallRoute {
  int before, after;   // expert of the slot, before and after re-routing (-1: no slot)
  int pos;             // place in the sorted list
  int rank, count;     // ... and among its expert's slots; how many these are
  int item;            // rank of its expert among the active ones
  int active;          // their number (uniform)
};

struct SmallRouteShared {
  uint64_t key[kSmallSlots];                      // of the slot's logit
  uint8_t id[kSmallSlots];
  float best[kSmallWaves][kSmallSlots];     // each wavefront's most similar primary expert
  int to[kSmallWaves][kSmallSlots];         // ... and its number, kSmallPrimary where the slot's own expert is primary
};
constexpr int kSmallPrimary = 0x100;

// Top-K: a wavefront takes a token, a lane one of the first eight entries of each of its sorted lists (16 lists: of two).  An
// entry's rank is the number of larger keys, counted by their upper halves (rules.hpp); if two of these are equal, the whole keys are
// compared, and equal ones go in the order of the experts, which is the order of (list, place).  (A merge of the list heads,
// one round after the other, takes 2.3 us for K = 8; comparing whole keys throughout 3.7; this 1.5.)
template <int N>
__device__ __forceinline__ void small_topk(const uint64_t* __restrict__ list_key, const uint8_t* __restrict__ list_id, const RouteArgs& p,
                                           SmallRouteShared& s) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, K = p.K, nlists = (p.M + 15) >> 4;
  for (int t = wave; t < p.T; t += kSmallWaves) {
    uint64_t key[N];
    uint32_t word[N], rank[N];
    int id[N];
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int list = lane / 8 + 8 * n;
      const size_t at = (static_cast<size_t>(t) * nlists + min(list, nlists - 1)) * 16 + lane % 8;
      key[n] = list_key[at];
      id[n] = list_id[at];
    }
    uint32_t sum = 0;
#pragma unroll
    for (int n = 0; n < N; ++n) {
      if (lane / 8 + 8 * n >= nlists) key[n] = 0;
      word[n] = rank_word(key[n], lane + 64 * n, 64 * N);
      rank[n] = 0;
    }
#pragma unroll
    for (int n = 0; n < N; ++n)
      for (int l = 0; l < min(8, nlists - 8 * n); ++l)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const uint32_t other = read_lane(word[n], 8 * l + j);
#pragma unroll
          for (int m = 0; m < N; ++m) rank[m] += other > word[m] ? 1u : 0u;
        }
    const int entries = 8 * nlists;
#pragma unroll
    for (int n = 0; n < N; ++n) sum += lane + 64 * n < entries ? rank[n] : 0u;
    if (read_lane(wave_scan(static_cast<int>(sum)), 63) != entries * (entries - 1) / 2) {   // two are equal (uniform)
#pragma unroll
      for (int n = 0; n < N; ++n) rank[n] = 0;
      for (int b = 0; b < entries; ++b) {
        const uint64_t mine = N == 2 && b >= 64 ? key[N - 1] : key[0];
        const uint64_t other = static_cast<uint64_t>(static_cast<uint32_t>(read_lane(static_cast<int>(mine >> 32), b & 63))) << 32 |
                               static_cast<uint32_t>(read_lane(static_cast<int>(mine), b & 63));
#pragma unroll
        for (int n = 0; n < N; ++n) rank[n] += ranks_before(other, b, key[n], lane + 64 * n) ? 1u : 0u;
      }
    }
#pragma unroll
    for (int n = 0; n < N; ++n)
      if (lane + 64 * n < entries && rank[n] < static_cast<uint32_t>(K)) {
        s.key[t * K + rank[n]] = key[n];
        s.id[t * K + rank[n]] = static_cast<uint8_t>(id[n]);
      }
  }
}

// All wavefronts of the workgroup, with barriers.
template <int N>
__device__ __forceinline__ SmallRoute small_route(const uint64_t* __restrict__ list_key, const uint8_t* __restrict__ list_id, const RouteArgs& p,
                                                  SmallRouteShared& s) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int K = p.K, M = p.M, S = p.S, A = p.T * K;
  small_topk<N>(list_key, list_id, p, s);
  if (p.reroute && S < K && wave != 0) {
    // The lines of the similarity matrix, shared out among a die's workgroups, so that the few values that are wanted come
    // from its L2.
    const int lines = (M * M + 31) / 32, share = (kSmallWaves - 1) * kWave;
    for (int i = blockIdx.x / 8 % 4 * share + (wave - 1) * kWave + lane; i < lines; i += 4 * share) {
      const float touched = p.sim[32 * i];
      asm volatile("" ::"v"(touched));
    }
  }
  __syncthreads();
  SmallRoute r;
  const bool slot = lane < A;
  r.before = slot ? s.id[lane] : -1;
  r.after = r.before;
  if (p.reroute && S < K) {
    // the most similar primary expert: larger similarity first, then the lower index, from (-inf, expert 0) on; a NaN
    // never wins (what remap_secondary finds)
    constexpr int kMost = 8;
    static_assert(kMost * kSmallWaves >= kSmallSlots, "eight primary slots a wavefront");
    float bs = -INFINITY;
    int bv = 0;
    bool primary = false;
    const bool secondary = slot && lane % K >= S;
    const int P = p.T * S, first = P <= kMost ? 0 : wave, stride = P <= kMost ? 1 : kSmallWaves;
    const float* row = p.sim + static_cast<size_t>(secondary ? r.before : 0) * M;
    int v[kMost];
    float sv[kMost];
#pragma unroll
    for (int j = 0; j < kMost; ++j) {
      const int i = first + stride * j, q = i < P ? i : 0;   // beyond the last: the first one
      v[j] = read_lane(r.before, q / S * K + q % S);
      if (i < P) {   // uniform
        primary |= v[j] == r.before;
        sv[j] = secondary ? row[v[j]] : 0.0f;
      } else {
        sv[j] = -INFINITY;
      }
    }
    auto better = [&](float s1, int v1) {
      if (s1 > bs || (s1 == bs && v1 < bv)) {
        bs = s1;
        bv = v1;
      }
    };
#pragma unroll
    for (int j = 0; j < kMost; ++j) better(sv[j], v[j]);
    if (P > kMost) {   // every wavefront has looked at an eighth of the primary slots
      s.best[wave][lane] = bs;
      s.to[wave][lane] = primary ? kSmallPrimary : bv;
      __syncthreads();
      bs = -INFINITY;
      bv = 0;
      primary = false;
#pragma unroll
      for (int w = 0; w < kSmallWaves; ++w) {
        const int vw = s.to[w][lane];
        primary |= vw == kSmallPrimary;
        better(s.best[w][lane], vw);
      }
    }
    if (secondary && !primary && !(p.rho > 0.0f && bs < p.rho)) r.after = bv;
  }
  // slots of the same expert and of lower ones, by the bits of the expert's number from the highest one on
  uint64_t same = __ballot(slot), lower = 0;
#pragma unroll
  for (int bit = 7; bit >= 0; --bit) {
    const bool set = (r.after >> bit) & 1;
    const uint64_t with = __ballot(set);
    if (set) lower |= same & ~with;
    same &= set ? with : ~with;
  }
  r.rank = __popcll(same & ((1ull << lane) - 1ull));
  r.count = __popcll(same);
  r.pos = __popcll(lower) + r.rank;
  const uint64_t leads = __ballot(slot && r.rank == 0);
  r.item = __popcll(lower & leads);
  r.active = __popcll(leads);
  return r;
}

// Everything about the routing that the down launch and the caller read; 256 threads and more, each wavefront with the same `r`.
__device__ __forceinline__ void write_small_route(const RouteArgs& p, const SmallRoute& r, const SmallRouteShared& s, int32_t* topk_ids,
                                                  float* topk_w) {
  static_assert(SERE_MAX_EXPERTS <= kSmallThreads, "a thread per expert");
  const int tid = threadIdx.x, A = p.T * p.K, M = p.M;
  int before = 0, after = 0, less = 0, primary = 0, distinct = 0;
  const int e = tid;
  for (int b = 0; b < A; ++b) {
    const int eb = read_lane(r.before, b), ea = read_lane(r.after, b);
    const bool mine = eb == e;
    before += mine ? 1 : 0;
    primary |= mine && b % p.K < p.S ? 1 : 0;
    after += ea == e ? 1 : 0;
    less += ea < e ? 1 : 0;
    distinct += !__ballot(static_cast<int>(threadIdx.x & 63) < b && r.before == eb) ? 1 : 0;
  }
  if (e < M) {
    p.count_before[e] = before;
    p.count_after[e] = after;
    p.primary_mask[e] = primary;
    p.expert_offsets[e] = less;
  }
  if (tid < A) {   // the first wavefront
    const int t = tid / p.K, k = tid % p.K;
    topk_ids[tid] = r.before;
    const double top = key_to_double(s.key[t * p.K]);
    double sum = 0.0;
    for (int j = 0; j < p.K; ++j) sum += exp(key_to_double(s.key[t * p.K + j]) - top);
    topk_w[tid] = static_cast<float>(exp(key_to_double(s.key[tid]) - top) / sum);
    p.rerouted_ids[tid] = r.after;
    p.slot_pos[tid] = r.pos;
    p.sorted_token[r.pos] = t;
    p.sorted_slot[r.pos] = k;
    if (p.sorted_token_out != nullptr) p.sorted_token_out[r.pos] = t;
    if (r.rank == 0) {
      p.work_expert[r.item] = r.after;
      p.work_off[r.item] = r.pos;
      p.work_cnt[r.item] = r.count;
    }
  }
  if (tid < p.n_sh) {
    p.work_expert[r.active + tid] = M + tid;
    p.work_off[r.active + tid] = A + tid * p.T;
    p.work_cnt[r.active + tid] = p.T;
  }
  for (int i = tid; i < p.n_sh * p.T; i += kSmallThreads) p.sorted_token[A + i] = i % p.T;
  if (tid == 0) {
    p.expert_offsets[M] = A;
    p.num_active[0] = distinct;
    p.num_active[1] = r.active;
    p.n_work[0] = r.active + p.n_sh;
    p.n_work[1] = 0;
    p.n_work[2] = 0;
  }
}

// One wavefront's sums of a tile of 16 weight rows and 16 token rows.  fp32: every 8 products are summed on their own, a
// block's four sums pairwise, and what each addition to the running sum rounds away is kept in a second one (as in
// ffn_tile.hpp).
template <int DT>
struct SmallSums {
  f32x4 acc = {0.f, 0.f, 0.f, 0.f}, low = {0.f, 0.f, 0.f, 0.f};   // low: what acc has lost (fp32)
  // the even and the odd 16-byte pieces of a block of 128 bytes
  __device__ __forceinline__ void add(u32x4 w0, u32x4 w1, u32x4 x0, u32x4 x1) {
    if constexpr (DT == SERE_BF16) {
      acc = mfma_bf16(w0, x0, acc);
      acc = mfma_bf16(w1, x1, acc);
    } else {
      f32x4 s[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        s[j / 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w0[j]), __uint_as_float(x0[j]), j % 2 == 0 ? zero : s[j / 2], 0, 0, 0);
        s[2 + j / 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w1[j]), __uint_as_float(x1[j]), j % 2 == 0 ? zero : s[2 + j / 2], 0, 0, 0);
      }
      const f32x4 add = (s[0] + s[1]) + (s[2] + s[3]), next = acc + add;
      low += add - (next - acc);
      acc = next;
    }
  }
};

// The same for one element, added up over wavefronts: each addition's rounding error goes to `low` as well.
template <int DT>
struct SmallTotal {
  float sum, low;
  __device__ __forceinline__ void add(float v, float l) {
    const float next = sum + v;
    if constexpr (DT == SERE_F32) {
      const float part = next - sum;
      low += l + ((sum - (next - part)) + (v - part));
    }
    sum = next;
  }
  __device__ __forceinline__ float value() const {
    if constexpr (DT == SERE_BF16) return sum;
    const float all = sum + low;
    return __builtin_amdgcn_fmed3f(all, all, sum);   // sum where that is a NaN
  }
};

// W[16 rows] * x over blocks [b0, b1) of 128 bytes.  `wx`, `wy`: this lane's address (row i & 7, piece 2 g + (i >> 3)) in the upper
// and the lower eight weight rows; HALF: there are no lower ones, and rows 8 to 15 of the result are not used.  `xt`:
// this lane's token row (row i) at piece 2 g.  All loads of N blocks go out together; AHEAD: and those of the next N before
// they are multiplied.
template <int DT, bool HALF, int N, bool AHEAD>
__device__ __forceinline__ SmallSums<DT> small_contract(const char* wx, const char* wy, const char* xt, int b0, int b1) {
  SmallSums<DT> sums;
  if (b0 >= b1) return sums;
  struct Set {
    u32x4 x[N], y[HALF ? 1 : N], even[N], odd[N];
  };
  auto load = [&](Set& s, int first) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const size_t at = static_cast<size_t>(min(first + u, b1 - 1)) * kSmallBlock;   // beyond the last: that one again, not used
      s.x[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wx + at));
      if (!HALF) s.y[HALF ? 0 : u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wy + at));
      s.even[u] = *reinterpret_cast<const u32x4*>(xt + at);
      s.odd[u] = *reinterpret_cast<const u32x4*>(xt + at + 16);
    }
  };
  auto multiply = [&](const Set& s, int first) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (first + u < b1) {
        if constexpr (HALF)
          sums.add(s.x[u], rotate8(s.x[u]), s.even[u], s.odd[u]);
        else
          sums.add(upper_from(s.x[u], s.y[u]), lower_from(s.y[u], s.x[u]), s.even[u], s.odd[u]);
      }
  };
  if constexpr (AHEAD) {
    Set s0, s1;
    load(s0, b0);
#pragma unroll 1
    for (int first = b0; first < b1; first += 2 * N) {
      load(s1, first + N);
      multiply(s0, first);
      if (first + 2 * N < b1) load(s0, first + 2 * N);
      multiply(s1, first + N);
    }
  } else {
#pragma unroll 1
    for (int first = b0; first < b1; first += N) {
      Set s;
      load(s, first);
      multiply(s, first);
    }
  }
  return sums;
}

// grid: workgroup 0 writes the routing down, the others walk the units (item, eight intermediate indices); 512 threads
template <int DT, int LISTS>
__global__ __launch_bounds__(kSmallThreads, 4) void ffn_small_gate_up(FfnArgs f, RouteArgs p, const uint64_t* __restrict__ list_key,
                                                                         const uint8_t* __restrict__ list_id,
                                                                         int32_t* __restrict__ topk_ids, float* __restrict__ topk_w,
                                                                         int split) {
  constexpr int EB = Store<DT>::bytes, W = kSmallWaves, kPlanes = DT == SERE_F32 ? 2 : 1;
  __shared__ float s_part[2][kPlanes][W][4][kWave];   // [unit, in turn][sum, what it has lost][wavefront][register][lane]
  __shared__ SmallRouteShared s_route;
  __shared__ uint8_t s_token[W][kSmallSlots];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int i = lane & 15, g = lane >> 4;
  const int dh = f.dh, dm = f.dm, A = p.T * p.K;
  const bool writer = blockIdx.x == 0;
  const SmallRoute r = small_route<LISTS>(list_key, list_id, p, s_route);
  if (writer) {
    write_small_route(p, r, s_route, topk_ids, topk_w);
    return;
  }
  // a wavefront takes one of `split` slices of the contraction for one of the unit's W / split groups of eight indices
  const int blocks = dh * EB / kSmallBlock, per = (blocks + split - 1) / split;
  const int tile = wave / split, slice = wave % split, b0 = slice * per, b1 = min(b0 + per, blocks);
  const int outs = kSmallOut * (W / split), parts = dm / outs;
  const size_t ld = static_cast<size_t>(dh) * EB;
  int buf = 0;
  for (int unit = blockIdx.x - 1; unit < (r.active + p.n_sh) * parts; unit += gridDim.x - 1) {
    const int item = unit / parts, j0 = unit % parts * outs;
    int e, off, cnt;
    if (item < r.active) {
      const bool mine = lane < A && r.item == item;
      const int lead = __ffsll(static_cast<long long>(__ballot(mine))) - 1;
      e = read_lane(r.after, lead);
      off = read_lane(r.pos, lead);
      cnt = read_lane(r.count, lead);
      if (mine) s_token[wave][r.rank] = static_cast<uint8_t>(lane / p.K);
    } else {
      e = p.M + item - r.active;
      off = A + (item - r.active) * p.T;
      cnt = p.T;
      s_token[wave][lane] = static_cast<uint8_t>(lane);
    }
    wave_lds_fence();
    const char* rows = static_cast<const char*>(expert_base<DT>(f.w_gate_up, f.shared_gate_up, e, f.M, static_cast<size_t>(2) * dm * dh));
    const char* wx = rows + static_cast<size_t>(j0 + tile * kSmallOut + (i & 7)) * ld + 16 * (2 * g + (i >> 3));
    for (int n0 = 0; n0 < cnt; n0 += kTile, buf ^= 1) {
      const char* xt = static_cast<const char*>(f.hidden) + s_token[wave][min(n0 + i, cnt - 1)] * ld + 32 * g;
      const SmallSums<DT> v = small_contract<DT, false, kSmallAhead, false>(wx, wx + static_cast<size_t>(dm) * ld, xt, b0, b1);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        s_part[buf][0][wave][c][lane] = v.acc[c];
        if constexpr (DT == SERE_F32) s_part[buf][kPlanes - 1][wave][c][lane] = v.low[c];
      }
      __syncthreads();   // (the next sums go to the other half, and the ones behind them come after the next barrier)
      // lane (g, n) of a tile holds D[4 g + c][n]: gate rows 0 to 7, the matching up rows 8 to 15
      for (int at = threadIdx.x; at < outs * min(kTile, cnt - n0); at += kSmallThreads) {
        const int j = at % outs, n = at / outs, w0 = j / kSmallOut * split, c = j & 3, l = 16 * ((j >> 2) & 1) + n;
        SmallTotal<DT> gate{0.0f, 0.0f}, up{0.0f, 0.0f};
        for (int w = w0; w < w0 + split; ++w) {
          gate.add(s_part[buf][0][w][c][l], s_part[buf][kPlanes - 1][w][c][l]);
          up.add(s_part[buf][0][w][c][l + 32], s_part[buf][kPlanes - 1][w][c][l + 32]);
        }
        const size_t to = static_cast<size_t>(off + n0 + n) * dm + j0 + j;
        if constexpr (DT == SERE_F32)
          f.h[to] = silu(gate.value()) * up.value();
        else
          reinterpret_cast<uint16_t*>(f.h)[to] = f32_to_bf16(silu_for_bf16(gate.value()) * up.value());
      }
    }
  }
}

// grid dh / kSmallOut, 512 threads.  Down projection of every item for eight output rows, and the weighted sum over slots,
// shared experts and the residual in combine_columns_kernel's order.
template <int DT>
__global__ __launch_bounds__(kSmallThreads, 2) void ffn_small_down(FfnArgs f, CombineArgs c) {
  constexpr int EB = Store<DT>::bytes, W = kSmallWaves, kPlanes = DT == SERE_F32 ? 2 : 1;
  __shared__ __attribute__((aligned(16))) float s_y[kPlanes][kSmallSums][kSmallOut];   // [sum, what it has lost][slice, row]
  __shared__ int s_pos[kSmallSlots];
  __shared__ float s_w[kSmallSlots];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int i = lane & 15, g = lane >> 4;
  const int dh = f.dh, dm = f.dm, A = c.T * c.K;
  const int n = f.n_work[0];
  // At most 64 items, one to a lane, requested together with their number: lanes beyond it hold nothing of use.  (Every array
  // of the workspace has room for 64 integers.)
  const int at = min(lane, A + c.n_sh - 1);
  const int item_e = f.work_expert[at], item_off = f.work_off[at], item_cnt = f.work_cnt[at];
  if (threadIdx.x < kSmallSlots) {
    const int a = min(static_cast<int>(threadIdx.x), A - 1);
    s_pos[threadIdx.x] = c.slot_pos[a];
    s_w[threadIdx.x] = c.topk_w[a];
  }
  const int blocks = dm * EB / kSmallBlock;
  const int slices = max(1, min(min(W / n, blocks), kSmallSums / c.rows)), per = (blocks + slices - 1) / slices;
  const int r0 = blockIdx.x * kSmallOut;
  const size_t ld = static_cast<size_t>(dm) * EB;
  for (int task = wave; task < n * slices; task += W) {
    const int item = task / slices, slice = task % slices;
    const int e = read_lane(item_e, item), off = read_lane(item_off, item), cnt = read_lane(item_cnt, item);
    const char* rows = static_cast<const char*>(expert_base<DT>(f.w_down, f.shared_down, e, f.M, static_cast<size_t>(dh) * dm));
    const char* wx = rows + static_cast<size_t>(r0 + (i & 7)) * ld + 16 * (2 * g + (i >> 3));
    for (int n0 = 0; n0 < cnt; n0 += kTile) {
      const char* xt = reinterpret_cast<const char*>(f.h) + static_cast<size_t>(off + min(n0 + i, cnt - 1)) * ld + 32 * g;
      const SmallSums<DT> v = small_contract<DT, true, kSmallAhead, true>(wx, wx, xt, slice * per, min((slice + 1) * per, blocks));
      if (g < 2 && n0 + i < cnt) {
        const int to = slice * c.rows + off + n0 + i;
        *reinterpret_cast<f32x4*>(&s_y[0][to][4 * g]) = v.acc;
        if constexpr (DT == SERE_F32) *reinterpret_cast<f32x4*>(&s_y[kPlanes - 1][to][4 * g]) = v.low;
      }
    }
  }
  __syncthreads();
  const int t = threadIdx.x / kSmallOut, r = threadIdx.x % kSmallOut;
  if (t >= c.T) return;
  auto value = [&](int row) {
    SmallTotal<DT> v{0.0f, 0.0f};
    for (int s = 0; s < slices; ++s) v.add(s_y[0][s * c.rows + row][r], s_y[kPlanes - 1][s * c.rows + row][r]);
    return v.value();
  };
  float acc = 0.0f;
  for (int k = 0; k < c.K; ++k) acc = fmaf(s_w[t * c.K + k], value(s_pos[t * c.K + k]), acc);
  for (int sh = 0; sh < c.n_sh; ++sh) acc += value(A + sh * c.T + t);
  const size_t to = static_cast<size_t>(t) * dh + r0 + r;
  if constexpr (DT == SERE_F32) {
    if (c.residual != nullptr) acc += static_cast<const float*>(c.residual)[to];
    static_cast<float*>(c.out)[to] = acc;
  } else {
    if (c.residual != nullptr) acc += bf16_to_f32(static_cast<const uint16_t*>(c.residual)[to]);
    static_cast<uint16_t*>(c.out)[to] = f32_to_bf16(acc);
  }
}

}  // namespace sere
