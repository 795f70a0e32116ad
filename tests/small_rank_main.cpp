// Top-K of one token as ffn_small.hpp ranks it, lane by lane.  Reads "K M key[0] .. key[M-1]" (the experts' keys, hexadecimal) and
// prints the K chosen experts; the lists are made as the router kernels leave them.  Host code only.
#include <algorithm>
#include <cinttypes>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "../paper_2602_07616_amd/csrc/rules.hpp"

int main() {
  int K = 0, M = 0;
  while (std::scanf("%d %d", &K, &M) == 2) {
    std::vector<uint64_t> keys(M);
    for (uint64_t& k : keys)
      if (std::scanf("%" SCNx64, &k) != 1) return 1;
    const int nlists = (M + 15) / 16, N = nlists <= 8 ? 1 : 2, entries = 8 * nlists;
    std::vector<uint64_t> key(64 * N, 0);
    std::vector<int> id(64 * N, -1);
    for (int l = 0; l < nlists; ++l) {   // a list: its 16 experts by descending key, equal ones in their order, places beyond M with key 0
      std::vector<int> e(16);
      for (int j = 0; j < 16; ++j) e[j] = 16 * l + j;
      const auto key_of = [&](int x) { return x < M ? keys[x] : 0; };
      std::stable_sort(e.begin(), e.end(), [&](int a, int b) { return key_of(a) > key_of(b); });
      for (int j = 0; j < 8; ++j) key[8 * l + j] = key_of(e[j]), id[8 * l + j] = e[j];
    }
    std::vector<int> rank(entries, 0), chosen(K, -1);
    int sum = 0;
    for (int a = 0; a < entries; ++a) {
      for (int b = 0; b < entries; ++b) rank[a] += sere::rank_word(key[b], b, 64 * N) > sere::rank_word(key[a], a, 64 * N);
      sum += rank[a];
    }
    if (sum != entries * (entries - 1) / 2)
      for (int a = 0; a < entries; ++a) {
        rank[a] = 0;
        for (int b = 0; b < entries; ++b) rank[a] += sere::ranks_before(key[b], b, key[a], a);
      }
    for (int a = 0; a < entries; ++a)
      if (rank[a] < K) chosen[rank[a]] = id[a];
    for (int k = 0; k < K; ++k) std::printf("%d ", chosen[k]);
    std::printf("\n");
  }
  return 0;
}
