// Host build of the persistent kernel's first claims: blocks come one after
// the other to a queue of n entries; each entry a block claims must be taken by
// one lane of one of its waves, and the waves it counts as used must be those
// that got some.  Prints, per case: entries, blocks, entries claimed, mistakes,
// waves used.
#define AVM_HOST_DEBUG 1
#include <cstdio>
#include <vector>

#include "avm_internal.hpp"

int main() {
  constexpr uint32_t kWaves = 16, kMost = 64 * kWaves;
  for (uint32_t blocks : {1u, 2u, 3u, 7u, 128u, 255u, 256u, 257u, 304u, 512u})
    for (uint32_t n : {0u, 1u, 2u, 15u, 16u, 17u, 63u, 64u, 65u, 255u, 256u, 257u, 1000u, 1023u, 1024u, 1025u, 4095u, 4096u,
                       4097u, 8192u, 10000u, 16383u, 16384u, 16385u, 65537u, 262143u, 262144u, 262145u, 1000000u, 4294967280u}) {
      unsigned long long head = 0, used_waves = 0;
      long bad = 0;
      for (uint32_t b = 0; b < blocks; ++b) {
        const uint32_t k = n > head ? avm::block_share(n, n - (uint32_t)head, blocks, kMost) : 0u, s = avm::wave_share(n, blocks * kWaves);
        head += k;
        std::vector<int> taken(k, 0);
        const uint32_t used = (k + s - 1u) / s;
        bad += s < 1 || s > 64 || used > kWaves;
        for (uint32_t w = 0; w < kWaves; ++w) {
          uint32_t got = 0;
          for (uint32_t lane = 0; lane < 64; ++lane) {
            const uint32_t i = w * s + lane;
            if (lane < s && i < k) {
              ++taken[i];
              ++got;
            }
          }
          bad += (got > 0) != (w < used);
        }
        for (int t : taken) bad += t != 1;
        used_waves += used;
      }
      std::printf("%u %u %llu %ld %llu\n", n, blocks, head, bad, used_waves);
    }
}
