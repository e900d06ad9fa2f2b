// Host build of the rules by which waves hand their secondaries on: for
// numbers of waves and of waves with electrons, what one look at them decides.
#define AVM_HOST_DEBUG 1
#include <cstdio>
#include <initializer_list>

#include "avm_internal.hpp"

int main() {
  for (uint32_t waves : {16u, 17u, 1024u, 2048u, 4096u, 8192u})
    for (uint32_t k = 0; k <= 16; ++k) {
      const avm::WaveLoad w{waves, waves * k / 16u};
      std::printf("%u %u %d %d %d %d\n", w.waves, w.busy, w.full(), w.spare(), w.spread(false), w.spread(true));
    }
}
