// Host build of the persistent kernel's pass lengths: for each number of
// flights that a caller may ask for, the flights of a pass and the most that
// a wave flies in one go, with a short and a long queue.
#define AVM_HOST_DEBUG 1
#include <cstdio>
#include <initializer_list>

#include "avm_internal.hpp"

int main() {
  for (int32_t n : {1, 2, 3, 48, 1000, (1 << 28) - 1, 1 << 28, (1 << 29) - 1, 1 << 29, 1 << 30, 0x7FFFFFFE, 0x7FFFFFFF})
    for (bool long_queue : {false, true}) {
      const int32_t pass = avm::pass_flights(avm::clamp_flights_per_pass(n), long_queue);
      std::printf("%d %d %d %d %d\n", n, long_queue, pass, avm::pass_limit(pass, false), avm::pass_limit(pass, true));
    }
}
