// Host-side check of the hashing chunks of a two-phase flush (no GPU, no HIP):
// compiled several times with g++ by tests/test_host_chunks.py, which compares
// what the compilations print.
#include <stdio.h>

#include "build_plan.hpp"

using namespace compass;

int main() {
  uint64_t sum = 0;
  long long wrong = 0, rounds = 0;
  for (int n_cu : {1, 8, 256, 304})
    for (int n_slices : {1, 3, 7, 15, 21, 66, 512})
      for (int w : {1, 1000, 3000, 8192, 16383, 65536, 65537, 70001, 1 << 20})
        for (int64_t chunks : {1, 2, 15, 48, 146, 1024}) {
          const int items = n_slices * ((w + 65535) / 65536);
          for (int64_t n = 0; n < (int64_t)1 << 33; n += n / 7 + 4097) {
            const int c = hash_chunks(n, chunks, n_slices, w, n_cu);
            // the buffer's slab rows, and no more chunks than survivors fill
            const int64_t need = n < 16384 ? 1 : (n + 16383) / 16384;
            wrong += c < 1 || c > chunks || c > need;
            // one round: as many as there are
            const int64_t most = need < chunks ? need : chunks;
            if (most * items <= n_cu) wrong += c != most;
            rounds += (int64_t)c * items > n_cu;
            sum = sum * 0x9E3779B97F4A7C15ull + (uint64_t)c;
          }
        }
  // times within a rounding of each other: in fp32, 11 chunks with separate
  // multiplies and adds and 8 with fused ones
  sum = sum * 31 + (uint64_t)hash_chunks(3133542, 48, 86, 15398, 256);
  printf("wrong %lld, more than one round %s, sum %016llx\n", wrong, rounds ? "too" : "never",
         (unsigned long long)sum);
  return wrong != 0;
}
