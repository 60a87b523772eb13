// The ranges of entries that the block copies go out in: all entries, each once, no launch of 2^32 threads or more, and one launch
// wherever one can hold them.
#include <algorithm>
#include <cstdio>

#include "ps_internal.h"

int main() {
  for (int64_t per_workgroup : {4, 16})                            // pieces
    for (int64_t heads : {1, 2, 8, 32})
      for (int64_t tile_bytes : {16, 2048, 4096, 4112, 4352, 8192, 65536, 1 << 28}) {
        const int64_t pieces = 2 * heads * ((tile_bytes + 4095) / 4096);
        for (int64_t entries : {int64_t(1), int64_t(3), int64_t(100000), int64_t(1) << 24, (int64_t(1) << 30) / heads}) {
          const int64_t step = entries_per_launch(entries, pieces, per_workgroup);
          int64_t done = 0, launches = 0;
          for (int64_t first = 0; first < entries && launches < 1000000; first += step, ++launches) {
            const int64_t n = std::min(step, entries - first);
            const int64_t workgroups = (n * pieces + per_workgroup - 1) / per_workgroup;
            if (n <= 0 || workgroups * 256 >= int64_t(1) << 32) {
              std::printf("FAILED: %lld entries of %lld pieces: %lld workgroups\n", (long long)n, (long long)pieces, (long long)workgroups);
              return 1;
            }
            done += n;
          }
          const bool one = (entries * pieces + per_workgroup - 1) / per_workgroup * 256 < int64_t(1) << 32;
          if (step <= 0 || (launches < 1000000 && done != entries) || (one && launches != 1)) {
            std::printf("FAILED: %lld entries of %lld pieces: %lld launches\n", (long long)entries, (long long)pieces, (long long)launches);
            return 1;
          }
        }
      }
  std::puts("ok");
  return 0;
}
