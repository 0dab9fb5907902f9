// Runs the last workgroups of counts_subtile_kernel with totals from the rows on host threads,
// n = 6 .. 8, the counts ending at a guard page.  Totals and row-sum parts are compared with
// the rows.
#include <cstdio>
#include <thread>
#include <vector>

#include "guarded.hpp"
#include "lre_kernels.hpp"
#undef __shared__
#define __shared__ static
#include "lre_tile.hpp"

using namespace lre;

int main() {
  for (int n = 6; n <= 8; ++n) {
    const int64_t rows = ipow3(n), cols = (int64_t)1 << n, blocks = ipow3(n - 5) << (n - 6);
    uint16_t* counts = guarded<uint16_t>((size_t)(rows * cols));
    uint32_t* nb = guarded<uint32_t>((size_t)rows);
    double* out = guarded<double>((size_t)((ipow3(n - 5) << (n - 5)) * 1024));
    uint32_t* part = guarded<uint32_t>((size_t)(blocks * kTileRows));
    for (int64_t i = 0; i < rows * cols; ++i) counts[i] = (uint16_t)(1 + (i * 2654435761u >> 9) % 60000);
    const int64_t tiles = (int64_t)1 << (n - 6);
    for (int64_t blk : {blocks - tiles, blocks - 1}) {
      std::barrier<> bar(256);
      host_barrier = &bar;
      std::vector<std::thread> group;
      for (unsigned t = 0; t < 256; ++t)
        group.emplace_back([=] {
          threadIdx.x = t;
          blockIdx.x = (unsigned)blk;
          blockIdx.y = 0;
          counts_subtile_kernel<true, double>(counts, n, n, nullptr, nb, out, part, 0, 0, 0);
        });
      for (auto& t : group) t.join();
    }
    for (int r = 0; r < kTileRows; ++r) {
      const int64_t b = rows - kTileRows + r;
      uint32_t total = 0, last = 0;
      for (int64_t s = 0; s < cols; ++s) {
        total += counts[b * cols + s];
        if (s >= cols - 64) last += counts[b * cols + s];
      }
      if (nb[b] != total || part[(blocks - 1) * kTileRows + r] != last) {
        std::printf("n %d row %ld: %u and %u, not %u and %u\n", n, (long)b, nb[b], part[(blocks - 1) * kTileRows + r],
                    total, last);
        return 1;
      }
    }
  }
  return 0;
}
