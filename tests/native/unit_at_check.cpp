// Host-side check of the 3-way units' closed form (unit_at, grid_unit_count)
// against the enumeration pair by pair (unit_coords over a table of offsets):
// every unit of every row range, tile of 16, 32 and 64 rows, runs of 1 and 4.
// Prints "ok <units>" and exits 0, or names the first difference.
#include <stdio.h>

#include <vector>

#include "../../paper_1705_08213_amd/csrc/kernels.h"

using namespace ccc;

int main() {
  long total = 0;
  for (int64_t run : {1, 4})
    for (int64_t b : {16, 32, 64})
      for (int64_t n : {3, 4, 17, 31, 32, 33, 34, 63, 64, 65, 66, 67, 96, 97, 98, 99, 130, 161, 200})
        for (int64_t ib = 0; ib < n - 2; ib += 1 + n / 40)
          for (int64_t ie : {ib + 1, ib + 2, ib + 33, n - 2}) {
            if (ie > n - 2) continue;
            const UnitGrid g = unit_grid(n, b, ib, ie, run);
            const int64_t P = grid_pairs(g);
            std::vector<int64_t> offs(P + 1, 0);
            for (int64_t p = 0; p < P; ++p) {
              int64_t it, kt;
              pair_tiles(g, p, it, kt);
              offs[p + 1] = offs[p] + pair_units(g, it, kt);
            }
            if (grid_unit_count(g) != offs[P]) {
              printf("FAIL count n=%ld b=%ld run=%ld ib=%ld ie=%ld: %ld, want %ld\n", (long)n, (long)b,
                     (long)run, (long)ib, (long)ie, (long)grid_unit_count(g), (long)offs[P]);
              return 1;
            }
            for (int64_t u = 0; u < offs[P]; ++u, ++total) {
              int64_t j0, i0, k0, j1, i1, k1;
              unit_coords(u, g, offs.data(), j0, i0, k0);
              unit_at(u, g, j1, i1, k1);
              if (j0 != j1 || i0 != i1 || k0 != k1) {
                printf("FAIL unit %ld n=%ld b=%ld run=%ld ib=%ld ie=%ld\n", (long)u, (long)n, (long)b,
                       (long)run, (long)ib, (long)ie);
                return 1;
              }
            }
          }
  printf("ok %ld\n", total);
  return 0;
}
