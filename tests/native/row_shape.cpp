// The default row-pass shape of 3-D grids read from stdin as "N0 N1 N2 bytes"
// (bytes of a complex element): prints rows per block, components split, and
// points per block.
#include <iostream>

#include "plan.hpp"

int main() {
  using namespace lshom;
  int64_t N[3];
  int elem;
  while (std::cin >> N[0] >> N[1] >> N[2] >> elem) {
    FftPlan plans[3];
    for (int a = 0; a < 3; ++a) plans[a] = default_plan((int)N[a]);
    const PassShape s = default_shape(3, N, plans, elem, 64 * 1024, 128, false, 2, true);
    std::cout << s.rows_per_block << ' ' << s.row_split << ' '
              << (s.row_split ? 1 : 3) * (s.rows_per_block / 2) * N[2] << ' '
              << shape_fits(3, N, plans, s, elem, 64 * 1024, 2) << '\n';
  }
}
