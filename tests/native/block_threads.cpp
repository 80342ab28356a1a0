// The block size of a pass launch, for lines "n points lds blocks bytes" read
// from stdin (an axis of n nodes, points and LDS bytes of a block, blocks of
// the launch, bytes of a complex element).
#include <iostream>

#include "plan.hpp"

int main() {
  using namespace lshom;
  int n, points, elem;
  long long lds, blocks;
  while (std::cin >> n >> points >> lds >> blocks >> elem)
    std::cout << pick_threads(points, default_plan(n), (size_t)lds, blocks, elem) << '\n';
}
