// The row pass that also writes the field (ROW_FUSED_OUT) exists in FP64: the
// FP32 launchers of the block, 2-D wave and 3-D wave passes refuse it, on the
// host, before any launch.  Prints one status per launcher; exits nonzero
// unless each is hipErrorInvalidValue.
#include <cstdio>

#include "kernels.hpp"
#include "plan.hpp"

int main() {
  using namespace lshom;
  RowArgs<float> row{};
  row.mode = ROW_FUSED_OUT;
  row.d = 2;
  row.n = 60;
  row.h = 31;
  row.nrows = 60;
  row.rows_per_block = 2;
  row.plan = default_plan(60);
  const hipError_t block = launch_row(row, nullptr);
  row.n = 81;
  row.h = 41;
  row.row_fast = 1;
  row.plan = default_plan(81);
  const hipError_t wave2 = launch_row(row, nullptr);
  const hipError_t wave2_direct = launch_w2_row(row, nullptr);
  W3Args<float> w3{};
  w3.mode = ROW_FUSED_OUT;
  w3.N0 = w3.N1 = w3.N2 = 27;
  w3.h = 14;
  w3.G = w3_groups(14);
  const hipError_t wave3 = launch_w3(W3_ROW, w3, nullptr);
  std::printf("%d %d %d %d\n", (int)block, (int)wave2, (int)wave2_direct, (int)wave3);
  return !(block == hipErrorInvalidValue && wave2 == hipErrorInvalidValue && wave2_direct == hipErrorInvalidValue &&
           wave3 == hipErrorInvalidValue);
}
