// Host tier of the test suite: prints the launch arithmetic and the dispatch
// rules of the library for tests/test_launch_rules.py; host code only.
//   near NNZ                "q0 blocks" of each launch of the near-field build
//   fused N F32 NR PAIRS T  whether the row pass takes the anterpolation along
//                           in a product that times (T = 1) one of the two
//   few N PK NACT NR        whether the row passes sum over PK kept pairs of columns
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "../../paper_2606_10784_amd/csrc/aim_internal.h"

int main(int argc, char** argv) {
  if (argc == 3 && !std::strcmp(argv[1], "near")) {
    const int64_t nnz = std::atoll(argv[2]);
    std::printf("%d %d\n", aim::kNG, aim::kNearBlock);
    for (int64_t q0 = 0; q0 < nnz; q0 += aim::kNearLaunch)
      std::printf("%lld %u\n", (long long)q0, aim::near_blocks(q0, nnz));
    return 0;
  }
  if (argc == 7 && !std::strcmp(argv[1], "fused")) {
    std::printf("%d\n", (int)aim::anterp_in_rows(std::atoi(argv[2]), std::atoi(argv[3]) != 0, std::atoi(argv[4]),
                                                 std::atoi(argv[5]), std::atoi(argv[6]) != 0));
    return 0;
  }
  if (argc == 6 && !std::strcmp(argv[1], "few")) {
    std::printf("%d\n", (int)aim::few_columns_pay(std::atoi(argv[2]), std::atoi(argv[3]), std::atoi(argv[4]),
                                                  std::atoi(argv[5])));
    return 0;
  }
  return 2;
}
