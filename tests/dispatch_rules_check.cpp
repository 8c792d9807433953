// The host side of csrc/launch.hpp's dispatch rules, printed or checked for
// tests/test_dispatch_rules.py.  CPU only.
#include <cstdio>

#include "launch.hpp"

int main() {
  using namespace mhl;
  // dw T Nh dff form: the weight-gradient kernel's form at d_h 128
  for (int dff = 32; dff <= 512; dff += 32)
    for (const int Nh : {1, 3, 8})
      for (const int64_t T : {int64_t(0), int64_t(1), int64_t(4096), (int64_t(1) << 24) / Nh - 1,
                              (int64_t(1) << 24) / Nh, (int64_t(1) << 24) / Nh + 1, int64_t(1) << 27})
        std::printf("dw %lld %d %d %d\n", (long long)T, Nh, dff, (int)bwd_dw_form(T, Nh, dff));
  return 0;
}
