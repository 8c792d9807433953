// The host side of csrc/launch.hpp's dispatch rules, printed or checked for
// tests/test_dispatch_rules.py.  CPU only.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <vector>

#include "launch.hpp"

using namespace mhl;

namespace {

// The shares of the weight-stationary FFN's tile list, written tile by tile as
// scatter_kernel does: every boundary once, in order, from 0 to ntot, and no
// share dearer than an equal one by more than the weights at its two ends.
void check_shares(const char* what, const std::vector<int64_t>& counts, int sw) {
  std::vector<int> owner;  // expert of each tile
  for (size_t e = 0; e < counts.size(); ++e)
    for (int64_t n = 0; n < ceil_div(counts[e], kWsTileRows); ++n) owner.push_back((int)e);
  const int64_t ntot = (int64_t)owner.size();
  int64_t nexp = 0;
  for (const int64_t c : counts) nexp += c > 0;
  std::vector<int64_t> share(kWsGrid + 1, -1);
  int bad = 0;
  auto put = [&](int m, int64_t i) {
    if (m < 0 || m > kWsGrid || share[m] != -1) ++bad;
    else share[m] = i;
  };
  int64_t rank = 0;
  for (int64_t i = 0; i < ntot; ++i) {
    const bool first = i == 0 || owner[i] != owner[i - 1];
    rank += first;
    const WsShares s = ws_shares_at(i, first, rank, ntot, nexp, sw);
    for (int m = s.begin; m < s.end; ++m) put(m, i);
    if (i == ntot - 1)
      for (int m = s.end; m <= kWsGrid; ++m) put(m, ntot);
  }
  int64_t dearest = 0;
  for (int m = 0; m <= kWsGrid; ++m) {
    if (share[m] < 0 || (m > 0 && share[m] < share[m - 1])) ++bad;
    if (m == 0) continue;
    int64_t cost = 0;
    for (int64_t i = share[m - 1]; i < share[m]; ++i)
      cost += 1 + (i == share[m - 1] || owner[i] != owner[i - 1] ? sw : 0);
    dearest = std::max(dearest, cost);
  }
  if (share[0] != 0 || share[kWsGrid] != ntot) ++bad;
  const double equal = double(ntot + sw * nexp) / kWsGrid;
  std::printf("shares %s %lld %lld %d %d %.3f %lld\n", what, (long long)ntot, (long long)nexp, sw,
              bad, equal, (long long)dearest);
}

}  // namespace

int main() {
  // dw T Nh dff form: the weight-gradient kernel's form at d_h 128
  for (int dff = 32; dff <= 512; dff += 32)
    for (const int Nh : {1, 3, 8})
      for (const int64_t T : {int64_t(0), int64_t(1), int64_t(4096), (int64_t(1) << 24) / Nh - 1,
                              (int64_t(1) << 24) / Nh, (int64_t(1) << 24) / Nh + 1, int64_t(1) << 27})
        std::printf("dw %lld %d %d %d\n", (long long)T, Nh, dff, (int)bwd_dw_form(T, Nh, dff));
  for (const int sw : {0, 2}) {
    check_shares("one_slot", {0, 0, 1, 0}, sw);
    check_shares("one_expert", {0, 70000, 0}, sw);
    check_shares("short", {64, 65, 1, 0, 127, 128, 129}, sw);
    check_shares("even", std::vector<int64_t>(2048, 512), sw);
    check_shares("many", std::vector<int64_t>(16384, 256), sw);
    std::vector<int64_t> zipf, hot(8192, 0);
    for (int h = 0; h < 8; ++h)
      for (int e = 0; e < 256; ++e) {
        const int place = (e * 97 + 31 * h) % 256;  // the experts in some order
        zipf.push_back((int64_t)(131072 * 0.2 / std::pow(1.0 + place, 1.1)));
      }
    for (int e = 0; e < 8192; e += 300) hot[e] = e % 900 == 0 ? 60000 : 3;
    check_shares("zipf", zipf, sw);
    check_shares("hot", hot, sw);
  }
  return 0;
}
