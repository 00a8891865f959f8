// Host-only driver of the automatic route's choice (choose_rebuilt): reads cases
// "n_kv d n_q_heads n_q n_blocks n_already (T rk rv)..." and prints how many blocks
// each call rebuilds; the first n_already blocks are rebuilt whatever the model says.
#include <cstdio>
#include <numeric>
#include <vector>

#include "milo_plan.h"

using namespace milo;

int main() {
  int n_kv, d, hq, n_q, nb, already;
  while (std::scanf("%d %d %d %d %d %d", &n_kv, &d, &hq, &n_q, &nb, &already) == 6) {
    std::vector<BlockMeta> meta(nb);
    for (BlockMeta& m : meta) {
      int rk, rv;
      if (std::scanf("%d %d %d", &m.T, &rk, &rv) != 3) return 2;
      m.T_pad = (m.T + kTile - 1) / kTile * kTile;
      m.rk_pad = (rk + 31) / 32 * 32;
      m.rv_pad = (rv + 31) / 32 * 32;
    }
    std::vector<int32_t> table(nb);
    std::iota(table.begin(), table.end(), 0);
    std::vector<char> recon(nb, 0);
    for (int j = 0; j < already; ++j) recon[j] = 1;
    choose_rebuilt(meta.data(), table.data(), nb, (int64_t)n_q * hq, n_kv * d, d, recon.data());
    std::printf("%d\n", std::accumulate(recon.begin(), recon.end(), 0));
  }
  return 0;
}
