// Host time of plans whose items are dealt out to work lists: per batch, the
// best of many build_plan calls in bf16 (lists) and of as many in fp32 (the same
// batch without lists) in turn.  Prints both in us.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "plan.h"

int main() {
  // pages, kv heads, paged with fork points
  const int cases[][3] = {{16, 2, 0}, {24, 2, 1}, {21, 8, 1}, {12, 2, 1}};
  for (const auto &c : cases) {
    std::mt19937 rng(7);
    auto in = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    std::normal_distribution<double> normal;
    std::vector<int32_t> prefix, page, num_new, past, fork, blocks, page0, branch0;
    for (int p = 0; p < c[0]; ++p) {
      prefix.push_back(in(1024, 4096));
      for (int b = in(4, 32); b > 0; --b) {
        page.push_back(p);
        num_new.push_back(4);
        past.push_back(std::min(1024, std::max(8, (int)(128 * std::exp(normal(rng))))));
        fork.push_back(in(prefix[p] / 4, prefix[p]));
      }
    }
    auto add = [&](int rows, std::vector<int32_t> &first) {
      first.push_back((int)blocks.size());
      for (int i = 0; i < rows; i += 64) blocks.push_back((int)blocks.size());
    };
    for (int p : prefix) add(p, page0);
    for (size_t i = 0; i < page.size(); ++i) add(past[i] + num_new[i], branch0);
    hpd_paged_kv pg{64, (int)blocks.size(), (int)blocks.size(), blocks.data(), page0.data(), branch0.data()};
    hpd_batch_desc b{};
    b.num_pages = c[0];
    b.num_branches = (int)page.size();
    b.prefix_len = prefix.data();
    b.branch_page = page.data();
    b.num_new = num_new.data();
    b.past_len = past.data();
    b.fork_len = c[2] ? fork.data() : nullptr;
    b.paged = c[2] ? &pg : nullptr;
    double best[2] = {1e9, 1e9};
    int lists = 0;
    for (int i = 0; i < 600; ++i) {
      hpd_attn_desc a{};
      a.num_q_heads = 16;
      a.num_kv_heads = c[1];
      a.head_dim = 64;
      a.dtype = a.out_dtype = i % 2 ? HPD_BF16 : HPD_F32;
      std::string err;
      hpd::Plan P;
      const auto t0 = std::chrono::steady_clock::now();
      if (hpd::build_plan(&a, &b, &P, &err) != HPD_OK) return 1;
      const std::chrono::duration<double, std::micro> dt = std::chrono::steady_clock::now() - t0;
      best[i % 2] = std::min(best[i % 2], dt.count());
      lists = P.num_wg;
    }
    std::printf("%.1f %.1f %d\n", best[0], best[1], lists);
  }
  return 0;
}
