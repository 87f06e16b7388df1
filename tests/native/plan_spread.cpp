// Private items of plans just over one round of workgroups, whose histories are
// short (a few pages of many branches): workgroups with the same shared work
// differ by at most kPrivateWaves / 2 private items (in whole rounds of
// kPrivateWaves some had 8 and others none, and the layer was slower than with the
// hardware handing them out).  Prints how many plans had lists.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <vector>

#include "plan.h"

int main(int argc, char **argv) {
  std::mt19937 rng(argc > 1 ? std::atoi(argv[1]) : 0);
  auto in = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  int lists = 0;
  for (int n = 0; n < 200; ++n) {
    std::vector<int32_t> prefix, page, num_new, past, fork;
    const int np = in(2, 16), hkv = n % 2 ? 8 : 2;
    for (int p = 0; p < np; ++p) {
      prefix.push_back(in(1024, 4096));
      for (int b = in(10, 30); b > 0; --b) {
        page.push_back(p);
        num_new.push_back(4);
        past.push_back(in(8, 48));
        fork.push_back(in(prefix[p] / 4, prefix[p]));
      }
    }
    hpd_batch_desc b{};
    b.num_pages = np;
    b.num_branches = (int)page.size();
    b.prefix_len = prefix.data();
    b.branch_page = page.data();
    b.num_new = num_new.data();
    b.past_len = past.data();
    b.fork_len = in(0, 1) ? fork.data() : nullptr;
    hpd_attn_desc a{};
    a.num_q_heads = 16;
    a.num_kv_heads = hkv;
    a.head_dim = 64;
    a.dtype = a.out_dtype = HPD_BF16;
    hpd::Plan P;
    std::string err;
    if (hpd::build_plan(&a, &b, &P, &err) != HPD_OK) return 1;
    if (P.num_wg == 0) continue;
    ++lists;
    std::map<std::vector<int>, std::pair<int, int>> range;   // shared items' units -> least, most private items
    for (int w = 0; w < P.num_wg; ++w) {
      const int32_t *l = &P.wg[4 * (size_t)w];
      std::vector<int> key{l[1] - l[0], 0};
      for (int i = l[0]; i < l[1]; ++i) {
        const int32_t *it = &P.wg_shared[(size_t)i * hpd::SI_NFIELDS];
        key[1] += (it[hpd::SI_KEY1] - it[hpd::SI_KEY0] + hpd::kSharedSplitUnit - 1) / hpd::kSharedSplitUnit;
      }
      // (the last private items fill no whole deal)
      const int priv = (l[3] - l[2] + hpd::kPrivateWaves / 2 - 1) / (hpd::kPrivateWaves / 2) * (hpd::kPrivateWaves / 2);
      auto [at, fresh] = range.try_emplace(key, priv, priv);
      at->second.first = std::min(at->second.first, priv);
      at->second.second = std::max(at->second.second, priv);
      if (at->second.second - at->second.first > hpd::kPrivateWaves / 2) {
        std::printf("plan %d: %d and %d private items beside %d pairs of key tiles\n", n, at->second.first,
                    at->second.second, key[1]);
        return 1;
      }
    }
  }
  std::printf("%d\n", lists);
  return 0;
}
