// Scratch of plans whose items are dealt out to work lists (bf16), over random
// ragged batches whose scratch is near HPD_NOALLOC_SCRATCH_BYTES: where the plan
// without lists (the same batch in fp32) fits the library's own scratch, the
// plan with lists does too.  Prints how many plans without lists fitted, and of
// them how many had lists and how many went without.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "plan.h"

int main(int argc, char **argv) {
  std::mt19937 rng(argc > 1 ? std::atoi(argv[1]) : 0);
  auto in = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  int fitted = 0, lists = 0, without = 0;
  for (int n = 0; n < 400; ++n) {
    const int np = in(16, 30), least = in(4, 24), most = in(least, 32), past_hi = in(64, 1024);
    std::vector<int32_t> prefix, page, num_new, past, fork;
    for (int p = 0; p < np; ++p) {
      prefix.push_back(in(1024, 4096));
      for (int b = in(least, most); b >= 0; --b) {
        page.push_back(p);
        num_new.push_back(4);
        past.push_back(in(8, past_hi));
        fork.push_back(in(prefix[p] / 2, prefix[p]));
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
    a.num_kv_heads = n % 3 ? 2 : 8;
    a.head_dim = 64;
    hpd::Plan P[2];
    for (int i = 0; i < 2; ++i) {
      a.dtype = a.out_dtype = i ? HPD_BF16 : HPD_F32;
      std::string err;
      if (hpd::build_plan(&a, &b, &P[i], &err) != HPD_OK) {
        std::printf("plan %d: %s\n", n, err.c_str());
        return 1;
      }
    }
    if (P[0].workspace_bytes > HPD_NOALLOC_SCRATCH_BYTES) continue;
    ++fitted;
    ++(P[1].num_wg > 0 ? lists : without);
    if (P[1].workspace_bytes > HPD_NOALLOC_SCRATCH_BYTES) {
      std::printf("plan %d: %zu bytes without lists, %zu with\n", n, P[0].workspace_bytes, P[1].workspace_bytes);
      return 1;
    }
  }
  std::printf("%d %d %d\n", fitted, lists, without);
  return 0;
}
