// launch_gemm's argument check, on the host: operands in different layouts are
// refused for every kernel (skinny and many-token, packed and row-major
// weights, all epilogues) before anything is launched.
#include <cstdio>

#include "gemm.h"

int main() {
  static float buf[16];
  int refused = 0, calls = 0;
  for (int wide : {0, 1, 2, 4})
    for (int epi : {(int)hpd::kEpiQKV, (int)hpd::kEpiResidual, (int)hpd::kEpiSwiGLU})
      for (bool a_packed : {false, true}) {
        hpd::GemmArgs g{};
        g.K = 256;
        g.N = 256;
        g.rg = 2;
        g.wide = wide;
        g.n_slices = 4;
        g.T = g.Tpad = 32;
        g.n_ttiles = 1;
        g.I = 128;
        g.h = buf;
        g.ss_in = buf;
        g.n_ss = 8;
        g.a_packed = a_packed;
        g.act_packed = !a_packed;
        const hipError_t e = hpd::launch_gemm(g, epi == hpd::kEpiSwiGLU, epi, hpd::KK_GEMM_QKV, nullptr);
        if (e != hipErrorInvalidValue)
          std::printf("wide %d epi %d a_packed %d: %s\n", wide, epi, a_packed, hipGetErrorString(e));
        refused += e == hipErrorInvalidValue;
        ++calls;
      }
  std::printf("%d of %d refused\n", refused, calls);
  return refused == calls ? 0 : 1;
}
