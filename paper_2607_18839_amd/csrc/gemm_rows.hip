// Projection kernel for packed operands and many tokens.
//
// The skinny kernels (gemm_kernels.hip) give a wave one 32 x 32 output tile and
// let every wave load its own operands: at 129 tokens that is a launch's fixed
// cost, but with hundreds of tokens each CU pulls the same rows in over and
// over (gate/up at 1,256 tokens: 7.5 workgroups of 512 KB per CU, 51 us).
// Here a workgroup of 4 waves owns 128 weight rows (32 per wave) x NT token
// tiles.  The weights, which no other wave needs, go straight into a register
// ring; the token tiles, which all 4 waves multiply, go through an LDS ring
// (direct global -> LDS copies), both 3 to 4 steps of 64 K ahead.  Token
// fragments are read one piece (16 K) ahead of their MFMAs, also across the
// steps' barrier.  Per step a CU then moves 16 + 4 NT KB for 16 NT MFMAs:
// NT = 4 is bound by the matrix cores (16 MFMAs of a wave in about 770 clocks,
// 630 without the weight loads), NT = 1 and 2 by the vector-memory path (371
// and 430 clocks per step), and they take the shapes that give NT = 4 too few
// workgroups (choose_gemm).  256 weight rows per workgroup with NT = 4 was no
// faster (22.8 against 22.5 us).
//
// Epilogue: a finished tile goes through LDS so that its output rows are
// stored in 64- and 128-byte runs (in the MFMA layout a store touches 32 rows
// by 16 or 32 bytes), and everything it needs besides is loaded during the
// loop.  gate/up + SwiGLU at 272 tokens: 14.5 us in the skinny kernel, 9.6 us
// with the MFMA-layout epilogue, 8.0 us so.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "gemm.h"
#include "gemm_dev.h"

namespace hpd {
namespace {

// Sum over each group of 8 lanes, in every lane of it (lane exchanges within
// the vector unit: pairs, quads, then the two quads mirrored).
__device__ __forceinline__ float sum8(float v) {
  auto dpp = [](float x, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  v += dpp(v, std::integral_constant<int, 0xB1>{});    // quad_perm [1,0,3,2]
  v += dpp(v, std::integral_constant<int, 0x4E>{});    // quad_perm [2,3,0,1]
  v += dpp(v, std::integral_constant<int, 0x141>{});   // row_half_mirror
  return v;
}

template <int NT, bool F16, int EPI>
__global__ __launch_bounds__(256) void gemm_rows_kernel(GemmArgs g) {
  asm volatile("" ::"s"(g.N), "s"(g.n_ttiles), "s"(g.K), "s"(g.w0), "s"(g.x), "s"(g.T), "s"(g.dest),
               "s"(g.scale_in), "s"(g.ss_in), "s"(g.n_ss), "s"(gridDim.x));
  constexpr int BM = 4, S = 4, kTileBytes = 4096, kStage = NT * kTileBytes;
  constexpr int kLoads = 4 + NT;   // per wave and step: weight pieces and token copies
  constexpr int kTailLoads = EPI == kEpiResidual ? 4 * NT + 1 : 0;   // issued before the last S steps
  static_assert((S - 1) * kLoads < 64 && (S - 2) * kLoads + kTailLoads < 64, "vmcnt range");
  constexpr int kScratch = 4 * 4608, kRing = S * kStage > kScratch ? S * kStage : kScratch;
  // the ring (after the loop: the waves' epilogue scratch), then two values
  // per token: RMSNorm factor or s_t, cache row.  One array: with a second one
  // the compiler waits for every copy in flight before each LDS read.
  __shared__ __attribute__((aligned(16))) unsigned char lds[kRing + 2 * NT * kGemmTile * 4];
  float *tok_f = (float *)(lds + kRing);
  int *tok_dest = (int *)(tok_f + NT * kGemmTile);

  const int n_rt = g.N / kGemmTile, n_tg = (g.n_ttiles + NT - 1) / NT, n_sl = (n_rt + BM - 1) / BM;
  const int per_xcd = gridDim.x / 8;
  const int logical = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (logical >= n_sl * n_tg) return;
  const int slice = logical / n_tg, tt0 = (logical % n_tg) * NT;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int frow = lane & 31, half = lane >> 5;
  const int nsteps = g.K / kGemmKStep;
  const int tile = slice * BM + wave;   // this wave's row tile

  const __amdgpu_buffer_rsrc_t rx = buffer_rsrc(g.x, (uint64_t)g.Tpad * g.K * 2);
  unsigned sb[NT];   // token copies: piece `wave` of each token tile
#pragma unroll
  for (int n = 0; n < NT; ++n) sb[n] = (unsigned)min(tt0 + n, g.n_ttiles - 1) * (unsigned)nsteps * 4096u + wave * 1024;
  auto issue_b = [&](int c, int slot) {
#pragma unroll
    for (int n = 0; n < NT; ++n)
      bdma16(rx, lane * 16, sb[n] + (unsigned)c * 4096u, lds + slot * kStage + n * kTileBytes + wave * 1024);
  };
  const __bf16 *arow = g.w0 + (int64_t)min(tile, n_rt - 1) * nsteps * 2048 + lane * 8;
  u32x4 a[S][4];   // weight pieces of step c in a[c % S]
  auto load_a = [&](int c, int slot) {
#pragma unroll
    for (int j = 0; j < 4; ++j) a[slot][j] = *(const u32x4 *)(arow + (int64_t)c * 2048 + 512 * j);
  };
  f32x16 acc[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[n][r] = 0.f;

  u32x4 b[2][NT];
  auto read_b = [&](int slot, int j, int buf) {
#pragma unroll
    for (int n = 0; n < NT; ++n) b[buf][n] = *(const u32x4 *)(lds + slot * kStage + n * kTileBytes + 1024 * j + 16 * lane);
  };
  auto mma = [&](const u32x4 &av, int buf) {
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      if constexpr (F16)
        acc[n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, av),
                                                        __builtin_bit_cast(f16x8, b[buf][n]), acc[n], 0, 0, 0);
      else
        acc[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av),
                                                         __builtin_bit_cast(bf16x8, b[buf][n]), acc[n], 0, 0, 0);
    }
  };
  issue_b(0, 0);
  load_a(0, 0);
  // Per-token operands of the epilogue (TP threads per token), loaded here,
  // behind step 0 and ahead of the later steps, and reduced after the loop, so
  // that neither the first step nor the epilogue waits for them.
  constexpr int TP = 256 / (NT * kGemmTile) >= 8 ? 8 : 256 / (NT * kGemmTile) >= 4 ? 4 : 256 / (NT * kGemmTile) >= 2 ? 2 : 1;
  const int st = min(tt0 * kGemmTile + (int)threadIdx.x / TP, g.Tpad - 1), spart = 4 * (threadIdx.x % TP);
  const float *sr = g.ss_in + (int64_t)st * g.n_ss;
  f32x4 sv[4];
  float s_t = 1.f;
  int dest = 0;
  if constexpr (EPI != kEpiResidual) {
#pragma unroll
    for (int u = 0; u < 4; ++u) sv[u] = *(const f32x4 *)(sr + min(spart + 4 * TP * u, g.n_ss - 4));
  }
  if constexpr (EPI == kEpiQKV) dest = g.dest[min(st, g.T - 1)];
  else if (g.scale_in) s_t = g.scale_in[min(st, g.T - 1)];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int c = 1; c < S; ++c) {
    issue_b(c, c);
    load_a(c, c);
    __builtin_amdgcn_sched_barrier(0);
  }
  wait_vm<(S - 1) * kLoads>();
  ring_barrier();
  read_b(0, 0, 0);
  // One step in ring slot SLOT: its last piece's MFMAs run while the next
  // step's first token fragments are read.  AHEAD: whole steps still in flight
  // when the next one is needed (-1: there is none); MORE: refill the slot.
  auto step = [&](int c, auto slot_, auto ahead, auto more) {
    constexpr int SLOT = decltype(slot_)::value, AHEAD = decltype(ahead)::value;
    constexpr bool MORE = decltype(more)::value;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j < 3) {
        read_b(SLOT, j + 1, (j + 1) & 1);
      } else if constexpr (AHEAD >= 0) {
        wait_vm<AHEAD * kLoads + (MORE ? 0 : kTailLoads)>();
        ring_barrier();   // step c + 1 visible to every wave; every wave has read step c
        if constexpr (MORE) issue_b(c + S, SLOT);
        read_b((SLOT + 1) % S, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      mma(a[SLOT][j], j & 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (MORE) {
      load_a(c + S, SLOT);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using std::integral_constant;
  for (int c = 0; c + S < nsteps; c += S) {   // nsteps is a multiple of S
    step(c, integral_constant<int, 0>{}, integral_constant<int, S - 2>{}, std::true_type{});
    step(c + 1, integral_constant<int, 1>{}, integral_constant<int, S - 2>{}, std::true_type{});
    step(c + 2, integral_constant<int, 2>{}, integral_constant<int, S - 2>{}, std::true_type{});
    step(c + 3, integral_constant<int, 3>{}, integral_constant<int, S - 2>{}, std::true_type{});
  }
  // Residual: this lane's slices of h and gamma in the epilogue's layout
  // (token 8 k + lane / 8, 4 columns from 4 (lane % 8)), behind every ring load.
  const int qcol = 4 * (lane & 7), qrow = lane >> 3;
  f32x4 hv[EPI == kEpiResidual ? NT : 1][4];
  bf16x4 gv;
  if constexpr (EPI == kEpiResidual) {
    const int col = min(tile, n_rt - 1) * kGemmTile + qcol;
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        hv[n][k] = *(const f32x4 *)(g.h + (int64_t)min((tt0 + n) * kGemmTile + 8 * k + qrow, g.T - 1) * g.N + col);
    gv = *(const bf16x4 *)((g.x_out && g.gamma ? g.gamma : (const __bf16 *)g.h) + col);   // (unused without gamma)
    __builtin_amdgcn_sched_barrier(0);
  }
  step(0, integral_constant<int, 0>{}, integral_constant<int, 2>{}, std::false_type{});
  step(0, integral_constant<int, 1>{}, integral_constant<int, 1>{}, std::false_type{});
  step(0, integral_constant<int, 2>{}, integral_constant<int, 0>{}, std::false_type{});
  step(0, integral_constant<int, 3>{}, integral_constant<int, -1>{}, std::false_type{});

  // per token: RMSNorm factor (SwiGLU: / s_t, exact: a power of two) or s_t
  if constexpr (EPI == kEpiResidual) {
    if (threadIdx.x % TP == 0 && threadIdx.x / TP < NT * kGemmTile) tok_f[threadIdx.x / TP] = s_t;
  } else {
    float sum = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (spart + 4 * TP * u < g.n_ss) sum += (sv[u][0] + sv[u][1]) + (sv[u][2] + sv[u][3]);
    for (int i = spart + 16 * TP; i < g.n_ss; i += 4 * TP) {   // hidden > 512 TP
      const f32x4 v = *(const f32x4 *)(sr + i);
      sum += (v[0] + v[1]) + (v[2] + v[3]);
    }
#pragma unroll
    for (int off = 1; off < TP; off <<= 1) sum += __shfl_xor(sum, off);
    if (threadIdx.x % TP == 0 && threadIdx.x / TP < NT * kGemmTile) {
      const float inv = 1.0f / sqrtf(sum * g.inv_H + g.eps);
      tok_f[threadIdx.x / TP] = EPI == kEpiSwiGLU ? inv / s_t : inv;
      if constexpr (EPI == kEpiQKV) {
        tok_dest[threadIdx.x / TP] = dest;
        if (g.scale_out && slice == 0 && tt0 * kGemmTile + (int)threadIdx.x / TP < g.T) g.scale_out[st] = pow2_scale(inv);
      }
    }
  }
  ring_barrier();   // also: every wave is done with the ring; its LDS becomes scratch
  // A tile goes through the wave's scratch as [32 tokens][32 rows] (row pitch
  // 144 bytes), so that whole 64- and 128-byte runs of its output rows are
  // finished and stored at once.
  if (tile >= n_rt) return;   // (past the last barrier)
  unsigned char *sc = lds + wave * 4608;
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const int tt = tt0 + n;
    if (tt >= g.n_ttiles) break;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f32x4 v;
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = acc[n][4 * i + r];
      *(f32x4 *)(sc + frow * 144 + 32 * i + 16 * half) = v;
    }
    if constexpr (EPI == kEpiSwiGLU) {
      _Float16 *mrow = (_Float16 *)g.m_out + packed_offset(tt * kGemmTile + (lane >> 2), tile * 16 + 4 * (lane & 3), g.I);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int row = 16 * k + (lane >> 2), q = lane & 3, t = tt * kGemmTile + row;
        const f32x4 gt = *(const f32x4 *)(sc + row * 144 + 16 * q), up = *(const f32x4 *)(sc + row * 144 + 64 + 16 * q);
        const float f = tok_f[n * kGemmTile + row];
        f16x4 mv;
#pragma unroll
        for (int r = 0; r < 4; ++r) mv[r] = (_Float16)(t < g.T ? swiglu(gt[r] * f, up[r] * f) : 0.f);
        *(f16x4 *)(mrow + 128 * k) = mv;   // 16 rows on: 16 pieces of 8 elements further
      }
    } else {
      const int col = tile * kGemmTile + qcol;
      f32x4 v[4];
      float f[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        v[k] = *(const f32x4 *)(sc + (8 * k + qrow) * 144 + 4 * qcol);
        f[k] = tok_f[n * kGemmTile + 8 * k + qrow];
      }
      const int t0 = tt * kGemmTile + qrow;   // token of k: t0 + 8 k
      if constexpr (EPI == kEpiQKV) {
        // n_q and n_kv are multiples of 64: a tile is of q, k or v (a uniform branch)
        const bool is_q = tile * kGemmTile < g.n_q, is_k = tile * kGemmTile < g.n_q + g.n_kv;
        __bf16 *base = is_q ? g.q_out + col : is_k ? g.k_cache + (col - g.n_q) : g.v_cache + (col - g.n_q - g.n_kv);
        const int width = is_q ? g.n_q : g.n_kv;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          bf16x4 o;
#pragma unroll
          for (int r = 0; r < 4; ++r) o[r] = (__bf16)(v[k][r] * f[k]);
          const int t = t0 + 8 * k, row = is_q ? t : tok_dest[n * kGemmTile + 8 * k + qrow];
          if (t < g.T) *(bf16x4 *)(base + (int64_t)row * width) = o;
        }
      } else {
        float ss[4];
        float *hrow = g.h + (int64_t)t0 * g.N + col;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          v[k] += hv[n][k];
          ss[k] = fmaf(v[k][0], v[k][0], fmaf(v[k][1], v[k][1], fmaf(v[k][2], v[k][2], v[k][3] * v[k][3])));
          if (t0 + 8 * k < g.T) *(f32x4 *)(hrow + (int64_t)8 * k * g.N) = v[k];
        }
        if (g.x_out) {
          // 8 rows on: 8 pieces of 8 elements further within the packed tile
          __bf16 *xrow = g.x_out + packed_offset(t0, col, g.N);
          float *srow = g.ss_out + (int64_t)t0 * n_rt + tile;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int t = t0 + 8 * k;
            ss[k] = sum8(ss[k]);
            f32x4 xv;
#pragma unroll
            for (int r = 0; r < 4; ++r) xv[r] = v[k][r] * (g.gamma ? (float)gv[r] : 1.f) * f[k];
            bf16x4 o;   // bf16, or fp16 bits
            if (g.x_out_f16) {
              f16x4 oh;
#pragma unroll
              for (int r = 0; r < 4; ++r) oh[r] = (_Float16)xv[r];
              o = __builtin_bit_cast(bf16x4, oh);
            } else {
#pragma unroll
              for (int r = 0; r < 4; ++r) o[r] = (__bf16)xv[r];
            }
            if (t < g.T) {
              *(bf16x4 *)(xrow + 64 * k) = o;
              if ((lane & 7) == 0) srow[(int64_t)8 * k * n_rt] = ss[k];
            }
          }
        }
      }
    }
  }
}

template <int NT, bool F16, int EPI>
hipError_t launch_rows(const GemmArgs &g, int kind, hipStream_t stream) {
  const int64_t n = (int64_t)((g.N / kGemmTile + 3) / 4) * ((g.n_ttiles + NT - 1) / NT);
  launch(kind, gemm_rows_kernel<NT, F16, EPI>, dim3((unsigned)((n + 7) / 8 * 8)), dim3(256), stream, g);
  return hipGetLastError();
}

template <bool F16, int EPI>
hipError_t launch_nt(const GemmArgs &g, int kind, hipStream_t stream) {
  switch (g.wide) {
    case 1: return launch_rows<1, F16, EPI>(g, kind, stream);
    case 2: return launch_rows<2, F16, EPI>(g, kind, stream);
    case 4: return launch_rows<4, F16, EPI>(g, kind, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_gemm_rows(const GemmArgs &g, bool f16, int epi, int kind, hipStream_t stream) {
  // K: whole rings of 4 steps; buffer addressing of the activations is 32-bit
  if (!g.a_packed || g.K % 256 || (uint64_t)g.Tpad * g.K * 2 >= (1ull << 32)) return hipErrorInvalidValue;
  if (epi == kEpiSwiGLU) return launch_nt<true, kEpiSwiGLU>(g, kind, stream);
  if (epi == kEpiQKV) return launch_nt<false, kEpiQKV>(g, kind, stream);
  return f16 ? launch_nt<true, kEpiResidual>(g, kind, stream) : launch_nt<false, kEpiResidual>(g, kind, stream);
}

}  // namespace hpd
