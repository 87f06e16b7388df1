// Device code shared by the projection kernels: operand types, the epilogues
// and the direct global -> LDS copies.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "gemm.h"

namespace hpd {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// ------------------------------------------------------------ GEMM

// 8 bf16 -> 8 fp16 (round to nearest even; exact for |w| >= 2^-14).
__device__ __forceinline__ u32x4 bf16x8_to_f16x8(u32x4 v) {
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float lo = __uint_as_float(v[i] << 16), hi = __uint_as_float(v[i] & 0xffff0000u);
    const _Float16 l16 = (_Float16)lo, h16 = (_Float16)hi;
    r[i] = (unsigned)__builtin_bit_cast(unsigned short, l16) | ((unsigned)__builtin_bit_cast(unsigned short, h16) << 16);
  }
  return r;
}

// Epilogue operands of a tile.  The token's cache row (QKV, plan data) and
// scale are loaded before the main loop; the residual row slice, the next
// norm's weights and the per-token sums of squares after the loads of the
// first pipeline steps (packed kernel, load_pre) or after the loop.
constexpr int kSsPrefetch = 32;   // sums of squares per token held in registers (hidden <= 1024)
struct EpilogueIn {
  f32x4 h[4], gamma[4];   // residual: h row slice and gamma (ones if none)
  f32x4 ss[kSsPrefetch / 4];   // QKV, SwiGLU: the token's sums of squares (load_pre)
  int dest;               // QKV: private cache row of the token
  float inv_rms;          // QKV, SwiGLU: RMSNorm factor of the token
  float scale;            // residual, SwiGLU: s_t of the fp16 norm input (scale_in), else 1
};

// Loaded before the main loop: plan data and the per-token scale, which were
// written at least two launches earlier.
template <int EPI>
__device__ __forceinline__ void load_early(const GemmArgs &g, int t, EpilogueIn &in) {
  if constexpr (EPI == kEpiQKV) in.dest = t < g.T ? g.dest[t] : 0;
  else in.scale = g.scale_in ? g.scale_in[min(t, g.T - 1)] : 1.f;
}

template <int EPI>
__device__ __forceinline__ void load_late(const GemmArgs &g, int t, int tile, int half, EpilogueIn &in) {
  if constexpr (EPI == kEpiResidual) {
    const float *hr = g.h + (int64_t)min(t, g.T - 1) * g.N + tile * kGemmTile + 4 * half;
#pragma unroll
    for (int i = 0; i < 4; ++i) in.h[i] = *(const f32x4 *)(hr + 8 * i);
    if (g.x_out && g.gamma) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bf16x4 gv = *(const bf16x4 *)(g.gamma + tile * kGemmTile + 8 * i + 4 * half);
        in.gamma[i] = f32x4{(float)gv[0], (float)gv[1], (float)gv[2], (float)gv[3]};
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) in.gamma[i] = f32x4{1.f, 1.f, 1.f, 1.f};
    }
  } else {
    // per-token RMSNorm factor from the partial sums of squares
    const float *sr = g.ss_in + (int64_t)t * g.n_ss;
    float sum = 0.f;
    for (int i = 0; i < g.n_ss; i += 4) {
      const f32x4 v = *(const f32x4 *)(sr + i);
      sum += (v[0] + v[1]) + (v[2] + v[3]);
    }
    in.inv_rms = 1.0f / sqrtf(sum * g.inv_H + g.eps);
  }
}

// The packed kernel's epilogue loads, split around its main loop: load_pre
// issues them right after the loads of the first pipeline steps, so that the
// waits for those steps do not cover them and their latency overlaps the
// loop; load_post reduces them.  (Issued before the first steps' loads they
// delayed the loop: loads retire in order.)  Every buffer they read was
// written at least two launches earlier (h by the residual projection
// before the previous kernel, the sums of squares and gamma earlier still).
// Sums of squares beyond kSsPrefetch values per token are loaded late.
template <int EPI>
__device__ __forceinline__ void load_pre(const GemmArgs &g, int t, int tile, int half, EpilogueIn &in) {
  if constexpr (EPI == kEpiResidual) {
    load_late<EPI>(g, t, tile, half, in);
  } else if (g.n_ss <= kSsPrefetch) {
    const float *sr = g.ss_in + (int64_t)t * g.n_ss;
    // unconditional loads (an index past the row repeats its last four
    // values, unused): a load under a condition would be followed by a wait
#pragma unroll
    for (int i = 0; i < kSsPrefetch / 4; ++i) in.ss[i] = *(const f32x4 *)(sr + min(4 * i, g.n_ss - 4));
  }
}
template <int EPI>
__device__ __forceinline__ void load_post(const GemmArgs &g, int t, int tile, int half, EpilogueIn &in) {
  if constexpr (EPI != kEpiResidual) {
    if (g.n_ss <= kSsPrefetch) {   // the sum in load_late's order
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < kSsPrefetch / 4; ++i)
        if (4 * i < g.n_ss) sum += (in.ss[i][0] + in.ss[i][1]) + (in.ss[i][2] + in.ss[i][3]);
      in.inv_rms = 1.0f / sqrtf(sum * g.inv_H + g.eps);
    } else {
      load_late<EPI>(g, t, tile, half, in);
    }
  }
}

// SwiGLU of one gate / up pair, the same in every kernel.
__device__ __forceinline__ float swiglu(float gate, float up) { return gate / (1.0f + __expf(-gate)) * up; }

// Writes the finished 32 x 32 tile `tile` for token t (this lane: rows
// 8 (r / 4) + 4 half + r % 4 of the tile, see below) through epilogue EPI.
template <int EPI>
__device__ __forceinline__ void epilogue(const GemmArgs &g, const f32x16 &acc, EpilogueIn &in, int t, int tile,
                                         int half) {
  if constexpr (EPI == kEpiResidual) {
    // h += Y; x_out = h * gamma (the next norm's input, unnormalised) and the
    // sum of squares of h over this 32-column tile
    if (t >= g.T) return;
    float *hr = g.h + (int64_t)t * g.N + tile * kGemmTile + 4 * half;
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        in.h[i][r] += acc[4 * i + r];
        ss = fmaf(in.h[i][r], in.h[i][r], ss);
      }
      *(f32x4 *)(hr + 8 * i) = in.h[i];
    }
    if (!g.x_out) return;
    ss += __shfl_xor(ss, 32);
    if (half == 0) g.ss_out[(int64_t)t * (g.N / kGemmTile) + tile] = ss;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int n = tile * kGemmTile + 8 * i + 4 * half;
      const f32x4 v = in.h[i] * in.gamma[i] * in.scale;
      const int64_t off = g.act_packed ? packed_offset(t, n, g.N) : (int64_t)t * g.N + n;
      if (g.x_out_f16) {
        f16x4 o;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = (_Float16)v[r];
        *(f16x4 *)((_Float16 *)g.x_out + off) = o;
      } else {
        bf16x4 o;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = (__bf16)v[r];
        *(bf16x4 *)(g.x_out + off) = o;
      }
    }
  } else {
    const float inv_rms = in.inv_rms;
    if constexpr (EPI == kEpiQKV) {
      if (t >= g.T) return;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int n = tile * kGemmTile + 8 * i + 4 * half;   // 4-runs never straddle q / k / v
        bf16x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = (__bf16)(acc[4 * i + r] * inv_rms);
        if (n < g.n_q) *(bf16x4 *)(g.q_out + (int64_t)t * g.n_q + n) = v;
        else if (n < g.n_q + g.n_kv) *(bf16x4 *)(g.k_cache + (int64_t)in.dest * g.n_kv + (n - g.n_q)) = v;
        else *(bf16x4 *)(g.v_cache + (int64_t)in.dest * g.n_kv + (n - g.n_q - g.n_kv)) = v;
      }
      if (g.scale_out && tile == 0 && half == 0) g.scale_out[t] = pow2_scale(inv_rms);
    } else {   // SwiGLU: m = silu(gate) * up, fp16; rows t >= T are written as zeros
      const float f = inv_rms / in.scale;   // exact: s_t is a power of two
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        f16x4 mv;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          mv[r] = (_Float16)(t < g.T ? swiglu(acc[4 * i + r] * f, acc[4 * i + 8 + r] * f) : 0.f);
        }
        const int col = tile * 16 + 8 * i + 4 * half;
        const int64_t off = g.act_packed ? packed_offset(t, col, g.I) : (int64_t)t * g.I + col;
        *(f16x4 *)((_Float16 *)g.m_out + off) = mv;
      }
    }
  }
}

// LDS rows are 128 bytes (64 K values); 16-byte piece q of row r is stored at
// piece q ^ ((r >> 1) & 7), so the 16 lanes of one LDS cycle (16 consecutive
// rows, same logical piece) cover all 64 banks.
__device__ __forceinline__ int swz(int row, int q) { return q ^ ((row >> 1) & 7); }

// Direct global -> LDS copy of 16 bytes per lane: lane i of the wave writes
// lds_base + 16 i (the LDS address must be wave-uniform).
__device__ __forceinline__ void dma16(const void *src, void *lds_base) {
  __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)lds_base, 16, 0, 0);
}

// Direct global -> LDS copy of 16 bytes per lane in its buffer form.  With
// the flat form (global_load_lds) in flight the compiler waits for every
// outstanding LDS read (lgkmcnt(0)) before the first use of any of them; with
// this one it counts them, so the next fragments can be read under the MFMAs.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void *p, uint64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (int)(unsigned)bytes, 0x00027000);
}
__device__ __forceinline__ void bdma16(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, void *lds_base) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)lds_base, 16, voff, soff, 0, 0);
}

// s_waitcnt vmcnt(n) with expcnt and lgkmcnt left free.
template <int N> __device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// Workgroup barrier of the LDS ring: completes this wave's LDS reads but not
// its in-flight global -> LDS copies (those are waited for by count).
__device__ __forceinline__ void ring_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace
}  // namespace hpd
