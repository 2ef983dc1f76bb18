// Formation of B's operand straight from B (K x N, row-major) for calls of one
// scheme: the block sums' maxima, then their codes transposed on the way out.
// Such a call forms each block sum of B twice and is bound by reading B; a
// transposed copy of B, which an orbit makes once for hundreds of gauges,
// would cost it a read and a write of B more.  4096 x 14336 under two-level
// Strassen: transpose 137, maxima 52 and codes 77 us from the copy; from B
// itself maxima 84 and codes 85 us in place of all three.
#pragma once

#include "fm_device.h"

namespace fm {
namespace dev {

// Families whose operand blocks and running maxima fit in registers.
template <class P>
constexpr bool direct_family() {
  return P::NB <= 16 && P::R <= 64;
}

// Block sums of product r at one thread's VW positions: the fused
// multiply-adds of form_static_gauges, in its order.
template <class P, int VW, class C, int r>
__device__ __forceinline__ void direct_sum(const float (&xv)[P::NB][VW], C coef, int so,
                                           std::integral_constant<int, r>, float (&acc)[VW]) {
#pragma unroll
  for (int v = 0; v < VW; ++v) acc[v] = 0.0f;
  sfor<P::rowptr[r], P::rowptr[r + 1]>([&](auto ec) {
    constexpr int e = decltype(ec)::value;
    constexpr int b = P::idx[e];
    const float c = coef[e + so];
#pragma unroll
    for (int v = 0; v < VW; ++v) acc[v] = __builtin_fmaf(c, xv[b][v], acc[v]);
  });
}

// Maxima.  A workgroup takes 128 columns z of the blocks and a strip of rows
// k; a lane owns 2 columns and keeps every product's maximum over its rows in
// registers (per column for GRAN 1), so nothing crosses lanes until the strip
// ends; then LDS, then one atomic per maximum and strip.  GRAN: 0 one scale
// per tensor, 1 per column, 3 per 128 x 128 block (values rounded to bf16;
// strips lie within a block).  84 us for 4096 x 14336 under two-level Strassen
// (2.8 TB/s of B), 62 per column for 4096 x 11008.
template <class P, int GRAN>
__global__ __launch_bounds__(kThreads) void form_direct_max_kernel(FormArgs a,
                                                                   const float* __restrict__ B,
                                                                   int N, int strip) {
  constexpr int W = GRAN == 1 ? 2 : 1;  // maxima per product and lane
  constexpr int SLOTS = GRAN == 1 ? 128 : 16;
  __shared__ uint32_t smax[P::R * SLOTS];
  const int Nb = a.br, Kb = a.bc;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int z0 = blockIdx.x * 128, z = z0 + 2 * lane;
  const bool active = z < Nb;
  const int k0 = blockIdx.y * strip, k1 = min(Kb, k0 + strip);
  for (int i = threadIdx.x; i < P::R * SLOTS; i += kThreads) smax[i] = 0u;
  __syncthreads();
  const auto coef = ro(a.coef) + ro(a.off)[0];
  float mx[P::R][W];
#pragma unroll
  for (int r = 0; r < P::R; ++r)
#pragma unroll
    for (int w = 0; w < W; ++w) mx[r][w] = 0.0f;
  for (int k = k0 + 2 * wave; k < k1; k += 8) {
    float xv[P::NB][4];  // rows k, k + 1 of columns z, z + 1
#pragma unroll
    for (int b = 0; b < P::NB; ++b) {
      const int j = b / a.gc, l = b - (b / a.gc) * a.gc;
      const float* src = B + (size_t)(l * Kb + k) * N + (size_t)j * Nb + (active ? z : 0);
      const float2 t0 = *reinterpret_cast<const float2*>(src);
      const float2 t1 = *reinterpret_cast<const float2*>(src + N);
      xv[b][0] = t0.x, xv[b][1] = t0.y, xv[b][2] = t1.x, xv[b][3] = t1.y;
    }
    int so = 0;
    sfor<0, P::R>([&](auto rc) {
      constexpr int r = decltype(rc)::value;
      // (as in form_static_gauges: the coefficients are read group by group)
      if constexpr (r % 8 == 0) {
        so = 0;
        asm volatile("" : "+s"(so));
      }
      float acc[4];
      direct_sum<P, 4>(xv, coef, so, rc, acc);
      if constexpr (GRAN == 3) round_bf16<4>(acc);
      if constexpr (GRAN == 1) {
        mx[r][0] = __builtin_elementwise_maximum(mx[r][0], __builtin_fabsf(acc[0]));
        mx[r][1] = __builtin_elementwise_maximum(mx[r][1], __builtin_fabsf(acc[1]));
        mx[r][0] = __builtin_elementwise_maximum(mx[r][0], __builtin_fabsf(acc[2]));
        mx[r][1] = __builtin_elementwise_maximum(mx[r][1], __builtin_fabsf(acc[3]));
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          mx[r][0] = __builtin_elementwise_maximum(mx[r][0], __builtin_fabsf(acc[v]));
      }
    });
  }
  if (active) {
    sfor<0, P::R>([&](auto rc) {
      constexpr int r = decltype(rc)::value;
      if constexpr (GRAN == 1) {
        atomicMax(&smax[r * 128 + 2 * lane], __float_as_uint(mx[r][0]));
        atomicMax(&smax[r * 128 + 2 * lane + 1], __float_as_uint(mx[r][1]));
      } else {
        atomicMax(&smax[r * 16 + (lane & 15)], __float_as_uint(mx[r][0]));
      }
    });
  }
  __syncthreads();
  if constexpr (GRAN == 1) {
    for (int i = threadIdx.x; i < P::R * 128; i += kThreads) {
      const int r = i >> 7, zl = i & 127;
      if (z0 + zl < Nb && smax[i]) atomicMax(&a.amax[(size_t)r * Nb + z0 + zl], smax[i]);
    }
  } else {
    for (int r = threadIdx.x; r < P::R; r += kThreads) {
      uint32_t m = 0u;
#pragma unroll
      for (int t = 0; t < 16; ++t) m = max(m, smax[r * 16 + t]);
      const size_t at = GRAN == 0 ? (size_t)r
                                  : ((size_t)r * (Kb / 128) + k0 / 128) * (Nb / 128) + z0 / 128;
      if (m) atomicMax(&a.amax[at], m);
    }
  }
}

// Codes.  A workgroup takes 32 columns z x 64 rows k of the blocks; a thread
// owns one column and 4 rows, whose codes are one dword of the transposed
// tensor.  The dwords of a group of products meet in LDS (rows of 64 bytes,
// their 16-byte pieces XOR-swizzled by the column: 2-way conflicts on the
// writes, none on the reads) and leave as 16-byte stores; two LDS buffers, one
// barrier per group.  Workgroups with consecutive k are on one XCD, whose L2
// joins the halves of a 128-byte line.  85 us for 4096 x 14336 under two-level
// Strassen (235 MB read and 180 MB of codes written: 4.9 TB/s).
template <class P, int FMT, int GRAN>
__global__ __launch_bounds__(512, 4) void form_direct_quant_kernel(FormArgs a,
                                                                   const float* __restrict__ B,
                                                                   int N, int tiles_k) {
  constexpr int GR = P::R % 7 == 0 ? 7 : 8, NG = (P::R + GR - 1) / GR;
  __shared__ __attribute__((aligned(16))) uint32_t lds[2][GR][32 * 16];
  const int Nb = a.br, Kb = a.bc;
  int w = blockIdx.x;
  const int total = gridDim.x;
  if ((total & 7) == 0) w = (w & 7) * (total >> 3) + (w >> 3);
  const int tz = w / tiles_k, tk = w - tz * tiles_k;
  const int z0 = tz * 32, k0 = tk * 64;
  const int tid = threadIdx.x, zl = tid & 31, kq = tid >> 5;
  const int z = z0 + zl, k = k0 + 4 * kq;
  const bool active = z < Nb && k < Kb;  // (Kb is a multiple of 16)
  float xv[P::NB][4];
#pragma unroll
  for (int b = 0; b < P::NB; ++b) {
    const int j = b / a.gc, l = b - (b / a.gc) * a.gc;
    const float* src = B + (size_t)(l * Kb + (active ? k : 0)) * N + (size_t)j * Nb + (active ? z : 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) xv[b][i] = src[(size_t)i * N];
  }
  const auto coef = ro(a.coef) + ro(a.off)[0];
  const int wr = zl * 16 + ((((kq >> 2) ^ (zl >> 2)) & 3) << 2 | (kq & 3));
  sfor<0, NG>([&](auto gc) {
    constexpr int gi = decltype(gc)::value;
    int so = 0;
    asm volatile("" : "+s"(so));
    sfor<0, GR>([&](auto jc) {
      constexpr int j = decltype(jc)::value, r = gi * GR + j;
      if constexpr (r < P::R) {
        float acc[4];
        direct_sum<P, 4>(xv, coef, so, std::integral_constant<int, r>{}, acc);
        if constexpr (GRAN == 3) round_bf16<4>(acc);
        float q;
        if constexpr (GRAN == 0) q = ro(a.q)[r + so];
        else if constexpr (GRAN == 1) q = a.q[(size_t)r * Nb + (active ? z : 0)];
        else q = ro(a.q)[((size_t)(r + so) * (Kb / 128) + k0 / 128) * (Nb / 128) + z0 / 128];
        uint32_t c;
        if constexpr (FMT == FM_E4M3) {
          c = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(acc[0] * q, acc[1] * q, 0, false);
          c = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(acc[2] * q, acc[3] * q, (int)c, true);
        } else {
          c = (uint32_t)__builtin_amdgcn_cvt_pk_bf8_f32(acc[0] * q, acc[1] * q, 0, false);
          c = (uint32_t)__builtin_amdgcn_cvt_pk_bf8_f32(acc[2] * q, acc[3] * q, (int)c, true);
        }
        lds[gi & 1][j][wr] = c;
      }
    });
    // (the other buffer's reads, a group ago, are before this barrier)
    __syncthreads();
    constexpr int NJ = (gi * GR + GR <= P::R) ? GR : P::R - gi * GR;
#pragma unroll
    for (int i = 0; i < (NJ * 128 + 511) / 512; ++i) {
      const int p = tid + 512 * i;  // product, column and 16-byte piece
      const int j = p >> 7, zr = (p >> 2) & 31, pc = p & 3;
      if (j < NJ && z0 + zr < Nb && k0 + 16 * pc < Kb) {
        const uint4 v = *reinterpret_cast<const uint4*>(
            &lds[gi & 1][j][zr * 16 + ((pc ^ (zr >> 2)) & 3) * 4]);
        *reinterpret_cast<uint4*>(a.codes + ((size_t)(gi * GR + j) * Nb + z0 + zr) * Kb + k0 +
                                  16 * pc) = v;
      }
    }
  });
}

// Both passes of one scheme (a.G = 1, a as for B's transposed copy but for
// a.X) from B: 1, launching nothing, when the arguments do not fit (the
// caller then makes the copy).  mode -1 only asks.
template <class P>
int launch_form_direct(const FormArgs& a, const float* B, int mode, hipStream_t st) {
  if constexpr (!direct_family<P>()) {
    return 1;
  } else {
    const int Nb = a.br, Kb = a.bc, N = a.rows;
    // 2 columns per 8-byte load, 16-byte code stores; whole blocks of scales
    if (a.G != 1 || a.R != P::R || a.gr * a.gc != P::NB || Kb % 16 || Nb % 2 || N % 2 ||
        ((uintptr_t)B & 7u) || ((uintptr_t)a.codes & 15u) ||
        (a.per_row && a.gran == 3 && (Kb % 128 || Nb % 128)))
      return 1;
    const long long tz = (Nb + 31) / 32, tk = (Kb + 63) / 64;
    // strips of at most 128 rows for the maxima, shorter while the launch has
    // less than 1024 workgroups (but 16 rows: four per wave)
    int strip = 128;
    const int nz = (Nb + 127) / 128;
    while (strip > 16 && (long long)nz * ((Kb + strip - 1) / strip) < 1024) strip /= 2;
    const int strips = (Kb + strip - 1) / strip;
    // a grid holds 65535 workgroups along y and fewer than 2^32 threads along x
    if (strips > 65535 || tz * tk >= (1LL << 32) / 512) return 1;
    if (mode < 0) return FM_OK;
    const int gran = a.per_row ? a.gran : 0;
    if (mode == 0) {
      const dim3 grid(nz, strips);
      if (gran == 0) form_direct_max_kernel<P, 0><<<grid, kThreads, 0, st>>>(a, B, N, strip);
      else if (gran == 1) form_direct_max_kernel<P, 1><<<grid, kThreads, 0, st>>>(a, B, N, strip);
      else form_direct_max_kernel<P, 3><<<grid, kThreads, 0, st>>>(a, B, N, strip);
      return launched("form_direct_max_kernel");
    }
    const unsigned grid = (unsigned)(tz * tk);
    auto go = [&](auto fc) {
      constexpr int F = decltype(fc)::value;
      if (gran == 0) form_direct_quant_kernel<P, F, 0><<<grid, 512, 0, st>>>(a, B, N, (int)tk);
      else if (gran == 1) form_direct_quant_kernel<P, F, 1><<<grid, 512, 0, st>>>(a, B, N, (int)tk);
      else form_direct_quant_kernel<P, F, 3><<<grid, 512, 0, st>>>(a, B, N, (int)tk);
    };
    if (a.fmt == FM_E4M3) go(std::integral_constant<int, FM_E4M3>{});
    else go(std::integral_constant<int, FM_E5M2>{});
    return launched("form_direct_quant_kernel");
  }
}

}  // namespace dev

#define FM_DECLARE_DIRECT(P) \
  int form_direct_family_##P(const FormArgs& a, const float* B, int mode, hipStream_t st);
FM_PATTERN_FAMILIES(FM_DECLARE_DIRECT)
#undef FM_DECLARE_DIRECT

#define FM_DEFINE_DIRECT(P)                                                                  \
  int form_direct_family_##P(const FormArgs& a, const float* B, int mode, hipStream_t st) {  \
    return dev::launch_form_direct<pat::P::B>(a, B, mode, st);                               \
  }

}  // namespace fm
