// Batched FP8 block products of libfm for CDNA4 (gfx950), wave64:
// M_r = (sum_k Tq_r[x,k] Sq_r[z,k]) * dT_r * dS_r for a batch of products
// (the block products of eq. (1); Sec. 2.1 and the FP8 schedule of App. B.1).
//
//  gemm_dma_kernel   persistent, 256 x 128 tiles, a 3-stage LDS ring filled
//                    by direct global-to-LDS loads; inner lengths that are
//                    multiples of 128.
//  gemm_small_kernel one 32 x 32 tile per wave; products of at most 64 x 64
//                    with few bytes to load (small_products).
//  gemm_tile_kernel  one 128 x 128 tile per workgroup, double-buffered LDS;
//                    any inner length that is a multiple of 16.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>

#include "fm_device.h"
#include "fm_lds_ring.h"

namespace fm {
namespace {
using namespace dev;
using namespace ring;

// ------------------------------------------------------ FP8 block GEMM
// Workgroup tile 128 x 128, K step 128 bytes, 4 waves in 2 x 2, each wave
// 64 x 64 = 4 x 4 tiles of 16 x 16.  FP8 operands are staged through
// double-buffered LDS, rows of 128 bytes with the 16-byte chunk index
// XOR-swizzled by a function of the row so that the fragment reads (16 rows
// x one chunk per instruction) hit distinct banks.
//
// Lane (i, q) = (lane % 16, lane / 16) of a wave holds the 32 bytes
// [32q, 32q + 32) of row i of a 16-row fragment, for both operands, so every
// k of the step is paired with the same k of the other operand.
//
// Two arithmetics for the products:
//   ACC_BF16 (default): every FP8 value is widened exactly to bf16
//     (v_cvt_scalef32_pk_bf16_{fp8,bf8}, scale 1) and multiplied on the bf16
//     matrix cores, v_mfma_f32_16x16x32_bf16: exact products, fp32 sums.
//   ACC_FP8: v_mfma_scale_f32_16x16x128_f8f6f4 with unit scales, twice the
//     rate; its sums of small products beside large ones are truncated
//     (about 5e-5 relative on random FP8 data), so it is not the default.
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));

constexpr int GT = 128;  // tile rows / cols

// Two FP8 codes (bytes 0-1 or 2-3 of w) -> two bf16 values, exactly.
template <int FMT, bool HI>
__device__ __forceinline__ v2bf widen2(int w) {
  if constexpr (FMT == FM_E4M3) return __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, HI);
  else return __builtin_amdgcn_cvt_scalef32_pk_bf16_bf8(w, 1.0f, HI);
}

// 8 FP8 codes (two dwords, little-endian byte order) -> 8 bf16 values
template <int FMT>
__device__ __forceinline__ v8bf widen8(int d0, int d1) {
  const v2bf a = widen2<FMT, false>(d0), b = widen2<FMT, true>(d0);
  const v2bf c = widen2<FMT, false>(d1), d = widen2<FMT, true>(d1);
  return (v8bf){a[0], a[1], b[0], b[1], c[0], c[1], d[0], d[1]};
}

// Scales of the epilogue: SC = 0 one scale per product (dT[b], dS[b]);
// SC = 1 one per row of Tq_b (dT[b * Mb + x]) and per row of Sq_b, i.e. per
// column of the product (dS[b * Nb + z]).  Either way M = (acc * dT) * dS.

// Non-persistent variant: one 128 x 128 tile per workgroup, 4 waves.
template <int FMT, int ACC, int SC>
__global__ __launch_bounds__(kThreads) void gemm_tile_kernel(const uint8_t* __restrict__ Tq,
                                                            const uint8_t* __restrict__ Sq,
                                                            const float* __restrict__ dT,
                                                            const float* __restrict__ dS,
                                                            float* __restrict__ Mout, int Mb,
                                                            int Nb, int Kb, int tiles_m,
                                                            int tiles_n, int total) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[2][2][GT * GK];
  // Workgroups are dispatched round-robin over the 8 XCDs; remap so that
  // each XCD works through a contiguous range of tiles (whole products),
  // keeping a product's operand panels in one L2.
  int w = blockIdx.x;
  if ((total & 7) == 0) w = (w & 7) * (total >> 3) + (w >> 3);
  const int tiles = tiles_m * tiles_n;
  const int b = w / tiles;
  const int t = w - b * tiles;
  const int tm = t / tiles_n, tn = t - (t / tiles_n) * tiles_n;
  const int m0 = tm * GT, n0 = tn * GT;
  const uint8_t* Ab = Tq + (size_t)b * Mb * Kb;
  const uint8_t* Bb = Sq + (size_t)b * Nb * Kb;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;

  uint4 ra[4], rb[4];
  auto gload = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = tid + kThreads * i;
      const int row = c >> 3, ch = c & 7;
      const int kk = k0 + ch * 16;
      ra[i] = make_uint4(0, 0, 0, 0);
      rb[i] = make_uint4(0, 0, 0, 0);
      if (kk < Kb) {
        if (m0 + row < Mb) ra[i] = *reinterpret_cast<const uint4*>(Ab + (size_t)(m0 + row) * Kb + kk);
        if (n0 + row < Nb) rb[i] = *reinterpret_cast<const uint4*>(Bb + (size_t)(n0 + row) * Kb + kk);
      }
    }
  };
  auto lstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = tid + kThreads * i;
      const int row = c >> 3, ch = c & 7;
      const int o = row * GK + ((ch ^ swz(row)) << 4);
      *reinterpret_cast<uint4*>(&lds[buf][0][o]) = ra[i];
      *reinterpret_cast<uint4*>(&lds[buf][1][o]) = rb[i];
    }
  };

  v4f acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};

  const int nk = (Kb + GK - 1) / GK;
  gload(0);
  lstore(0);
  __syncthreads();
  const int q = lane >> 4, l16 = lane & 15;
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < nk) gload((kt + 1) * GK);
    v8i fa[4], fb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = wm * 64 + i * 16 + l16;
      const uint8_t* base = &lds[cur][0][row * GK];
      const uint4 lo = *reinterpret_cast<const uint4*>(base + (((2 * q) ^ swz(row)) << 4));
      const uint4 hi = *reinterpret_cast<const uint4*>(base + (((2 * q + 1) ^ swz(row)) << 4));
      fa[i] = (v8i){(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = wn * 64 + j * 16 + l16;
      const uint8_t* base = &lds[cur][1][row * GK];
      const uint4 lo = *reinterpret_cast<const uint4*>(base + (((2 * q) ^ swz(row)) << 4));
      const uint4 hi = *reinterpret_cast<const uint4*>(base + (((2 * q + 1) ^ swz(row)) << 4));
      fb[j] = (v8i){(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
    }
    if constexpr (ACC == 1) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fa[i], fb[j], acc[i][j], FMT,
                                                                       FMT, 0, 127, 0, 127);
    } else {
#pragma unroll
      for (int sub = 0; sub < 4; ++sub) {
        v8bf wa[4], wb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) wa[i] = widen8<FMT>(fa[i][2 * sub], fa[i][2 * sub + 1]);
#pragma unroll
        for (int j = 0; j < 4; ++j) wb[j] = widen8<FMT>(fb[j][2 * sub], fb[j][2 * sub + 1]);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[i], wb[j], acc[i][j], 0, 0, 0);
      }
    }
    if (kt + 1 < nk) lstore(cur ^ 1);
    __syncthreads();
  }

  float* Mo = Mout + (size_t)b * Mb * Nb;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int col = n0 + wn * 64 + j * 16 + l16;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = m0 + wm * 64 + i * 16 + 4 * q + v;
        if (row < Mb && col < Nb) {
          const float sT = SC ? dT[(size_t)b * Mb + row] : dT[b];
          const float sS = SC ? dS[(size_t)b * Nb + col] : dS[b];
          float m = acc[i][j][v] * sT;
          m = m * sS;
          Mo[(size_t)row * Nb + col] = m;
        }
      }
    }
}

// Small products (at most 64 x 64; bf16 arithmetic): a wave per 32 x 32 tile,
// its operand rows loaded straight into fragments.  Lane (r, h) = (lane % 32,
// lane / 32) takes bytes [16 h, 16 h + 16) of row r per 32 of the inner
// dimension, for both operands alike.  Such products are bound by launch and
// memory, not by the matrix cores: a 128 x 128 tile would be mostly padding
// (512 gauges of 49 products of 32 x 32 x 32: 282 us against 40).
template <int FMT, int SC>
__global__ __launch_bounds__(kThreads) void gemm_small_kernel(const uint8_t* __restrict__ Tq,
                                                             const uint8_t* __restrict__ Sq,
                                                             const float* __restrict__ dT,
                                                             const float* __restrict__ dS,
                                                             float* __restrict__ Mout, int Mb,
                                                             int Nb, int Kb, int tiles_m,
                                                             int tiles_n, long long total) {
  typedef float acc16 __attribute__((ext_vector_type(16)));
  const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
  const long long blk = (long long)blockIdx.y * gridDim.x + blockIdx.x;
  const long long w = blk * (kThreads / 64) + (threadIdx.x >> 6);
  if (w >= total) return;
  const int tiles = tiles_m * tiles_n;
  const long long b = w / tiles;
  const int t = (int)(w - b * tiles);
  const int m0 = t / tiles_n * 32, n0 = (t - t / tiles_n * tiles_n) * 32;
  // rows beyond the operand read row 0: they only feed outputs never stored
  const int ar = m0 + r < Mb ? m0 + r : 0, br = n0 + r < Nb ? n0 + r : 0;
  const uint8_t* pa = Tq + ((size_t)b * Mb + ar) * Kb + 16 * h;
  const uint8_t* pb = Sq + ((size_t)b * Nb + br) * Kb + 16 * h;
  acc16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
#pragma unroll 4
  for (int k = 0; k < Kb; k += 32) {
    uint4 a = make_uint4(0, 0, 0, 0), c = a;
    if (k + 16 * h < Kb) {
      a = *reinterpret_cast<const uint4*>(pa + k);
      c = *reinterpret_cast<const uint4*>(pb + k);
    }
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(widen8<FMT>((int)c.x, (int)c.y),
                                                  widen8<FMT>((int)a.x, (int)a.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(widen8<FMT>((int)c.z, (int)c.w),
                                                  widen8<FMT>((int)a.z, (int)a.w), acc, 0, 0, 0);
  }
  // element v of lane (r, h): row r, column 8 (v / 4) + 4 h + v % 4
  const int row = m0 + r;
  if (row >= Mb) return;
  const float sT = SC ? dT[(size_t)b * Mb + row] : dT[b];
  float* out = Mout + ((size_t)b * Mb + row) * Nb;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int col = n0 + 8 * g + 4 * h;
    float o[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float sS = SC ? dS[(size_t)b * Nb + (col + v < Nb ? col + v : 0)] : dS[b];
      o[v] = (acc[4 * g + v] * sT) * sS;
    }
    if ((Nb & 3) == 0) {
      if (col < Nb) *reinterpret_cast<float4*>(out + col) = make_float4(o[0], o[1], o[2], o[3]);
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (col + v < Nb) out[col + v] = o[v];
    }
  }
}

// Pipelined persistent kernel (inner block length a multiple of 128):
// workgroup tile 256 x 128, 8 waves of 64 x 64 (4 x 2), K step 128 bytes, a
// ring of 3 LDS stages of 48 KB filled by direct global-to-LDS loads
// (global_load_lds_dwordx4: lane L of a wave writes the 16 bytes it fetched
// at M0 + 16 L, so the XOR swizzle is applied by choosing each lane's source
// chunk).  Each workgroup walks a flattened sequence of (tile, K-step) pairs
// with two pairs in flight while it computes a third, so the next tile's
// loads run under the current tile's epilogue.  Rows beyond the operand
// (ragged M or N) read row 0 instead: they only feed outputs never stored.
//
// SW: the tile is 128 x 256, its 256 side along the columns, for products
// whose rows would leave half of a 256-row tile empty.
//
// The ring, its direct loads and their vmcnt accounting are in
// fm_lds_ring.h.  The products are accumulated transposed (operands swapped
// in the MFMA) so that each lane holds 4 consecutive output columns and the
// epilogue writes 16-byte stores.
template <int FMT, int ACC, int SC, bool OB, bool SW>
__global__ __launch_bounds__(DNT) void gemm_dma_kernel(const uint8_t* __restrict__ Tq,
                                                       const uint8_t* __restrict__ Sq,
                                                       const float* __restrict__ dT,
                                                       const float* __restrict__ dS,
                                                       float* __restrict__ Mout, int Mb, int Nb,
                                                       int Kb, int tiles_m, int tiles_n, int total,
                                                       int tiled) {
  // SC = 2 (group scales): every K step is one group of 128; its scales ride
  // the ring in a 2 KB slot after the stage (dT of the tile's 256 rows, then
  // the tile's one dS)
  constexpr int STG = SC == 2 ? DSTAGE + 2048 : DSTAGE;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[DNS * STG];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int q = lane >> 4, l16 = lane & 15;
  const int tiles = tiles_m * tiles_n;
  const int nk = Kb / GK;
  // the operands of the tile's 256 and 128 sides (rows Ra and Rb)
  const uint8_t* Pa = SW ? Sq : Tq;
  const uint8_t* Pb = SW ? Tq : Sq;
  const int Ra = SW ? Nb : Mb, Rb = SW ? Mb : Nb;
  const bool vec_store = (Nb & 3) == 0;

  const int G = gridDim.x;
  // (XCD x takes tiles [x per, (x + 1) per), per = ceil(total / 8))
  const bool xcd_split = (G & 7) == 0;
  const int per = (total + 7) >> 3;
  const int t = xcd_split ? (blockIdx.x & 7) * per + (blockIdx.x >> 3) : blockIdx.x;
  const int tstep = xcd_split ? (G >> 3) : G;
  const int t_end = xcd_split ? min(total, ((blockIdx.x & 7) + 1) * per) : total;
  if (t >= t_end) return;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;

  auto issue = [&](int tile, int kt, int buf) {
    const int b = tile / tiles, tt = tile - b * tiles;
    const int tmi = tt / tiles_n;
    const int m0 = tmi * DBM, n0 = (tt - tmi * tiles_n) * DBN;
    const uint8_t* Ab = Pa + (size_t)b * Ra * Kb + (size_t)kt * GK;
    const uint8_t* Bb = Pb + (size_t)b * Rb * Kb + (size_t)kt * GK;
#pragma unroll
    for (int j = 0; j < DLOADS; ++j) {
      const int r0 = (wave * DLOADS + j) * 8;  // first of the 8 rows this wave-load fills
      const int r = r0 + (lane >> 3);
      const int ch = (lane & 7) ^ swz(r);
      const uint8_t* src;
      if (r0 < DBM) {  // uniform: a wave-load never straddles the A/B boundary
        int row = m0 + r;
        row = row < Ra ? row : 0;
        src = Ab + (size_t)row * Kb + ch * 16;
      } else {
        int row = n0 + r - DBM;
        row = row < Rb ? row : 0;
        src = Bb + (size_t)row * Kb + ch * 16;
      }
      dma16(src, lds_base + (uint32_t)(buf * STG + r0 * GK));
    }
    if constexpr (SC == 2) {
      // wave 0: dT[b][kt] of the tile's rows, 4 per lane (Mb a multiple of
      // 4; with SW lanes 32-63 repeat 0-31); wave 1: the 16-byte-aligned
      // chunk holding the tile's dS[b][kt][column / 128], with SW lane 1 the
      // one of its second 128 columns (the scale arrays are padded to whole
      // chunks)
      if (wave < 2) {
        const size_t grp = (size_t)b * nk + kt;
        const float* src;
        if (wave == 0) {
          const int row = SW ? n0 + 4 * (lane & 31) : m0 + 4 * lane;
          src = dT + grp * Mb + (row < Mb ? row : 0);
        } else {
          const size_t blk = grp * (Nb / 128) + (SW ? m0 : n0) / 128;
          const bool second = SW && lane == 1 && m0 + 128 < Nb;
          src = dS + ((blk + (second ? 1 : 0)) & ~(size_t)3);
        }
        dma16(src, lds_base + (uint32_t)(buf * STG + DSTAGE + wave * 1024));
      }
    }
  };
  // Half h of a K step: lane (l16, q) of fragment i holds bytes
  // [32q + 16h, 32q + 16h + 16) of its row, i.e. the k values of two 16x16x32
  // sub-steps (2h and 2h + 1).
  uint4 fa[2][4], fb[2][4];
  auto read_half = [&](int h, int buf) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = wm * 64 + i * 16 + l16;
      fa[h][i] = *reinterpret_cast<const uint4*>(lds + buf * STG + row * GK +
                                                 (((2 * q + h) ^ swz(row)) << 4));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = DBM + wn * 64 + j * 16 + l16;
      fb[h][j] = *reinterpret_cast<const uint4*>(lds + buf * STG + row * GK +
                                                 (((2 * q + h) ^ swz(row)) << 4));
    }
  };

  v4f acc[4][4];
  v4f ofl[4][4];  // SC = 2: the fp32 sum over the groups so far
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
      ofl[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
    }
  // SC = 2: the step's scales, read from its ring slot before the barrier
  float gs[4];
  auto read_scales = [&](int buf, int tile, int kt) {
    const float* sA = reinterpret_cast<const float*>(lds + buf * STG + DSTAGE);
    const float* sB = reinterpret_cast<const float*>(lds + buf * STG + DSTAGE + 1024);
    const int b = tile / tiles, tt = tile - b * tiles;
    const int tmi = tt / tiles_n;
    const size_t grp = ((size_t)b * nk + kt) * (Nb / 128);
    if constexpr (SW) {
      const int half = (tmi * DBM + 128 < Nb) ? wm >> 1 : 0;
      const float ds = sB[4 * half + (int)((grp + tmi * (DBM / 128) + half) & 3)];
#pragma unroll
      for (int j = 0; j < 4; ++j) gs[j] = sA[wn * 64 + j * 16 + l16] * ds;
    } else {
      const float ds = sB[(grp + (tt - tmi * tiles_n)) & 3];
#pragma unroll
      for (int i = 0; i < 4; ++i) gs[i] = sA[wm * 64 + i * 16 + l16] * ds;
    }
  };
  // out = fmaf(group sum, dT dS, out), then the next group starts from zero
  auto rescale = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          ofl[i][j][v] = __builtin_fmaf(acc[i][j][v], gs[SW ? j : i], ofl[i][j][v]);
        acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
      }
  };

  // acc[i][j] holds the transposed 16 x 16 product: element (4q+v, l16) is
  // output row i*16 + l16, column j*16 + 4q + v of the wave's 64 x 64 block;
  // with SW (columns on the 256 side) the operands are the other way round,
  // and it is output row j*16 + l16, column i*16 + 4q + v
  auto compute_half = [&](int h) {
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      if constexpr (ACC == 1) {
        long xa[4], xb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          xa[i] = sub ? (long)(((unsigned long)(uint32_t)fa[h][i].w << 32) | (uint32_t)fa[h][i].z)
                      : (long)(((unsigned long)(uint32_t)fa[h][i].y << 32) | (uint32_t)fa[h][i].x);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          xb[j] = sub ? (long)(((unsigned long)(uint32_t)fb[h][j].w << 32) | (uint32_t)fb[h][j].z)
                      : (long)(((unsigned long)(uint32_t)fb[h][j].y << 32) | (uint32_t)fb[h][j].x);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if constexpr (FMT == FM_E4M3)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(SW ? xa[i] : xb[j], SW ? xb[j] : xa[i], acc[i][j], 0, 0, 0);
            else
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf8_bf8(SW ? xa[i] : xb[j], SW ? xb[j] : xa[i], acc[i][j], 0, 0, 0);
          }
      } else {
        v8bf wa[4], wb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          wa[i] = sub ? widen8<FMT>((int)fa[h][i].z, (int)fa[h][i].w) : widen8<FMT>((int)fa[h][i].x, (int)fa[h][i].y);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          wb[j] = sub ? widen8<FMT>((int)fb[h][j].z, (int)fb[h][j].w) : widen8<FMT>((int)fb[h][j].x, (int)fb[h][j].y);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(SW ? wa[i] : wb[j], SW ? wb[j] : wa[i], acc[i][j], 0, 0, 0);
      }
    }
  };
  // this lane's output row and first of 4 columns of acc[i][j], from the
  // tile's origin
  const int rl = (SW ? wn : wm) * 64 + l16, cl = (SW ? wm : wn) * 64 + 4 * q;
  auto row_of = [&](int i, int j) { return rl + (SW ? j : i) * 16; };
  auto col_of = [&](int i, int j) { return cl + (SW ? i : j) * 16; };
  auto epilogue = [&](int tile) -> int {  // returns the number of stores counted
    const int b = tile / tiles, tt = tile - b * tiles;
    const int tmi = tt / tiles_n;
    const int a0 = tmi * DBM, b0 = (tt - tmi * tiles_n) * DBN;
    const int r0 = SW ? b0 : a0, c0 = SW ? a0 : b0;
    const bool whole = a0 + DBM <= Ra && b0 + DBN <= Rb;
    float* Mo = Mout + (size_t)b * Mb * Nb;
    if constexpr (SC == 2) {
      // products returned in bf16 (nearest even), held as fp32
      auto bf = [](float x) {
        const uint32_t u = __float_as_uint(x);
        return __uint_as_float((u + 0x7fffu + ((u >> 16) & 1u)) & 0xffff0000u);
      };
      // OB: stored as bf16 (the values' high halves, 8-byte stores)
      uint16_t* Mh = reinterpret_cast<uint16_t*>(Mout) + (size_t)b * Mb * Nb;
      auto hi = [](float x) { return __float_as_uint(x) >> 16; };
      // (columns are whole 128s, so 4 of them are in or out together)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int row = r0 + row_of(i, j), col = c0 + col_of(i, j);
          const float v0 = bf(ofl[i][j][0]), v1 = bf(ofl[i][j][1]);
          const float v2 = bf(ofl[i][j][2]), v3 = bf(ofl[i][j][3]);
          if (whole || (row < Mb && col < Nb)) {
            if constexpr (OB)
              *reinterpret_cast<uint2*>(Mh + (size_t)row * Nb + col) =
                  make_uint2(hi(v0) | (hi(v1) << 16), hi(v2) | (hi(v3) << 16));
            else
              *reinterpret_cast<float4*>(Mo + (size_t)row * Nb + col) =
                  make_float4(v0, v1, v2, v3);
          }
          ofl[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
        }
      }
    } else if (vec_store) {
      // 16-byte stores; in a ragged tile 4 columns are in or out together
      // (storing its values one by one took half the time of 49 products of
      // 250 x 1024 x 2752: 190 us)
      auto emit = [&](auto tc, auto wc) {
        constexpr bool TILED = decltype(tc)::value, WHOLE = decltype(wc)::value;
        float sT[4];
        float4 sS[4];
        if constexpr (SC) {
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const int row = r0 + rl + t * 16, col = c0 + cl + t * 16;
            sT[t] = dT[(size_t)b * Mb + (WHOLE || row < Mb ? row : 0)];
            // (single loads: behind an odd number of row scales dS is only
            // 4-byte aligned)
            const float* ps = dS + (size_t)b * Nb + (WHOLE || col < Nb ? col : 0);
            sS[t] = make_float4(ps[0], ps[1], ps[2], ps[3]);
          }
        } else {
          const float t = dT[b], u = dS[b];
#pragma unroll
          for (int i = 0; i < 4; ++i) sT[i] = t;
#pragma unroll
          for (int j = 0; j < 4; ++j) sS[j] = make_float4(u, u, u, u);
        }
        // tiled layout (full tiles only): the 16-byte pieces of a tile in
        // the order (wave, i, j, row l16, column group q), so each store of a
        // wave is one contiguous kilobyte
        float* tbase = Mo + (size_t)tt * (DBM * DBN) + (size_t)wave * 4096 + (l16 * 4 + q) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int row = r0 + row_of(i, j), col = c0 + col_of(i, j);
            const float t = sT[SW ? j : i];
            const float4 u = sS[SW ? i : j];
            float4 o;
            o.x = (acc[i][j][0] * t) * u.x;
            o.y = (acc[i][j][1] * t) * u.y;
            o.z = (acc[i][j][2] * t) * u.z;
            o.w = (acc[i][j][3] * t) * u.w;
            // whole lines of products read once, by the reconstruction:
            // non-temporal
            if constexpr (TILED)
              __builtin_nontemporal_store((v4f){o.x, o.y, o.z, o.w},
                                          reinterpret_cast<v4f*>(tbase + (i * 4 + j) * 256));
            else if (WHOLE || (row < Mb && col < Nb))
              *reinterpret_cast<float4*>(Mo + (size_t)row * Nb + col) = o;
          }
        }
      };
      using T = std::true_type;
      using F = std::false_type;
      if (whole && tiled) {
        if constexpr (!SW && SC == 0) emit(T{}, T{});
      } else if (whole) {
        emit(F{}, T{});
      } else {
        emit(F{}, F{});
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int row = r0 + row_of(i, j), col = c0 + col_of(i, j) + v;
            if (row < Mb && col < Nb) {
              const float sT = SC ? dT[(size_t)b * Mb + row] : dT[b];
              const float sS = SC ? dS[(size_t)b * Nb + col] : dS[b];
              Mo[(size_t)row * Nb + col] = (acc[i][j][v] * sT) * sS;
            }
          }
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
    // (a ragged tile's number of stores depends on the lane: counted as none,
    // a lower bound)
    return whole && (SC == 2 || vec_store) ? DSTORES : 0;
  };

  // Sequence of (tile, K-step) pairs p_0, p_1, ...; p_s lives in LDS buffer
  // s mod 3.  Iteration s: read the high half of p_s while the matrix cores
  // work on its low half; wait until p_{s+1} has landed and every wave is done
  // reading p_s; start the loads of p_{s+3} into the buffer of p_s; read the
  // low half of p_{s+1} while the matrix cores work on the high half of p_s.
  auto advance = [&](int& tt, int& kk) {
    if (++kk == nk) {
      kk = 0;
      tt += tstep;
    }
  };
  int t1 = t, k1 = 0;  // p_{s+1}
  advance(t1, k1);
  int t2 = t1, k2 = k1;  // p_{s+2}
  advance(t2, k2);
  int t3 = t2, k3 = k2;  // p_{s+3}
  advance(t3, k3);
  int ct = t, ck = 0;  // p_s
  issue(ct, ck, 0);
  int after1 = 0;  // vector-memory operations issued after the group of p_{s+1}
  if (t1 < t_end) issue(t1, k1, 1);
  if (t2 < t_end) {
    issue(t2, k2, 2);
    after1 = DLOADS;
  }
  wait_vm(t1 < t_end ? after1 + DLOADS : 0);  // p_0 has landed
  FM_COMPILER_FENCE();
  __builtin_amdgcn_s_barrier();
  FM_COMPILER_FENCE();
  read_half(0, 0);
  int cb = 0;  // buffer of p_s
  while (true) {
    read_half(1, cb);
    if constexpr (SC == 2) read_scales(cb, ct, ck);
    compute_half(0);
    wait_vm(after1);                     // p_{s+1} has landed (this wave's share)
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave's reads of p_s are done
    FM_COMPILER_FENCE();
    __builtin_amdgcn_s_barrier();
    FM_COMPILER_FENCE();
    const int nb = cb == 2 ? 0 : cb + 1;
    int after2 = 0;  // operations issued after the group of p_{s+2}
    if (t3 < t_end) {
      issue(t3, k3, cb);
      after2 = DLOADS;
    }
    FM_COMPILER_FENCE();
    const bool more = t1 < t_end;
    if (more) read_half(0, nb);
    compute_half(1);
    if constexpr (SC == 2) rescale();
    if (ck == nk - 1) after2 += epilogue(ct);
    FM_COMPILER_FENCE();
    if (!more) break;
    ct = t1;
    ck = k1;
    t1 = t2;
    k1 = k2;
    t2 = t3;
    k2 = k3;
    advance(t3, k3);
    after1 = after2;
    cb = nb;
  }
}


// Wide persistent kernel (tensor or row/column scales, bf16 products, Kb a
// multiple of 64): workgroup tile 256 x 256 (WN = 4) or 512 x 128 (WN = 2), K
// step 64 bytes, a ring of 4 LDS stages (512 or 640 rows of 64 bytes: 32 or
// 40 KB) filled by direct global-to-LDS loads two to three K steps ahead, 8
// waves, two per SIMD.  Each wave computes 128 rows x 64 columns = 4 x 2
// tiles of 32 x 32 (v_mfma_f32_32x32x16_bf16, 128 accumulators), so a widened
// A fragment feeds 2 matrix instructions and a B fragment 4, and the two
// waves of a SIMD share its matrix unit: while one issues its loads, LDS
// reads or conversions (which stall a wave, and with one wave per SIMD the
// matrix unit with it), the other's matrix instructions run.  Wave w takes
// the 128 A rows w % (8 / WN) and the 64 columns w / (8 / WN).
//
// Bound by the matrix cores at the clock they hold and by the operand loads
// from L2 (about 19 bytes per cycle and CU when loading alone): the square
// tile loads 512 rows per K step for the 65536 outputs the other loads 640
// for, and where both fit it was the faster: 49 x 32 products of 512 x 1024 x
// 1024 in 1.46 against 1.55 ms, 23 x 32 of 1024 x 1536 x 4096 in 8.05 against
// 8.5 ms.  The 512 x 128 tile serves column counts that are whole 128s only.
// Per stage a wave loads its share of the A and B rows (4 or 5 wave-loads of
// 1 KB).  The raw codes of a stage
// are read from LDS in two halves (the first 16 bytes of each lane's 32,
// sub-steps 0 and 1; then the second), each as soon as the previous stage's
// half is widened, so one stage of raw codes and two sub-steps of widened
// fragments are held.
//
// Within a K step, lane (r, h) = (lane % 32, lane / 32) of a 32-row fragment
// holds the 32 bytes [32h, 32h + 32) of row r; sub-step t (16 k values)
// takes bytes [8t, 8t + 8) of them, for both operands alike (the 64 k values
// of the step are summed in another order than in gemm_dma_kernel: the
// products are exact, the fp32 sums differ only by rounding).  Rows of 64
// bytes hold their 4 chunks XOR-swizzled by (row / 4) % 4: the 16 lanes
// served per LDS cycle of a 16-byte fragment read (16 consecutive rows, 4
// rows per 256-byte bank window) then hit 16 distinct 16-byte bank groups.
namespace wide {
constexpr int KS = 64;

// global_load_lds_dwordx4 with a scalar base and a 32-bit per-lane offset:
// lane L writes the 16 bytes it fetched at M0 + 16 L (M0 written by SALU
// then read by an LDS-DMA load needs one wait state).  Device scope (sc1):
// the codes are used once, from LDS, so the CU's vector L1 need not keep
// them (measured a few percent faster than the default scope)
__device__ __forceinline__ void dma16s(const void* sbase, uint32_t voff, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 sc1"
               :
               : "v"(voff), "s"(sbase), "s"(lds_addr)
               : "memory", "m0");
}
}  // namespace wide

typedef float v16f __attribute__((ext_vector_type(16)));

namespace wide8 {
constexpr int KS = 64, NT = 512, NSTG = 4;
constexpr int STORES = 32;  // 16-byte stores per lane per tile

// WN waves side by side: 2 for 512 x 128 tiles, 4 for 256 x 256
template <int WN>
struct Tile {
  static constexpr int BM = 8 / WN * 128, BN = WN * 64;
  static constexpr int ROWS = BM + BN;         // rows of KS bytes per stage
  static constexpr int STAGE = ROWS * KS;      // 40 KB or 32 KB
  static constexpr int LA = BM / 16 / 8;       // 1 KB wave-loads per wave per stage of A
  static constexpr int LOADS = ROWS / 16 / 8;  // and of both operands (5 or 4)
  // loads of the stage three ahead issued in the first of an iteration's four
  // phases; the others issue one each
  static constexpr int L0 = LOADS - 3;
};

// the counts used: after a tile's stores, or not; anything less waits for
// everything (a count above the one needed waits for more than needed)
template <int WN>
__device__ __forceinline__ void wait_vm(int n) {
  constexpr int N1 = Tile<WN>::LOADS + Tile<WN>::L0;
  if (n >= N1 + STORES) ring::wait_vm_n<N1 + STORES>();
  else if (n >= N1) ring::wait_vm_n<N1>();
  else ring::wait_vm_n<0>();
}
}  // namespace wide8

template <int FMT, int SC, int WN>
__global__ __launch_bounds__(wide8::NT) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_wide8_kernel(const uint8_t* __restrict__ Tq, const uint8_t* __restrict__ Sq,
                       const float* __restrict__ dT, const float* __restrict__ dS,
                       float* __restrict__ Mout, int Mb, int Nb, int Kb, int tiles_m, int tiles_n,
                       int total, int tiled) {
  using namespace wide8;
  using TL = Tile<WN>;
  constexpr int BM = TL::BM, BN = TL::BN, STAGE = TL::STAGE, LOADS = TL::LOADS, LA = TL::LA;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[NSTG * STAGE];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % (8 / WN), wn = wave / (8 / WN);
  const int r32 = lane & 31, h = lane >> 5;
  const int tiles = tiles_m * tiles_n;
  const int nk = Kb / KS;

  // workgroups go round-robin over the 8 XCDs: give each XCD a contiguous
  // range of tiles (whole products), so a product's operand panels stay in
  // one L2: XCD x takes tiles [x per, (x + 1) per), per = ceil(total / 8)
  const int G = gridDim.x;
  const bool xcd_split = (G & 7) == 0;
  const int per = (total + 7) >> 3;
  const int t = xcd_split ? (blockIdx.x & 7) * per + (blockIdx.x >> 3) : blockIdx.x;
  const int tstep = xcd_split ? (G >> 3) : G;
  const int t_end = xcd_split ? min(total, ((blockIdx.x & 7) + 1) * per) : total;
  if (t >= t_end) return;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;

  // A wave-load fills 16 rows of 64 bytes: lane L writes row L / 4, slot L %
  // 4, and fetches the chunk (L % 4) ^ ((row / 4) % 4); rows start at
  // multiples of 16, so the chunk and the row's offset in the operand depend
  // on the lane alone (one 32-bit offset), and the row block's address is
  // uniform (a scalar base)
  const uint32_t dma_off =
      (uint32_t)(lane >> 2) * (uint32_t)Kb + (uint32_t)(((lane & 3) ^ ((lane >> 4) & 3)) << 4);
  const size_t kb16 = (size_t)16 * Kb;
  // this wave's first A row (16 LA wave) and B row of a tile's panels
  auto tile_base = [&](int tile, const uint8_t*& Ab, const uint8_t*& Bb) {
    const int b = tile / tiles, tt = tile - b * tiles;
    const int tmi = tt / tiles_n;
    Ab = Tq + ((size_t)b * Mb + (size_t)tmi * BM + (size_t)wave * (16 * LA)) * Kb;
    Bb = Sq + ((size_t)b * Nb + (size_t)(tt - tmi * tiles_n) * BN + (size_t)wave * (16 * (LOADS - LA))) * Kb;
  };
  // wave-load j of a stage: j < LA 16 A rows, otherwise 16 B rows
  auto dma_one = [&](const uint8_t* Ab, const uint8_t* Bb, int kt, int buf, int j) {
    const uint32_t l0 = lds_base + (uint32_t)(buf * STAGE);
    if (j < LA)
      wide::dma16s(Ab + j * kb16 + kt * KS, dma_off, l0 + (uint32_t)((wave * LA + j) * 16 * KS));
    else
      wide::dma16s(Bb + (j - LA) * kb16 + kt * KS, dma_off,
                   l0 + (uint32_t)((BM + (wave * (LOADS - LA) + j - LA) * 16) * KS));
  };
  auto issue = [&](const uint8_t* Ab, const uint8_t* Bb, int kt, int buf) {
#pragma unroll
    for (int j = 0; j < LOADS; ++j) dma_one(Ab, Bb, kt, buf, j);
  };

  // one stage's raw codes: A rows 128 wm + 32 i + r32, B rows 64 wn + 32 j +
  // r32, 32 bytes each (two 16-byte chunks: sub-steps 0-1 and 2-3)
  uint4 ra[4][2], rb[2][2];
  const uint32_t rd0 = (uint32_t)r32 * KS + (uint32_t)(((2 * h) ^ ((r32 >> 2) & 3)) << 4);
  const uint32_t rd1 = (uint32_t)r32 * KS + (uint32_t)(((2 * h + 1) ^ ((r32 >> 2) & 3)) << 4);
  auto read_half = [&](int buf, auto cc) {
    constexpr int c = decltype(cc)::value;
    const uint32_t rd = c ? rd1 : rd0;
    const uint8_t* sa = lds + buf * STAGE + wm * 128 * KS;
    const uint8_t* sb = lds + buf * STAGE + (BM + wn * 64) * KS;
#pragma unroll
    for (int i = 0; i < 4; ++i) ra[i][c] = *reinterpret_cast<const uint4*>(sa + i * 32 * KS + rd);
#pragma unroll
    for (int j = 0; j < 2; ++j) rb[j][c] = *reinterpret_cast<const uint4*>(sb + j * 32 * KS + rd);
  };
  using C0 = std::integral_constant<int, 0>;
  using C1 = std::integral_constant<int, 1>;
  auto sel = [](const uint4 (&r)[2], int tsub, int d) -> int {
    const uint4& c = r[tsub >> 1];
    return (tsub & 1) ? (d ? (int)c.w : (int)c.z) : (d ? (int)c.y : (int)c.x);
  };
  v8bf wa[2][4], wb[2][2];  // widened fragments of two sub-steps
  auto widen_sub = [&](int tsub, int slot) {
#pragma unroll
    for (int i = 0; i < 4; ++i) wa[slot][i] = widen8<FMT>(sel(ra[i], tsub, 0), sel(ra[i], tsub, 1));
#pragma unroll
    for (int j = 0; j < 2; ++j) wb[slot][j] = widen8<FMT>(sel(rb[j], tsub, 0), sel(rb[j], tsub, 1));
  };
  auto pin = [&](int slot) {
#pragma unroll
    for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(wa[slot][i]));
#pragma unroll
    for (int j = 0; j < 2; ++j) asm volatile("" : "+v"(wb[slot][j]));
  };

  // acc[i][j]: the transposed 32 x 32 product, element v of lane (r32, h)
  // at row i*32 + r32, column j*32 + 8 (v / 4) + 4 h + v % 4 of the wave's
  // 128 x 64 block
  v16f acc[4][2];
  auto epilogue = [&](int tile) {
    const int b = tile / tiles, tt = tile - b * tiles;
    const int tmi = tt / tiles_n;
    const int m0 = tmi * BM, n0 = (tt - tmi * tiles_n) * BN;
    float* Mo = Mout + (size_t)b * Mb * Nb;
    const int r_base = m0 + wm * 128 + r32, c_base = n0 + wn * 64 + 4 * h;
    // tiled layout: the 128 x 128 piece this wave has half of, its values in
    // the order (i, column tile of 32, column group g, lane), one contiguous
    // kilobyte per wave store
    const int pr = tmi * (BM / 128) + wm, pc = n0 / 128 + (wn >> 1);
    float* tbase = Mo + ((size_t)pr * (Nb / 128) + pc) * (128 * 128) + lane * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = r_base + i * 32;
      const float sT = SC == 1 ? dT[(size_t)b * Mb + row] : dT[b];
      float* prow = Mo + (size_t)row * Nb + c_base;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          float4 sS;
          if constexpr (SC == 1) {
            sS = *reinterpret_cast<const float4*>(dS + (size_t)b * Nb + c_base + j * 32 + 8 * g);
          } else {
            const float u = dS[b];
            sS = make_float4(u, u, u, u);
          }
          v4f o;
          o[0] = (acc[i][j][4 * g + 0] * sT) * sS.x;
          o[1] = (acc[i][j][4 * g + 1] * sT) * sS.y;
          o[2] = (acc[i][j][4 * g + 2] * sT) * sS.z;
          o[3] = (acc[i][j][4 * g + 3] * sT) * sS.w;
          if (tiled)
            __builtin_nontemporal_store(
                o, reinterpret_cast<v4f*>(tbase + ((i * 4 + 2 * (wn & 1) + j) * 4 + g) * 256));
          else
            *reinterpret_cast<v4f*>(prow + j * 32 + 8 * g) = o;
        }
      }
    }
  };

  // Iteration s over the (tile, K step) pairs p_s, in four phases of 8
  // matrix instructions (one sub-step each), with the wave-loads of
  // p_{s+3} (into the buffer of p_{s-1}) after matrix instructions 1 and 5:
  //   A: sub-step 0 (slot 0), widening sub-step 1 into slot 1; 1 or 2 loads;
  //   wait until p_{s+1} has landed and every wave's reads of p_s are done;
  //   B: sub-step 1 (slot 1), widening sub-step 2 into slot 0, reading the
  //      first half of p_{s+1}; 1 load;
  //   C: sub-step 2 (slot 0), widening sub-step 3 into slot 1; 1 load;
  //   D: sub-step 3 (slot 1), reading the second half of p_{s+1}, widening
  //      its sub-step 0 into slot 0; 1 load.
  auto advance = [&](int& tt, int& kk) {
    if (++kk == nk) {
      kk = 0;
      tt += tstep;
    }
  };
  auto mma_dma = [&](int slot, const uint8_t* Ab, const uint8_t* Bb, int kt, int buf, auto j0c,
                     auto j1c) {
    constexpr int j0 = decltype(j0c)::value, j1 = decltype(j1c)::value;
    sfor<0, 8>([&](auto qc) {
      constexpr int q = decltype(qc)::value;
      acc[q >> 1][q & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wb[slot][q & 1], wa[slot][q >> 1], acc[q >> 1][q & 1], 0, 0, 0);
      if constexpr (q % 4 == 1 && j0 + q / 4 < j1) dma_one(Ab, Bb, kt, buf, j0 + q / 4);
    });
  };
  // 8 matrix instructions, each followed by N vector-ALU and R LDS-read
  // instructions (R for the first 6 only)
  auto groups = [](auto nc, auto rc) {
    constexpr int N = decltype(nc)::value, R = decltype(rc)::value;
    sfor<0, 8>([&](auto qc) {
      constexpr int q = decltype(qc)::value;
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if constexpr (R > 0 && q < 6) __builtin_amdgcn_sched_group_barrier(0x100, R, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, N, 0);
    });
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using J1 = std::integral_constant<int, TL::L0>;
  using J2 = std::integral_constant<int, TL::L0 + 1>;
  using J3 = std::integral_constant<int, TL::L0 + 2>;
  using J4 = std::integral_constant<int, LOADS>;
  int t1 = t, k1 = 0;  // p_{s+1}
  advance(t1, k1);
  int t2 = t1, k2 = k1;  // p_{s+2}
  advance(t2, k2);
  int t3 = t2, k3 = k2;  // p_{s+3}
  advance(t3, k3);
  const uint8_t *A0, *B0;
  tile_base(t, A0, B0);
  issue(A0, B0, 0, 0);
  int after1 = 0;  // vector-memory operations issued after the group of p_{s+1}
  if (t1 < t_end) {
    if (t1 != t) tile_base(t1, A0, B0);
    issue(A0, B0, k1, 1);
  }
  if (t2 < t_end) {
    if (t2 != t1) tile_base(t2, A0, B0);
    issue(A0, B0, k2, 2);
    after1 += LOADS;
  }
  const uint8_t *A3 = A0, *B3 = B0;  // panels of the tile of p_{s+3}
  if (t3 < t_end && t3 != t2) tile_base(t3, A3, B3);
  wait_vm<WN>(t1 < t_end ? after1 + LOADS : 0);  // p_0 has landed
  FM_COMPILER_FENCE();
  __builtin_amdgcn_s_barrier();
  FM_COMPILER_FENCE();
  read_half(0, C0{});
  read_half(0, C1{});
  widen_sub(0, 0);
  int cb = 0;  // buffer of p_s
  bool more = true;
  for (int tile = t; more; tile += tstep) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    for (int kk = 0; kk < nk; ++kk) {
      const int b3 = cb == 0 ? NSTG - 1 : cb - 1;  // buffer of p_{s+3} (that of p_{s-1})
      // A
      mma_dma(0, A3, B3, k3, b3, I0{}, J1{});
      widen_sub(1, 1);
      groups(std::integral_constant<int, 3>{}, I0{});
      pin(1);
      __builtin_amdgcn_sched_barrier(0);
      // p_{s+1} was issued before p_{s+2}'s loads and the first of p_{s+3}
      wait_vm<WN>(after1 + TL::L0);
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave's reads of p_s are done
      FM_COMPILER_FENCE();
      __builtin_amdgcn_s_barrier();
      FM_COMPILER_FENCE();
      const int nb = cb == NSTG - 1 ? 0 : cb + 1;
      more = t1 < t_end;
      // B
      mma_dma(1, A3, B3, k3, b3, J1{}, J2{});
      widen_sub(2, 0);
      read_half(nb, C0{});
      groups(std::integral_constant<int, 3>{}, I1{});
      pin(0);
      __builtin_amdgcn_sched_barrier(0);
      // C
      mma_dma(0, A3, B3, k3, b3, J2{}, J3{});
      widen_sub(3, 1);
      groups(std::integral_constant<int, 3>{}, I0{});
      pin(1);
      __builtin_amdgcn_sched_barrier(0);
      // D
      mma_dma(1, A3, B3, k3, b3, J3{}, J4{});
      read_half(nb, C1{});
      widen_sub(0, 0);
      groups(std::integral_constant<int, 3>{}, I1{});
      pin(0);
      __builtin_amdgcn_sched_barrier(0);
      t1 = t2;
      k1 = k2;
      t2 = t3;
      k2 = k3;
      advance(t3, k3);
      if (k3 == 0 && t3 < t_end) tile_base(t3, A3, B3);
      after1 = LOADS;
      cb = nb;
    }
    epilogue(tile);
    after1 += STORES;
  }
  ring::wait_vm_n<0>();  // the loads past the last pair land before the workgroup ends
}

}  // namespace

namespace {
int g_block_product_arith = FM_ACC_BF16;

// The wide kernel is the default where it applies; FM_BLOCK_GEMM=dma in the
// environment selects gemm_dma_kernel instead (for comparisons).
bool wide_enabled() {
  static const bool on = [] {
    const char* e = std::getenv("FM_BLOCK_GEMM");
    return !(e && std::strcmp(e, "dma") == 0);
  }();
  return on;
}

// Waves side by side of the wide kernel's tile for these arguments: 4 (256 x
// 256), 2 (512 x 128), or 0 when another kernel takes the products.  R:
// products of one gauge.  Rows in whole 512s are always the wide kernel's (both
// its tiles give the same bits).  Rows in an odd number of 256s are its only
// where the 256 x 256 tiles of one gauge are more than half of the 256 CUs: up
// to there the pipelined kernel's 256 x 128 tiles, twice as many, are one
// round on them and its round is the shorter (7 products of 256 x 1024 x 512
// in 13.9 against 18.7 us, one of 256 x 4096 x 4096 in 63 against 76, 49 of
// 256 x 512 x 1024 in 25 against 29; 49 of 256 x 768 x 1024, 147 square
// tiles, in 40 against 31).  Beyond, an inner length that is no multiple of
// 128 (whose products would go to the 128 x 128 tiles) gains at every length
// measured (49 products of 768 x 768 x 192 39 to 29 us, x 960 84 to 62), others
// from 768 on (49 of 768 x 768 x 1024 75 to 65 us, 1568 of 256 x 512 x 1024 523
// to 490, but x 256 226 to 253, x 640 376 to 390).  By one gauge's products, not by the
// launch's: the kernels' sums differ in rounding, and a gauge's bits are not
// to depend on how many others are evaluated with it.
int wide_waves(int Mb, int Nb, int Kb, int sc, bool out_bf16, int R) {
  if (!wide_enabled() || g_block_product_arith != FM_ACC_BF16 || (sc != 0 && sc != 1) ||
      out_bf16 || Kb % wide8::KS)
    return 0;
  const bool square = Mb % 256 == 0 && Nb % 256 == 0;
  if (Mb % 512 == 0) return square ? 4 : Nb % 128 == 0 ? 2 : 0;
  if (!square) return 0;
  const long long tiles = (long long)R * (Mb / 256) * (Nb / 256);
  return tiles > 128 && (Kb % 128 != 0 || Kb >= 768) ? 4 : 0;
}

// Products a wave per 32 x 32 tile takes.  It loads every operand row once
// per tile beside it, with no LDS in between; where a product's loads are
// more than 128 KB the 128 x 128 tile is the faster (orbits of 1, 32 and 128
// two-level gauges: 64 x 64 x 528 106, 254 and 689 us by waves against 107,
// 246 and 587 by tiles, x 2064 136, 637 and 1692 against 125, 498 and 1218; 64
// x 32 x 1040 109, 283 and 777 against 104, 273 and 734; 33 x 33 x 1040 129, 277
// and 738 against 124, 279 and 729; 32 x 32 x 2064 130, 312 and 1034 against
// 114, 333 and 933).  An inner length of whole 128s has the persistent kernel
// to fall back on, which took longer than the waves at every length (25088
// products of 64 x 64 x 2048 3.0 against 2.6 ms).  (Not by the launch's
// products: the kernels' sums differ in rounding, as in wide_waves.)
bool small_products(int Mb, int Nb, int Kb) {
  if (Mb > 64 || Nb > 64) return false;
  const int tm = (Mb + 31) / 32, tn = (Nb + 31) / 32;
  return Kb % 128 == 0 || (long long)(Mb * tn + Nb * tm) * Kb <= 131072;
}
}  // namespace

int block_gemm_tile_rows(int Mb, int Nb, int Kb, int scale_mode, bool out_bf16, int R) {
  const int sc = scale_mode == FM_SCALE_ROWCOL ? 1 : (scale_mode == FM_SCALE_GROUP ? 2 : 0);
  if (wide_waves(Mb, Nb, Kb, sc, out_bf16, R)) return 128;
  if (Kb % GK == 0) return DBM;
  return 0;
}

int set_block_product_arith(int a) {
  if (a != FM_ACC_BF16 && a != FM_ACC_FP8) return fail(FM_E_ARG, "unknown product arithmetic");
  g_block_product_arith = a;
  return FM_OK;
}

namespace {
template <int SC, bool OB = false>
int launch_block_gemm_sc(const uint8_t* Tq, const uint8_t* Sq, const float* dT, const float* dS,
                         float* Mout, int batch, int Mb, int Nb, int Kb, int fmt, int R,
                         hipStream_t st, int tiled = 0) {
  const bool fp8acc = g_block_product_arith == FM_ACC_FP8;
  if (const int wn = wide_waves(Mb, Nb, Kb, SC, OB, R)) {
    if constexpr (SC == 0 || SC == 1) {
      // persistent: one workgroup of 8 waves (160 or 128 KB of LDS) per CU
      const int tm = Mb / (8 / wn * 128), tn = Nb / (wn * 64);
      const long long total = (long long)batch * tm * tn;
      if (total > 0x7fffffffLL) return fail(FM_E_SHAPE, "too many GEMM tiles in one launch");
      const int T = (int)total;
      const int grid = (int)std::min<long long>(total, 256);
      if (tiled && SC != 0)
        return fail(FM_E_UNSUPPORTED, "the tiled product layout needs tensor scales");
#define FM_WIDE8(F, W)                                                                          \
  gemm_wide8_kernel<F, SC, W><<<grid, wide8::NT, 0, st>>>(Tq, Sq, dT, dS, Mout, Mb, Nb, Kb, tm, \
                                                          tn, T, tiled)
      if (fmt == FM_E4M3) {
        if (wn == 4) FM_WIDE8(FM_E4M3, 4);
        else FM_WIDE8(FM_E4M3, 2);
      } else {
        if (wn == 4) FM_WIDE8(FM_E5M2, 4);
        else FM_WIDE8(FM_E5M2, 2);
      }
#undef FM_WIDE8
      return launched("gemm_wide8_kernel");
    }
  }
  if constexpr (SC == 0 || SC == 1) {
    if (small_products(Mb, Nb, Kb) && !fp8acc && !tiled) {
      const int tm = (Mb + 31) / 32, tn = (Nb + 31) / 32;
      const long long total = (long long)batch * tm * tn;
      const long long blocks = (total + kThreads / 64 - 1) / (kThreads / 64);
      if (blocks > 0x7fffffffLL) return fail(FM_E_SHAPE, "too many GEMM tiles in one launch");
      // along x and y: a grid holds fewer than 2^32 threads along x
      const unsigned gx = (unsigned)std::min<long long>(blocks, 1 << 20);
      const dim3 grid(gx, (unsigned)((blocks + gx - 1) / gx));
      if (fmt == FM_E4M3)
        gemm_small_kernel<FM_E4M3, SC><<<grid, kThreads, 0, st>>>(Tq, Sq, dT, dS, Mout, Mb, Nb, Kb, tm, tn, total);
      else
        gemm_small_kernel<FM_E5M2, SC><<<grid, kThreads, 0, st>>>(Tq, Sq, dT, dS, Mout, Mb, Nb, Kb, tm, tn, total);
      return launched("gemm_small_kernel");
    }
  }
  if (Kb % GK == 0) {
    // pipelined persistent kernel: one 144 KB-LDS workgroup per CU, tiles of
    // 256 x 128, or 128 x 256 where those are fewer (49 products of 128 x 1024
    // x 1024 with group scales: 196 tiles instead of 392, 29 instead of 57 us)
    auto tiles_of = [](int r256, int r128) {
      return (long long)((r256 + DBM - 1) / DBM) * ((r128 + DBN - 1) / DBN);
    };
    const bool sw = !tiled && tiles_of(Nb, Mb) < tiles_of(Mb, Nb);
    const int ra = sw ? Nb : Mb, rb = sw ? Mb : Nb;
    const int tm = (ra + DBM - 1) / DBM, tn = (rb + DBN - 1) / DBN;
    const long long total = (long long)batch * tm * tn;
    if (total > 0x7fffffffLL) return fail(FM_E_SHAPE, "too many GEMM tiles in one launch");
    const int T = (int)total;
    const int grid = (int)std::min<long long>(total, 256);
    if (tiled && (SC != 0 || Mb % DBM || Nb % DBN))
      return fail(FM_E_UNSUPPORTED, "the tiled product layout needs whole tiles and tensor scales");
#define FM_DMA(F, A)                                                                            \
  (sw ? gemm_dma_kernel<F, A, SC, OB, true><<<grid, DNT, 0, st>>>(Tq, Sq, dT, dS, Mout, Mb, Nb, \
                                                                  Kb, tm, tn, T, tiled)         \
      : gemm_dma_kernel<F, A, SC, OB, false><<<grid, DNT, 0, st>>>(Tq, Sq, dT, dS, Mout, Mb,    \
                                                                   Nb, Kb, tm, tn, T, tiled))
    if (fmt == FM_E4M3) {
      if (fp8acc) FM_DMA(FM_E4M3, 1);
      else FM_DMA(FM_E4M3, 0);
    } else {
      if (fp8acc) FM_DMA(FM_E5M2, 1);
      else FM_DMA(FM_E5M2, 0);
    }
#undef FM_DMA
    return launched("gemm_dma_kernel");
  }
  if (tiled) return fail(FM_E_UNSUPPORTED, "the tiled product layout needs inner blocks of 128");
  if constexpr (SC == 2) {
    return fail(FM_E_SHAPE, "group scales need inner blocks of a multiple of 128");
  } else {
  // inner length a multiple of 16 only: one 128 x 128 tile per workgroup
  const int tm = (Mb + GT - 1) / GT, tn = (Nb + GT - 1) / GT;
  const long long total = (long long)batch * tm * tn;
  if (total > 0x7fffffffLL) return fail(FM_E_SHAPE, "too many GEMM tiles in one launch");
  const int T = (int)total;
  if (fmt == FM_E4M3) {
    if (fp8acc) gemm_tile_kernel<FM_E4M3, 1, SC><<<T, kThreads, 0, st>>>(Tq, Sq, dT, dS, Mout, Mb, Nb, Kb, tm, tn, T);
    else gemm_tile_kernel<FM_E4M3, 0, SC><<<T, kThreads, 0, st>>>(Tq, Sq, dT, dS, Mout, Mb, Nb, Kb, tm, tn, T);
  } else {
    if (fp8acc) gemm_tile_kernel<FM_E5M2, 1, SC><<<T, kThreads, 0, st>>>(Tq, Sq, dT, dS, Mout, Mb, Nb, Kb, tm, tn, T);
    else gemm_tile_kernel<FM_E5M2, 0, SC><<<T, kThreads, 0, st>>>(Tq, Sq, dT, dS, Mout, Mb, Nb, Kb, tm, tn, T);
  }
  return launched("gemm_tile_kernel");
  }
}
}  // namespace

int launch_block_gemm(const uint8_t* Tq, const uint8_t* Sq, const float* dT, const float* dS,
                      float* Mout, int batch, int Mb, int Nb, int Kb, int fmt, int scale_mode,
                      int R, hipStream_t st, bool out_bf16, bool tiled) {
  if (tiled && scale_mode != FM_SCALE_TENSOR)
    return fail(FM_E_UNSUPPORTED, "the tiled product layout needs tensor scales");
  if (scale_mode == FM_SCALE_ROWCOL)
    return launch_block_gemm_sc<1>(Tq, Sq, dT, dS, Mout, batch, Mb, Nb, Kb, fmt, R, st);
  if (scale_mode == FM_SCALE_GROUP) {
    if (Kb % 128 || Nb % 128 || Mb % 4)
      return fail(FM_E_SHAPE, "group scales need Kb, Nb multiples of 128 and Mb of 4");
    if (out_bf16)
      return launch_block_gemm_sc<2, true>(Tq, Sq, dT, dS, Mout, batch, Mb, Nb, Kb, fmt, R, st);
    return launch_block_gemm_sc<2>(Tq, Sq, dT, dS, Mout, batch, Mb, Nb, Kb, fmt, R, st);
  }
  return launch_block_gemm_sc<0>(Tq, Sq, dT, dS, Mout, batch, Mb, Nb, Kb, fmt, R, st, tiled ? 1 : 0);
}

}  // namespace fm
