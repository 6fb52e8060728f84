// Weight-streaming GEMM for few rows (M <= 80: the last-token tail, decode steps):
//   C[M,N] = A[M,K] * W[N,K]^T     (optionally a second weight for SwiGLU)
// HBM-bound: every weight byte is read once.  A workgroup owns 16*NB output
// columns; its 8 waves split K in interleaved 32-wide steps and each issues
// v_mfma_f32_16x16x32_bf16 with the weight rows as first operand, so a lane
// ends up with 4 consecutive output columns of one activation row per column
// block.  The eight partial sums meet in LDS.
// Every workgroup reads all of A (from L2), 16*MB rows against its 16*NB weight
// rows: with many rows the activation reads would outweigh the weights, so NB
// grows with MB (fewer, wider workgroups); with up to 16 rows NB = 1 keeps the
// most workgroups streaming.
// A CU sustains only a fraction of its share of HBM bandwidth on one such stream
// (loads in flight / latency), so every CU has to stream: when there are fewer
// column tiles than CUs, K is split over blockIdx.y, the splits write fp32
// partial sums and a second small kernel (or the consumer of the result) adds
// them in a fixed order and applies the epilogue (deterministic, unlike atomic
// accumulation).
// Four kernels: skinny_kernel (above; any K % 8 == 0, activations from L2),
// skinny_lds_kernel (one weight, up to 32 rows, K % 512 == 0: a workgroup's one slice
// of K in LDS), skinny_seq_kernel (K % 512 == 0: slices of K walked in sequence, the
// activation slice double-buffered in LDS by a producer wave) and skinny_res_kernel
// (the SwiGLU pair for up to 8 rows: all activation rows resident in LDS).
#include "../../include/swiftkv.h"
#include "common.h"

#include <algorithm>
#include <cmath>

namespace {

constexpr int SK_WAVES = 8;

template <int MB, int NB, int EPI>
__global__ __launch_bounds__(SK_WAVES * 64) void skinny_kernel(SkinnyParams p) {
  constexpr int NW = (EPI == EPI_SWIGLU) ? 2 : 1;
  constexpr int NJ = NW * NB;                       // weight-row blocks per workgroup
  constexpr int UN = NJ >= 4 ? 2 : 4;               // k steps in flight per wave
  __shared__ float red[SK_WAVES][NJ][64][4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, kq = lane >> 4;
  const int n0 = blockIdx.x * 16 * NB;
  const bf16_t *wrow[NJ];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    wrow[nb] = (p.wtab ? p.wtab[n0 / 16 + nb] + (int64_t)l16 * p.K : p.W + (int64_t)(n0 + nb * 16 + l16) * p.K) + kq * 8;
    if constexpr (EPI == EPI_SWIGLU) wrow[NB + nb] = p.W2 + (int64_t)(n0 + nb * 16 + l16) * p.K + kq * 8;
  }
  const bf16_t *arow[MB];
  bool avalid[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    int m = mb * 16 + l16;
    avalid[mb] = m < p.M;
    arow[mb] = p.A + (int64_t)(avalid[mb] ? m : 0) * p.K + kq * 8;
  }
  floatx4 acc[MB][NJ];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[mb][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  // k steps of this split
  const int all_steps = (p.K + 31) / 32;
  const int per_split = (all_steps + (int)gridDim.y - 1) / (int)gridDim.y;
  const int s_begin = blockIdx.y * per_split;
  const int nsteps = (s_begin + per_split) < all_steps ? (s_begin + per_split) : all_steps;
  // (a wave takes UN consecutive steps: both 64-byte halves of a 128-byte line of a weight row are then
  // requested by the same wave back to back; with the steps dealt out one by one, two waves fetched each line)
  for (int s0 = s_begin + wave * UN; s0 < nsteps; s0 += SK_WAVES * UN) {
    uint4 wv[UN][NJ], av[UN][MB];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int s = s0 + u;
      const int k = s * 32;
      const bool ok = (s < nsteps) && (k + kq * 8 + 8 <= p.K);
#pragma unroll
      for (int j = 0; j < NJ; ++j) wv[u][j] = ok ? *(const uint4 *)(wrow[j] + k) : make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) av[u][mb] = (ok && avalid[mb]) ? *(const uint4 *)(arow[mb] + k) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[mb][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wv[u][j]), __builtin_bit_cast(bf16x8, av[u][mb]), acc[mb][j], 0, 0, 0);
  }

  // acc[mb][w*NB + nb][v] = C[m = mb*16 + l16][n = n0 + nb*16 + 4*kq + v] (weight w) partial over this wave's k steps
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[wave][j][lane][v] = acc[mb][j][v];
    __syncthreads();
    if (wave < NB) {   // wave nb finishes column block nb
      const int nb = wave;
      float x[NW][4];
#pragma unroll
      for (int w = 0; w < NW; ++w)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          float sum = 0.f;
#pragma unroll
          for (int ww = 0; ww < SK_WAVES; ++ww) sum += red[ww][w * NB + nb][lane][v];
          x[w][v] = sum;
        }
      const int m = mb * 16 + l16, n = n0 + nb * 16 + 4 * kq;
      if (gridDim.y > 1) {   // partial[split][w][m][n]
        if (m < p.M) {
#pragma unroll
          for (int w = 0; w < NW; ++w)
            *(float4 *)(p.partial + (((int64_t)blockIdx.y * NW + w) * p.M + m) * p.N + n) = make_float4(x[w][0], x[w][1], x[w][2], x[w][3]);
        }
      } else if (m < p.M) {
        if constexpr (EPI == EPI_STORE_F32) {
          *(float4 *)((float *)p.C + (int64_t)m * p.N + n) = make_float4(x[0][0], x[0][1], x[0][2], x[0][3]);
        } else if constexpr (EPI == EPI_RESID) {
          float4 *dst = (float4 *)((float *)p.C + (int64_t)m * p.N + n);
          const float4 r = *dst;
          *dst = make_float4(r.x + x[0][0], r.y + x[0][1], r.z + x[0][2], r.w + x[0][3]);
        } else {
          bf16_t *dst = (bf16_t *)p.C + (int64_t)m * p.N + n;
          float o[4] = {x[0][0], x[0][1], x[0][2], x[0][3]};
          if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] = x[0][v] / (1.f + __expf(-x[0][v])) * x[NW - 1][v];
          }
          *(uint2 *)dst = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
        }
      }
    }
    __syncthreads();
  }
}

// sum of the K splits in split order + epilogue, 4 columns per thread
template <int EPI>
__global__ void skinny_reduce_kernel(SkinnyParams p, int ksplit) {
  constexpr int NW = (EPI == EPI_SWIGLU) ? 2 : 1;
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i >= (int64_t)p.M * p.N) return;
  float x[NW][4];
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int ks = 0; ks < ksplit; ++ks) {
      const float4 v = *(const float4 *)(p.partial + ((int64_t)ks * NW + w) * p.M * p.N + i);
      sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
    }
    x[w][0] = sum.x; x[w][1] = sum.y; x[w][2] = sum.z; x[w][3] = sum.w;
  }
  if constexpr (EPI == EPI_STORE_F32) {
    *(float4 *)((float *)p.C + i) = make_float4(x[0][0], x[0][1], x[0][2], x[0][3]);
  } else if constexpr (EPI == EPI_RESID) {
    float4 *dst = (float4 *)((float *)p.C + i);
    const float4 r = *dst;
    *dst = make_float4(r.x + x[0][0], r.y + x[0][1], r.z + x[0][2], r.w + x[0][3]);
  } else {
    bf16_t *dst = (bf16_t *)p.C + i;
    float o[4] = {x[0][0], x[0][1], x[0][2], x[0][3]};
    if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
      for (int v = 0; v < 4; ++v) o[v] = x[0][v] / (1.f + __expf(-x[0][v])) * x[NW - 1][v];
    }
    *(uint2 *)dst = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
  }
}

__device__ __forceinline__ void lds_dma16(const void *gptr, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(gptr) : "memory");
}

// ---------------------------------------------------------------------------
// One K slice per workgroup (one weight, no row-block table, up to 32 rows, K % 512 == 0): the slice's activations sit in LDS in MFMA operand
// order (filled by LDS-DMA, one 1 KB fragment per request: lane (row l16, quarter kq) lands at 16 * lane), the
// waves split the output columns (16-column blocks, `nbw` in a row per wave) and stream their weight rows through
// registers two groups of U k steps ahead, both steps of a 128-byte line in the same wave.  No cross-wave
// reduction and no barrier after the fill.  K slices go to blockIdx.y and meet in skinny_reduce_kernel in a fixed
// order.  Against skinny_seq_kernel, whose workgroups walk their slices in sequence: no barrier in
// the stream and longer load groups, but a slice is a split, so more partial sums (us per call, this form /
// skinny_seq_kernel at its best shape: 1 row 28672 x 8192 90 / 101, 24 rows 5120 x 5120 17.7 / 20.2, but 12 rows 5120 x
// 13824 41 / 32).
constexpr int LDS_WAVES = 8;
template <int MB, int EPI>
__global__ __launch_bounds__(LDS_WAVES * 64) void skinny_lds_kernel(SkinnyParams p, int ks_steps, int nbw) {
  constexpr int U = 8;                                     // k steps (of 32) per group of loads
  extern __shared__ __align__(16) unsigned char a_lds[];   // [k step][MB][64 lanes][16 bytes]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kq = lane >> 4;
  const int all_steps = p.K / 32;
  const int s_begin = blockIdx.y * ks_steps;
  const int steps = (all_steps - s_begin) < ks_steps ? (all_steps - s_begin) : ks_steps;   // a multiple of 2U
  const int k0 = s_begin * 32;
  const int groups = steps / U;

  const int nblocks = p.N / 16;
  const int nb0 = (blockIdx.x * LDS_WAVES + wave) * nbw;
  const int nb_end = (nb0 + nbw) < nblocks ? (nb0 + nbw) : nblocks;
  const int total = nb0 < nblocks ? (nb_end - nb0) * groups : 0;   // groups of this wave, an even number

  // weight rows of this lane: group g of column block nb covers k steps g * U ...; the groups of a wave's
  // blocks are walked in order, (l_nb, l_g) being the next one to request
  int l_nb = nb0, l_g = 0;
  auto load_group = [&](uint4 (&dst)[U]) {
    const int64_t koff = k0 + l_g * (U * 32) + kq * 8;
    const bf16_t *src = p.W + ((int64_t)(l_nb * 16 + l16) * p.K + koff);
    if (++l_g == groups) { l_g = 0; ++l_nb; }
#pragma unroll
    for (int u = 0; u < U; ++u) dst[u] = *(const uint4 *)(src + u * 32);
  };
  uint4 wa[U], wb[U];
  if (total > 0) load_group(wa);   // on its way while the activations arrive

  // activation slice -> LDS: fragment (k step s, row block mb) at (s * MB + mb) * 1024; rows past M repeat row M-1
  {
    typedef __attribute__((address_space(3))) void *lds_ptr_t;
    const unsigned lds_base = (unsigned)(size_t)(lds_ptr_t)a_lds;
    for (int f = wave; f < steps * MB; f += LDS_WAVES) {
      const int s = f / MB, mb = f % MB;
      int m = mb * 16 + l16;
      m = m < p.M ? m : p.M - 1;
      lds_dma16(p.A + ((int64_t)m * p.K + k0 + s * 32 + kq * 8), lds_base + f * 1024);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    __syncthreads();
  }
  if (total == 0) return;

  floatx4 acc[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) acc[mb] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto compute_group = [&](const uint4 (&src)[U], int g) {
    const unsigned char *fr = a_lds + (size_t)(g * U) * (MB * 1024) + lane * 16;
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
        acc[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, src[u]), *(const bf16x8 *)(fr + (u * MB + mb) * 1024), acc[mb], 0, 0, 0);
  };
  // acc[mb][v] = C[m = mb*16 + l16][n = nb*16 + 4*kq + v] over this K slice
  auto flush = [&](int nb) {
    const int n = nb * 16 + 4 * kq;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int m = mb * 16 + l16;
      if (m < p.M) {
        if (gridDim.y > 1) {   // partial[split][m][n]
          *(float4 *)(p.partial + ((int64_t)blockIdx.y * p.M + m) * p.N + n) = make_float4(acc[mb][0], acc[mb][1], acc[mb][2], acc[mb][3]);
        } else if constexpr (EPI == EPI_STORE_F32) {
          *(float4 *)((float *)p.C + (int64_t)m * p.N + n) = make_float4(acc[mb][0], acc[mb][1], acc[mb][2], acc[mb][3]);
        } else if constexpr (EPI == EPI_RESID) {
          float4 *dst = (float4 *)((float *)p.C + (int64_t)m * p.N + n);
          const float4 r = *dst;
          *dst = make_float4(r.x + acc[mb][0], r.y + acc[mb][1], r.z + acc[mb][2], r.w + acc[mb][3]);
        } else {
          *(uint2 *)((bf16_t *)p.C + (int64_t)m * p.N + n) = make_uint2(pack_bf16x2(acc[mb][0], acc[mb][1]), pack_bf16x2(acc[mb][2], acc[mb][3]));
        }
      }
      acc[mb] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
  };
  // two groups per iteration, one register set in flight while the other is consumed; `groups` is even, so
  // a block ends after the second group of an iteration
  int c_nb = nb0, c_g = 0;
  for (int idx = 0; idx < total; idx += 2) {
    load_group(wb);
    compute_group(wa, c_g);
    if (idx + 2 < total) load_group(wa);
    compute_group(wb, c_g + 1);
    c_g += 2;
    if (c_g == groups) { flush(c_nb); ++c_nb; c_g = 0; }
  }
}

// ---------------------------------------------------------------------------
// The SwiGLU pair for few rows: the M rows (not their padding to 16) are resident in LDS over the whole of K, row
// after row with 64 bytes between them, lanes of columns past M read the last row.  A wave owns one column block of
// both weights and walks K from end to end, two groups of eight 32-wide steps in flight; nothing is split, so there are
// no partial sums and no second launch, and no slice boundary either.  us per launch with 1 / 2 / 4 / 8 rows, this kernel against
// what plan_skinny takes without it: 2 x 14336 x 4096 44 / 45 / 46 / 49 (5.3 TB/s with one) against 53 / 56 / 56 / 51, 2 x 13824 x
// 5120 50 / 50 / 51 / 54 against 58 / 59 / 60 / 61, 2 x 13312 x 8192 82 / 85 / 88 / 95 against 95 / 96 / 100 / 102.  Beyond: 12 rows
// of 2 x 14336 x 4096 51 against 51, 16 rows 54 against 52.
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
constexpr int RES_WAVES = 4;
__global__ __launch_bounds__(RES_WAVES * 64) void skinny_res_kernel(SkinnyParams p, int stride) {
  constexpr int NW = 2, U = 8, WAVES = RES_WAVES;
  extern __shared__ __align__(16) unsigned char a_lds[];   // [M][stride bytes]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kq = lane >> 4;
  const int nblocks = p.N / 16;
  int nb = blockIdx.x * WAVES + wave;
  const bool live = nb < nblocks;
  nb = live ? nb : nblocks - 1;   // (a wave past the end re-reads the last block and stores nothing)
  const int groups = p.K / (32 * U);   // even
  const unsigned char *wp[NW];         // uniform; a lane adds its row's offset
#pragma unroll
  for (int w = 0; w < NW; ++w) wp[w] = (const unsigned char *)((w ? p.W2 : p.W) + (int64_t)nb * 16 * p.K);
  const uint64_t w_lane = (uint64_t)l16 * p.K * 2 + kq * 16;
  auto load_group = [&](u32x4_t (&dst)[NW][U], int g) __attribute__((always_inline)) {
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
      for (int u = 0; u < U; ++u) dst[w][u] = *(const u32x4_t *)(wp[w] + (int64_t)(g * U + u) * 64 + w_lane);
  };
  u32x4_t wa[NW][U], wb[NW][U];
  load_group(wa, 0);   // on their way while the activations arrive
  load_group(wb, 1);
  const int row_chunks = p.K / 8;
  for (int i = tid; i < p.M * row_chunks; i += WAVES * 64) {
    const int r = i / row_chunks, c = i % row_chunks;
    *(uint4 *)(a_lds + r * stride + c * 16) = *(const uint4 *)(p.A + (int64_t)r * p.K + c * 8);
  }
  __syncthreads();
  floatx4 acc[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) acc[w] = floatx4{0.f, 0.f, 0.f, 0.f};
  const unsigned char *fr = a_lds + (l16 < p.M ? l16 : p.M - 1) * stride + kq * 16;
  auto compute_group = [&](const u32x4_t (&src)[NW][U], int g) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bf16x8 a = *(const bf16x8 *)(fr + (g * U + u) * 64);
#pragma unroll
      for (int w = 0; w < NW; ++w) acc[w] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, src[w][u]), a, acc[w], 0, 0, 0);
    }
  };
  for (int g = 0; g < groups; g += 2) {
    compute_group(wa, g);
    if (g + 2 < groups) load_group(wa, g + 2);
    compute_group(wb, g + 1);
    if (g + 3 < groups) load_group(wb, g + 3);
  }
  // acc[w][v] = C[m = l16][n = nb*16 + 4*kq + v] (weight w)
  const int m = l16, n = nb * 16 + 4 * kq;
  if (!live || m >= p.M) return;
  float o[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) o[v] = acc[0][v] / (1.f + __expf(-acc[0][v])) * acc[1][v];
  *(uint2 *)((bf16_t *)p.C + (int64_t)m * p.N + n) = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
}
// Whether the form above runs this shape: up to 8 rows, and four column blocks to a workgroup fill one round of the 256
// CUs to at least four fifths (with half of the CUs idle too few loads are in flight: 2 x 8192 x 2048, 128 workgroups,
// 18.0 us against 15.6 of the first kernel; with several rounds skinny_seq_kernel is ahead: 2 x 28672 x 8192 168
// against 176).
bool res_fits(const SkinnyParams &p, int epi) {
  if (epi != EPI_SWIGLU || p.wtab || p.M > 8 || (p.N % 16) != 0 || (p.K % 512) != 0 || (size_t)p.M * (p.K * 2 + 64) > 160 * 1024) return false;
  const int wgs = (p.N / 16 + RES_WAVES - 1) / RES_WAVES;
  return wgs <= 256 && wgs * 5 >= 256 * 4;
}
int launch_res(const SkinnyParams &p, hipStream_t st) {
  static bool attr = false;
  if (!attr) {
    if (hipFuncSetAttribute((const void *)skinny_res_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) return -1;
    attr = true;
  }
  const int stride = p.K * 2 + 64, nblocks = p.N / 16;
  hipLaunchKernelGGL(skinny_res_kernel, dim3((nblocks + RES_WAVES - 1) / RES_WAVES), dim3(RES_WAVES * 64), (size_t)p.M * stride, st, p, stride);
  return 0;
}

// ---------------------------------------------------------------------------
// The activations through LDS (K % 512 == 0).  Measured on the first kernel: the activation fragments, which every
// wave fetches from L2 for every k step, take as many vector-memory requests as the weights and cost 20-30 % of the
// achieved HBM rate.  Here a workgroup walks slices of its K range one after the other: the activation slice sits in
// LDS in MFMA operand order, double-buffered and filled by a producer wave of its own (LDS-DMA, then a wait for
// everything it requested, then the workgroup barrier), so the consumer waves never wait for an LDS-DMA request and
// their weight stream runs on across slice boundaries; a consumer keeps the accumulators of its NBW column blocks in
// registers over the whole K range.  One barrier per slice.
template <int MB, int EPI, int WAVES, int NBW>
__global__ __launch_bounds__((WAVES + 1) * 64) void skinny_seq_kernel(SkinnyParams p, int ks_steps, int n_slices) {
  constexpr int NW = (EPI == EPI_SWIGLU) ? 2 : 1;
  constexpr int U = (NBW * NW >= 4) ? 2 : 4;                                      // k steps (of 32) per group of loads
  extern __shared__ __align__(16) unsigned char a_lds[];   // [2][k step][MB][64 lanes][16 bytes]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kq = lane >> 4;
  const int all_slices = p.K / (32 * ks_steps);
  const int sl_begin = blockIdx.y * n_slices;
  const int my_slices = (all_slices - sl_begin) < n_slices ? (all_slices - sl_begin) : n_slices;   // >= 1 by the grid
  const int k0 = sl_begin * ks_steps * 32;
  const int buf_bytes = ks_steps * MB * 1024;

  if (wave == WAVES) {
    // producer: slice s -> buffer s & 1, fragment (k step j, row block mb) at (j * MB + mb) * 1024; rows past M repeat row M-1
    typedef __attribute__((address_space(3))) void *lds_ptr_t;
    const unsigned lds_base = (unsigned)(size_t)(lds_ptr_t)a_lds;
    for (int s = 0; s <= my_slices; ++s) {
      if (s < my_slices) {
        for (int f = 0; f < ks_steps * MB; ++f) {
          const int j = f / MB, mb = f % MB;
          int m = mb * 16 + l16;
          m = m < p.M ? m : p.M - 1;
          lds_dma16(p.A + ((int64_t)m * p.K + k0 + (s * ks_steps + j) * 32 + kq * 8), lds_base + (s & 1) * buf_bytes + f * 1024);
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the slice is in LDS
      }
      __builtin_amdgcn_s_barrier();           // slice s is ready / the consumers have left slice s - 1
    }
    return;
  }

  const int nblocks = p.N / 16;
  const int gps = ks_steps / U;                                       // groups per slice, even
  const int nb0 = (blockIdx.x * WAVES + wave) * NBW;
  const int total = my_slices * gps;                                  // groups of this wave
  // weight rows of this lane: a group is U k steps of all NBW column blocks (an activation fragment read from
  // LDS then feeds NBW * NW products); groups are requested in the order they are consumed.
  // (a column block past N re-reads the last one; its results are dropped)
  int64_t woff[NBW];
  const bf16_t *wt[NBW];
#pragma unroll
  for (int b = 0; b < NBW; ++b) {
    int nb = nb0 + b;
    nb = nb < nblocks ? nb : nblocks - 1;
    woff[b] = (int64_t)(nb * 16 + l16) * p.K + k0 + kq * 8;
    wt[b] = p.wtab ? p.wtab[nb] + ((int64_t)l16 * p.K + k0 + kq * 8) : nullptr;   // (one weight, never SwiGLU)
  }
  int l_idx = 0;
  auto load_group = [&](uint4 (&dst)[NBW][NW][U]) {
    const int koff = l_idx * (U * 32);
    ++l_idx;
#pragma unroll
    for (int b = 0; b < NBW; ++b)
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const bf16_t *src = (wt[b] ? wt[b] : (w ? p.W2 : p.W) + woff[b]) + koff;
#pragma unroll
        for (int u = 0; u < U; ++u) dst[b][w][u] = *(const uint4 *)(src + u * 32);
      }
  };
  uint4 wa[NBW][NW][U], wb[NBW][NW][U];
  load_group(wa);   // on its way while the first slice arrives

  floatx4 acc[NBW][NW][MB];
#pragma unroll
  for (int b = 0; b < NBW; ++b)
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) acc[b][w][mb] = floatx4{0.f, 0.f, 0.f, 0.f};

  int idx = 0;
  __builtin_amdgcn_s_barrier();   // slice 0 is in LDS
  for (int s = 0; s < my_slices; ++s) {
    const unsigned char *buf = a_lds + (s & 1) * buf_bytes + lane * 16;
    for (int g = 0; g < gps; g += 2) {
      load_group(wb);
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const unsigned char *fr = buf + (size_t)((g + half) * U) * (MB * 1024);
        if (half == 1 && idx + 2 < total) load_group(wa);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          bf16x8 a[MB];
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) a[mb] = *(const bf16x8 *)(fr + (u * MB + mb) * 1024);
#pragma unroll
          for (int b = 0; b < NBW; ++b)
#pragma unroll
            for (int w = 0; w < NW; ++w)
#pragma unroll
              for (int mb = 0; mb < MB; ++mb)
                acc[b][w][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, half ? wb[b][w][u] : wa[b][w][u]), a[mb], acc[b][w][mb], 0, 0, 0);
        }
      }
      idx += 2;
    }
    // every LDS read of this slice has returned (its values went into the products above); no wait for the
    // weight loads in flight
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
  }

  // acc[b][w][mb][v] = C[m = mb*16 + l16][n = (nb0 + b)*16 + 4*kq + v] (weight w), over this K range
#pragma unroll
  for (int b = 0; b < NBW; ++b) {
    const int nb = nb0 + b;
    if (nb >= nblocks) continue;
    const int n = nb * 16 + 4 * kq;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int m = mb * 16 + l16;
      if (m >= p.M) continue;
      if (gridDim.y > 1) {   // partial[split][w][m][n]
#pragma unroll
        for (int w = 0; w < NW; ++w)
          *(float4 *)(p.partial + (((int64_t)blockIdx.y * NW + w) * p.M + m) * p.N + n) =
              make_float4(acc[b][w][mb][0], acc[b][w][mb][1], acc[b][w][mb][2], acc[b][w][mb][3]);
      } else if constexpr (EPI == EPI_STORE_F32) {
        *(float4 *)((float *)p.C + (int64_t)m * p.N + n) = make_float4(acc[b][0][mb][0], acc[b][0][mb][1], acc[b][0][mb][2], acc[b][0][mb][3]);
      } else if constexpr (EPI == EPI_RESID) {
        float4 *dst = (float4 *)((float *)p.C + (int64_t)m * p.N + n);
        const float4 r = *dst;
        *dst = make_float4(r.x + acc[b][0][mb][0], r.y + acc[b][0][mb][1], r.z + acc[b][0][mb][2], r.w + acc[b][0][mb][3]);
      } else {
        float o[4] = {acc[b][0][mb][0], acc[b][0][mb][1], acc[b][0][mb][2], acc[b][0][mb][3]};
        if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
          for (int v = 0; v < 4; ++v) o[v] = o[v] / (1.f + __expf(-o[v])) * acc[b][NW - 1][mb][v];
        }
        *(uint2 *)((bf16_t *)p.C + (int64_t)m * p.N + n) = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
      }
    }
  }
}

struct LdsPlan {
  bool ok;
  int ks_steps, ksplit, nbw;
  size_t lds_bytes, partial_bytes;
  double cost;   // as SeqPlan's
};
// How skinny_lds_kernel would run this shape (up to 32 rows), with slices of up to 2048 columns of K (1024 beyond 16 rows) or
// of 1024 where those leave one workgroup to a CU (16 rows x 8192 x 8192 33 us -> 28 with 512 workgroups).  ok = false: it
// cannot, has fewer than 1024 (column block, K slice) pairs, where the first kernel, whose workgroups split K among their
// waves, keeps more CUs busy, or weights beyond 500 MB (28672 x 8192, 470 MB, is ahead; 24 rows x 128256 x 4096, 1050 MB, 238
// us against 187 of skinny_seq_kernel).
LdsPlan plan_lds(int M, int N, int K, size_t partial_cap) {
  LdsPlan best{};
  if (M < 1 || M > 32 || (N % 16) != 0 || (K % 512) != 0 || 2.0 * N * K > 0.5e9) return best;
  const int MB = (M + 15) / 16, all_steps = K / 32, nblocks = N / 16;
  const int even = (all_steps + 64 / MB - 1) / (64 / MB);   // slices of at most 64 KB of LDS, of one length
  const int lengths[2] = {((all_steps + even - 1) / even + 15) / 16 * 16, MB == 1 && all_steps % 32 == 0 ? 32 : 0};
  if ((int64_t)nblocks * ((all_steps + lengths[0] - 1) / lengths[0]) < 1024) return best;
  for (const int ks_steps : lengths) {
    if (ks_steps == 0) continue;
    const int ksplit = (all_steps + ks_steps - 1) / ks_steps;
    const size_t partial = ksplit > 1 ? (size_t)ksplit * M * N * 4 : 0;
    if (partial > partial_cap || ksplit > SKINNY_MAX_SPLIT) continue;
    const int nbw = (int64_t)nblocks * ksplit >= 3200 ? 2 : 1;   // pairs a wave takes in a row
    const int64_t n_cg = (nblocks + LDS_WAVES * nbw - 1) / (LDS_WAVES * nbw), wgs = n_cg * ksplit;
    const double uneven = (double)((wgs + 255) / 256) * 256 / (double)wgs - 1;
    const double cost = (2.0 * N * K + 0.49 * n_cg * M * K * 2 + 1.9 * partial + (ksplit > 1 ? 11e6 : 0)) * (1 + 0.49 * uneven) * (MB == 1 ? 0.873 : 0.84);
    if (!best.ok || cost < best.cost) best = LdsPlan{true, ks_steps, ksplit, nbw, (size_t)ks_steps * MB * 1024, partial, cost};
  }
  return best;
}

struct SeqPlan {
  bool ok;
  int waves, nbw, ks_steps, n_slices, ksplit;
  size_t lds_bytes, partial_bytes;
  double cost;   // bytes at the streaming rate
};
// Shape of the launch: column blocks per workgroup (waves x nbw), slice length and K ranges, chosen by the bytes that
// move besides the weights -- every workgroup fetches the activation rows of its K range from L2 (n_cg * M * K * 2
// bytes in total over n_cg column groups, whatever the K split), K splits write and re-read fp32 partial sums (2 *
// ksplit * nw * M * N * 4 bytes) and, for the epilogues that cannot leave the sum to their consumer, need a second
// launch.  Beyond 32 rows the two activation buffers take most of LDS, one workgroup runs per CU, and what counts is
// how evenly the workgroups fill whole rounds of 256.  Up to 32 rows several fit, and what counts is the bytes in
// flight per CU (two load groups per consumer wave): below 64 KB the stream slows down.  Where the consumer adds the splits
// (Q/K/V, O, down and the fused K/V projection of a prefill), each one also lengthens the pass that adds them, about 0.25 us;
// the terms' larger weights there stand for that.
// Measured, us per call (before -> this form): 64 rows: 128256 x 4096 296 -> 196, 28672 x 4096 64.4 -> 61.2 and no second
// launch, 4096 x 4096 18.0 -> 16.5, 4096 x 14336 36.8 -> 36.8; 24 rows: 2 x 28672 x 8192 233 -> 171, 128256 x 4096 285 ->
// 184, 8192 x 28672 101 -> 93, 4096 x 14336 26.4 -> 28.0; 1 row: 6144 x 4096 14.3 -> 11.7, 8192 x 28672 90 -> 82,
// 2048 x 8192 12.8 -> 9.3, 4096 x 14336 26.6 -> 25.3 (4 ranges of 7 slices, 32 KB in flight per CU: 28.9).
SeqPlan plan_seq(int M, int N, int K, int nw, bool consumer_sums, size_t partial_cap) {
  SeqPlan best{};
  if (M < 1 || M > 80 || (N % 16) != 0 || (K % 512) != 0) return best;
  const int MB = (M + 15) / 16, nblocks = N / 16;
  const bool few = M <= 32;
  // up to 16 rows, where skinny_lds_kernel has too few (column block, K slice) pairs: no second launch (4096 x 4096 in bf16, 1
  // row: 13.0 us against 9.9 of the first kernel)
  const bool one_launch = M <= 16 && !consumer_sums && (nw == 2 || !plan_lds(M, N, K, partial_cap).ok);
  const double w_bytes = 2.0 * nw * N * K;
  int64_t best_wgs = 0;
  // The first of equals wins: beyond 32 rows eight waves with a block each are ahead of four with two (64 rows x 6144 x
  // 4096 18.0 us against 19.0, 4096 x 4096 13.0 / 13.7), four waves with four blocks of eight with two (8192 x 8192 33.4 / 35.3).
  static const int few_shapes[6][2] = {{4, 1}, {4, 2}, {4, 4}, {8, 1}, {8, 2}, {8, 4}};
  static const int many_shapes[6][2] = {{8, 1}, {4, 1}, {4, 2}, {4, 4}, {8, 2}, {8, 4}};
  for (const auto &shape : few ? few_shapes : many_shapes) {
    const int waves = shape[0], nbw = shape[1];
    if (nw == 2 && nbw * waves > 8) continue;               // (two weights: register budget of the instantiations below)
    const int n_cg = (nblocks + waves * nbw - 1) / (waves * nbw);
    for (int ks_steps = 16; ks_steps >= 8; ks_steps /= 2) {
      // 2 x 48 to 64 KB of LDS; at 65 to 80 rows 2 x 40, where the weights are large 2 x 80 (us per call with 256 / 512
      // columns, 80 rows: 2048 x 2048 12.1 / 13.3, 8192 x 3072 22.7 / 24.9, 13824 x 5120 47.6 / 52.4, but 8192 x 28672 120.6 /
      // 113.3; 228 products of 2 to 940 MB: from 430 MB on 512 columns are 1 % slower to 8 % faster)
      if (!few && ks_steps != (MB <= 4 || w_bytes >= 4.3e8 ? 16 : 8)) continue;
      const int all_slices = K / (32 * ks_steps);
      const size_t lds = (size_t)2 * ks_steps * MB * 1024;
      for (int want = 1; want <= std::min(SKINNY_MAX_SPLIT, all_slices); ++want) {
        const int n_slices = (all_slices + want - 1) / want;
        const int ksplit = (all_slices + n_slices - 1) / n_slices;
        if (ksplit != want) continue;
        const int64_t wgs = (int64_t)n_cg * ksplit;
        const size_t partial = ksplit > 1 ? (size_t)ksplit * nw * M * N * 4 : 0;
        if (partial > partial_cap) continue;
        const double a_bytes = (double)n_cg * M * K * 2;
        const bool second = ksplit > 1 && !consumer_sums;   // a launch, below in bytes at the streaming rate
        const int64_t n_rounds = (wgs + 255) / 256;
        const double uneven = (double)n_rounds * 256 / (double)wgs - 1;
        double cost;
        if (few) {
          if (!consumer_sums && (wgs < 192 || (second && one_launch))) continue;
          // (resident: by LDS and by the registers of the instantiations)
          const int per_simd = nbw * nw == 1 ? 8 : nbw * nw == 4 || (nw == 1 && MB == 2) ? 4 : 5;
          const int64_t fit = (160 << 10) / lds, resident = std::max<int64_t>(1, std::min<int64_t>(fit, 4 * per_simd / (waves + 1)));
          const double in_flight = (double)std::min(n_rounds, consumer_sums ? fit : resident) * waves * (nbw * nw == 1 ? 8 : 16);   // KB per CU
          cost = consumer_sums ? (w_bytes + 0.75 * a_bytes + 2.0 * partial) * (1 + 0.3 * uneven) * (1 + 0.35 * std::max(0.0, 1 - in_flight / 64))
                               : (w_bytes + 0.26 * a_bytes + 1.9 * partial + (second ? 11e6 : 0)) * (1 + 0.31 * uneven) * (1 + 0.19 * std::max(0.0, 1 - in_flight / 52)) +
                                     0.06e6 * n_slices * ((n_rounds + resident - 1) / resident);
        } else {   // L2 hits: cheaper than the partial sums' trip to memory; every further round pays its own fill and uneven end
          cost = (w_bytes + 0.75 * a_bytes + 2.0 * partial + (second ? 25e6 : 0)) * (1 + uneven) * (1.0 + 0.15 * (double)(n_rounds - 1));
        }
        if (!best.ok || cost < best.cost) {
          best = SeqPlan{true, waves, nbw, ks_steps, n_slices, ksplit, lds, partial, cost};
          best_wgs = wgs;
        }
      }
    }
  }
  // too few workgroups: the first kernel is ahead, which splits K among the waves of a workgroup (2048 x 2048, 1 row: 6.5 us
  // against 5.5)
  if (few && best_wgs < 192) best.ok = false;
  return best;
}
template <int MB, int EPI, int WAVES, int NBW>
int launch_seq_k(const SkinnyParams &p, const SeqPlan &pl, hipStream_t st) {
  auto kern = skinny_seq_kernel<MB, EPI, WAVES, NBW>;
  static bool attr = false;
  if (!attr) {
    if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 2 * 16 * MB * 1024) != hipSuccess) return -1;   // the longest slices
    attr = true;
  }
  const int nblocks = p.N / 16;
  dim3 grid((nblocks + WAVES * NBW - 1) / (WAVES * NBW), pl.ksplit);
  hipLaunchKernelGGL(kern, grid, dim3((WAVES + 1) * 64), pl.lds_bytes, st, p, pl.ks_steps, pl.n_slices);
  if (pl.ksplit > 1 && p.n_splits_out) *p.n_splits_out = pl.ksplit;   // the consumer adds the splits
  else if (pl.ksplit > 1) {
    const int64_t quads = (int64_t)p.M * p.N / 4;
    hipLaunchKernelGGL((skinny_reduce_kernel<EPI>), dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, st, p, pl.ksplit);
  }
  return 0;
}
template <int MB, int EPI>
int launch_seq_e(const SkinnyParams &p, const SeqPlan &pl, hipStream_t st) {
  if constexpr (EPI != EPI_SWIGLU) {
    if (pl.nbw == 4) return pl.waves == 4 ? launch_seq_k<MB, EPI, 4, 4>(p, pl, st) : launch_seq_k<MB, EPI, 8, 4>(p, pl, st);
    if (pl.waves == 8 && pl.nbw == 2) return launch_seq_k<MB, EPI, 8, 2>(p, pl, st);
  }
  if (pl.waves == 8 && pl.nbw == 1) return launch_seq_k<MB, EPI, 8, 1>(p, pl, st);
  if (pl.waves == 4 && pl.nbw == 2) return launch_seq_k<MB, EPI, 4, 2>(p, pl, st);
  if (pl.waves == 4 && pl.nbw == 1) return launch_seq_k<MB, EPI, 4, 1>(p, pl, st);
  return -1;
}
template <int MB>
int launch_seq_m(const SkinnyParams &p, int epi, const SeqPlan &pl, hipStream_t st) {
  switch (epi) {
    case EPI_STORE_BF16: return launch_seq_e<MB, EPI_STORE_BF16>(p, pl, st);
    case EPI_STORE_F32: return launch_seq_e<MB, EPI_STORE_F32>(p, pl, st);
    case EPI_RESID: return launch_seq_e<MB, EPI_RESID>(p, pl, st);
    case EPI_SWIGLU: return launch_seq_e<MB, EPI_SWIGLU>(p, pl, st);
  }
  return -1;
}
int launch_seq(const SkinnyParams &p, int epi, const SeqPlan &pl, hipStream_t st) {
  switch ((p.M + 15) / 16) {
    case 1: return launch_seq_m<1>(p, epi, pl, st);
    case 2: return launch_seq_m<2>(p, epi, pl, st);
    case 3: return launch_seq_m<3>(p, epi, pl, st);
    case 4: return launch_seq_m<4>(p, epi, pl, st);
    default: return launch_seq_m<5>(p, epi, pl, st);
  }
}

template <int MB, int EPI>
int launch_lds_k(const SkinnyParams &p, const LdsPlan &pl, hipStream_t st) {
  auto kern = skinny_lds_kernel<MB, EPI>;
  static bool attr = false;
  if (!attr) {
    if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024) != hipSuccess) return -1;   // the longest slices
    attr = true;
  }
  const int nblocks = p.N / 16;
  dim3 grid((nblocks + LDS_WAVES * pl.nbw - 1) / (LDS_WAVES * pl.nbw), pl.ksplit);
  hipLaunchKernelGGL(kern, grid, dim3(LDS_WAVES * 64), pl.lds_bytes, st, p, pl.ks_steps, pl.nbw);
  if (pl.ksplit > 1) {
    const int64_t quads = (int64_t)p.M * p.N / 4;
    hipLaunchKernelGGL((skinny_reduce_kernel<EPI>), dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, st, p, pl.ksplit);
  }
  return 0;
}
template <int EPI>
int launch_lds_e(const SkinnyParams &p, const LdsPlan &pl, hipStream_t st) {
  return p.M <= 16 ? launch_lds_k<1, EPI>(p, pl, st) : launch_lds_k<2, EPI>(p, pl, st);
}
int launch_lds(const SkinnyParams &p, int epi, const LdsPlan &pl, hipStream_t st) {   // never with n_splits_out
  switch (epi) {
    case EPI_STORE_BF16: return launch_lds_e<EPI_STORE_BF16>(p, pl, st);
    case EPI_STORE_F32: return launch_lds_e<EPI_STORE_F32>(p, pl, st);
    case EPI_RESID: return launch_lds_e<EPI_RESID>(p, pl, st);
  }
  return -1;
}

// The first kernel's shape: column blocks of a workgroup (two weight matrices count double: at most four weight-row
// blocks), and K splits where the column tiles of more than 32 rows leave CUs idle, each of at least 16 k steps per wave.
int first_blocks(const SkinnyParams &p, int epi) {
  if (p.M > 32 && epi != EPI_SWIGLU && p.N % 64 == 0) return 4;
  return p.M > 16 && p.N % 32 == 0 ? 2 : 1;
}
int first_splits(const SkinnyParams &p, int epi, int nb) {
  const int tiles = p.N / (16 * nb), nw = epi == EPI_SWIGLU ? 2 : 1;
  if (!p.partial || p.M <= 32 || tiles >= 256) return 1;
  const int ksplit = std::min({SKINNY_MAX_SPLIT, 256 / tiles, std::max(1, p.K / (32 * SK_WAVES * 4))});
  return (size_t)ksplit * nw * p.M * p.N * 4 > p.partial_bytes ? 1 : ksplit;
}
template <int MB, int NB, int EPI>
int launch_kernels(const SkinnyParams &p, hipStream_t st) {
  const int tiles = p.N / (16 * NB), ksplit = first_splits(p, EPI, NB);
  dim3 grid(tiles, ksplit), block(SK_WAVES * 64);
  hipLaunchKernelGGL((skinny_kernel<MB, NB, EPI>), grid, block, 0, st, p);
  if (ksplit > 1 && p.n_splits_out) *p.n_splits_out = ksplit;   // the consumer adds the splits
  else if (ksplit > 1) {
    const int64_t quads = (int64_t)p.M * p.N / 4;
    hipLaunchKernelGGL((skinny_reduce_kernel<EPI>), dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, st, p, ksplit);
  }
  return 0;
}

template <int MB, int NB>
int launch_mb(const SkinnyParams &p, int epi, hipStream_t st) {
  switch (epi) {
    case EPI_STORE_BF16: return launch_kernels<MB, NB, EPI_STORE_BF16>(p, st);
    case EPI_STORE_F32: return launch_kernels<MB, NB, EPI_STORE_F32>(p, st);
    case EPI_RESID: return launch_kernels<MB, NB, EPI_RESID>(p, st);
    case EPI_SWIGLU:
      if constexpr (NB <= 2) return launch_kernels<MB, NB, EPI_SWIGLU>(p, st);
      break;
  }
  return -1;
}

template <int MB>
int launch_wide(const SkinnyParams &p, int epi, hipStream_t st) {
  switch (first_blocks(p, epi)) {
    case 4: return launch_mb<MB, 4>(p, epi, st);
    case 2: return launch_mb<MB, 2>(p, epi, st);
  }
  return launch_mb<MB, 1>(p, epi, st);
}

// Which kernel runs this shape.  Up to 32 rows, where the result is final, three of them compete by the bytes they move at
// the streaming rate: the weights, a share of the activation rows' way from L2, the partial sums' trip to memory, a second
// launch; times what an uneven last round costs.  The terms' weights are fitted to the times of 565 products (2 to 940 MB of
// weights, 1 to 32 rows, one weight or two).  us per call, skinny_lds_kernel wherever it has enough pairs and the first kernel
// elsewhere / skinny_seq_kernel wherever it needs no second launch (up to 16 rows) or at all / this choice: 16 rows 13824 x
// 5120 37 / 51 / 33, 14336 x 4096 30 / 36 / 26, 8192 x 28672 105 / 129 / 105, 1 row 28672 x 8192 93 / 103 / 91, 24 rows 11008 x
// 4096 28 / 37 / 28; over 490 products of 1 to 32 rows 6 % ahead of the first and 4 % of the second rule, behind the first by
// more than 3 % only at 32000 x 2048 in fp32 (28.1 -> 29.0).  Two weights: without skinny_lds_kernel, which is nowhere ahead by
// more than 5 % there.
struct SkinnyRoute {
  int kernel;   // SWIFTKV_GEMM_STREAM_*
  SeqPlan seq;
  LdsPlan lds;
};
SkinnyRoute plan_skinny(const SkinnyParams &p, int epi) {
  SkinnyRoute r{};
  if (res_fits(p, epi)) { r.kernel = SWIFTKV_GEMM_STREAM_RESIDENT; return r; }
  const int nw = epi == EPI_SWIGLU ? 2 : 1;
  const bool adds = p.n_splits_out != nullptr;
  const size_t cap = p.partial ? p.partial_bytes : 0;
  r.seq = plan_seq(p.M, p.N, p.K, nw, adds, cap);
  r.kernel = r.seq.ok ? SWIFTKV_GEMM_STREAM_SEQ : SWIFTKV_GEMM_STREAM_FIRST;
  if (p.M > 32 || adds) return r;
  const double wgs = p.N / (16.0 * first_blocks(p, epi));   // of the first kernel
  const double first = (2.0 * nw * p.N * p.K + 0.68 * wgs * p.M * p.K * 2) * (1 + 0.88 * (std::ceil(wgs / 256) * 256 / wgs - 1)) * 0.913;
  double best = first;
  if (r.seq.ok && r.seq.cost < first) best = r.seq.cost;
  else r.kernel = SWIFTKV_GEMM_STREAM_FIRST;
  if (nw == 1 && !p.wtab) r.lds = plan_lds(p.M, p.N, p.K, cap);
  if (r.lds.ok && r.lds.cost < best) r.kernel = SWIFTKV_GEMM_STREAM_SLICE;
  return r;
}

}  // namespace

GemmRoute route_skinny(const SkinnyParams &p, int epi) {
  const SkinnyRoute r = plan_skinny(p, epi);
  const int nb = first_blocks(p, epi);
  switch (r.kernel) {
    case SWIFTKV_GEMM_STREAM_RESIDENT: return GemmRoute{r.kernel, RES_WAVES, 1, 0};
    case SWIFTKV_GEMM_STREAM_SEQ: return GemmRoute{r.kernel, r.seq.waves * r.seq.nbw, r.seq.ksplit, r.seq.ks_steps * 32};
    case SWIFTKV_GEMM_STREAM_SLICE: return GemmRoute{r.kernel, LDS_WAVES * r.lds.nbw, r.lds.ksplit, r.lds.ks_steps * 32};
  }
  return GemmRoute{r.kernel, nb, first_splits(p, epi, nb), 0};
}
int launch_skinny(const SkinnyParams &p, int epi, hipStream_t st) {
  if (p.M <= 0 || p.N <= 0) return 0;
  if (p.M > 80 || (p.N % 16) != 0 || (p.K % 8) != 0) return -1;
  if (p.n_splits_out) {
    if (epi != EPI_STORE_F32 && epi != EPI_RESID) return -1;
    *p.n_splits_out = 1;
  }
  const SkinnyRoute r = plan_skinny(p, epi);
  switch (r.kernel) {
    case SWIFTKV_GEMM_STREAM_RESIDENT: return launch_res(p, st);
    case SWIFTKV_GEMM_STREAM_SEQ: return launch_seq(p, epi, r.seq, st);
    case SWIFTKV_GEMM_STREAM_SLICE: return launch_lds(p, epi, r.lds, st);
  }
  if (p.M <= 16) return launch_mb<1, 1>(p, epi, st);
  if (p.M <= 32) return first_blocks(p, epi) == 2 ? launch_mb<2, 2>(p, epi, st) : launch_mb<2, 1>(p, epi, st);
  if (p.M <= 48) return launch_wide<3>(p, epi, st);
  if (p.M <= 64) return launch_wide<4>(p, epi, st);
  return launch_wide<5>(p, epi, st);
}
