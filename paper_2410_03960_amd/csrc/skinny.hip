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
// skinny_ring_kernel (K % 512 == 0: weights and activations through LDS, slices of K walked in sequence;
// everything but final results of up to 32 rows over one weight), and for those skinny_lds_kernel (K % 512 == 0: a
// workgroup's one slice of K in LDS) and skinny_seq_kernel (K % 512 == 0: slices walked in sequence, weights to registers).
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

// acc[mb][v] = C[m = mb*16 + l16][n + v] of one weight, whole or over K range `split`: to partial[split][m][n] or through the epilogue
template <int MB, int EPI>
__device__ __forceinline__ void store_blocks(const SkinnyParams &p, const floatx4 (&acc)[MB], int n, int l16, int split, bool partial) {
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int m = mb * 16 + l16;
    if (m >= p.M) continue;
    if (partial) {
      *(float4 *)(p.partial + ((int64_t)split * p.M + m) * p.N + n) = make_float4(acc[mb][0], acc[mb][1], acc[mb][2], acc[mb][3]);
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
    store_blocks<MB, EPI>(p, acc, nb * 16 + 4 * kq, l16, blockIdx.y, gridDim.y > 1);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[mb] = floatx4{0.f, 0.f, 0.f, 0.f};
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
// The activations through LDS (K % 512 == 0).  Measured on the first kernel: the activation fragments, which every
// wave fetches from L2 for every k step, take as many vector-memory requests as the weights and cost 20-30 % of the
// achieved HBM rate.  Here a workgroup walks slices of its K range one after the other: the activation slice sits in
// LDS in MFMA operand order, double-buffered and filled by a producer wave of its own (LDS-DMA, then a wait for
// everything it requested, then the workgroup barrier), so the consumer waves never wait for an LDS-DMA request and
// their weight stream runs on across slice boundaries; a consumer keeps the accumulators of its NBW column blocks in
// registers over the whole K range.  One barrier per slice.
template <int MB, int EPI, int WAVES, int NBW>
__global__ __launch_bounds__((WAVES + 1) * 64) void skinny_seq_kernel(SkinnyParams p, int ks_steps, int n_slices) {
  constexpr int U = NBW >= 4 ? 2 : 4;                                             // k steps (of 32) per group of loads
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
  // LDS then feeds NBW products); groups are requested in the order they are consumed.
  // (a column block past N re-reads the last one; its results are dropped)
  const bf16_t *wt[NBW];
#pragma unroll
  for (int b = 0; b < NBW; ++b) {
    int nb = nb0 + b;
    nb = nb < nblocks ? nb : nblocks - 1;
    wt[b] = p.W + ((int64_t)(nb * 16 + l16) * p.K + k0 + kq * 8);
  }
  int l_idx = 0;
  auto load_group = [&](uint4 (&dst)[NBW][U]) {
    const int koff = l_idx * (U * 32);
    ++l_idx;
#pragma unroll
    for (int b = 0; b < NBW; ++b)
#pragma unroll
      for (int u = 0; u < U; ++u) dst[b][u] = *(const uint4 *)(wt[b] + koff + u * 32);
  };
  uint4 wa[NBW][U], wb[NBW][U];
  load_group(wa);   // on its way while the first slice arrives

  floatx4 acc[NBW][MB];
#pragma unroll
  for (int b = 0; b < NBW; ++b)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[b][mb] = floatx4{0.f, 0.f, 0.f, 0.f};

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
            for (int mb = 0; mb < MB; ++mb)
              acc[b][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, half ? wb[b][u] : wa[b][u]), a[mb], acc[b][mb], 0, 0, 0);
        }
      }
      idx += 2;
    }
    // every LDS read of this slice has returned (its values went into the products above); no wait for the
    // weight loads in flight
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
  }

  // acc[b][mb][v] = C[m = mb*16 + l16][n = (nb0 + b)*16 + 4*kq + v], over this K range
#pragma unroll
  for (int b = 0; b < NBW; ++b) {
    if (nb0 + b < nblocks) store_blocks<MB, EPI>(p, acc[b], (nb0 + b) * 16 + 4 * kq, l16, blockIdx.y, gridDim.y > 1);
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
// Shape of a launch of skinny_seq_kernel: column blocks per workgroup (waves x nbw), slice length and K ranges, chosen by the
// bytes that move besides the weights -- every workgroup fetches the activation rows of its K range from L2 (n_cg * M * K * 2
// bytes in total over n_cg column groups, whatever the K split), K splits write and re-read fp32 partial sums (2 *
// ksplit * M * N * 4 bytes) and need a second launch.  Several workgroups fit a CU, and what counts is the bytes in
// flight per CU (two load groups per consumer wave): below 52 KB the stream slows down.
SeqPlan plan_seq(int M, int N, int K, size_t partial_cap) {
  SeqPlan best{};
  if (M < 1 || M > 32 || (N % 16) != 0 || (K % 512) != 0) return best;
  const int MB = (M + 15) / 16, nblocks = N / 16;
  // up to 16 rows, where skinny_lds_kernel has too few (column block, K slice) pairs: no second launch (4096 x 4096 in bf16, 1
  // row: 13.0 us against 9.9 of the first kernel)
  const bool one_launch = M <= 16 && !plan_lds(M, N, K, partial_cap).ok;
  const double w_bytes = 2.0 * N * K;
  static const int shapes[6][2] = {{4, 1}, {4, 2}, {4, 4}, {8, 1}, {8, 2}, {8, 4}};
  for (const auto &shape : shapes) {
    const int waves = shape[0], nbw = shape[1];
    const int n_cg = (nblocks + waves * nbw - 1) / (waves * nbw);
    for (int ks_steps = 16; ks_steps >= 8; ks_steps /= 2) {
      const int all_slices = K / (32 * ks_steps);
      const size_t lds = (size_t)2 * ks_steps * MB * 1024;
      for (int want = 1; want <= std::min(SKINNY_MAX_SPLIT, all_slices); ++want) {
        const int n_slices = (all_slices + want - 1) / want;
        const int ksplit = (all_slices + n_slices - 1) / n_slices;
        if (ksplit != want) continue;
        const int64_t wgs = (int64_t)n_cg * ksplit;
        const size_t partial = ksplit > 1 ? (size_t)ksplit * M * N * 4 : 0;
        // (too few workgroups: the first kernel is ahead, which splits K among the waves of a workgroup; 2048 x 2048, 1 row: 6.5 us
        // against 5.5)
        if (partial > partial_cap || wgs < 192 || (ksplit > 1 && one_launch)) continue;
        const double a_bytes = (double)n_cg * M * K * 2;
        const int64_t n_rounds = (wgs + 255) / 256;
        const double uneven = (double)n_rounds * 256 / (double)wgs - 1;
        // (resident: by LDS and by the registers of the instantiations)
        const int per_simd = nbw == 1 ? 8 : nbw == 4 || MB == 2 ? 4 : 5;
        const int64_t resident = std::max<int64_t>(1, std::min<int64_t>((160 << 10) / lds, 4 * per_simd / (waves + 1)));
        const double in_flight = (double)std::min(n_rounds, resident) * waves * (nbw == 1 ? 8 : 16);   // KB per CU
        const double cost = (w_bytes + 0.26 * a_bytes + 1.9 * partial + (ksplit > 1 ? 11e6 : 0)) * (1 + 0.31 * uneven) * (1 + 0.19 * std::max(0.0, 1 - in_flight / 52)) +
                            0.06e6 * n_slices * ((n_rounds + resident - 1) / resident);
        if (!best.ok || cost < best.cost) best = SeqPlan{true, waves, nbw, ks_steps, n_slices, ksplit, lds, partial, cost};
      }
    }
  }
  return best;
}
template <int EPI>
void launch_reduce(const SkinnyParams &p, int ksplit, hipStream_t st) {
  const int64_t quads = (int64_t)p.M * p.N / 4;
  hipLaunchKernelGGL((skinny_reduce_kernel<EPI>), dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, st, p, ksplit);
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
  if (pl.ksplit > 1) launch_reduce<EPI>(p, pl.ksplit, st);
  return 0;
}
template <int MB, int EPI>
int launch_seq_e(const SkinnyParams &p, const SeqPlan &pl, hipStream_t st) {
  if (pl.nbw == 4) return pl.waves == 4 ? launch_seq_k<MB, EPI, 4, 4>(p, pl, st) : launch_seq_k<MB, EPI, 8, 4>(p, pl, st);
  if (pl.nbw == 2) return pl.waves == 4 ? launch_seq_k<MB, EPI, 4, 2>(p, pl, st) : launch_seq_k<MB, EPI, 8, 2>(p, pl, st);
  return pl.waves == 4 ? launch_seq_k<MB, EPI, 4, 1>(p, pl, st) : launch_seq_k<MB, EPI, 8, 1>(p, pl, st);
}
template <int EPI>
int launch_seq_m(const SkinnyParams &p, const SeqPlan &pl, hipStream_t st) {
  return p.M <= 16 ? launch_seq_e<1, EPI>(p, pl, st) : launch_seq_e<2, EPI>(p, pl, st);
}
int launch_seq(const SkinnyParams &p, int epi, const SeqPlan &pl, hipStream_t st) {   // one weight, never with n_splits_out
  switch (epi) {
    case EPI_STORE_BF16: return launch_seq_m<EPI_STORE_BF16>(p, pl, st);
    case EPI_STORE_F32: return launch_seq_m<EPI_STORE_F32>(p, pl, st);
    case EPI_RESID: return launch_seq_m<EPI_RESID>(p, pl, st);
  }
  return -1;
}

// ---------------------------------------------------------------------------
// Weights and activations through LDS (K % 512 == 0).  A wave owns one 16-column block of one weight and streams it through a
// ring of its own, R steps of 64 columns of K, by LDS-DMA in whole 128-byte pieces of its rows; it issues no other
// vector-memory request, so they complete in order and a counted wait is exact.  A producer wave brings the
// activations, 256 columns of K at a time, into two buffers shared by the workgroup; one barrier per buffer.
// What bounds such a stream, measured on it:
//  - The address unit serves a request four lanes at a time, one 128-byte line per cycle.  With a row per lane, the
//    order in which the matrix instruction wants weights in registers, a 1 KB request takes 64 cycles instead of 16: an
//    L2-resident stream ends at 7.8 TB/s so loaded and at 20 with eight lanes to a row, and the activations' requests come on top.
//  - Rows 2^13 or 2^14 bytes apart at the same column lie on few memory channels, and all workgroups walk K in step.  So those of
//    a die start at different columns (`rot` buffers further round their K range): 28672 x 4096, 64 rows, 52.0 -> 42.4 us.
// With both, us per call (register form before -> this one): 64 rows 2 x 14336 x 4096 58.9 -> 42.0 (5.6 TB/s), 6144 x
// 4096 17.5 -> 13.8, 4096 x 4096 12.6 -> 9.8, 4096 x 14336 31.3 -> 25.5, 2048 x 2048 9.0 -> 5.4; 24 rows 2 x 28672 x 8192 171 -> 157, 8192 x
// 28672 92 -> 80; one row 2 x 14336 x 4096 44.6 (all rows resident in LDS) -> 39.5, 4096 x 14336 25.2 -> 21.2.
// Chunk c (16 bytes) of row r of a 16 x 64 piece lies at chunk c ^ ((r >> 1) & 7) of its 128 bytes, so that fragment reads meet
// every bank once.
template <int R>
__device__ __forceinline__ void wait_ring(int younger) {   // step i is in LDS: no more than the requests of `younger` later steps in flight
  static_assert(R <= 4, "cases below");
  if (younger >= R - 1) wait_vm<2 * (R - 1)>();
  else if (younger == 2) wait_vm<4>();
  else if (younger == 1) wait_vm<2>();
  else wait_vm<0>();
}
constexpr int RING_BUF = 256;                                       // columns of K in an activation buffer
constexpr int ring_steps(int waves) { return waves == 8 ? 3 : 4; }   // 48 and 32 KB per workgroup; more in flight is no faster (8 waves, 64 rows, 6 steps: 51.7 us against 48.8)
constexpr int ring_lds(int MB, int waves) { return 2 * MB * 16 * RING_BUF * 2 + waves * ring_steps(waves) * 2048 + (MB == 1 ? SKINNY_RESID_ROWS * 4 : 0); }
template <int MB, int EPI, int WAVES>
__global__ __launch_bounds__((WAVES + 1) * 64) void skinny_ring_kernel(SkinnyParams p, int n_bufs, int stride) {
  constexpr int R = ring_steps(WAVES);
  constexpr int CW = EPI == EPI_SWIGLU ? WAVES / 2 : WAVES;   // column blocks of a workgroup (SwiGLU: gate waves, then up waves)
  constexpr int ABUF = MB * 16 * RING_BUF * 2;
  extern __shared__ __align__(16) unsigned char lds[];   // [2][MB][4 steps][2 KB] activations, [WAVES][R][2 KB] weights, 1/rms of up to 8 rows
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, kq = lane >> 4;
  const int b0 = blockIdx.y * n_bufs, all = p.K / RING_BUF;
  const int bufs = all - b0 < n_bufs ? all - b0 : n_bufs;   // of this K range, >= 1 by the grid
  const int rot = (blockIdx.x / 8 * stride) % bufs;         // (workgroup ids go round the eight dies)
  typedef __attribute__((address_space(3))) void *lds_ptr_t;
  const unsigned lds_base = (unsigned)(size_t)(lds_ptr_t)lds;
  // request h of a piece: rows 8 h + r8, and the chunk that lies at this lane's place
  const int r8 = lane >> 3, c0 = (lane & 7) ^ (lane >> 4), c1 = c0 ^ 4;
  const unsigned row_bytes = p.K * 2;

  if (wave == WAVES) {
    for (int s = 0; s <= bufs; ++s) {
      if (s < bufs) {
        const int at = s + rot < bufs ? s + rot : s + rot - bufs;
        const unsigned char *base = (const unsigned char *)(p.A + (int64_t)(b0 + at) * RING_BUF);
        for (int mb = 0; mb < MB; ++mb) {
          const int m0 = mb * 16 + r8, m1 = m0 + 8;   // rows past M repeat row M - 1
          const unsigned o0 = (m0 < p.M ? m0 : p.M - 1) * row_bytes + c0 * 16, o1 = (m1 < p.M ? m1 : p.M - 1) * row_bytes + c1 * 16;
          const unsigned dst = lds_base + (s & 1) * ABUF + mb * 8192;
#pragma unroll
          for (int st = 0; st < 4; ++st) {
            lds_dma16_at(base + st * 128, o0, dst + st * 2048);
            lds_dma16_at(base + st * 128, o1, dst + st * 2048 + 1024);
          }
        }
        wait_vm<0>();
      }
      __builtin_amdgcn_s_barrier();   // buffer s is ready / the consumers have left buffer s - 1
    }
    if constexpr (EPI == EPI_SWIGLU) { if (gridDim.y == 1) __builtin_amdgcn_s_barrier(); }
    return;
  }

  const int nblocks = p.N / 16;
  const int my = blockIdx.x * CW + wave % CW, nb = my < nblocks ? my : nblocks - 1;   // (past N: the last block again, results dropped)
  const bf16_t *w0 = p.wtab ? p.wtab[nb] : (EPI == EPI_SWIGLU && wave >= CW ? p.W2 : p.W) + (int64_t)nb * 16 * p.K;
  const unsigned char *wbase = (const unsigned char *)(w0 + (int64_t)b0 * RING_BUF);
  const unsigned o0 = r8 * row_bytes + c0 * 16, o1 = (8 + r8) * row_bytes + c1 * 16;
  const int ring_off = 2 * ABUF + wave * (R * 2048);
  const int steps = bufs * 4;
  int next = rot * 4;   // column (in steps) of the next request
  auto request = [&](int slot) __attribute__((always_inline)) {
    const unsigned char *src = wbase + (int64_t)next * 128;
    lds_dma16_at(src, o0, lds_base + ring_off + slot * 2048);
    lds_dma16_at(src, o1, lds_base + ring_off + slot * 2048 + 1024);
    next = next + 1 == steps ? 0 : next + 1;
  };
#pragma unroll
  for (int i = 0; i < R; ++i) request(i);   // (steps >= 4 >= R)

  // 1/rms of the rows, where A lacks it: two rows to a wave at most, while the ring fills
  float *const rms = (float *)(lds + 2 * ABUF + WAVES * R * 2048);
  if (MB == 1 && p.ssq) {
    static_assert(2 * WAVES >= SKINNY_RESID_ROWS, "two rows to a wave");
    const int m0 = wave, m1 = wave + WAVES, n = p.K / 16;
    float q0 = 0.f, q1 = 0.f;
    for (int i = lane; i < n; i += 64) {
      if (m0 < p.M) q0 += p.ssq[m0 * n + i];
      if (m1 < p.M) q1 += p.ssq[m1 * n + i];
    }
    q0 = wave_sum(q0); q1 = wave_sum(q1);
    if (lane == 0) {
      if (m0 < p.M) rms[m0] = rsqrtf(q0 / (float)p.K + p.eps);
      if (m1 < p.M) rms[m1] = rsqrtf(q1 / (float)p.K + p.eps);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (read behind the barriers below)
  }
  floatx4 acc[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) acc[mb] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int frag = l16 * 128 + ((kq ^ (l16 >> 1)) << 4);   // (second half of a step: four chunks on, XOR 64)
  int slot = 0;
  __builtin_amdgcn_s_barrier();   // buffer 0 is in LDS
  for (int s = 0; s < bufs; ++s) {
    const unsigned char *buf = lds + (s & 1) * ABUF;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int left = steps - 1 - (s * 4 + j);   // steps after this one
      wait_ring<R>(left);
      asm volatile("" ::: "memory");
      bf16x8 w[2], a[2][MB];
#pragma unroll
      for (int u = 0; u < 2; ++u) w[u] = *(const bf16x8 *)(lds + ring_off + slot * 2048 + (frag ^ (u * 64)));
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) a[u][mb] = *(const bf16x8 *)(buf + mb * 8192 + j * 2048 + (frag ^ (u * 64)));
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[u], a[u][mb], acc[mb], 0, 0, 0);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // every read of the slot (and of the buffer) has returned
      if (left >= R) request(slot);
      slot = slot + 1 == R ? 0 : slot + 1;
    }
    __builtin_amdgcn_s_barrier();
  }
  if (MB == 1 && p.ssq) {
    asm volatile("" ::: "memory");
    const float f = rms[l16 < p.M ? l16 : 0];
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[0][v] *= f;
  }
  const int n = nb * 16 + 4 * kq;
  if constexpr (EPI == EPI_SWIGLU) {
    if (gridDim.y > 1) {   // partial[split][weight][m][n]
      if (my < nblocks) store_blocks<MB, EPI_STORE_F32>(p, acc, n, l16, blockIdx.y * 2 + (wave >= CW ? 1 : 0), true);
      return;
    }
    // the up waves hand their sums to the gate waves
    float4 *up = (float4 *)lds + (wave % CW) * (MB * 64) + lane;
    if (wave >= CW) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) up[mb * 64] = make_float4(acc[mb][0], acc[mb][1], acc[mb][2], acc[mb][3]);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (wave >= CW || my >= nblocks) return;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int m = mb * 16 + l16;
      if (m >= p.M) continue;
      const float4 u = up[mb * 64];
      float o[4] = {acc[mb][0], acc[mb][1], acc[mb][2], acc[mb][3]};
#pragma unroll
      for (int v = 0; v < 4; ++v) o[v] = o[v] / (1.f + __expf(-o[v])) * (v == 0 ? u.x : v == 1 ? u.y : v == 2 ? u.z : u.w);
      *(uint2 *)((bf16_t *)p.C + (int64_t)m * p.N + n) = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
    }
  } else {
    if (my < nblocks) store_blocks<MB, EPI>(p, acc, n, l16, blockIdx.y, gridDim.y > 1);
  }
}

struct RingPlan {
  bool ok;
  int waves, slice, n_slices, ksplit;   // slice: columns of K; K ranges are whole slices
  double cost;                          // us
};
// Shape of the launch: eight or four waves and the K ranges, by a time model fitted to 29 products of 2 to 1050 MB with 1 to 80 rows in
// every shape (median error 4 %; the choice costs 1 % against the best of each): launch and first fill; the weights, the
// activations' way from L2 (n_cg * M * K * 2 bytes over n_cg column groups) and the partial sums' way at 6.7 TB/s, lengthened by
// an uneven last round; a start for each further round of workgroups that fit; a wave's own chain of fragment reads and
// products.  K splits whose consumer adds them lengthen its pass by about a third of a microsecond each, others need a launch.
RingPlan plan_ring(int M, int N, int K, int nw, bool consumer_sums, size_t partial_cap) {
  RingPlan best{};
  if (M < 1 || M > 80 || (N % 16) != 0 || (K % 512) != 0) return best;
  if ((uint64_t)std::max(M, 16) * (uint64_t)K * 2 > 0xffffffffull) return best;   // (32-bit row offsets, of activations and of a block's 16 weight rows)
  const int MB = (M + 15) / 16, nblocks = N / 16;
  const double w_bytes = 2.0 * nw * N * K;
  // K ranges in steps of 512 columns; of 256 at 65 to 80 rows, whose longer rounds of a wave an even split evens out, but for
  // large weights
  const int slice = M > 64 && w_bytes < 4.3e8 ? 256 : 512, all_slices = K / slice;
  for (int waves = 8; waves >= 4; waves -= 4) {
    const int cw = waves / nw, n_cg = (nblocks + cw - 1) / cw;
    const int resident = (160 << 10) / ring_lds(MB, waves);
    for (int want = 1; want <= std::min(SKINNY_MAX_SPLIT, all_slices); ++want) {
      const int n_slices = (all_slices + want - 1) / want, ksplit = (all_slices + n_slices - 1) / n_slices;
      if (ksplit != want) continue;
      const size_t partial = ksplit > 1 ? (size_t)ksplit * nw * M * N * 4 : 0;
      if (partial > partial_cap) continue;
      const double wgs = (double)n_cg * ksplit, rounds = std::ceil(wgs / 256);
      const double bytes = w_bytes + 0.15 * n_cg * M * K * 2 + 1.6 * (double)partial;
      const double cost = 2.6 + bytes / 6.67e6 * (1 + 0.385 * (rounds * 256 / wgs - 1)) + 1.73 * (std::ceil(rounds / resident) - 1) +
                          1.33e-6 * w_bytes / wgs * MB * rounds + (ksplit == 1 ? 0 : consumer_sums ? 0.35 * (ksplit - 1) : 3.0);
      if (!best.ok || cost < best.cost) best = RingPlan{true, waves, slice, n_slices, ksplit, cost};
    }
  }
  return best;
}
template <int MB, int EPI, int WAVES>
int launch_ring_k(const SkinnyParams &p, const RingPlan &pl, hipStream_t st) {
  auto kern = skinny_ring_kernel<MB, EPI, WAVES>;
  constexpr int lds = ring_lds(MB, WAVES);
  static bool attr = false;
  if (!attr) {
    if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess) return -1;
    attr = true;
  }
  constexpr int CW = EPI == EPI_SWIGLU ? WAVES / 2 : WAVES;
  // Five buffers from one workgroup of a die to its next, where the activations (M rows of K) stay in a die's L2 all the same; else one,
  // so that neighbours still share them (64 rows: 2 x 28672 x 8192 162 us with five, 169 with one; 8192 x 28672, 3.7 MB, 98 and 89).
  const int stride = (int64_t)p.M * p.K * 2 <= (3 << 19) ? 5 : 1;
  const dim3 grid((p.N / 16 + CW - 1) / CW, pl.ksplit);
  hipLaunchKernelGGL(kern, grid, dim3((WAVES + 1) * 64), lds, st, p, pl.n_slices * (pl.slice / RING_BUF), stride);
  if (pl.ksplit > 1 && p.n_splits_out) *p.n_splits_out = pl.ksplit;   // the consumer adds the splits
  else if (pl.ksplit > 1) launch_reduce<EPI>(p, pl.ksplit, st);
  return 0;
}
template <int MB>
int launch_ring_m(const SkinnyParams &p, int epi, const RingPlan &pl, hipStream_t st) {
  switch (epi) {
    case EPI_STORE_BF16: return pl.waves == 8 ? launch_ring_k<MB, EPI_STORE_BF16, 8>(p, pl, st) : launch_ring_k<MB, EPI_STORE_BF16, 4>(p, pl, st);
    case EPI_STORE_F32: return pl.waves == 8 ? launch_ring_k<MB, EPI_STORE_F32, 8>(p, pl, st) : launch_ring_k<MB, EPI_STORE_F32, 4>(p, pl, st);
    case EPI_RESID: return pl.waves == 8 ? launch_ring_k<MB, EPI_RESID, 8>(p, pl, st) : launch_ring_k<MB, EPI_RESID, 4>(p, pl, st);
    case EPI_SWIGLU: return pl.waves == 8 ? launch_ring_k<MB, EPI_SWIGLU, 8>(p, pl, st) : launch_ring_k<MB, EPI_SWIGLU, 4>(p, pl, st);
  }
  return -1;
}
int launch_ring(const SkinnyParams &p, int epi, const RingPlan &pl, hipStream_t st) {
  switch ((p.M + 15) / 16) {
    case 1: return launch_ring_m<1>(p, epi, pl, st);
    case 2: return launch_ring_m<2>(p, epi, pl, st);
    case 3: return launch_ring_m<3>(p, epi, pl, st);
    case 4: return launch_ring_m<4>(p, epi, pl, st);
    default: return launch_ring_m<5>(p, epi, pl, st);
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
  if (pl.ksplit > 1) launch_reduce<EPI>(p, pl.ksplit, st);
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
  else if (ksplit > 1) launch_reduce<EPI>(p, ksplit, st);
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
// weights, 1 to 32 rows).  us per call, skinny_lds_kernel wherever it has enough pairs and the first kernel
// elsewhere / skinny_seq_kernel wherever it needs no second launch (up to 16 rows) or at all / this choice: 16 rows 13824 x
// 5120 37 / 51 / 33, 14336 x 4096 30 / 36 / 26, 8192 x 28672 105 / 129 / 105, 1 row 28672 x 8192 93 / 103 / 91, 24 rows 11008 x
// 4096 28 / 37 / 28; over 490 products of 1 to 32 rows 6 % ahead of the first and 4 % of the second rule, behind the first by
// more than 3 % only at 32000 x 2048 in fp32 (28.1 -> 29.0).
struct SkinnyRoute {
  int kernel;   // SWIFTKV_GEMM_STREAM_*
  RingPlan ring;
  SeqPlan seq;
  LdsPlan lds;
};
SkinnyRoute plan_skinny(const SkinnyParams &p, int epi) {
  SkinnyRoute r{};
  const int nw = epi == EPI_SWIGLU ? 2 : 1;
  const size_t cap = p.partial ? p.partial_bytes : 0;
  r.kernel = SWIFTKV_GEMM_STREAM_FIRST;
  if (p.ssq) {   // (the one kernel that takes the rows' factor)
    r.ring = plan_ring(p.M, p.N, p.K, nw, p.n_splits_out != nullptr, cap);
    if (r.ring.ok) r.kernel = SWIFTKV_GEMM_STREAM_SEQ;
    return r;
  }
  if (p.M > 32 || p.n_splits_out || nw == 2) {
    // (up to 8 rows of a SwiGLU pair with no more column blocks than CUs the first kernel is ahead, whose workgroups split K among
    // their waves: one row 2 x 4096 x 4096 15.0 us against 16.2, 2 x 2048 x 2048 7.9 / 8.6)
    if (nw == 2 && p.M <= 8 && p.N <= 4096) return r;
    r.ring = plan_ring(p.M, p.N, p.K, nw, p.n_splits_out != nullptr, cap);
    if (r.ring.ok) r.kernel = SWIFTKV_GEMM_STREAM_SEQ;
    return r;
  }
  r.seq = plan_seq(p.M, p.N, p.K, cap);
  const double wgs = p.N / (16.0 * first_blocks(p, epi));   // of the first kernel
  const double first = (2.0 * p.N * p.K + 0.68 * wgs * p.M * p.K * 2) * (1 + 0.88 * (std::ceil(wgs / 256) * 256 / wgs - 1)) * 0.913;
  double best = first;
  if (r.seq.ok && r.seq.cost < first) { best = r.seq.cost; r.kernel = SWIFTKV_GEMM_STREAM_SEQ; }
  r.lds = plan_lds(p.M, p.N, p.K, cap);
  if (r.lds.ok && r.lds.cost < best) r.kernel = SWIFTKV_GEMM_STREAM_SLICE;
  return r;
}

}  // namespace

GemmRoute route_skinny(const SkinnyParams &p, int epi) {
  const SkinnyRoute r = plan_skinny(p, epi);
  const int nb = first_blocks(p, epi);
  switch (r.kernel) {
    case SWIFTKV_GEMM_STREAM_SEQ:
      if (r.ring.ok) return GemmRoute{r.kernel, r.ring.waves / (epi == EPI_SWIGLU ? 2 : 1), r.ring.ksplit, r.ring.slice};
      return GemmRoute{r.kernel, r.seq.waves * r.seq.nbw, r.seq.ksplit, r.seq.ks_steps * 32};
    case SWIFTKV_GEMM_STREAM_SLICE: return GemmRoute{r.kernel, LDS_WAVES * r.lds.nbw, r.lds.ksplit, r.lds.ks_steps * 32};
  }
  return GemmRoute{r.kernel, nb, first_splits(p, epi, nb), 0};
}
bool skinny_takes_ssq(int M, int N, int K) {
  return M <= SKINNY_RESID_ROWS && plan_ring(M, N, K, 1, true, 0).ok;
}
int launch_skinny(const SkinnyParams &p, int epi, hipStream_t st) {
  if (p.M <= 0 || p.N <= 0) return 0;
  if (p.ssq && !skinny_takes_ssq(p.M, p.N, p.K)) return -1;
  if (p.M > 80 || (p.N % 16) != 0 || (p.K % 8) != 0) return -1;
  if (p.wtab && !p.n_splits_out) return -1;   // (the kernels of final results know no row-block table)
  if (p.n_splits_out) {
    if (epi == EPI_SWIGLU) return -1;
    *p.n_splits_out = 1;
  }
  const SkinnyRoute r = plan_skinny(p, epi);
  switch (r.kernel) {
    case SWIFTKV_GEMM_STREAM_SEQ: return r.ring.ok ? launch_ring(p, epi, r.ring, st) : launch_seq(p, epi, r.seq, st);
    case SWIFTKV_GEMM_STREAM_SLICE: return launch_lds(p, epi, r.lds, st);
  }
  if (p.M <= 16) return launch_mb<1, 1>(p, epi, st);
  if (p.M <= 32) return first_blocks(p, epi) == 2 ? launch_mb<2, 2>(p, epi, st) : launch_mb<2, 1>(p, epi, st);
  if (p.M <= 48) return launch_wide<3>(p, epi, st);
  if (p.M <= 64) return launch_wide<4>(p, epi, st);
  return launch_wide<5>(p, epi, st);
}
