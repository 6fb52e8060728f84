// bf16 MFMA GEMM for tens to thousands of rows:  C[M,N] = A[M,K] * W[N,K]^T.
//
// Decode batches beyond 80 rows, short prompts, prompt chunks: too many rows for the weight-streaming
// kernels, too few 256 x 256 tiles for the 256 CUs.  What bounds these products is the bytes a CU fetches
// per step: with a bounded number of requests in flight per CU a 64-wide step of a 128 x 256 tile (48 KB)
// takes 0.65 to 0.85 us of fetching and 0.70 of matrix and LDS work alone, 1.0 together, whatever the
// prefetch distance (two or four register sets, one or two workgroups per CU measured alike).  So the lever
// is the shape of the work: the tallest tile whose tiles, times K splits, fill the CUs in whole rounds.
// plan_gemm_mid chooses kernel, tile height and splits; the splits' fp32 partial sums meet in the norm pass
// that reads the residual rows anyway or in a finishing pass with the epilogue's arithmetic.
//
// gemm_mid_kernel: 4 waves side by side along N (wave tile 32 FM x 64), activations through registers into
// two LDS stages, weights in fragment order straight into registers, or row-major through a wave-private
// part of LDS.  Everything is an ordinary load, so loads return in order and the compiler's counted waits are
// exact.  In fragment order it serves the short tiles (FM = 2, 3: at most 256 registers, two workgroups per
// CU; 96 x 4096 x 14336 28 us against 33 with the LDS-DMA loop of gemm_wreg.hip, which is ahead from FM = 4
// on); row-major it serves every height (the tail of more than 80 sequences, contexts without packed copies).
#include "gemm_epilogue.h"

#include <algorithm>
#include <type_traits>

namespace {

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

template <int EPI, int FM, bool PACKED, bool NORM_OUT>
__global__ __launch_bounds__(256) void gemm_mid_kernel(GemmParams p) {
  constexpr int BM = 32 * FM, STAGE = BM * 128;
  constexpr int W_LDS = PACKED ? 0 : 8192;          // bytes of LDS per wave and stage for row-major weights
  extern __shared__ __align__(16) unsigned char smem[];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g = lane >> 5;

  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + 255) / 256;
  const int per_split = tiles_m * tiles_n, total = per_split * p.n_splits;
  const int per_xcd = (total + 7) / 8;
  const int logical = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (logical >= total) return;
  const int split = logical / per_split, tile = logical % per_split;
  constexpr int GM = 8;
  const int group = tile / (GM * tiles_n);
  const int first_m = group * GM;
  const int gsz = (tiles_m - first_m) < GM ? (tiles_m - first_m) : GM;
  const int in_group = tile % (GM * tiles_n);
  const int tm = first_m + in_group % gsz, tn = in_group / gsz;
  const int m0 = tm * BM, n0 = tn * 256 + wave * 64;   // n0: first column of this wave

  const int all_steps = p.K / 64, s0 = split * p.split_steps;
  const int nk = (all_steps - s0) < p.split_steps ? (all_steps - s0) : p.split_steps;   // >= 1 by the plan

  // Activations: request i of this wave covers rows (wave*FM + i)*8 .. +7, 128 bytes each, 8 lanes to a row; chunk c
  // of row r sits at LDS chunk c ^ ((r >> 1) & 7).  Addresses are a uniform base plus a 32-bit offset per lane.
  unsigned a_off[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int m = m0 + (wave * FM + i) * 8 + (lane >> 3);
    a_off[i] = (unsigned)(m < p.M ? m : p.M - 1) * (unsigned)(p.lda * 2) + (lane & 7) * 16;
  }
  const unsigned a_st0 = wave * FM * 1024 + (lane >> 3) * 128 + (((lane & 7) ^ (lane >> 4) ^ ((wave * FM & 1) * 4)) << 4);
  const unsigned char *a_base = (const unsigned char *)p.A + (int64_t)s0 * 128;
  // Weights (blocks past N re-read the last one; their results are dropped).  In fragment order a request is one
  // fragment, 1 KB contiguous: request 2*kk + nb is the sub-step's fragment of the wave's 32-row block nb.  Row-major
  // rows go through LDS like the activations, but through a part of it that only this wave touches: request i
  // covers the wave's rows 8 i .. 8 i + 7, 128 bytes each (fetched as fragments, 32 bytes of 32 rows per request,
  // the same rows took 1.5 to 1.8 times as long).  Bases are wave-uniform.
  const unsigned char *w_base[PACKED ? 2 : 8];
#pragma unroll
  for (int i = 0; i < (PACKED ? 2 : 8); ++i) {
    int blk = n0 / 32 + (PACKED ? i : i / 4);
    blk = blk < p.N / 32 ? blk : p.N / 32 - 1;
    if constexpr (PACKED) {
      w_base[i] = (const unsigned char *)(p.wpack + ((int64_t)blk * (p.K / 16) + (int64_t)s0 * 4) * 512);
    } else {
      if ((EPI == EPI_QKV || EPI == EPI_KV || EPI == EPI_PARTIAL) && p.head_dim == 128) {   // rotary partner blocks side by side, as in the packed order
        const int b = blk & 3;
        blk = (blk & ~3) | (b == 1 ? 2 : b == 2 ? 1 : b);
      }
      const int n16 = blk * 2 + ((i >> 1) & 1);
      w_base[i] = (const unsigned char *)((p.wtab ? p.wtab[n16] : p.W + (int64_t)n16 * 16 * p.ldw) + (i & 1) * 8 * p.ldw + (int64_t)s0 * 64);
    }
  }
  const unsigned w_lane = PACKED ? lane * 16 : (lane >> 3) * (unsigned)(p.ldw * 2) + (lane & 7) * 16;
  unsigned char *w_lds = smem + 2 * STAGE + wave * 8192;
  const unsigned w_st0 = (lane >> 3) * 128 + (((lane & 7) ^ (lane >> 4)) << 4);

  floatx16 acc[2][FM];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int bm = 0; bm < FM; ++bm)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[nb][bm][v] = 0.f;

  const unsigned a_lane = l32 * 128 + ((g ^ ((l32 >> 1) & 7)) << 4);

  u32x4_t wr[2][8];       // weights of the step in use and of the next one (fragment order), or of the next two (row-major, on their way to LDS)
  u32x4_t ar[2][FM];      // activation rows of the next two steps on their way to LDS
  bf16x8 af[2][FM], wf[2][2];

  auto load_a = [&](u32x4_t &dst, int i, int step) { dst = *(const u32x4_t *)(a_base + (int64_t)step * 128 + (uint64_t)a_off[i]); };
  auto load_w = [&](u32x4_t &dst, int i, int step) {
    if constexpr (PACKED) dst = *(const u32x4_t *)(w_base[i & 1] + ((int64_t)step * 4 + (i >> 1)) * 1024 + (uint64_t)w_lane);
    else dst = *(const u32x4_t *)(w_base[PACKED ? 0 : i] + (int64_t)step * 128 + (uint64_t)w_lane);
  };
  auto store_a = [&](int stage, int i, const u32x4_t &v) { *(u32x4_t *)(smem + stage * STAGE + (a_st0 ^ ((i & 1) * 64u)) + i * 1024) = v; };
  auto store_w = [&](int stage, int i, const u32x4_t &v) { *(u32x4_t *)(w_lds + stage * 4 * W_LDS + (w_st0 ^ ((i & 1) * 64u)) + i * 1024) = v; };
  auto frag_a = [&](int stage, int kk, int bm) { return *(const bf16x8 *)(smem + stage * STAGE + (a_lane ^ (unsigned)(kk * 32)) + bm * 4096); };
  auto frag_w = [&](int stage, int kk, int nb) { return *(const bf16x8 *)(w_lds + stage * 4 * W_LDS + (a_lane ^ (unsigned)(kk * 32)) + nb * 4096); };

  // prologue: the activations of steps 0 and 1, the weights of step 0 (row-major: also of step 1) requested, step 0 into LDS
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int step = s < nk ? s : nk - 1;
#pragma unroll
    for (int i = 0; i < FM; ++i) load_a(ar[s][i], i, step);
    if (s == 0 || !PACKED) {
#pragma unroll
      for (int i = 0; i < 8; ++i) load_w(wr[s][i], i, step);
    }
  }
#pragma unroll
  for (int i = 0; i < FM; ++i) store_a(0, i, ar[0][i]);
  if constexpr (!PACKED) {
#pragma unroll
    for (int i = 0; i < 8; ++i) store_w(0, i, wr[0][i]);
  }
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
  for (int bm = 0; bm < FM; ++bm) af[0][bm] = frag_a(0, 0, bm);
  if constexpr (!PACKED) {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) wf[0][nb] = frag_w(0, 0, nb);
  }

  // One 64-wide step in stage `cur` (it mod 2).  Between its MFMAs: the fragments of the next sub-step, the requests of
  // step it + 2 (fragment-order weights: it + 1), and in the first three sub-steps the LDS writes of step it + 1.
  // Plain loads and LDS accesses throughout: the compiler places the waits, and loads return in order.
  auto step_fn = [&](auto cur_c, const int it) __attribute__((always_inline)) {
    constexpr int cur = decltype(cur_c)::value, nxt = cur ^ 1;
    const int ka = it + 2 < nk ? it + 2 : nk - 1, kw = PACKED ? (it + 1 < nk ? it + 1 : nk - 1) : ka;   // past the end: repeated, never used
    constexpr int NMF = 2 * FM, NST = PACKED ? FM : FM + 8;   // LDS writes per step
    constexpr int SPK = (NST + 2) / 3;                        // ... per sub-step 0..2
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      if (kk == 3) {   // every wave's rows of step it+1 are in LDS, and every read of this step's stage has been issued and has returned
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
      const int a_lo = kk * FM / 4, a_hi = (kk + 1) * FM / 4;   // activation requests of this sub-step
#pragma unroll
      for (int i = 0; i < NMF; ++i) {
        const int nb = i / FM, bm = i % FM;
        const bf16x8 w = PACKED ? __builtin_bit_cast(bf16x8, wr[cur][kk * 2 + nb]) : wf[kk & 1][nb];
        acc[nb][bm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, af[kk & 1][bm], acc[nb][bm], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (i < FM) af[(kk + 1) & 1][i] = frag_a(kk < 3 ? cur : nxt, (kk + 1) & 3, i);
        if constexpr (!PACKED) { if (i == FM || i == FM + 1) wf[(kk + 1) & 1][i - FM] = frag_w(kk < 3 ? cur : nxt, (kk + 1) & 3, i - FM); }
        if (kk < 3) {   // writes NST per step, spread over the MFMAs of three sub-steps
#pragma unroll
          for (int w0 = i * SPK / NMF; w0 < (i + 1) * SPK / NMF; ++w0) {
            const int j = kk * SPK + w0;
            if (j < FM) store_a(nxt, j, ar[nxt][j]);
            else if (j < NST) store_w(nxt, j - FM, wr[nxt][j - FM]);
          }
        }
        if (i == FM / 2 && a_lo < a_hi) load_a(ar[cur][a_lo], a_lo, ka);
        if (i == FM / 2 + FM && a_lo + 1 < a_hi) load_a(ar[cur][a_lo + 1], a_lo + 1, ka);
        if (i == FM - 1) load_w(wr[PACKED ? nxt : cur][kk * 2], kk * 2, kw);
        if (i == NMF - 1) load_w(wr[PACKED ? nxt : cur][kk * 2 + 1], kk * 2 + 1, kw);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  for (int it = 0;; it += 2) {
    step_fn(std::integral_constant<int, 0>{}, it);
    if (it + 1 >= nk) break;
    step_fn(std::integral_constant<int, 1>{}, it + 1);
    if (it + 2 >= nk) break;
  }
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // every wave is done with the stages before the epilogue reuses them
  if (n0 >= p.N) return;
  unsigned char *slab = smem + wave * ((EPI == EPI_QKV || EPI == EPI_KV) ? FM * 32 * (64 * 2 + 16) : 32 * (64 * 4 + 16));
  gemm_epilogue_n64<EPI, FM, NORM_OUT>(p, acc, m0, n0, lane, slab, EPI == EPI_PARTIAL ? (int64_t)split * p.M * p.N : 0);
}

template <int EPI, int FM, bool PACKED, bool NORM_OUT = false>
int launch_k(const GemmParams &p, hipStream_t st) {
  constexpr int SLAB = 4 * ((EPI == EPI_QKV || EPI == EPI_KV) ? FM * 32 * (64 * 2 + 16) : 32 * (64 * 4 + 16));
  constexpr int STAGES = 2 * 32 * FM * 128 + (PACKED ? 0 : 2 * 4 * 8192);
  constexpr int SMEM = SLAB > STAGES ? SLAB : STAGES;
  auto kern = gemm_mid_kernel<EPI, FM, PACKED, NORM_OUT>;
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
    if (e != hipSuccess) return (int)e;
    attr_set = true;
  }
  const int total = ((p.M + 32 * FM - 1) / (32 * FM)) * ((p.N + 255) / 256) * p.n_splits;
  hipLaunchKernelGGL(kern, dim3(((total + 7) / 8) * 8), dim3(256), SMEM, st, p);
  return 0;
}

template <int EPI, int FM>
int launch_e(const GemmParams &p, MidKernel k, hipStream_t st) {
  if (k == MID_PACKED) {
    if constexpr (EPI != EPI_STORE_F32 && FM <= 3) {
      if constexpr (EPI == EPI_RESID) {
        if (p.hb && p.ssq) return launch_k<EPI, FM, true, true>(p, st);
      }
      return launch_k<EPI, FM, true>(p, st);
    }
    return -1;
  }
  return launch_k<EPI, FM, false>(p, st);
}
template <int FM>
int launch_f(const GemmParams &p, int epi, MidKernel k, hipStream_t st) {
  switch (epi) {
    case EPI_STORE_BF16: return launch_e<EPI_STORE_BF16, FM>(p, k, st);
    case EPI_STORE_F32: return launch_e<EPI_STORE_F32, FM>(p, k, st);
    case EPI_RESID: return launch_e<EPI_RESID, FM>(p, k, st);
    case EPI_SWIGLU: return launch_e<EPI_SWIGLU, FM>(p, k, st);
    case EPI_QKV: return launch_e<EPI_QKV, FM>(p, k, st);
    case EPI_KV: return launch_e<EPI_KV, FM>(p, k, st);
    case EPI_PARTIAL: return launch_e<EPI_PARTIAL, FM>(p, k, st);
  }
  return -1;
}
int launch_one(const GemmParams &p, int epi, const MidPlan &pl, hipStream_t st) {
  if (pl.kernel == MID_WREG) return launch_gemm_wreg(p, epi, pl.fm, pl.fm_low, st);
  if (pl.kernel == MID_STREAM) return launch_gemm_stream(p, epi, pl.fm, p.wpack != nullptr, st);
  switch (pl.fm) {
    case 2: return launch_f<2>(p, epi, pl.kernel, st);
    case 3: return launch_f<3>(p, epi, pl.kernel, st);
    case 4: return launch_f<4>(p, epi, pl.kernel, st);
    case 5: return launch_f<5>(p, epi, pl.kernel, st);
  }
  return -1;
}

// ---- K splits added up in split order, then the epilogue; 4 columns of C per thread ----
__device__ __forceinline__ float4 sum_splits(const float *p, int64_t stride, int n) {
  float4 s = *(const float4 *)p;
  for (int k = 1; k < n; ++k) {
    const float4 v = *(const float4 *)(p + k * stride);
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  return s;
}
template <int EPI>
__global__ void splits_finish_kernel(GemmParams p) {
  const int ncol = EPI == EPI_SWIGLU ? p.N / 2 : p.N;   // output columns
  const int64_t id = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4, stride = (int64_t)p.M * p.N;
  if (id >= (int64_t)p.M * ncol) return;
  const int m = (int)(id / ncol), n = (int)(id % ncol);
  if constexpr (EPI == EPI_SWIGLU) {   // every 32 virtual columns = 16 gate columns, then the matching 16 up columns
    const float *src = p.partial + (int64_t)m * p.N + (n / 16) * 32 + n % 16;
    const float rs = p.rstd ? p.rstd[m] : 1.f;
    const float4 g4 = sum_splits(src, stride, p.n_splits), u4 = sum_splits(src + 16, stride, p.n_splits);
    const float g[4] = {g4.x * rs, g4.y * rs, g4.z * rs, g4.w * rs}, u[4] = {u4.x * rs, u4.y * rs, u4.z * rs, u4.w * rs};
    float o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = g[e] * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g[e])) * u[e];   // silu(gate) * up
    *(uint2 *)((bf16_t *)p.C + (int64_t)m * p.ldc + n) = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
  } else {
    const float4 s = sum_splits(p.partial + id, stride, p.n_splits);
    if constexpr (EPI == EPI_STORE_F32) {
      *(float4 *)((float *)p.C + (int64_t)m * p.ldc + n) = s;
    } else if constexpr (EPI == EPI_RESID) {
      float4 *dst = (float4 *)((float *)p.C + (int64_t)m * p.ldc + n);
      const float4 r = *dst;
      *dst = make_float4(r.x + s.x, r.y + s.y, r.z + s.z, r.w + s.w);
    } else {
      *(uint2 *)((bf16_t *)p.C + (int64_t)m * p.ldc + n) = make_uint2(pack_bf16x2(s.x, s.y), pack_bf16x2(s.z, s.w));
    }
  }
}
// The same where an FP8 cache's scales are computed from all values of a head: rotation, rounding, bf16 rows and the absmax as in the
// GEMM's own epilogue (without absmax: launch_kv_finish).  A wave takes one head of a row, a rotary pair per lane (half of
// them idle at head_dim 64).  Grid (groups of `rows` rows, heads), the rows dealt to the four
// waves, and one atomic per workgroup: all heads' maxima share a few cache lines, and the atomics on them run one after
// the other at about 5 ns each (one per row and head: 512 rows x 64 heads took 200 us).
template <int EPI, int HD>
__global__ __launch_bounds__(256) void rope_finish_kernel(GemmParams p, int rows) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int hs = blockIdx.y;
  const int n_kv = p.kv_dim / HD, n_q = EPI == EPI_QKV ? p.q_dim / HD : 0;
  int kind, head, proj = 0;                              // kind 0 = q, 1 = k, 2 = v
  if constexpr (EPI == EPI_QKV) {
    kind = hs < n_q ? 0 : (hs < n_q + n_kv ? 1 : 2);
    head = kind == 0 ? hs : (hs - n_q) % n_kv;
  } else {
    proj = hs / (2 * n_kv);
    kind = 1 + (hs % (2 * n_kv)) / n_kv;
    head = hs % n_kv;
  }
  const int64_t stride = (int64_t)p.M * p.N;
  const int i = lane;
  const auto finish_row = [&](int row) __attribute__((always_inline)) {   // absmax of the lane's pair, as stored
    bf16_t *dst;
    if constexpr (EPI == EPI_QKV) dst = (kind == 0 ? p.q_out + (int64_t)row * p.q_dim : (kind == 1 ? p.k_out : p.v_out) + (int64_t)row * p.kv_dim) + head * HD;
    else dst = p.stage + (int64_t)row * p.N + hs * HD;
    const float *src = p.partial + (int64_t)row * p.N + hs * HD;
    const float rs = p.rstd ? p.rstd[row] : 1.f;
    if (i >= HD / 2) return 0.f;
    float x0 = src[i], x1 = src[i + HD / 2];
    for (int k = 1; k < p.n_splits; ++k) { x0 += src[k * stride + i]; x1 += src[k * stride + i + HD / 2]; }
    x0 *= rs; x1 *= rs;
    if (kind != 2) {
      const float2 cs = p.cos_sin[(int64_t)row * (HD / 2) + i];
      rotate_pair(x0, x1, cs.x, cs.y);
    }
    const bf16_t b0 = f32_to_bf16(x0), b1 = f32_to_bf16(x1);
    dst[i] = b0;
    dst[i + HD / 2] = b1;
    return fmaxf(fabsf(bf16_to_f32(b0)), fabsf(bf16_to_f32(b1)));
  };
  __shared__ float of_wave[4];
  const int row0 = blockIdx.x * rows, row_end = row0 + rows < p.M ? row0 + rows : p.M;
  float a = 0.f;
  for (int row = row0 + wave; row < row_end; row += 4) a = fmaxf(a, finish_row(row));
  a = wave_max(a);
  if (lane == 0) of_wave[wave] = a;
  __syncthreads();
  if (threadIdx.x == 0 && kind != 0) {
    a = fmaxf(fmaxf(of_wave[0], of_wave[1]), fmaxf(of_wave[2], of_wave[3]));
    atomicMax(p.amax + ((int64_t)(p.first_cache_layer + proj) * 2 + (kind == 2 ? 1 : 0)) * n_kv + head, __float_as_uint(a));
  }
}

template <int EPI>
void launch_finish(const GemmParams &p, hipStream_t st) {
  const int64_t quads = (int64_t)p.M * (EPI == EPI_SWIGLU ? p.N / 2 : p.N) / 4;
  hipLaunchKernelGGL(splits_finish_kernel<EPI>, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, st, p);
}
template <int EPI, int HD>
void launch_rope_finish_hd(const GemmParams &p, hipStream_t st) {
  const int heads = p.N / HD;
  // about 1024 workgroups (5 us of atomics), but no wave with more than 8 rows one after the other (2048 and 4096 workgroups: 4
  // and 15 us slower over 512 rows x 64 heads)
  const int64_t want = ((int64_t)p.M * heads + 1023) / 1024;
  const int rows = (int)std::min<int64_t>(32, std::max<int64_t>(4, (want + 3) / 4 * 4));
  hipLaunchKernelGGL((rope_finish_kernel<EPI, HD>), dim3((p.M + rows - 1) / rows, heads), dim3(256), 0, st, p, rows);
}
template <int EPI>
void launch_rope_finish(const GemmParams &p, hipStream_t st) {
  if (!p.amax) launch_kv_finish(p, EPI, st);
  else if (p.head_dim == 128) launch_rope_finish_hd<EPI, 128>(p, st);
  else launch_rope_finish_hd<EPI, 64>(p, st);
}

constexpr int MID_MAX_SPLIT = 16;

}  // namespace

// Time model, us: a fixed part (launch, the first loads) and, per round of workgroups, its 64-wide steps and its
// epilogue.  The per-step times are those measured with every CU busy on products of 4096 and 14336 columns of K and
// 2048 to 28672 columns of N over 96 to 2048 rows, weights from HBM; the epilogues those of 16384 rows.  K splits add
// the partial sums' trip (written and read once more, about 4 TB/s) and, unless the consumer of the residual rows adds
// them in a pass it makes anyway, a launch.  What the choice is worth, us (256 x 256 tile only -> this choice): 2048 x
// 4096 x 14336 264 -> 206, 1024 x 4096 x 14336 265 -> 107, 8831 x 4096 x 14336 1010 -> 765; below 1024 rows (128 x 128
// tile -> this choice): 333 x 28672 x 4096 160 -> 77, 333 x 4096 x 14336 190 -> 53, 160 x 6144 x 4096 73 -> 22.
MidPlan plan_gemm_mid(const GemmParams &p, int epi) {
  MidPlan best{};
  best.kernel = MID_NONE;
  const bool packed = p.wpack && p.K % 256 == 0 && p.N % 256 == 0 && epi != EPI_STORE_F32 && (uint64_t)p.lda * 512 <= 0xffffffffull;   // (32-bit row offsets inside a 256-row tile)
  if (p.M <= 80) return best;
  const bool far = (uint64_t)p.M * (uint64_t)p.lda * 2 >= 0xffffffffull;   // beyond the 32-bit row offsets of gemm_mid_kernel (gemm_wreg_kernel's start at its tile)
  if (!packed && (p.M >= 1024 || p.K % 64 != 0 || p.N % 64 != 0 || ((epi == EPI_QKV || epi == EPI_KV) && p.N % 128 != 0))) return best;
  const bool norm_out = epi == EPI_RESID && p.hb && p.ssq;
  const bool consumer = p.n_splits_out != nullptr;
  const int all_steps = p.K / 64, unit = packed ? 4 : 1;
  const int tiles_n = (p.N + 255) / 256;
  // us per step of a round of up to 256 workgroups (t1); the forms that fit two workgroups to a CU: per 256 of more (t2)
  struct Form { MidKernel kernel; int fm; double t1, t2; };
  const Form forms[] = {
      {MID_WREG, 8, 1.46, 0}, {MID_WREG, 7, 1.27, 0}, {MID_WREG, 6, 1.12, 0}, {MID_WREG, 5, 0.99, 0}, {MID_WREG, 4, 0.89, 0},
      {MID_PACKED, 3, 0.82, 0.73}, {MID_PACKED, 2, 0.76, 0.66},
      {MID_ROWS, 5, 1.45, 0}, {MID_ROWS, 4, 1.33, 0}, {MID_ROWS, 3, 1.27, 0}, {MID_ROWS, 2, 1.20, p.partial ? 0.76 : 0.92}};   // (the last: 0.80 to 0.92 over a whole long K)
  // epilogue of a 256-row tile
  const double epi_us = norm_out ? 25 : epi == EPI_RESID || epi == EPI_QKV ? 12 : epi == EPI_KV ? 10 : 4;
  // Beyond 24 rounds of the full height an uneven last one is under 4 %, less than a lower height throughout loses in a run that long
  // (more bytes per product on a power-limited chip; gate/up of 32832 rows, a whole launch over its steps: 1.34 us per step
  // of 224 rows against 1.45 of 256, where the table has 1.27 and 1.46; 6.02 ms per launch -> 5.85).
  const bool full = packed && ((int64_t)((p.M + 255) / 256) * tiles_n + 255) / 256 > 24;
  for (const Form &f : forms) {
    if ((f.kernel == MID_ROWS) == packed || (full && f.fm < 8) || (far && f.kernel != MID_WREG)) continue;
    const int64_t tiles = (int64_t)((p.M + 32 * f.fm - 1) / (32 * f.fm)) * tiles_n;
    for (int want = 1; want <= std::min(MID_MAX_SPLIT, all_steps / unit); ++want) {
      if (want > 1 && (!p.partial || norm_out)) break;
      const int steps = ((all_steps / unit + want - 1) / want) * unit, s = (all_steps + steps - 1) / steps;
      if (s != want) continue;
      const size_t bytes = s > 1 ? (size_t)s * p.M * p.N * 4 : 0;
      if (bytes > p.partial_bytes) break;
      const double wgs = (double)(tiles * s);
      const double rounds = f.t2 > 0 && wgs > 256 ? std::max(2.0, wgs / 256) : (double)((tiles * s + 255) / 256);
      const double round_us = steps * (f.t2 > 0 && wgs > 256 ? f.t2 : f.t1) + 4 + (s > 1 ? 0 : epi_us * f.fm / 8);
      const double cost = 7 + rounds * round_us + (s > 1 ? 2.0 * bytes / 4.0e6 + (consumer ? 0 : 5) : 0);
      if (best.kernel == MID_NONE || cost < best.cost) best = MidPlan{f.kernel, f.fm, s, steps, cost};
    }
  }
  // Two tile heights in a launch (gate and up, the widest product of a layer: without K splits its rounds rarely come out even): 256-row
  // tiles over the first columns fill whole rounds, lower ones the time that is left.  By the same table: `tall` rounds of the full
  // height hold some columns of tiles, the rest go to CUs that have no tile of the last tall round and then to rounds of their own.
  // us per launch, 28672 columns, K 4096, one height -> two: 900 rows 203 -> 189, 1300 266 -> 262, 2048 421 -> 393, 3300 638 -> 617,
  // 4700 878 -> 853, 13000 2278 -> 2207; 16384 columns, K 2048, 5000 rows 299 and 308 were about the worst of the others (not taken).
  // Beyond 24 rounds the lower tiles are the last few columns only, and it still pays: 14300 rows 2490 -> 2481, 14600 2587 -> 2562, 15700
  // 2760 -> 2715, 18000 3171 -> 3129, 24000 4194 -> 4137, 32832 5673 -> 5628, 64000 11347 and 11357.
  if (packed && epi == EPI_SWIGLU && best.kernel == MID_WREG && best.n_splits == 1) {
    const int rows_n = (p.M + 255) / 256, most = (int)std::min<int64_t>((int64_t)rows_n * tiles_n / 256, 1 << 20);
    const double a = all_steps * forms[0].t1 + 4 + epi_us;
    for (const Form &f : {forms[2], forms[4]}) {
      const double b = all_steps * f.t1 + 4 + epi_us * f.fm / 8;
      for (int tall = std::max(1, most - 2); tall <= most; ++tall) {
        const int cols = tall * 256 / rows_n, spare = tall * 256 - cols * rows_n;
        if (cols < 1 || cols >= tiles_n) continue;
        const int64_t low = (int64_t)((p.M + 32 * f.fm - 1) / (32 * f.fm)) * (tiles_n - cols) - (int64_t)spare * (int)(a / b);
        const double cost = 7 + tall * a + (double)((std::max<int64_t>(low, 0) + 255) / 256) * b;
        if (cost < best.cost) best = MidPlan{MID_WREG, 8, 1, all_steps, cost, f.fm, tiles_n - cols};
      }
    }
  }
  // gemm_stream_kernel: 128-column tiles of 64 to 192 rows, alone on a CU.  A 128-column slice of K takes what its LDS traffic or
  // the workgroups' share of the weight stream takes (row tiles after the first find most of it in L2); every term fitted to
  // 5600 timings of 16 products of 81 to 512 rows (median error 5 %).  Rotary operands always leave as partial sums, so a form that
  // needs no K ranges and no second pass keeps them (700 x 4096 x 2048, K and V of 8 layers: 35.4 us a call, 38.8 here; 130 x
  // 8192 x 1024 24.2 and 27.5; with K ranges in the other form this one was ahead in all of 57 products).
  // What it is worth, us (the forms above -> this one), fragment order: 160 x 28672 x 4096 67 -> 56, 192 x 4096 x 4096 18.9 -> 13.8,
  // 256 x 3072 x 2048 10.0 -> 8.6, but 256 x 28672 x 4096 68 against 81; row-major: 160 x 28672 x 4096 84 -> 56, 160 x 4096 x
  // 4096 20.7 -> 13.4, 160 x 4096 x 14336 39 -> 33, 333 x 8192 x 4096 53 -> 32.
  const bool rope = epi == EPI_QKV || epi == EPI_KV;
  if ((packed || p.streamed) && p.M < 1024 && p.K % 128 == 0 && !far && !norm_out && !(packed && epi == EPI_STORE_F32) && !(rope && best.n_splits == 1)) {
    static const double slice_us[] = {0.83, 0.92, 1.09, 1.32, 1.44};
    const int slices = p.K / 128;
    // (the fixed part of the packed forms' model is 12 us above what 600 products of these sizes take; of 376 of 520 to 1023 rows this
    // choice makes 3 slower by more than 2 %, all together 0.91 of the time)
    const double other = best.kernel == MID_NONE ? 1e30 : packed ? 1.05 * best.cost - 11.5 : best.cost;
    MidPlan stream{};
    for (int fm = 2; fm <= 6; ++fm) {
      const int64_t rows_n = (p.M + 32 * fm - 1) / (32 * fm), tiles = rows_n * ((p.N + 127) / 128);
      for (int want = 1; want <= std::min(MID_MAX_SPLIT, slices); ++want) {
        if ((want > 1 || rope) && !p.partial) break;
        const int per = (slices + want - 1) / want, s = (slices + per - 1) / per;
        if (s != want) continue;
        const size_t bytes = s > 1 || rope ? (size_t)s * p.M * p.N * 4 : 0;
        if (bytes > p.partial_bytes) break;
        const double wgs = (double)(tiles * s), rounds = std::ceil(wgs / 256);
        const double hbm_us = std::min(wgs, 256.0) * 32768 * (0.23 + 0.77 / rows_n) / 5.2e6;
        const double out = bytes ? 1.7 * bytes + (consumer ? 0 : 20e6) : (double)p.M * p.N * (epi == EPI_RESID ? 8 : epi == EPI_STORE_F32 ? 4 : 1);   // at 4 TB/s
        const double cost = 1.7 + rounds * per * std::max(slice_us[fm - 2], hbm_us) + out / 4.0e6;
        if (stream.kernel == MID_NONE || cost < stream.cost) stream = MidPlan{MID_STREAM, fm, s, 2 * per, cost};
      }
    }
    if (stream.kernel != MID_NONE && 1.05 * stream.cost < other) return stream;
  }
  // Row-major weights also have the 128 x 128 tile of gemm.hip (no K splits).  With scratch for splits it keeps up only
  // over many columns.  Without, it is the better one nearly everywhere: a lone workgroup on a CU takes 1.03 us per step,
  // the forms above 1.2 and more, two on one CU 1.31 (us, forms above -> tile: 128 x 8192 x 8192 155 -> 137, 333 x 11008 x
  // 4096 93 -> 78, 1023 x 4096 x 11008 203 -> 179), unless its last round is nearly empty (700 x 11008 x 4096 103 against 138).
  if (!packed && best.kernel != MID_NONE) {
    const int64_t tiles = (int64_t)((p.M + 127) / 128) * ((p.N + 127) / 128), last = tiles % 512;
    if (p.partial) {
      if (tiles >= 384 && 10 + (double)((tiles + 511) / 512) * all_steps * 1.22 < best.cost) best.kernel = MID_NONE;
    } else {
      const double rounds = 1.31 * (tiles / 512) + (last == 0 ? 0 : 1.03 + 0.28 * std::max<int64_t>(0, last - 256) / 256);
      if (8 + all_steps * rounds < 1.03 * best.cost) best.kernel = MID_NONE;
    }
  }
  return best;
}

int launch_gemm_mid(const GemmParams &p0, int epi, const MidPlan &pl, hipStream_t st) {
  GemmParams p = p0;
  p.n_splits = pl.n_splits; p.split_steps = pl.split_steps; p.low_tiles_n = pl.low_tiles_n;
  if (p.n_splits_out) *p.n_splits_out = 1;
  const bool rope = epi == EPI_QKV || epi == EPI_KV;
  if (pl.n_splits == 1 && !(rope && pl.kernel == MID_STREAM)) return launch_one(p, epi, pl, st);
  GemmParams q = p;
  q.C = p.partial; q.ldc = p.N;
  if (!rope) q.head_dim = 0;   // the packed order of rotary operands is theirs alone
  if (int e = launch_one(q, EPI_PARTIAL, pl, st)) return e;
  if (p.n_splits_out) { *p.n_splits_out = pl.n_splits; return 0; }
  if (rope && p.sums_left) { *p.sums_left = pl.n_splits; return 0; }
  return launch_splits_finish(p, epi, st);
}

// p.partial holds p.n_splits partial results [split][M][N] of C: added in split order, then the epilogue
int launch_splits_finish(const GemmParams &p, int epi, hipStream_t st) {
  switch (epi) {
    case EPI_STORE_BF16: launch_finish<EPI_STORE_BF16>(p, st); return 0;
    case EPI_STORE_F32: launch_finish<EPI_STORE_F32>(p, st); return 0;
    case EPI_RESID: launch_finish<EPI_RESID>(p, st); return 0;
    case EPI_SWIGLU: launch_finish<EPI_SWIGLU>(p, st); return 0;
    case EPI_QKV: launch_rope_finish<EPI_QKV>(p, st); return 0;
    case EPI_KV: launch_rope_finish<EPI_KV>(p, st); return 0;
  }
  return -1;
}
