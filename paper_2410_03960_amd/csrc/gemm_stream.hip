// bf16 MFMA GEMM for decode batches beyond 80 rows and short prompts:  C[M,N] = A[M,K] * W[N,K]^T, weights streamed.
//
// Up to 192 rows fit one tile of 32 FM rows x 128 columns, so every weight byte crosses the memory bus once and the launch is
// bound by that stream; what keeps it from its rate is the time a CU spends besides it.  The kernel is built like
// skinny_ring_kernel (skinny.hip): everything travels by LDS-DMA in whole 128-byte lines or 1 KB fragments, eight consumer
// waves each with a ring of its own for the weights, a producer wave for the activations, one barrier per 128
// columns of K.  Four waves side by side (32 columns each), twice: the two groups take alternate 64-column steps of K and meet in
// LDS at the end, so that on every SIMD a wave's fragment reads run under the other's products.
// Bounds: up to 128 rows the weight stream (128 x 28672 x 4096: 47 us, 5.0 TB/s), above the CU's LDS traffic -- a 128-column
// slice of 160 rows writes 72 KB and reads 192 KB, 1.0 us at 128 bytes per cycle, and takes 1.3.
#include "gemm_epilogue.h"

#include <algorithm>

namespace {


constexpr int ST_R = 2;   // 64-column steps in a wave's ring
constexpr int st_bufs(int FM) { return FM <= 4 ? 3 : 2; }   // activation buffers of 128 columns
constexpr int st_lds(int FM) { return st_bufs(FM) * 2 * 32 * FM * 128 + 8 * ST_R * 4096; }

template <int EPI, int FM, bool PACKED>
__global__ __launch_bounds__(9 * 64) void gemm_stream_kernel(GemmParams p) {
  constexpr int BM = 32 * FM, ASTEP = BM * 128, ABUF = 2 * ASTEP, NB = st_bufs(FM);
  extern __shared__ __align__(16) unsigned char lds[];   // [NB][2 steps][BM][128 bytes] activations, [8 waves][ST_R][4 KB] weights
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, g = lane >> 5;

  // Workgroup ids go round the eight dies.  Without K ranges so do the column tiles (neighbours in memory are read at the same
  // time; the row tiles of one share a die's L2), and a die's tiles start one slice apart.  With K ranges each die gets a run of
  // (K range, column tile, row tile), so that it needs few ranges of the activations (160 x 8192 x 28672: 138 -> 105 us; without
  // ranges the runs cost 2 to 10 %); runs are apart in memory by themselves, row-major ones less so.
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + 127) / 128, tiles = tiles_n * tiles_m;
  int split = 0, tm, tn, first;
  if (p.n_splits == 1) {
    first = blockIdx.x / 8 / tiles_m; tm = blockIdx.x / 8 % tiles_m; tn = first * 8 + blockIdx.x % 8;
    if (tn >= tiles_n) return;
  } else {
    const int total = tiles * p.n_splits, logical = blockIdx.x % 8 * ((total + 7) / 8) + blockIdx.x / 8;
    if (logical >= total) return;
    split = logical / tiles; tm = logical % tiles % tiles_m; tn = logical % tiles / tiles_m;
    first = PACKED ? 0 : tn;
  }
  const int m0 = tm * BM;
  const int all = p.K / 128, per = p.split_steps / 2, s0 = split * per;
  const int slices = all - s0 < per ? all - s0 : per;   // of 128 columns, >= 1 by the plan
  const int rot = first % slices;   // slice this workgroup starts with
  typedef __attribute__((address_space(3))) void *lds_ptr_t;
  const unsigned lds_base = (unsigned)(size_t)(lds_ptr_t)lds;
  // a request: 8 rows of 128 bytes; chunk c of row r lies at chunk c ^ ((r >> 1) & 7)
  const int r8 = lane >> 3, c0 = (lane & 7) ^ (lane >> 4), c1 = c0 ^ 4;   // even and odd requests

  if (wave == 8) {
    const unsigned lda = (unsigned)(p.lda * 2);
    int buf = 0, at = rot;
    auto fill = [&]() __attribute__((always_inline)) {
      const unsigned char *base = (const unsigned char *)p.A + (int64_t)(s0 + at) * 256;
#pragma unroll
      for (int i = 0; i < BM / 16; ++i) {
        const int ma = m0 + i * 16 + r8, mb = ma + 8;   // rows past M repeat row M - 1
        const unsigned oa = (unsigned)(ma < p.M ? ma : p.M - 1) * lda + c0 * 16, ob = (unsigned)(mb < p.M ? mb : p.M - 1) * lda + c1 * 16;
        const unsigned dst = lds_base + buf * ABUF + i * 2048;
#pragma unroll
        for (int st = 0; st < 2; ++st) {
          lds_dma16_at(base + st * 128, oa, dst + st * ASTEP);
          lds_dma16_at(base + st * 128, ob, dst + st * ASTEP + 1024);
        }
      }
      buf = buf + 1 == NB ? 0 : buf + 1;
      at = at + 1 == slices ? 0 : at + 1;
    };
#pragma unroll
    for (int s = 0; s < NB - 1; ++s) if (s < slices) fill();
    for (int s = 0; s <= slices; ++s) {
      if (s + NB - 2 < slices) wait_vm<(NB - 2) * 8 * FM>();   // slice s is in LDS, the younger ones may be on their way
      else wait_vm<0>();
      __builtin_amdgcn_s_barrier();   // buffer s is ready / the consumers have left buffer s - 1
      if (s + NB - 1 < slices) fill();
    }
    __builtin_amdgcn_s_barrier();   // (the meeting of the groups below)
    return;
  }

  const int cw = wave & 3, kg = wave >> 2;
  const int n0 = tn * 128 + cw * 32;
  const int n32 = (n0 < p.N ? n0 : p.N - 32) / 32;   // (blocks past N re-read the last one; their results are dropped)
  const unsigned char *wb[2];   // of the block's rows 0..15 and 16..31, or of its fragments
  unsigned o0, o1;
  if constexpr (PACKED) {
    wb[0] = (const unsigned char *)(p.wpack + ((int64_t)n32 * (p.K / 16) + (int64_t)s0 * 8 + kg * 4) * 512);
    o0 = o1 = lane * 16;
  } else {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      wb[h] = (const unsigned char *)((p.wtab ? p.wtab[n32 * 2 + h] : p.W + (int64_t)(n32 * 32 + h * 16) * p.ldw) + (int64_t)s0 * 128 + kg * 64);
    o0 = r8 * (unsigned)(p.ldw * 2) + c0 * 16; o1 = (8 + r8) * (unsigned)(p.ldw * 2) + c1 * 16;
  }
  const int ring_off = NB * ABUF + wave * (ST_R * 4096);
  int next = rot;   // slice of the next request
  auto request = [&](int slot) __attribute__((always_inline)) {
    const unsigned dst = lds_base + ring_off + slot * 4096;
    if constexpr (PACKED) {
      const unsigned char *src = wb[0] + (int64_t)next * 8192;
#pragma unroll
      for (int h = 0; h < 4; ++h) lds_dma16_at(src + h * 1024, o0, dst + h * 1024);
    } else {
#pragma unroll
      for (int h = 0; h < 4; ++h) lds_dma16_at(wb[h >> 1] + (int64_t)next * 256, h & 1 ? o1 : o0, dst + h * 1024);
    }
    next = next + 1 == slices ? 0 : next + 1;
  };
#pragma unroll
  for (int i = 0; i < ST_R; ++i) if (i < slices) request(i);

  floatx16 acc[FM];
#pragma unroll
  for (int bm = 0; bm < FM; ++bm)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[bm][v] = 0.f;
  const int a_lane = l32 * 128 + ((g ^ ((l32 >> 1) & 7)) << 4), w_lane = PACKED ? lane * 16 : a_lane;   // sub-step kk: XOR 32 kk
  int slot = 0, abuf = 0;
  __builtin_amdgcn_s_barrier();   // buffer 0 is in LDS
  for (int s = 0; s < slices; ++s) {
    const unsigned char *buf = lds + abuf * ABUF + kg * ASTEP;
    if (s + 1 < slices) wait_vm<4 * (ST_R - 1)>();
    else wait_vm<0>();
    asm volatile("" ::: "memory");
    const unsigned char *wr = lds + ring_off + slot * 4096;
    bf16x8 w[4], a[2][FM];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) w[kk] = *(const bf16x8 *)(wr + (PACKED ? w_lane + kk * 1024 : (w_lane ^ (kk * 32))));
#pragma unroll
    for (int bm = 0; bm < FM; ++bm) a[0][bm] = *(const bf16x8 *)(buf + a_lane + bm * 4096);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      if (kk < 3) {
#pragma unroll
        for (int bm = 0; bm < FM; ++bm) a[(kk + 1) & 1][bm] = *(const bf16x8 *)(buf + (a_lane ^ ((kk + 1) * 32)) + bm * 4096);
      }
#pragma unroll
      for (int bm = 0; bm < FM; ++bm) acc[bm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[kk], a[kk & 1][bm], acc[bm], 0, 0, 0);
      if (kk == 2) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // every read of the slot and of the buffer has returned
        if (s + ST_R < slices) request(slot);
      }
    }
    slot = slot + 1 == ST_R ? 0 : slot + 1;
    abuf = abuf + 1 == NB ? 0 : abuf + 1;
    __builtin_amdgcn_s_barrier();
  }

  // The two groups meet: group 1 hands over the first FM / 2 row blocks, group 0 the others, each finishes its own.
  constexpr int H = FM / 2;
  float4 *const low = (float4 *)lds + cw * H * 256 + lane, *const high = (float4 *)lds + (4 * H + cw * (FM - H)) * 256 + lane;
  float4 *const ex = kg == 0 ? high : low;
  const float4 *const in = kg == 0 ? low : high;
#pragma unroll
  for (int bm = 0; bm < FM; ++bm) {
    if ((bm < H) == (kg == 0)) continue;
    const int at = bm < H ? bm : bm - H;
#pragma unroll
    for (int q = 0; q < 4; ++q) ex[(at * 4 + q) * 64] = make_float4(acc[bm][4 * q], acc[bm][4 * q + 1], acc[bm][4 * q + 2], acc[bm][4 * q + 3]);
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  if (n0 >= p.N) return;
  // Rows leave through 32 x 32 blocks of fp32 in the wave's ring (row stride padded by 16 bytes), as whole row pieces.
  constexpr int RS = 32 * 4 + 16;
  static_assert(4 * FM * 4096 <= 2 * ABUF && 32 * RS <= ST_R * 4096, "exchange and slab");
  unsigned char *slab = lds + ring_off;
  // (the fragment order of rotary operands of 128-wide heads lists a head's 32-row blocks as 0, 2, 1, 3)
  int col = n0;
  if (PACKED && EPI == EPI_PARTIAL && p.head_dim == 128 && (((n0 >> 5) ^ (n0 >> 6)) & 1)) col = n0 ^ 96;
#pragma unroll
  for (int bm = 0; bm < FM; ++bm) {
    if ((bm < H) != (kg == 0)) continue;
    const int at = bm < H ? bm : bm - H;
#pragma unroll
    for (int q = 0; q < 4; ++q) {   // columns 8 q + 4 g .. + 3 of row l32; group 0's sum first
      const float4 o = in[(at * 4 + q) * 64];
      *(float4 *)(slab + l32 * RS + (8 * q + 4 * g) * 4) =
          make_float4(acc[bm][4 * q] + o.x, acc[bm][4 * q + 1] + o.y, acc[bm][4 * q + 2] + o.z, acc[bm][4 * q + 3] + o.w);
    }
    // a wave's LDS operations execute in order: the reads below see the writes above
    if constexpr (EPI == EPI_SWIGLU) {   // 16 gate columns, then the matching 16 up columns
      const int c4 = lane & 3;
#pragma unroll
      for (int it = 0; it < 2; ++it) {
        const int row = it * 16 + (lane >> 2), m = m0 + bm * 32 + row;
        const float4 g4 = *(const float4 *)(slab + row * RS + c4 * 16), u4 = *(const float4 *)(slab + row * RS + 64 + c4 * 16);
        const float rs = p.rstd ? p.rstd[m < p.M ? m : p.M - 1] : 1.f;
        const float gt[4] = {g4.x * rs, g4.y * rs, g4.z * rs, g4.w * rs}, up[4] = {u4.x * rs, u4.y * rs, u4.z * rs, u4.w * rs};
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = gt[e] * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * gt[e])) * up[e];   // silu(gate) * up
        if (m < p.M) *(uint2 *)((bf16_t *)p.C + (int64_t)m * p.ldc + n0 / 2 + c4 * 4) = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
      }
    } else {
      const int ch = lane & 7;
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int row = it * 8 + (lane >> 3), m = m0 + bm * 32 + row;
        const float4 x = *(const float4 *)(slab + row * RS + ch * 16);
        if (m >= p.M) continue;
        if constexpr (EPI == EPI_PARTIAL) {
          *(float4 *)((float *)p.C + ((int64_t)split * p.M + m) * p.N + col + ch * 4) = x;
        } else if constexpr (EPI == EPI_STORE_F32) {
          *(float4 *)((float *)p.C + (int64_t)m * p.ldc + n0 + ch * 4) = x;
        } else if constexpr (EPI == EPI_RESID) {
          float4 *dst = (float4 *)((float *)p.C + (int64_t)m * p.ldc + n0 + ch * 4);
          const float4 r = *dst;
          *dst = make_float4(r.x + x.x, r.y + x.y, r.z + x.z, r.w + x.w);
        } else {
          *(uint2 *)((bf16_t *)p.C + (int64_t)m * p.ldc + n0 + ch * 4) = make_uint2(pack_bf16x2(x.x, x.y), pack_bf16x2(x.z, x.w));
        }
      }
    }
  }
}

template <int EPI, int FM, bool PACKED>
int launch_k(const GemmParams &p, hipStream_t st) {
  auto kern = gemm_stream_kernel<EPI, FM, PACKED>;
  static bool attr = false;
  if (!attr) {
    if (hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, st_lds(FM)); e != hipSuccess) return (int)e;
    attr = true;
  }
  const int tiles_m = (p.M + 32 * FM - 1) / (32 * FM), tiles_n = (p.N + 127) / 128;
  const int dies = p.n_splits == 1 ? (tiles_n + 7) / 8 * tiles_m : (tiles_n * tiles_m * p.n_splits + 7) / 8;   // workgroups of each
  hipLaunchKernelGGL(kern, dim3(dies * 8), dim3(9 * 64), st_lds(FM), st, p);
  return 0;
}
template <int EPI>
int launch_e(const GemmParams &p, int fm, bool packed, hipStream_t st) {
  switch (fm) {
    case 2: return packed ? launch_k<EPI, 2, true>(p, st) : launch_k<EPI, 2, false>(p, st);
    case 3: return packed ? launch_k<EPI, 3, true>(p, st) : launch_k<EPI, 3, false>(p, st);
    case 4: return packed ? launch_k<EPI, 4, true>(p, st) : launch_k<EPI, 4, false>(p, st);
    case 5: return packed ? launch_k<EPI, 5, true>(p, st) : launch_k<EPI, 5, false>(p, st);
    case 6: return packed ? launch_k<EPI, 6, true>(p, st) : launch_k<EPI, 6, false>(p, st);
  }
  return -1;
}

}  // namespace

// tile of 32 * fm rows, p.n_splits K ranges of p.split_steps (even) 64-wide steps
int launch_gemm_stream(const GemmParams &p, int epi, int fm, bool packed, hipStream_t st) {
  switch (epi) {
    case EPI_STORE_BF16: return launch_e<EPI_STORE_BF16>(p, fm, packed, st);
    case EPI_STORE_F32: return packed ? -1 : launch_e<EPI_STORE_F32>(p, fm, false, st);
    case EPI_RESID: return launch_e<EPI_RESID>(p, fm, packed, st);
    case EPI_SWIGLU: return launch_e<EPI_SWIGLU>(p, fm, packed, st);
    case EPI_PARTIAL: return launch_e<EPI_PARTIAL>(p, fm, packed, st);
  }
  return -1;
}
