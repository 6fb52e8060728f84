// Residual GEMM of very few rows (the last-token tail of a few sequences, small decode steps):
//   h[M, N] += A[M, K] * W[N, K]^T      (h fp32), and with it the operand of the projection behind the next RMSNorm.
//
// The weight-streaming kernels split K over workgroups here, whose partial sums a norm pass of one workgroup per row adds up: 3.9 to 5 us
// in which nothing streams, twice a layer.  Here the eight waves of a workgroup split K and meet in LDS, so a workgroup's 16
// columns are final: it updates h, leaves bf16(h * gain) for the next projection and each row's sum of squares over its columns, from
// which that projection (skinny_ring_kernel with SkinnyParams::ssq) takes 1/rms as a factor of its result.  No norm pass.
// A wave streams its K range of the block's 16 weight rows and of the activation rows through a ring of its own by LDS-DMA in
// whole 128-byte pieces (eight rows to a request) and issues no other vector-memory request in the loop, so a counted wait is exact; no
// barrier until the end.  Every workgroup reads all activation rows (from L2), which is why the rows are few.
#include "common.h"

#include <cmath>

namespace {

constexpr int SR_WAVES = 8;
constexpr int SR_STEPS = 3;                // 64-column steps in a wave's ring (two or four: no different)
constexpr int SR_SLOT = 3 * 1024;          // of a step: 16 weight rows, 8 activation rows
constexpr int SR_LDS = SR_WAVES * SR_STEPS * SR_SLOT;   // 72 KB: two workgroups to a CU

__global__ __launch_bounds__(SR_WAVES * 64) void skinny_resid_kernel(SkinnyResidParams p) {
  constexpr int R = SR_STEPS, NREQ = 3;
  extern __shared__ __align__(16) unsigned char lds[];   // [wave][R][2 KB weights, 1 KB activations]; at the end [wave][1 KB] sums
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kq = lane >> 4;
  const int n0 = blockIdx.x * 16;

  // what the finishing threads need besides the sums: requested first, used last
  const int fm = tid >> 4, fn = n0 + (tid & 15);   // this thread's row and column
  const bool fin = fm < p.M;
  float h = 0.f, g = 1.f, g_tail = 1.f;
  if (fin) {
    h = p.h[(int64_t)fm * p.N + fn];
    if (p.gain) g = bf16_to_f32(p.gain[fn]);
    if (p.h_tail) g_tail = bf16_to_f32(p.gain_tail[fn]);
  }

  const int all = p.K / 64, per = (all + SR_WAVES - 1) / SR_WAVES, s0 = wave * per;
  const int steps = all - s0 < per ? (all - s0 > 0 ? all - s0 : 0) : per;
  floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
  typedef __attribute__((address_space(3))) void *lds_ptr_t;
  const unsigned ring = (unsigned)(size_t)(lds_ptr_t)lds + wave * (R * SR_SLOT);
  const unsigned char *ring_p = lds + wave * (R * SR_SLOT);
  if (steps > 0) {
    // request h of a piece: rows 8 h + r8; chunk c of row r lies at chunk c ^ ((r >> 1) & 7)
    const int r8 = lane >> 3, c0 = (lane & 7) ^ (lane >> 4), c1 = c0 ^ 4;
    const unsigned row_bytes = (unsigned)p.K * 2;
    const unsigned w0 = r8 * row_bytes + c0 * 16, w1 = (8 + r8) * row_bytes + c1 * 16;
    const unsigned a0 = (unsigned)(r8 < p.M ? r8 : p.M - 1) * row_bytes + c0 * 16;   // rows past M repeat row M - 1
    const unsigned char *wb = (const unsigned char *)(p.W + (int64_t)n0 * p.K) + (int64_t)s0 * 128, *ab = (const unsigned char *)p.A + (int64_t)s0 * 128;
    int next = (int)(blockIdx.x / 8) % steps;   // (neighbours of a die start a step apart: rows 2^13 bytes apart lie on few memory channels)
    auto request = [&](int slot) __attribute__((always_inline)) {
      const unsigned dst = ring + slot * SR_SLOT;
      lds_dma16_at(wb + (int64_t)next * 128, w0, dst);
      lds_dma16_at(wb + (int64_t)next * 128, w1, dst + 1024);
      lds_dma16_at(ab + (int64_t)next * 128, a0, dst + 2048);
      next = next + 1 == steps ? 0 : next + 1;
    };
#pragma unroll
    for (int i = 0; i < R; ++i) if (i < steps) request(i);
    const int wf = l16 * 128 + ((kq ^ (l16 >> 1)) << 4), ar = l16 & 7, af = 2048 + ar * 128 + ((kq ^ (ar >> 1)) << 4);
    int slot = 0;
    for (int s = 0; s < steps; ++s) {
      const int younger = steps - 1 - s;
      if (younger >= R - 1) wait_vm<NREQ * (R - 1)>();
      else if (younger == 1) wait_vm<NREQ>();
      else wait_vm<0>();
      asm volatile("" ::: "memory");
      const unsigned char *at = ring_p + slot * SR_SLOT;
      bf16x8 w[2], x[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) { w[u] = *(const bf16x8 *)(at + (wf ^ (u * 64))); x[u] = *(const bf16x8 *)(at + (af ^ (u * 64))); }
#pragma unroll
      for (int u = 0; u < 2; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[u], x[u], acc, 0, 0, 0);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // every read of the slot has returned
      if (s + R < steps) request(slot);
      slot = slot + 1 == R ? 0 : slot + 1;
    }
  }
  // acc[v] = this K range's sum of C[m = l16][n0 + 4 kq + v]; columns m >= 8 of the product repeat the others
  float *mine = (float *)(lds + wave * (R * SR_SLOT));
  *(float4 *)(mine + l16 * 16 + 4 * kq) = make_float4(acc[0], acc[1], acc[2], acc[3]);
  __syncthreads();
  if (!fin) return;   // (whole groups of 16 lanes)
  float x = 0.f;
#pragma unroll
  for (int w = 0; w < SR_WAVES; ++w) x += ((const float *)(lds + w * (R * SR_SLOT)))[tid];   // tid = 16 fm + column
  h += x;
  p.h[(int64_t)fm * p.N + fn] = h;
  if (p.out) p.out[(int64_t)fm * p.N + fn] = f32_to_bf16(h * g);
  if (p.h_tail) {
    p.h_tail[(int64_t)fm * p.N + fn] = h;
    p.out_tail[(int64_t)fm * p.N + fn] = f32_to_bf16(h * g_tail);
  }
  if (p.ssq) {
    float q = h * h;
    q += __shfl_xor(q, 1); q += __shfl_xor(q, 2); q += __shfl_xor(q, 4); q += __shfl_xor(q, 8);
    if ((tid & 15) == 0) p.ssq[(int64_t)fm * (p.N / 16) + blockIdx.x] = q;
  }
}

}  // namespace

// us per product: skinny_ring_kernel with its K ranges left to the norm pass -> this kernel; the norm pass (3.9 to 5.4) falls away.  One
// row: 4096 x 4096 8.2 -> 7.7, 4096 x 14336 21.6 -> 21.0, 2048 x 8192 8.3 -> 8.8, 8192 x 8192 23.3 -> 24.9, 8192 x 28672 78.3 -> 77.8, but
// 5120 x 13824 25.7 -> 30.3: with 320 column blocks 64 CUs have two and the others one.  So the blocks have to be at most one per CU, or
// their last round nearly full.  Eight rows: 21.8 -> 21.4, 2048 x 8192 8.5 -> 10.5; 16 rows (two requests for activations) 22.0 -> 23.8
// and 8.7 -> 12.4, not taken.
// Fewer than 256 blocks leave CUs without work while a wave walks K / 8, which the ring kernel's K ranges do not; more so with more rows
// in a step.  So K is bounded by the CUs left over and the rows; where K is far longer than N the chain loses whatever the rows.  The
// norm of a width that 1024 does not divide is two launches here (K ranges added by one), so there more K pays.  A pass of four layers
// against the form with norm passes, 1, 2, 4, 8 rows, K of down over N: 1024, 8192 0.88 0.83 0.88 0.95, 14336 0.97 0.98 1.00 1.03, 20480
// 1.03 1.04 1.06 1.11; 2048, 8192 0.92 0.93 0.95 0.97, 16384 0.96 0.97 0.98 1.02, 40960 1.04 1.05 1.06 1.08; 3072, 49152 0.98 0.99 1.00
// 1.03; 512, 16384 0.85 0.85 0.86 0.89, 32768 1.04 1.05 1.09 1.13; 1536, 32768 0.89 0.89 0.90 0.95, 49152 0.97 0.96 0.97 1.02.
bool skinny_resid_pays(int M, int N, int K) {
  if (M < 1 || M > SKINNY_RESID_ROWS || N % 16 != 0 || K % 64 != 0 || (uint64_t)16 * (uint64_t)K * 2 > 0xffffffffull) return false;   // (32-bit row offsets)
  const int blocks = N / 16;
  if (blocks > 256) return (blocks + 255) / 256 * 256 <= 1.15 * blocks;
  const double idle = 1 - blocks / 256.0;
  const bool one_norm = N % 1024 == 0;
  return K <= (one_norm ? 16 : 40) * (int64_t)N && K * std::pow(idle, 1.5) * (1 + 0.3 * M) <= (one_norm ? 19500 : 56000);
}
int launch_skinny_resid(const SkinnyResidParams &p, hipStream_t st) {
  static bool attr = false;
  if (!attr) {
    if (hipFuncSetAttribute((const void *)skinny_resid_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, SR_LDS) != hipSuccess) return -1;
    attr = true;
  }
  if (p.M < 1 || p.M > SKINNY_RESID_ROWS || p.N % 16 || p.K % 64) return -1;
  hipLaunchKernelGGL(skinny_resid_kernel, dim3(p.N / 16), dim3(SR_WAVES * 64), SR_LDS, st, p);
  return 0;
}
