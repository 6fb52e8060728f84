// HBM-bound kernels of the SwiftKV prefill path: integer plan + RoPE table,
// embedding gather, row rstd, RMSNorm of a few rows, row gather, KV commit
// (paged scatter, FP8 quantise, V transpose), split-KV combine.
#include "common.h"

#include <algorithm>

// ---------------------------------------------------------------- plan -----
// One thread per (new token, rotary pair): sequence by binary search in
// cu_seqlens, absolute position, paged slot = block_table[b][p/16]*16 + p%16
// (written by the token's first thread), and the RoPE angle table
// cos/sin(p * theta^(-2i/hd)) formed in double precision.
__device__ __forceinline__ void plan_token(const PlanParams &p, const int64_t gid) {
  const int half = p.head_dim / 2;
  if (gid < p.B) p.last_rows[gid] = p.cu_seqlens[gid + 1] - 1;
  const int t = (int)(gid / half), i = (int)(gid % half);
  if (t >= p.T) return;
  int lo = 0, hi = p.B - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (p.cu_seqlens[mid] <= t) lo = mid; else hi = mid - 1;
  }
  const int b = lo;
  const int pos = p.context_lens[b] + (t - p.cu_seqlens[b]);
  if (i == 0) {
    int blk = p.block_tables[(int64_t)b * p.max_blocks_per_seq + pos / SKV_BLOCK];
    if (blk < 0 || blk >= p.n_blocks) {  // never let a bad table turn into a wild store
      atomicOr(p.err_flag, 1);
      blk = 0;
    }
    if (p.token_ids) {
      int id = p.token_ids[t];
      if (id < 0 || id >= p.vocab) atomicOr(p.err_flag, 2);
    }
    p.positions[t] = pos;
    p.seq_of[t] = b;
    p.slots[t] = (int64_t)blk * SKV_BLOCK + pos % SKV_BLOCK;
  }
  const double inv_freq = pow((double)p.rope_theta, -2.0 * (double)i / (double)p.head_dim);
  const double ang = (double)pos * inv_freq;
  p.cos_sin[(int64_t)t * half + i] = make_float2((float)cos(ang), (float)sin(ang));
}
__global__ void plan_kernel(PlanParams p) { plan_token(p, (int64_t)blockIdx.x * blockDim.x + threadIdx.x); }
static unsigned plan_blocks(const PlanParams &p) { return (unsigned)((std::max<int64_t>((int64_t)p.T * (p.head_dim / 2), p.B) + 255) / 256); }
int launch_plan(const PlanParams &p, hipStream_t st) {
  hipLaunchKernelGGL(plan_kernel, dim3(plan_blocks(p)), dim3(256), 0, st, p);
  return 0;
}

// --------------------------------------------------------------- embed -----
// h[t, :] = E[id[t], :] widened to fp32 (the residual stream is kept in fp32).
__global__ void embed_kernel(const int32_t *ids, const uint4 *E, float4 *h, int T, int chunks, int vocab) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)T * chunks) return;
  int t = (int)(i / chunks), c = (int)(i % chunks);
  int id = ids[t];
  id = id < 0 ? 0 : (id >= vocab ? vocab - 1 : id);
  const uint4 u = E[(int64_t)id * chunks + c];
  h[2 * i] = make_float4(bf16lo(u.x), bf16hi(u.x), bf16lo(u.y), bf16hi(u.y));
  h[2 * i + 1] = make_float4(bf16lo(u.z), bf16hi(u.z), bf16lo(u.w), bf16hi(u.w));
}
int launch_embed(const int32_t *ids, const bf16_t *E, float *h, int32_t T, int32_t d, int32_t vocab, hipStream_t st) {
  int chunks = d / 8;
  int64_t n = (int64_t)T * chunks;
  hipLaunchKernelGGL(embed_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, ids, (const uint4 *)E, (float4 *)h, T, chunks, vocab);
  return 0;
}

// ---------------------------------------------------------------- rstd -----
// rstd[t] = rsqrt(mean(h[t,:]^2) + eps); one wave per row.
__global__ void rstd_kernel(const uint4 *h, float *rstd, int T, int chunks, float eps, float inv_d) {
  int row = blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64;
  int lane = threadIdx.x & 63;
  if (row >= T) return;
  const uint4 *r = h + (int64_t)row * chunks;
  float s = 0.f;
  for (int c = lane; c < chunks; c += 64) {
    uint4 u = r[c];
    float a;
    a = bf16lo(u.x); s += a * a; a = bf16hi(u.x); s += a * a;
    a = bf16lo(u.y); s += a * a; a = bf16hi(u.y); s += a * a;
    a = bf16lo(u.z); s += a * a; a = bf16hi(u.z); s += a * a;
    a = bf16lo(u.w); s += a * a; a = bf16hi(u.w); s += a * a;
  }
  s = wave_sum(s);
  if (lane == 0) rstd[row] = rsqrtf(s * inv_d + eps);
}
int launch_rstd(const bf16_t *h, float *rstd, int32_t T, int32_t d, float eps, hipStream_t st) {
  hipLaunchKernelGGL(rstd_kernel, dim3((T + 3) / 4), dim3(256), 0, st, (const uint4 *)h, rstd, T, d / 8, eps, 1.0f / (float)d);
  return 0;
}

// 1/rms from the per-block sums of squares the residual epilogue of the packed-weight GEMM leaves:
// ssq[t][b], b < n_blocks (a multiple of 4), added in block order (fixed order: results do not change
// from run to run).  One thread per row; its loads are independent of each other.
__global__ void rstd_from_ssq_kernel(const float4 *ssq, int n_quads, float *rstd, int T, float eps, float inv_d) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  const float4 *r = ssq + (int64_t)t * n_quads;
  float s = 0.f;
  for (int q0 = 0; q0 < n_quads; q0 += 8) {
    float4 v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = q0 + i < n_quads ? r[q0 + i] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int i = 0; i < 8; ++i) { s += v[i].x; s += v[i].y; s += v[i].z; s += v[i].w; }
  }
  rstd[t] = rsqrtf(s * inv_d + eps);
}
int launch_rstd_from_ssq(const float *ssq, int32_t n_blocks, float *rstd, int32_t T, int32_t d, float eps, hipStream_t st) {
  hipLaunchKernelGGL(rstd_from_ssq_kernel, dim3((T + 63) / 64), dim3(64), 0, st, (const float4 *)ssq, n_blocks / 4, rstd, T, eps, 1.0f / (float)d);
  return 0;
}

// ------------------------------------------------------- RMSNorm of rows ----
// fp32 rows -> bf16 GEMM operand; one wave per row.  With rstd_out the row factor is left to the
// consumer: out = bf16(h * gain), rstd_out[row] = 1/rms; else out = bf16(h * 1/rms * gain).
__device__ __forceinline__ uint2 norm4(const float4 u, const float rs, const bf16_t *gain, int c) {
  float g0 = 1.f, g1 = 1.f, g2 = 1.f, g3 = 1.f;
  if (gain) {
    const uint2 g = *(const uint2 *)(gain + 4 * c);
    g0 = bf16lo(g.x); g1 = bf16hi(g.x); g2 = bf16lo(g.y); g3 = bf16hi(g.y);
  }
  return make_uint2(pack_bf16x2(u.x * rs * g0, u.y * rs * g1), pack_bf16x2(u.z * rs * g2, u.w * rs * g3));
}
__global__ void rmsnorm_rows_kernel(const float4 *h, const bf16_t *gain, uint2 *out, int rows, int chunks, float eps, float inv_d, float *rstd_out) {
  int row = blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64;
  int lane = threadIdx.x & 63;
  if (row >= rows) return;
  const float4 *r = h + (int64_t)row * chunks;
  float s = 0.f;
  for (int c = lane; c < chunks; c += 64) {
    const float4 u = r[c];
    s += u.x * u.x; s += u.y * u.y; s += u.z * u.z; s += u.w * u.w;
  }
  s = wave_sum(s);
  const float rs = rsqrtf(s * inv_d + eps);
  if (rstd_out && lane == 0) rstd_out[row] = rs;
  const float f = rstd_out ? 1.f : rs;
  for (int c = lane; c < chunks; c += 64) out[(int64_t)row * chunks + c] = norm4(r[c], f, gain, c);
}
// Single-pass variant: the row (d = 256 * CH elements) stays in registers between the reduction and the
// scaling; the gains are requested together with the row (asked for only after the reduction they were a
// second memory latency, which is most of the time of the few-row launches of decode steps and the tail).
template <int CH>
__global__ __launch_bounds__(256) void rmsnorm_rows_reg_kernel(const float4 *h, const bf16_t *gain, uint2 *out, int rows, float eps, float inv_d, float *rstd_out) {
  const int row = blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64;
  const int lane = threadIdx.x & 63;
  if (row >= rows) return;
  const float4 *r = h + (int64_t)row * (CH * 64);
  float4 u[CH];
  uint2 g[CH];
#pragma unroll
  for (int i = 0; i < CH; ++i) u[i] = r[i * 64 + lane];
#pragma unroll
  for (int i = 0; i < CH; ++i) g[i] = gain ? *(const uint2 *)(gain + 4 * (i * 64 + lane)) : make_uint2(0x3f803f80u, 0x3f803f80u);   // bf16 ones
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < CH; ++i) { s += u[i].x * u[i].x; s += u[i].y * u[i].y; s += u[i].z * u[i].z; s += u[i].w * u[i].w; }
  s = wave_sum(s);
  const float rs = rsqrtf(s * inv_d + eps);
  if (rstd_out && lane == 0) rstd_out[row] = rs;
  const float f = rstd_out ? 1.f : rs;
#pragma unroll
  for (int i = 0; i < CH; ++i)
    out[(int64_t)row * (CH * 64) + i * 64 + lane] =
        make_uint2(pack_bf16x2(u[i].x * f * bf16lo(g[i].x), u[i].y * f * bf16hi(g[i].x)), pack_bf16x2(u[i].z * f * bf16lo(g[i].y), u[i].w * f * bf16hi(g[i].y)));
}
// Few rows (decode steps, the tail): one workgroup per row, d = 256 * WAVES * CQ.  With n_splits > 1
// the row first takes the sums of the K splits a weight-streaming GEMM left in `partial` ([n_splits][rows][d]
// fp32): the splits are added in order, then to the row, which is written back.  The sum of squares is added
// over a lane's values in order, then over the wave, then over the waves in order.
// SRC: where the row comes from -- h itself; 1: the embedding row of its token id; 2: row idx[row] of another buffer.
// The latter two leave it in h: the first norm of a pass and of the tail need no launch in front of them that only
// copies (about 4.5 us each where rows are few; 8831 rows of 4096 from the embedding 70 us in two launches -> 46).
// TAIL: rows that are the last of their sequence leave their tail's rows and operand as well, a launch of 4.6 to 5.4 us less (SRC = 2); us
// per pass: 512 new rows 928.7 -> 924.5, 333 648.6 -> 646.0, 160 decode rows 870.3 -> 868.0, 64 868.1 -> 866.8.
template <int CQ, int SRC, int WAVES, bool TAIL = false>
__device__ __forceinline__ void rmsnorm_row_wg(const int row, float4 *h, const bf16_t *gain, uint2 *out, int rows, float eps, float inv_d,
                                               float *rstd_out, const float4 *partial, int n_splits, const RowSource &rs_in, const TailRows &tail = TailRows{}) {
  constexpr int TH = WAVES * 64;
  __shared__ float red[WAVES];
  const int tid = threadIdx.x;
  int seq = -1;
  if constexpr (TAIL) {
    const int s = tail.seq_of[row];
    if (tail.last_rows[s] == row) seq = s;
  }
  float4 *r = h + (int64_t)row * (CQ * TH);
  float4 u[CQ];
  uint2 g[CQ];
  if constexpr (SRC == 1) {
    int id = rs_in.idx[row];
    id = id < 0 ? 0 : (id >= rs_in.n ? rs_in.n - 1 : id);   // (the plan reported it)
    const uint2 *e = (const uint2 *)rs_in.rows + (int64_t)id * (CQ * TH) + tid;
#pragma unroll
    for (int i = 0; i < CQ; ++i) {
      const uint2 x = e[i * TH];
      u[i] = make_float4(bf16lo(x.x), bf16hi(x.x), bf16lo(x.y), bf16hi(x.y));
    }
  } else {
    const float4 *from = SRC == 2 ? (const float4 *)rs_in.rows + (int64_t)rs_in.idx[row] * (CQ * TH) : r;
#pragma unroll
    for (int i = 0; i < CQ; ++i) u[i] = from[i * TH + tid];
  }
#pragma unroll
  for (int i = 0; i < CQ; ++i) g[i] = gain ? *(const uint2 *)(gain + 4 * (i * TH + tid)) : make_uint2(0x3f803f80u, 0x3f803f80u);
  if (SRC != 0) {
#pragma unroll
    for (int i = 0; i < CQ; ++i) r[i * TH + tid] = u[i];
  } else if (n_splits > 1) {
    float4 sum[CQ];
#pragma unroll
    for (int i = 0; i < CQ; ++i) sum[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 *pr = partial + (int64_t)row * (CQ * TH) + tid;
    const int64_t step = (int64_t)rows * (CQ * TH);
    int ks = 0;
    constexpr int AT = CQ <= 2 && WAVES > 4 ? 4 : 2;
    for (; ks + AT <= n_splits; ks += AT) {   // AT splits' loads in flight, added in split order
      float4 v[AT][CQ];
#pragma unroll
      for (int j = 0; j < AT; ++j)
#pragma unroll
        for (int i = 0; i < CQ; ++i) v[j][i] = pr[(ks + j) * step + i * TH];
#pragma unroll
      for (int j = 0; j < AT; ++j)
#pragma unroll
        for (int i = 0; i < CQ; ++i) { sum[i].x += v[j][i].x; sum[i].y += v[j][i].y; sum[i].z += v[j][i].z; sum[i].w += v[j][i].w; }
    }
    for (; ks < n_splits; ++ks) {
#pragma unroll
      for (int i = 0; i < CQ; ++i) {
        const float4 v = pr[ks * step + i * TH];
        sum[i].x += v.x; sum[i].y += v.y; sum[i].z += v.z; sum[i].w += v.w;
      }
    }
#pragma unroll
    for (int i = 0; i < CQ; ++i) {
      u[i].x += sum[i].x; u[i].y += sum[i].y; u[i].z += sum[i].z; u[i].w += sum[i].w;
      r[i * TH + tid] = u[i];
    }
  }
  uint2 tg[CQ];
  if (TAIL && seq >= 0) {
#pragma unroll
    for (int i = 0; i < CQ; ++i) { tg[i] = *(const uint2 *)(tail.gain + 4 * (i * TH + tid)); tail.h[(int64_t)seq * (CQ * TH) + i * TH + tid] = u[i]; }
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < CQ; ++i) { s += u[i].x * u[i].x; s += u[i].y * u[i].y; s += u[i].z * u[i].z; s += u[i].w * u[i].w; }
  s = wave_sum(s);
  if ((tid & 63) == 0) red[tid >> 6] = s;
  __syncthreads();
  s = red[0];
#pragma unroll
  for (int w = 1; w < WAVES; ++w) s += red[w];
  const float rs = rsqrtf(s * inv_d + eps);
  if (rstd_out && tid == 0) rstd_out[row] = rs;
  const float f = rstd_out ? 1.f : rs;
#pragma unroll
  for (int i = 0; i < CQ; ++i)
    out[(int64_t)row * (CQ * TH) + i * TH + tid] =
        make_uint2(pack_bf16x2(u[i].x * f * bf16lo(g[i].x), u[i].y * f * bf16hi(g[i].x)), pack_bf16x2(u[i].z * f * bf16lo(g[i].y), u[i].w * f * bf16hi(g[i].y)));
  if (TAIL && seq >= 0) {
#pragma unroll
    for (int i = 0; i < CQ; ++i)
      tail.out[(int64_t)seq * (CQ * TH) + i * TH + tid] =
          make_uint2(pack_bf16x2(u[i].x * rs * bf16lo(tg[i].x), u[i].y * rs * bf16hi(tg[i].x)), pack_bf16x2(u[i].z * rs * bf16lo(tg[i].y), u[i].w * rs * bf16hi(tg[i].y)));
  }
}
template <int CQ, int SRC, int WAVES = 4>
__global__ __launch_bounds__(WAVES * 64) void rmsnorm_row_wg_kernel(float4 *h, const bf16_t *gain, uint2 *out, int rows, float eps, float inv_d,
                                                             float *rstd_out, const float4 *partial, int n_splits, RowSource rs_in) {
  rmsnorm_row_wg<CQ, SRC, WAVES>(blockIdx.x, h, gain, out, rows, eps, inv_d, rstd_out, partial, n_splits, rs_in);
}
template <int CQ, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void rmsnorm_row_tail_kernel(float4 *h, uint2 *out, int rows, float eps, float inv_d, float *rstd_out, const float4 *partial,
                                                               int n_splits, TailRows tail) {
  rmsnorm_row_wg<CQ, 0, WAVES, true>(blockIdx.x, h, nullptr, out, rows, eps, inv_d, rstd_out, partial, n_splits, RowSource{}, tail);
}
// The plan and the first norm of a pass in one launch: neither reads what the other writes.  The plan's workgroups come first, as a
// thread's power, sine and cosine in double precision outlast a row.  us of a whole pass, two launches ->
// one: one decode row 406.9 -> 404.4, 64 871.4 -> 867.9, 597 rows of 2048 over 16 layers 1350.7 -> 1344.7; 16384 rows of 4096 20 + 89 -> 103.
template <int CQ>
__global__ __launch_bounds__(256) void plan_norm_kernel(PlanParams p, int n_plan, float4 *h, const bf16_t *gain, uint2 *out, float eps, float inv_d, float *rstd_out,
                                                        RowSource rs_in) {
  if ((int)blockIdx.x < n_plan) plan_token(p, (int64_t)blockIdx.x * 256 + threadIdx.x);
  else rmsnorm_row_wg<CQ, 1, 4>(blockIdx.x - n_plan, h, gain, out, p.T, eps, inv_d, rstd_out, nullptr, 1, rs_in);
}
// the K-split sums of a weight-streaming GEMM added into fp32 rows (for row widths the kernel above does not cover)
__global__ void add_splits_kernel(float4 *h, const float4 *partial, int64_t n4, int n_splits) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n4) return;
  float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int ks = 0; ks < n_splits; ++ks) {
    const float4 v = partial[(int64_t)ks * n4 + i];
    sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
  }
  float4 u = h[i];
  u.x += sum.x; u.y += sum.y; u.z += sum.z; u.w += sum.w;
  h[i] = u;
}
#define SKV_EACH_CQ(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8)
int launch_plan_rmsnorm_embed(const PlanParams &p, const bf16_t *E, float *h, const bf16_t *gain, bf16_t *out, int32_t d, float eps, float *rstd_out,
                              hipStream_t st) {
  const float inv_d = 1.0f / (float)d;
  const unsigned n_plan = plan_blocks(p);
#define SKV_PLAN_NORM(CQ_)                                                                                                               \
  case CQ_ * 1024:                                                                                                                       \
    hipLaunchKernelGGL(plan_norm_kernel<CQ_>, dim3(n_plan + p.T), dim3(256), 0, st, p, (int)n_plan, (float4 *)h, gain, (uint2 *)out, eps, inv_d, \
                       rstd_out, RowSource{E, p.token_ids, p.vocab});                                                                    \
    return 0;
  switch (d) { SKV_EACH_CQ(SKV_PLAN_NORM) }
#undef SKV_PLAN_NORM
  launch_plan(p, st);   // (other row widths)
  launch_embed(p.token_ids, E, h, p.T, d, p.vocab, st);
  return launch_rmsnorm_rows(h, gain, out, p.T, d, eps, rstd_out, st);
}
int launch_rmsnorm_gather(const float *from, const int32_t *idx, float *h, const bf16_t *gain, bf16_t *out, int32_t rows, int32_t d, float eps,
                          hipStream_t st) {
  if (rows <= 0) return 0;
  const float inv_d = 1.0f / (float)d;
#define SKV_RMS_GATHER(CQ_)                                                                                                              \
  case CQ_ * 1024:                                                                                                                       \
    hipLaunchKernelGGL((rmsnorm_row_wg_kernel<CQ_, 2>), dim3(rows), dim3(256), 0, st, (float4 *)h, gain, (uint2 *)out, rows, eps, inv_d, \
                       (float *)nullptr, (const float4 *)nullptr, 1, RowSource{from, idx, 0});                                           \
    return 0;
  switch (d) { SKV_EACH_CQ(SKV_RMS_GATHER) }
#undef SKV_RMS_GATHER
  launch_gather_rows(from, idx, h, rows, d, st);
  return launch_rmsnorm_rows(h, gain, out, rows, d, eps, nullptr, st);
}
#undef SKV_EACH_CQ
int launch_rmsnorm_rows(float *h, const bf16_t *gain, bf16_t *out, int32_t rows, int32_t d, float eps, float *rstd_out, hipStream_t st,
                        const float *partial, int32_t n_splits, const TailRows *tail, bool *tail_done) {
  if (rows <= 0) return 0;
  const dim3 grid((rows + 3) / 4), block(256);
  const float inv_d = 1.0f / (float)d;
  if ((rows <= 256 || n_splits > 1) && d % 1024 == 0 && d / 1024 <= 8) {   // few rows, or K splits to add on the way: a workgroup per row
    // Bound by the latency of its loads, not by their bytes: up to 1024 rows (four workgroups per CU) one or two float4 per
    // thread and split, four splits in flight, instead of four waves with d / 1024 float4 and two splits (us, before -> now,
    // K ranges as the product in front leaves them: 24 rows of 8192 9.6 -> 5.1, 597 of 2048 8.0 -> 6.1, 64 of 4096 4.9 ->
    // 4.8).  Beyond, four waves: more rows than the CUs hold workgroups keep as many loads in flight.
    // (the tail's rows with a gain of one only: the norm in front of the fused K/V projection)
    const bool tails = tail && !gain;
    if (tails) *tail_done = true;
#define SKV_RMS_FORM(CQ_, WAVES_)                                                                                                  \
  do {                                                                                                                             \
    if (tails)                                                                                                                     \
      hipLaunchKernelGGL((rmsnorm_row_tail_kernel<CQ_, WAVES_>), dim3(rows), dim3(WAVES_ * 64), 0, st, (float4 *)h, (uint2 *)out, rows, eps, inv_d, rstd_out, \
                         (const float4 *)partial, n_splits, *tail);                                                                \
    else                                                                                                                           \
      hipLaunchKernelGGL((rmsnorm_row_wg_kernel<CQ_, 0, WAVES_>), dim3(rows), dim3(WAVES_ * 64), 0, st, (float4 *)h, gain, (uint2 *)out, rows, eps, inv_d, \
                         rstd_out, (const float4 *)partial, n_splits, RowSource{});                                                \
    return 0;                                                                                                                      \
  } while (0)
#define SKV_RMS_WIDE(D_, CQ_) case D_ / 1024: SKV_RMS_FORM(CQ_, D_ / 256 / CQ_);
    if (rows <= 1024) switch (d / 1024) {
      SKV_RMS_WIDE(2048, 1) SKV_RMS_WIDE(3072, 1) SKV_RMS_WIDE(4096, 1) SKV_RMS_WIDE(5120, 2) SKV_RMS_WIDE(6144, 2) SKV_RMS_WIDE(7168, 2) SKV_RMS_WIDE(8192, 2)
      default: break;
    }
#undef SKV_RMS_WIDE
#define SKV_RMS_WG(CQ_) case CQ_: SKV_RMS_FORM(CQ_, 4);
    switch (d / 1024) {
      SKV_RMS_WG(1) SKV_RMS_WG(2) SKV_RMS_WG(3) SKV_RMS_WG(4) SKV_RMS_WG(5) SKV_RMS_WG(6) SKV_RMS_WG(7) SKV_RMS_WG(8)
      default: break;
    }
#undef SKV_RMS_WG
#undef SKV_RMS_FORM
  }
  if (n_splits > 1) {   // otherwise: the splits in a pass of their own
    const int64_t n4 = (int64_t)rows * d / 4;
    hipLaunchKernelGGL(add_splits_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, st, (float4 *)h, (const float4 *)partial, n4, n_splits);
  }
#define SKV_RMS_CASE(CH_)                                                                                          \
  case CH_:                                                                                                        \
    hipLaunchKernelGGL(rmsnorm_rows_reg_kernel<CH_>, grid, block, 0, st, (const float4 *)h, gain, (uint2 *)out, rows, eps, inv_d, rstd_out); \
    return 0;
  if (d % 256 == 0) {
    switch (d / 256) {
      SKV_RMS_CASE(1) SKV_RMS_CASE(2) SKV_RMS_CASE(4) SKV_RMS_CASE(8) SKV_RMS_CASE(16) SKV_RMS_CASE(20) SKV_RMS_CASE(24) SKV_RMS_CASE(32)
      default: break;
    }
  }
#undef SKV_RMS_CASE
  hipLaunchKernelGGL(rmsnorm_rows_kernel, grid, block, 0, st, (const float4 *)h, gain, (uint2 *)out, rows, d / 4, eps, inv_d, rstd_out);
  return 0;
}

// ------------------------------------------- fold a norm gain into weights ----
// out[n, k] = bf16(W[n, k] * gain[k]): RMSNorm_j(x) W^T = rstd(x) * (x (W diag(g_j))^T), so the
// per-layer gain can live in the weights and only the row scale rstd is left for the GEMM epilogue.
__global__ void fold_gain_kernel(const uint4 *W, const uint4 *gain, uint4 *out, int64_t n_chunks, int chunks_per_row) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_chunks) return;
  uint4 u = W[i], g = gain[i % chunks_per_row], o;
  o.x = pack_bf16x2(bf16lo(u.x) * bf16lo(g.x), bf16hi(u.x) * bf16hi(g.x));
  o.y = pack_bf16x2(bf16lo(u.y) * bf16lo(g.y), bf16hi(u.y) * bf16hi(g.y));
  o.z = pack_bf16x2(bf16lo(u.z) * bf16lo(g.z), bf16hi(u.z) * bf16hi(g.z));
  o.w = pack_bf16x2(bf16lo(u.w) * bf16lo(g.w), bf16hi(u.w) * bf16hi(g.w));
  out[i] = o;
}
int launch_fold_gain(const bf16_t *W, const bf16_t *gain, bf16_t *out, int64_t rows, int32_t K, hipStream_t st) {
  int64_t n = rows * (K / 8);
  hipLaunchKernelGGL(fold_gain_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (const uint4 *)W, (const uint4 *)gain, (uint4 *)out, n, K / 8);
  return 0;
}

// -------------------------------------------------------------- gather -----
__global__ void gather_rows_kernel(const float4 *h, const int32_t *rows, float4 *out, int n_rows, int chunks) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)n_rows * chunks) return;
  int r = (int)(i / chunks), c = (int)(i % chunks);
  out[i] = h[(int64_t)rows[r] * chunks + c];
}
int launch_gather_rows(const float *h, const int32_t *rows, float *out, int32_t n_rows, int32_t d, hipStream_t st) {
  int chunks = d / 4;
  int64_t n = (int64_t)n_rows * chunks;
  hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (const float4 *)h, rows, (float4 *)out, n_rows, chunks);
  return 0;
}

__global__ void f32_to_bf16_kernel(const float4 *x, uint2 *out, int64_t n4) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n4) return;
  const float4 u = x[i];
  out[i] = make_uint2(pack_bf16x2(u.x, u.y), pack_bf16x2(u.z, u.w));
}
int launch_f32_to_bf16(const float *x, bf16_t *out, int64_t n, hipStream_t st) {   // n % 4 == 0
  if (n <= 0) return 0;
  hipLaunchKernelGGL(f32_to_bf16_kernel, dim3((unsigned)((n / 4 + 255) / 256)), dim3(256), 0, st, (const float4 *)x, (uint2 *)out, n / 4);
  return 0;
}

__global__ void fill_u32_kernel(uint32_t *p, uint32_t v, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
// One 16-byte chunk per thread: chunk id = ((block * K/16 + k16) * 64 + lane), lane = g*32 + l32.
// rope_hd == 128: inside every group of 128 rows (one head) the 32-row blocks are taken in the order
// 0, 2, 1, 3, so that a 64-row wave tile holds a block of the first half of the head next to its
// rotary partner block of the second half.
__global__ void pack_w_kernel(const bf16_t *const *wtab, const bf16_t *W, int64_t ldw, int32_t N, int32_t K, int32_t rope_hd, uint4 *out) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n_chunks = (int64_t)N * K / 8;
  if (id >= n_chunks) return;
  const int lane = (int)(id & 63);
  const int64_t frag = id >> 6;
  const int k16 = (int)(frag % (K / 16));
  int block = (int)(frag / (K / 16));
  if (rope_hd == 128) {
    const int b = block & 3;
    block = (block & ~3) | (b == 1 ? 2 : b == 2 ? 1 : b);
  }
  const int n = block * 32 + (lane & 31), k = k16 * 16 + (lane >> 5) * 8;
  const bf16_t *row = wtab ? wtab[n >> 4] + (int64_t)(n & 15) * ldw : W + (int64_t)n * ldw;
  const uint4 u = *(const uint4 *)(row + k);
  out[id] = u;
}
int launch_pack_w(const bf16_t *const *wtab, const bf16_t *W, int64_t ldw, int32_t N, int32_t K, int32_t rope_hd, bf16_t *out, hipStream_t st) {
  const int64_t n_chunks = (int64_t)N * K / 8;
  if (n_chunks <= 0) return 0;
  hipLaunchKernelGGL(pack_w_kernel, dim3((unsigned)((n_chunks + 255) / 256)), dim3(256), 0, st, wtab, W, ldw, N, K, rope_hd, (uint4 *)out);
  return 0;
}
int launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t st) {
  if (n <= 0) return 0;
  hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, v, n);
  return 0;
}

// ----------------------------------------------------------- KV commit -----
// One workgroup per (64-token tile, KV head).  Reads the tile's K and V rows
// (row-major, already rotated), stores them at their paged slots as bf16 or as
// e4m3 codes of x/scale, optionally writes the dequantised values back (so that
// attention sees exactly what the cache holds) and writes V transposed
// ([dim][token], 64-aligned columns, zero padded) for the prefill attention.
//
// What bounds it is instruction issue, so the conversions are the hardware's (x / scale below) and the transposition
// moves 16-byte chunks into LDS and 32-bit words out of it.  Before (IEEE division, codes by integer arithmetic, 16-bit
// LDS accesses) -> now, us: 512 tokens, 8 heads of 128, e4m3 13.7 -> 7.8, 8831 tokens 37.5 -> 21.1; V^T alone of 5666
// tokens 10.2 -> 7.4.

// x / s rounded as IEEE division does wherever the result decides an e4m3 code: two Newton steps on the product with the
// correctly rounded reciprocal leave the correctly rounded quotient (Markstein, IBM J. Res. Dev. 34, 1990).  From 1024
// on (infinities and NaN too) the code saturates whatever the last bits are.  Needs fast_scale(s).
__device__ __forceinline__ bool fast_scale(float s) { return s >= 0x1p-60f && s <= 0x1p60f; }
template <bool FAST>
__device__ __forceinline__ float quotient(float x, float s, float inv) {
  if (!FAST) return x / s;
  const float q0 = x * inv;
  const float q1 = __builtin_fmaf(__builtin_fmaf(-q0, s, x), inv, q0);
  const float q2 = __builtin_fmaf(__builtin_fmaf(-q1, s, x), inv, q1);
  return copysignf(fabsf(q0) < 1024.f ? q2 : q0, x);   // (the steps turn -0 into 0)
}
// the codes of four values, as f32_to_e4m3fn gives them (NaN and everything past 448 to the largest code of its sign)
__device__ __forceinline__ uint32_t four_codes(float a, float b, float c, float d) {
  auto sat = [](float x) { return copysignf(fminf(fabsf(x), 448.f), x); };
  const int lo = __builtin_amdgcn_cvt_pk_fp8_f32(sat(a), sat(b), 0, false);
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(sat(c), sat(d), lo, true);
}
// eight bf16 values -> eight codes of x / s, and the bf16 values they stand for in place
template <bool FAST>
__device__ __forceinline__ uint2 quantize8(uint4 &x, float s, float inv) {
  uint32_t w[4] = {x.x, x.y, x.z, x.w}, c[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    c[h] = four_codes(quotient<FAST>(bf16lo(w[2 * h]), s, inv), quotient<FAST>(bf16hi(w[2 * h]), s, inv),
                      quotient<FAST>(bf16lo(w[2 * h + 1]), s, inv), quotient<FAST>(bf16hi(w[2 * h + 1]), s, inv));
    w[2 * h] = pack_bf16x2(__builtin_amdgcn_cvt_f32_fp8((int)c[h], 0) * s, __builtin_amdgcn_cvt_f32_fp8((int)c[h], 1) * s);
    w[2 * h + 1] = pack_bf16x2(__builtin_amdgcn_cvt_f32_fp8((int)c[h], 2) * s, __builtin_amdgcn_cvt_f32_fp8((int)c[h], 3) * s);
  }
  x = make_uint4(w[0], w[1], w[2], w[3]);
  return make_uint2(c[0], c[1]);
}
// A 64-row tile of V in LDS, chunk c of row r at c ^ (r / 8): whole chunks are written, and the words that eight rows of
// one dim pair give to eight lanes lie in different banks.
template <int HD>
__device__ __forceinline__ int v_chunk(int r, int c) { return r * (HD / 8) + (c ^ (r >> 3)); }
// V^T of the tile: a thread writes 8 consecutive tokens (16 bytes) of two dims
template <int HD>
__device__ __forceinline__ void store_vt(const uint4 *sv, bf16_t *vt, int64_t vt_ld, int tid) {
  for (int i = tid; i < HD / 2 * 8; i += 256) {
    const int dp = i / 8, tc = i % 8;
    uint32_t x[8], lo[4], hi[4];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = ((const uint32_t *)(sv + v_chunk<HD>(tc * 8 + e, dp / 4)))[dp & 3];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      lo[e] = (x[2 * e] & 0xffffu) | (x[2 * e + 1] << 16);
      hi[e] = (x[2 * e] >> 16) | (x[2 * e + 1] & 0xffff0000u);
    }
    bf16_t *dst = vt + (int64_t)(2 * dp) * vt_ld + tc * 8;
    *(uint4 *)dst = make_uint4(lo[0], lo[1], lo[2], lo[3]);
    *(uint4 *)(dst + vt_ld) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
  }
}
template <int HD>
__global__ __launch_bounds__(256) void kv_commit_kernel(CommitParams p) {
  constexpr int CH = HD / 8;  // 16-byte chunks per row
  __shared__ uint4 sv[64 * CH];
  const KVTile tile = p.tiles[blockIdx.x];
  const int head = blockIdx.y;
  const int tid = threadIdx.x;
  float sk = 1.f, svs = 1.f;
  if (p.fp8 && !p.per_token) {
    if (p.compute_scale) {
      sk = fmaxf(__uint_as_float(p.amax[head]), 1e-12f) / 448.0f;
      svs = fmaxf(__uint_as_float(p.amax[p.n_kv_heads + head]), 1e-12f) / 448.0f;
      if (blockIdx.x == 0 && tid == 0) {
        p.scales[head] = sk;
        p.scales[p.n_kv_heads + head] = svs;
      }
    } else {
      sk = p.scales[head];
      svs = p.scales[p.n_kv_heads + head];
    }
  }
  // everything this thread reads is requested before its first store (loads and stores share one
  // counter: a load issued after a store would wait for that store to reach memory)
  constexpr int NI = 64 * CH / 256;
  uint4 kin[NI], vin[NI];
  int64_t slot_in[NI];
  float sk_in[NI], sv_in[NI];
#pragma unroll
  for (int ii = 0; ii < NI; ++ii) {
    const int i = tid + ii * 256, r = i / CH, c = i % CH;
    kin[ii] = make_uint4(0, 0, 0, 0); vin[ii] = make_uint4(0, 0, 0, 0);
    slot_in[ii] = 0; sk_in[ii] = sk; sv_in[ii] = svs;
    if (r < tile.n_valid) {
      const int64_t row = tile.row0 + r;
      if (p.cache_k) kin[ii] = *(const uint4 *)(p.k_src + row * p.ld_src + head * HD + c * 8);   // (no cache: only V^T is wanted)
      vin[ii] = *(const uint4 *)(p.v_src + row * p.ld_src + head * HD + c * 8);
      if (p.cache_k) slot_in[ii] = p.slots[row];
      if (p.per_token) { sk_in[ii] = p.scales[p.slots[row]]; sv_in[ii] = p.scales[p.n_slots + p.slots[row]]; }
    }
  }
  float isk = 1.f / sk, isv = 1.f / svs;
#pragma unroll
  for (int ii = 0; ii < NI; ++ii) {
    const int i = tid + ii * 256;
    int r = i / CH, c = i % CH;
    uint4 kq = kin[ii], vq = vin[ii];
    if (r < tile.n_valid) {
      int64_t row = tile.row0 + r;
      bf16_t *kp = p.k_src + row * p.ld_src + head * HD + c * 8;
      bf16_t *vp = p.v_src + row * p.ld_src + head * HD + c * 8;
      int64_t dst = (slot_in[ii] * p.n_kv_heads + head) * HD + c * 8;
      sk = sk_in[ii]; svs = sv_in[ii];
      if (!p.cache_k) {
        // no cache wanted (stand-alone attention): only V^T is produced
      } else if (!p.fp8) {
        *(uint4 *)((bf16_t *)p.cache_k + dst) = kq;
        *(uint4 *)((bf16_t *)p.cache_v + dst) = vq;
      } else {
        if (p.per_token) { isk = 1.f / sk; isv = 1.f / svs; }
        uint2 kc, vc;
        if (fast_scale(sk) && fast_scale(svs)) { kc = quantize8<true>(kq, sk, isk); vc = quantize8<true>(vq, svs, isv); }
        else { kc = quantize8<false>(kq, sk, isk); vc = quantize8<false>(vq, svs, isv); }
        *(uint2 *)((uint8_t *)p.cache_k + dst) = kc;
        *(uint2 *)((uint8_t *)p.cache_v + dst) = vc;
        if (p.writeback) {
          *(uint4 *)kp = kq;
          *(uint4 *)vp = vq;
        }
      }
    }
    if (p.vt) sv[v_chunk<HD>(r, c)] = vq;
  }
  if (!p.vt || tile.vt_col0 < 0) return;
  __syncthreads();
  store_vt<HD>(sv, p.vt + (int64_t)(head * HD) * p.vt_ld + tile.vt_col0, p.vt_ld, tid);
}
int launch_kv_commit(const CommitParams &p, hipStream_t st) {
  if (p.n_tiles <= 0) return 0;
  dim3 grid(p.n_tiles, p.n_kv_heads);
  if (p.head_dim == 128) hipLaunchKernelGGL(kv_commit_kernel<128>, grid, dim3(256), 0, st, p);
  else hipLaunchKernelGGL(kv_commit_kernel<64>, grid, dim3(256), 0, st, p);
  return 0;
}

// -------------------------------------------------------- token scales -----
// One wave per token: absmax of its K row and of its V row (bf16 values as they will be stored),
// scale = max(absmax, 1e-12) / 448 written at the token's cache slot.
__global__ __launch_bounds__(256) void token_scale_kernel(TokenScaleParams p) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= p.T) return;
  float ak = 0.f, av = 0.f;
  for (int c = lane; c < p.kv_dim / 8; c += 64) {
    const uint4 k = *(const uint4 *)(p.k_src + (int64_t)row * p.ld_src + c * 8);
    const uint4 v = *(const uint4 *)(p.v_src + (int64_t)row * p.ld_src + c * 8);
    const uint32_t kw[4] = {k.x, k.y, k.z, k.w}, vw[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      ak = fmaxf(ak, fmaxf(fabsf(bf16lo(kw[e])), fabsf(bf16hi(kw[e]))));
      av = fmaxf(av, fmaxf(fabsf(bf16lo(vw[e])), fabsf(bf16hi(vw[e]))));
    }
  }
  for (int o = 32; o > 0; o >>= 1) { ak = fmaxf(ak, __shfl_xor(ak, o)); av = fmaxf(av, __shfl_xor(av, o)); }
  if (lane == 0) {
    const int64_t slot = p.slots[row];
    p.scales[slot] = fmaxf(ak, 1e-12f) / 448.0f;
    p.scales[p.n_slots + slot] = fmaxf(av, 1e-12f) / 448.0f;
  }
}
int launch_token_scales(const TokenScaleParams &p, hipStream_t st) {
  if (p.T <= 0) return 0;
  hipLaunchKernelGGL(token_scale_kernel, dim3((p.T + 3) / 4), dim3(256), 0, st, p);
  return 0;
}

// --------------------------------------------- finishing pass of Q, K and V ----
// K-split Q, K, V (EPI_QKV) or later layers' K, V (EPI_KV): the partial sums added in split order, 1/rms, rotation, rounding
// once, and K and V straight to where they are read: bf16 rows, paged slots (bf16, e4m3 under given scales, e4m3 under the token's own
// scale, which the wave that holds the row finds on the way) and V^T columns.  Bound by the latency of its loads and stores.
// A wave takes 1024 columns of a row, 8 + 8 values of a rotary pair of chunks per lane, so that a row's partial sums are 32-byte pieces
// in flight together; V that is wanted transposed goes by 64-token tiles through LDS instead.  Before, a pass with one rotary pair per
// lane, a pass for the tokens' scales and the commit pass followed one another: 512 rows over an e4m3 cache with per-token scales,
// Q, K, V and two later layers 102 us in eight launches -> 25 in three, 333 rows in bf16 30 -> 18, 597 rows with 64-wide heads
// 12.7 a layer -> 6.0.
// NIT: rounds of 1024 columns a wave holds (per-token scales of more than 1024 K columns).
template <int EPI, int HD, int NIT>
__global__ __launch_bounds__(256) void kv_finish_kernel(GemmParams p, KvStore s, int vt_wgs, int q_units, int kv_units) {
  constexpr int CH = HD / 8, PAIRS = HD / 16;   // 16-byte chunks of a head; pairs of chunks (c, c + CH / 2)
  __shared__ uint4 sv[EPI == EPI_QKV ? 64 * CH : 1];
  const int tid = threadIdx.x, lane = tid & 63;
  const int n_kv = p.kv_dim / HD;
  const int64_t stride = (int64_t)p.M * p.N;
  // eight columns at each of N places, the splits' loads of all of them in flight together
  auto add_splits = [&](auto &src, auto &x) __attribute__((always_inline)) {
    constexpr int N = sizeof(x) / sizeof(x[0]);
    auto add = [&](int k, bool first) __attribute__((always_inline)) {
      float4 a[N][2];
#pragma unroll
      for (int i = 0; i < N; ++i) { a[i][0] = *(const float4 *)(src[i] + k * stride); a[i][1] = *(const float4 *)(src[i] + k * stride + 4); }
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const float v[8] = {a[i][0].x, a[i][0].y, a[i][0].z, a[i][0].w, a[i][1].x, a[i][1].y, a[i][1].z, a[i][1].w};
#pragma unroll
        for (int e = 0; e < 8; ++e) x[i][e] = first ? v[e] : x[i][e] + v[e];
      }
    };
    add(0, true);
    for (int k = 1; k < p.n_splits; ++k) add(k, false);
  };
  auto pack8 = [](const float (&x)[8]) __attribute__((always_inline)) {
    return make_uint4(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7]));
  };
  if constexpr (EPI == EPI_QKV) {
    if ((int)blockIdx.x < vt_wgs) {   // V of 64 tokens and one head: slots and V^T
      const KVTile tile = s.tiles[blockIdx.x / n_kv];
      const int head = blockIdx.x % n_kv;
      constexpr int NI = 64 * CH / 256;
      float x[NI][8], rs[NI];
      int64_t slot[NI];
      const float *src[NI];   // (rows past the tile's last repeat it)
#pragma unroll
      for (int ii = 0; ii < NI; ++ii) {
        const int i = tid + ii * 256, r = i / CH, c = i % CH, row = tile.row0 + (r < tile.n_valid ? r : tile.n_valid - 1);
        slot[ii] = p.slots[row];
        rs[ii] = p.rstd ? p.rstd[row] : 1.f;
        src[ii] = p.partial + (int64_t)row * p.N + p.q_dim + p.kv_dim + head * HD + c * 8;
      }
      add_splits(src, x);
#pragma unroll
      for (int ii = 0; ii < NI; ++ii)
#pragma unroll
        for (int e = 0; e < 8; ++e) x[ii][e] = (tid + ii * 256) / CH < tile.n_valid ? x[ii][e] * rs[ii] : 0.f;   // (V^T columns past the sequence are zero)
#pragma unroll
      for (int ii = 0; ii < NI; ++ii) {
        const int i = tid + ii * 256, r = i / CH, c = i % CH;
        const uint4 v = pack8(x[ii]);
        if (r < tile.n_valid) *(uint4 *)((bf16_t *)s.cache_v + (slot[ii] * n_kv + head) * HD + c * 8) = v;
        sv[v_chunk<HD>(r, c)] = v;
      }
      if (tile.vt_col0 < 0) return;
      __syncthreads();
      store_vt<HD>(sv, s.vt + (int64_t)(head * HD) * s.vt_ld + tile.vt_col0, s.vt_ld, tid);
      return;
    }
  }
  // a wave per (row, unit): units of q, then of K, then (V^T is not wanted) of V; EPI_KV: of K and of V of every projection
  const int units = EPI == EPI_QKV ? q_units + kv_units * (s.vt ? 1 : 2) : p.N / p.kv_dim * kv_units;
  const int id = __builtin_amdgcn_readfirstlane(((int)blockIdx.x - vt_wgs) * 4 + (tid >> 6));
  const int row = id / units, u = id % units;
  if (row >= p.M) return;
  int kind, part, proj = 0, col0;   // kind 0 = q, 1 = k, 2 = v; part: which 1024 columns; col0: column of the matrix in the sums
  if constexpr (EPI == EPI_QKV) {
    kind = u < q_units ? 0 : u < q_units + kv_units ? 1 : 2;
    part = u - (kind == 0 ? 0 : kind == 1 ? q_units : q_units + kv_units);
    col0 = kind == 0 ? 0 : kind == 1 ? p.q_dim : p.q_dim + p.kv_dim;
  } else {
    const int m = u / kv_units;
    proj = m / 2; kind = 1 + m % 2; part = u % kv_units;
    col0 = m * p.kv_dim;
  }
  const int dim = kind == 0 ? p.q_dim : p.kv_dim;
  const float rs = p.rstd ? p.rstd[row] : 1.f;
  const int64_t slot = kind == 0 ? 0 : p.slots[row];
  uint4 lo[NIT], hi[NIT];
  float amax = 0.f, head_scale = 1.f;   // (given scales: NIT = 1)
#pragma unroll
  for (int t = 0; t < NIT; ++t) {
    const int item = (part * NIT + t) * 64 + lane, head = item / PAIRS, c = item % PAIRS;
    lo[t] = hi[t] = make_uint4(0, 0, 0, 0);
    if (item * 16 >= dim) continue;
    const float *first = p.partial + (int64_t)row * p.N + col0 + head * HD + c * 8, *src[2] = {first, first + HD / 2};
    float4 cs[4];
    if (kind != 2) {
#pragma unroll
      for (int e = 0; e < 4; ++e) cs[e] = ((const float4 *)(p.cos_sin + (int64_t)row * (HD / 2) + c * 8))[e];
    }
    if (kind != 0 && s.kind == KV_STORE_GIVEN) head_scale = s.scales[(int64_t)proj * s.scale_stride + (kind == 2 ? n_kv : 0) + head];
    float x[2][8];
    add_splits(src, x);
    float(&x0)[8] = x[0], (&x1)[8] = x[1];
#pragma unroll
    for (int e = 0; e < 8; ++e) { x0[e] *= rs; x1[e] *= rs; }
    if (kind != 2) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        rotate_pair(x0[2 * e], x1[2 * e], cs[e].x, cs[e].y);
        rotate_pair(x0[2 * e + 1], x1[2 * e + 1], cs[e].z, cs[e].w);
      }
    }
    lo[t] = pack8(x0); hi[t] = pack8(x1);
    if (s.kind == KV_STORE_PER_TOKEN) {   // absmax of the values as stored
      const uint32_t w[8] = {lo[t].x, lo[t].y, lo[t].z, lo[t].w, hi[t].x, hi[t].y, hi[t].z, hi[t].w};
#pragma unroll
      for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fmaxf(fabsf(bf16lo(w[e])), fabsf(bf16hi(w[e]))));
    }
  }
  bf16_t *rows = nullptr;
  if (kind == 0) rows = p.q_out + (int64_t)row * p.q_dim;
  else if (EPI == EPI_QKV) rows = (kind == 1 ? p.k_out : p.v_out) + (int64_t)row * p.kv_dim;
  else if (p.stage) rows = p.stage + (int64_t)row * p.N + col0;
  const bool put_rows = rows && (kind == 0 || (s.rows & kind));
  float token_scale = 1.f;
  if (kind != 0 && s.kind == KV_STORE_PER_TOKEN) {
    token_scale = fmaxf(wave_max(amax), 1e-12f) / 448.0f;
    if (lane == 0 && s.cache_k) s.scales[(int64_t)proj * s.scale_stride + (kind == 2 ? s.n_slots : 0) + slot] = token_scale;
  }
#pragma unroll
  for (int t = 0; t < NIT; ++t) {
    const int item = (part * NIT + t) * 64 + lane, head = item / PAIRS, c = item % PAIRS, at = head * HD + c * 8;
    if (item * 16 >= dim) continue;
    if (put_rows) {
      *(uint4 *)(rows + at) = lo[t];
      *(uint4 *)(rows + at + HD / 2) = hi[t];
    }
    if (kind == 0 || !s.cache_k) continue;
    unsigned char *plane = (unsigned char *)(kind == 1 ? s.cache_k : s.cache_v) + (int64_t)proj * s.layer_bytes;
    const int64_t dst = slot * p.kv_dim + at;
    if (s.kind == KV_STORE_BF16) {
      *(uint4 *)((bf16_t *)plane + dst) = lo[t];
      *(uint4 *)((bf16_t *)plane + dst + HD / 2) = hi[t];
    } else {
      const float sc = s.kind == KV_STORE_PER_TOKEN ? token_scale : head_scale;
      const float inv = 1.f / sc;
      uint2 a, b;
      if (fast_scale(sc)) { a = quantize8<true>(lo[t], sc, inv); b = quantize8<true>(hi[t], sc, inv); }
      else { a = quantize8<false>(lo[t], sc, inv); b = quantize8<false>(hi[t], sc, inv); }
      *(uint2 *)(plane + dst) = a;
      *(uint2 *)(plane + dst + HD / 2) = b;
    }
  }
}
template <int EPI, int HD>
static void launch_kv_finish_hd(const GemmParams &p, const KvStore &s, hipStream_t st) {
  const bool wide = s.kind == KV_STORE_PER_TOKEN && p.kv_dim > 1024;
  const int cols = wide ? 4096 : 1024;
  const int q_units = EPI == EPI_QKV ? (p.q_dim + cols - 1) / cols : 0, kv_units = (p.kv_dim + cols - 1) / cols;
  const int units = EPI == EPI_QKV ? q_units + kv_units * (s.vt ? 1 : 2) : p.N / p.kv_dim * kv_units;
  const int vt_wgs = EPI == EPI_QKV && s.vt ? s.n_tiles * (p.kv_dim / HD) : 0;
  const dim3 grid((unsigned)(vt_wgs + ((int64_t)p.M * units + 3) / 4));
  if (wide) hipLaunchKernelGGL((kv_finish_kernel<EPI, HD, 4>), grid, dim3(256), 0, st, p, s, vt_wgs, q_units, kv_units);
  else hipLaunchKernelGGL((kv_finish_kernel<EPI, HD, 1>), grid, dim3(256), 0, st, p, s, vt_wgs, q_units, kv_units);
}
// (a token's own scale: its K or V row in one wave)
bool kv_store_fits(const KvStore &s, int kv_dim) { return s.kind != KV_STORE_PER_TOKEN || kv_dim <= 4096; }
int launch_kv_finish(const GemmParams &p, int epi, hipStream_t st) {
  KvStore s{};
  if (p.store) {
    s = *p.store;
  } else {
    s.rows = 3;
    if (epi == EPI_KV && !p.stage) {
      s.cache_k = p.cache + (int64_t)p.first_cache_layer * p.cache_layer_stride;
      s.cache_v = (bf16_t *)s.cache_k + p.cache_kv_stride;
      s.layer_bytes = p.cache_layer_stride * 2;
    }
  }
  if (epi == EPI_QKV) p.head_dim == 128 ? launch_kv_finish_hd<EPI_QKV, 128>(p, s, st) : launch_kv_finish_hd<EPI_QKV, 64>(p, s, st);
  else p.head_dim == 128 ? launch_kv_finish_hd<EPI_KV, 128>(p, s, st) : launch_kv_finish_hd<EPI_KV, 64>(p, s, st);
  return 0;
}

// ----------------------------------------------------------- QKV finish ----
// grid (T, Hq + 2*Hkv), hd/2 threads: thread i owns the rotary pair (i, i + hd/2) of one head of one row.
__global__ void qkv_finish_kernel(QkvFinishParams p) {
  const int row = blockIdx.x, hs = blockIdx.y, i = threadIdx.x;
  const int hd = p.head_dim, half = hd / 2;
  const int kind = hs < p.n_q_heads ? 0 : (hs < p.n_q_heads + p.n_kv_heads ? 1 : 2);
  const int head = kind == 0 ? hs : (kind == 1 ? hs - p.n_q_heads : hs - p.n_q_heads - p.n_kv_heads);
  const int64_t dim = (int64_t)(kind == 0 ? p.n_q_heads : p.n_kv_heads) * hd;
  const float *src = (kind == 0 ? p.q32 : kind == 1 ? p.k32 : p.v32) + row * (p.ld32 ? (int64_t)p.ld32 : dim) + head * hd;
  bf16_t *dst = (kind == 0 ? p.q : kind == 1 ? p.k : p.v) + row * dim + head * hd;
  float x0 = src[i], x1 = src[i + half];
  if (p.n_splits > 1) {   // the K splits of the projection, added in split order
    const int64_t step = (int64_t)p.T * p.ld32;
    for (int ks = 1; ks < p.n_splits; ++ks) { x0 += src[ks * step + i]; x1 += src[ks * step + i + half]; }
  }
  if (kind != 2) {
    const float2 cs = p.cos_sin[(int64_t)row * half + i];
    rotate_pair(x0, x1, cs.x, cs.y);
  }
  const bf16_t b0 = f32_to_bf16(x0), b1 = f32_to_bf16(x1);
  if (kind != 0 && p.cache_k) {
    const int64_t at = (p.slots[row] * p.n_kv_heads + head) * hd + i;
    void *plane = kind == 1 ? p.cache_k : p.cache_v;
    if (p.scales) {
      const float s = p.scales[(kind == 2 ? p.n_kv_heads : 0) + head];
      ((uint8_t *)plane)[at] = f32_to_e4m3fn(bf16_to_f32(b0) / s);
      ((uint8_t *)plane)[at + half] = f32_to_e4m3fn(bf16_to_f32(b1) / s);
    } else {
      ((bf16_t *)plane)[at] = b0;
      ((bf16_t *)plane)[at + half] = b1;
    }
    return;
  }
  dst[i] = b0;
  dst[i + half] = b1;
  if (p.amax && kind != 0) {   // absmax of the values as stored (bf16-rounded)
    float a = fmaxf(fabsf(bf16_to_f32(b0)), fabsf(bf16_to_f32(b1)));
    for (int o = 32; o > 0; o >>= 1) a = fmaxf(a, __shfl_xor(a, o));
    if ((i & 63) == 0) atomicMax(p.amax + (kind == 2 ? p.n_kv_heads : 0) + head, __float_as_uint(a));
  }
}
int launch_qkv_finish(const QkvFinishParams &p, hipStream_t st) {
  if (p.T <= 0) return 0;
  hipLaunchKernelGGL(qkv_finish_kernel, dim3(p.T, p.n_q_heads + 2 * p.n_kv_heads), dim3(p.head_dim / 2), 0, st, p);
  return 0;
}

// ----------------------------------------------------------- early exit ----
// One workgroup per row: max, then sum of exp(x - max); the largest probability is 1 / that sum.
__global__ __launch_bounds__(256) void early_exit_flags_kernel(const float *early, int32_t V, float threshold, int32_t *flags) {
  __shared__ float red[4];
  const float *x = early + (int64_t)blockIdx.x * V;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float mx = -INFINITY;
  for (int i = tid; i < V; i += 256) mx = fmaxf(mx, x[i]);
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
  if (lane == 0) red[wave] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  __syncthreads();
  float sum = 0.f;
  for (int i = tid; i < V; i += 256) sum += __expf(x[i] - mx);
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  if (lane == 0) red[wave] = sum;
  __syncthreads();
  if (tid == 0) flags[blockIdx.x] = (1.0f / (red[0] + red[1] + red[2] + red[3])) > threshold ? 1 : 0;
}
__global__ void early_exit_select_kernel(const float *early, const int32_t *flags, float *logits, int32_t V) {
  if (!flags[blockIdx.y]) return;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < V) logits[(int64_t)blockIdx.y * V + i] = early[(int64_t)blockIdx.y * V + i];
}
int launch_early_exit_flags(const float *early, int32_t B, int32_t V, float threshold, int32_t *flags, hipStream_t st) {
  if (B <= 0) return 0;
  hipLaunchKernelGGL(early_exit_flags_kernel, dim3(B), dim3(256), 0, st, early, V, threshold, flags);
  return 0;
}
int launch_early_exit_select(const float *early, const int32_t *flags, float *logits, int32_t B, int32_t V, hipStream_t st) {
  if (B <= 0) return 0;
  hipLaunchKernelGGL(early_exit_select_kernel, dim3((V + 255) / 256, B), dim3(256), 0, st, early, flags, logits, V);
  return 0;
}

// ----------------------------------------------------------- KV gather -----
// One workgroup per (64-position tile, KV head) of a sequence whose prompt continues over a cached
// prefix: copies the tile's K rows out of the paged cache into consecutive rows and its V rows
// into V^T columns (through LDS, as above), dequantising e4m3 codes with the layer's scales to
// the bf16 values every other reader of the cache sees.  Columns past n_valid are zero filled.
template <int HD>
__global__ __launch_bounds__(256) void kv_gather_kernel(GatherParams p) {
  constexpr int CH = HD / 8;  // 8-element chunks per row
  __shared__ uint4 sv[64 * CH];
  const GatherTile tile = p.tiles[blockIdx.x];
  const int head = blockIdx.y;
  const int tid = threadIdx.x;
  const int kv_dim = p.n_kv_heads * HD;
  float sk = 1.f, svs = 1.f;
  if (p.fp8 == 1) { sk = p.scales[head]; svs = p.scales[p.n_kv_heads + head]; }
  // three rounds of requests for the whole tile (block ids, scales and rows, then the stores), not one chain per chunk
  constexpr int NI = 64 * CH / 256;
  int64_t slot[NI];
#pragma unroll
  for (int ii = 0; ii < NI; ++ii) {
    const int r = (tid + ii * 256) / CH, pos = tile.pos0 + (r < tile.n_valid ? r : 0);
    int blk = p.block_tables[(int64_t)tile.seq * p.max_blocks_per_seq + pos / SKV_BLOCK];
    blk = blk < 0 ? 0 : (blk >= p.n_blocks ? p.n_blocks - 1 : blk);   // bad ids were reported by the plan; stay inside the pool
    slot[ii] = (int64_t)blk * SKV_BLOCK + pos % SKV_BLOCK;
  }
  uint4 kin[NI], vin[NI];   // (codes: the first two words)
  float sk_in[NI], sv_in[NI];
#pragma unroll
  for (int ii = 0; ii < NI; ++ii) {
    const int64_t src = (slot[ii] * p.n_kv_heads + head) * HD + ((tid + ii * 256) % CH) * 8;
    sk_in[ii] = sk; sv_in[ii] = svs;
    if (p.fp8 == 2) { sk_in[ii] = p.scales[slot[ii]]; sv_in[ii] = p.scales[(int64_t)p.n_blocks * SKV_BLOCK + slot[ii]]; }
    if (!p.fp8) {
      kin[ii] = *(const uint4 *)((const bf16_t *)p.cache_k + src);
      vin[ii] = *(const uint4 *)((const bf16_t *)p.cache_v + src);
    } else {
      const uint2 kc = *(const uint2 *)((const uint8_t *)p.cache_k + src), vc = *(const uint2 *)((const uint8_t *)p.cache_v + src);
      kin[ii] = make_uint4(kc.x, kc.y, 0, 0);
      vin[ii] = make_uint4(vc.x, vc.y, 0, 0);
    }
  }
#pragma unroll
  for (int ii = 0; ii < NI; ++ii) {
    const int i = tid + ii * 256, r = i / CH, c = i % CH;
    uint4 kq = kin[ii], vq = vin[ii];
    if (p.fp8) {
      const uint32_t kcw[2] = {kq.x, kq.y}, vcw[2] = {vq.x, vq.y};
      uint32_t kw[4], vw[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t k2 = kcw[e / 2] >> ((e & 1) * 16), v2 = vcw[e / 2] >> ((e & 1) * 16);
        kw[e] = pack_bf16x2(e4m3fn_to_f32((uint8_t)k2) * sk_in[ii], e4m3fn_to_f32((uint8_t)(k2 >> 8)) * sk_in[ii]);
        vw[e] = pack_bf16x2(e4m3fn_to_f32((uint8_t)v2) * sv_in[ii], e4m3fn_to_f32((uint8_t)(v2 >> 8)) * sv_in[ii]);
      }
      kq = make_uint4(kw[0], kw[1], kw[2], kw[3]);
      vq = make_uint4(vw[0], vw[1], vw[2], vw[3]);
    }
    if (r < tile.n_valid) *(uint4 *)(p.k_dst + (int64_t)(tile.k_row0 + r) * kv_dim + head * HD + c * 8) = kq;
    else vq = make_uint4(0, 0, 0, 0);
    sv[v_chunk<HD>(r, c)] = vq;
  }
  __syncthreads();
  store_vt<HD>(sv, p.vt + (int64_t)(head * HD) * p.vt_ld + tile.vt_col0, p.vt_ld, tid);
}
int launch_kv_gather(const GatherParams &p, hipStream_t st) {
  if (p.n_tiles <= 0) return 0;
  dim3 grid(p.n_tiles, p.n_kv_heads);
  if (p.head_dim == 128) hipLaunchKernelGGL(kv_gather_kernel<128>, grid, dim3(256), 0, st, p);
  else hipLaunchKernelGGL(kv_gather_kernel<64>, grid, dim3(256), 0, st, p);
  return 0;
}

__global__ void fp8_quantize_kernel(const float *x, float scale, uint8_t *codes, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    float y = x[i] / scale;
    codes[i] = f32_to_e4m3fn(y);
  }
}
int launch_fp8_quantize(const float *x, float scale, uint8_t *codes, int64_t n, hipStream_t st) {
  if (n <= 0) return 0;
  hipLaunchKernelGGL(fp8_quantize_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, x, scale, codes, n);
  return 0;
}

// ------------------------------------------------- split-KV combine --------
// partial layout: [row][head][split][hd + 2] = (o[hd] unnormalised, m, l), m in log2 units; n_split <= MAX_SPLIT.
// One latency-bound pass: every load is requested before the first use.  Lane s of each wave holds split s's m and l,
// so the weights come from wave reductions and are broadcast lane by lane (no second trip to memory, no barrier):
// one row of 25 splits 5.8 -> 3.9 us per launch.  An empty split carries m = -inf and enters with weight 0.
__global__ __launch_bounds__(128) void decode_combine_kernel(const float *partial, bf16_t *out, const DecodeRow *rows, int n_q_heads, int hd, int n_split) {
  const int row = blockIdx.x, head = blockIdx.y, d = threadIdx.x, lane = threadIdx.x & 63;
  const int64_t out_row = rows[row].out_row;
  const float *base = partial + ((int64_t)(row * n_q_heads + head) * n_split) * (hd + 2);
  const int ls = lane < n_split ? lane : n_split - 1;
  float mv = base[ls * (hd + 2) + hd];
  const float lv = base[ls * (hd + 2) + hd + 1];
  float ov[MAX_SPLIT];
#pragma unroll
  for (int c = 0; c < MAX_SPLIT / 8; ++c)
    if (c * 8 < n_split) {
#pragma unroll
      for (int i = c * 8; i < c * 8 + 8; ++i) ov[i] = i < n_split ? base[i * (hd + 2) + d] : 0.f;   // (0: what weighs nothing must not be infinite)
    }
  if (lane >= n_split) mv = -INFINITY;
  const float m = wave_max(mv);
  const float w = (mv == -INFINITY) ? 0.f : exp2f(mv - m);
  const float l = wave_sum(w * lv);
  float acc = 0.f;
#pragma unroll
  for (int c = 0; c < MAX_SPLIT / 8; ++c)
    if (c * 8 < n_split) {
#pragma unroll
      for (int i = c * 8; i < c * 8 + 8; ++i) acc += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), i)) * ov[i];   // (weight 0 past the last split)
    }
  out[out_row * n_q_heads * hd + head * hd + d] = f32_to_bf16(acc / l);
}
int launch_decode_combine(const float *partial, bf16_t *out, const DecodeRow *rows, int32_t n_rows,
                          int32_t n_q_heads, int32_t head_dim, int32_t n_split, hipStream_t st) {
  if (n_rows <= 0 || n_split == 1) return 0;   // (one split: the attention kernel wrote the result)
  if (n_split > MAX_SPLIT) return -1;
  hipLaunchKernelGGL(decode_combine_kernel, dim3(n_rows, n_q_heads), dim3(head_dim), 0, st, partial, out, rows, n_q_heads, head_dim, n_split);
  return 0;
}
