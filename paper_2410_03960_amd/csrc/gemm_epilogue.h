// Epilogue of the GEMM kernels whose waves own FM x 32 rows by 64 columns of C (the packed-weight loop for
// many rows and the loop for tens to thousands of rows): accumulators leave through a per-wave LDS slab as
// contiguous row pieces.
#pragma once
#include "common.h"

namespace {

template <int EPI, int FM, bool NORM_OUT = false>   // NORM_OUT (RESID only): also the next projection's bf16 operand and the rows' sums of squares
__device__ __forceinline__ void gemm_epilogue_n64(const GemmParams &p, floatx16 (&acc)[2][FM], const int m_base,
                                                  const int n_base, const int lane, unsigned char *slab, const int64_t c_off = 0) {
  // acc[bn][bm][4*jg + e] is C[m_base + bm*32 + l32][n_base + bn*32 + 8*jg + 4*g + e].  32 rows at a
  // time go through a per-wave LDS slab (row stride padded by 16 bytes) and leave as 16-byte stores
  // in which consecutive lanes cover a contiguous row segment.
  const int l32 = lane & 31, g = lane >> 5;
  if constexpr (EPI == EPI_STORE_F32 || EPI == EPI_PARTIAL) {
    // fp32 rows; a K split's partial sums go to C + c_off with their columns in true order (the packed order of
    // rotary operands of 128-wide heads has the tile's second block 64 columns behind its first)
    constexpr int RS = 64 * 4 + 16;
    const int ch = lane & 7, r8 = lane >> 3;
    int col = n_base + ch * 8;
    if (EPI == EPI_PARTIAL && p.head_dim == 128) col = (n_base & ~127) + ((n_base >> 6) & 1) * 32 + (ch >> 2) * 64 + (ch & 3) * 8;
    float *cbase = (float *)p.C + c_off + col;
#pragma unroll
    for (int bm = 0; bm < FM; ++bm) {
#pragma unroll
      for (int bn = 0; bn < 2; ++bn)
#pragma unroll
        for (int jg = 0; jg < 4; ++jg)
          *(float4 *)(slab + l32 * RS + (bn * 32 + 8 * jg + 4 * g) * 4) =
              make_float4(acc[bn][bm][4 * jg], acc[bn][bm][4 * jg + 1], acc[bn][bm][4 * jg + 2], acc[bn][bm][4 * jg + 3]);
      // a wave's LDS operations execute in order: the reads below see the writes above
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int row = it * 8 + r8;
        const int m = m_base + bm * 32 + row;
        const float4 lo = *(const float4 *)(slab + row * RS + ch * 32), hi = *(const float4 *)(slab + row * RS + ch * 32 + 16);
        if (m < p.M) {
          float4 *dst = (float4 *)(cbase + (int64_t)m * p.ldc);
          dst[0] = lo;
          dst[1] = hi;
        }
      }
    }
  } else if constexpr (EPI == EPI_RESID) {
    // C (fp32, the residual stream) += acc.  Optionally also the bf16 operand of the next projection,
    // hb = bf16(C_new * gain of that projection's RMSNorm), and the sum of squares of C_new over this
    // wave's 64 columns (the consumer's epilogue applies 1/rms as a row factor).
    constexpr int RS = 64 * 4 + 16;                // fp32 row stride in bytes
    float *cbase = (float *)p.C + n_base;
    const int ch = lane & 7, r8 = lane >> 3;       // this lane's 8 columns, its row inside a group of 8
    float gv[8] = {1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f};
    if (NORM_OUT && p.hb_gain) {
      const uint4 gq = *(const uint4 *)(p.hb_gain + n_base + ch * 8);
      gv[0] = bf16lo(gq.x); gv[1] = bf16hi(gq.x); gv[2] = bf16lo(gq.y); gv[3] = bf16hi(gq.y);
      gv[4] = bf16lo(gq.z); gv[5] = bf16hi(gq.z); gv[6] = bf16lo(gq.w); gv[7] = bf16hi(gq.w);
    }
    // The residual rows are requested for half of the wave tile at a time (128 registers; the operand
    // registers of the main loop are free by now), all of a half before its first store: loads and stores
    // share one counter, so a load issued between stores would wait for the stores before it.
    constexpr int HB = (FM + 1) / 2;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      float4 res[HB][4][2];
#pragma unroll
      for (int b = 0; b < HB && half * HB + b < FM; ++b)
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int m = m_base + (half * HB + b) * 32 + it * 8 + r8;
          const float4 *src = (const float4 *)(cbase + (int64_t)(m < p.M ? m : p.M - 1) * p.ldc + ch * 8);
          res[b][it][0] = src[0];
          res[b][it][1] = src[1];
        }
#pragma unroll
      for (int b = 0; b < HB && half * HB + b < FM; ++b) {
        const int bm = half * HB + b;
#pragma unroll
        for (int bn = 0; bn < 2; ++bn)
#pragma unroll
          for (int jg = 0; jg < 4; ++jg)
            *(float4 *)(slab + l32 * RS + (bn * 32 + 8 * jg + 4 * g) * 4) =
                make_float4(acc[bn][bm][4 * jg], acc[bn][bm][4 * jg + 1], acc[bn][bm][4 * jg + 2], acc[bn][bm][4 * jg + 3]);
        // a wave's LDS operations execute in order: the reads below see the writes above
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int row = it * 8 + r8;
          const int m = m_base + bm * 32 + row;
          const float4 lo = *(const float4 *)(slab + row * RS + ch * 32), hi = *(const float4 *)(slab + row * RS + ch * 32 + 16);
          const float4 r0 = res[b][it][0], r1 = res[b][it][1];
          const float x[8] = {r0.x + lo.x, r0.y + lo.y, r0.z + lo.z, r0.w + lo.w, r1.x + hi.x, r1.y + hi.y, r1.z + hi.z, r1.w + hi.w};
          if (m < p.M) {
            float4 *dst = (float4 *)(cbase + (int64_t)m * p.ldc + ch * 8);
            dst[0] = make_float4(x[0], x[1], x[2], x[3]);
            dst[1] = make_float4(x[4], x[5], x[6], x[7]);
            if constexpr (NORM_OUT)
              *(uint4 *)(p.hb + (int64_t)m * p.ldc + n_base + ch * 8) =
                  make_uint4(pack_bf16x2(x[0] * gv[0], x[1] * gv[1]), pack_bf16x2(x[2] * gv[2], x[3] * gv[3]),
                             pack_bf16x2(x[4] * gv[4], x[5] * gv[5]), pack_bf16x2(x[6] * gv[6], x[7] * gv[7]));
          }
          if constexpr (NORM_OUT) {   // fixed order: the lane's 8 columns left to right, then a butterfly over the row's 8 lanes
            float sq = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) sq += x[e] * x[e];
            sq += __shfl_xor(sq, 1);
            sq += __shfl_xor(sq, 2);
            sq += __shfl_xor(sq, 4);
            if (ch == 0 && m < p.M) p.ssq[(int64_t)m * (p.N >> 6) + (n_base >> 6)] = sq;
          }
        }
      }
    }
  } else if constexpr (EPI == EPI_QKV || EPI == EPI_KV) {
    // The wave's 64 (virtual) columns are one head (head_dim 64: blocks = first / second half) or, for
    // head_dim 128, half a head in the packed order: block 0 = columns s*32.. of the first half, block 1
    // = their rotary partners s*32 + 64.. (s = parity of the wave tile inside the head).  Either way
    // element v of block 0 and element v of block 1 are rotary partners.
    const int hd = p.head_dim;
    const int head_base = hd == 128 ? (n_base & ~127) : n_base;
    const int s = hd == 128 ? ((n_base >> 6) & 1) : 0;
    int kind, col0, proj = 0;                          // kind 0 = q, 1 = k, 2 = v; col0 = head's first column in its output
    if constexpr (EPI == EPI_QKV) {
      if (head_base < p.q_dim) { kind = 0; col0 = head_base; }
      else if (head_base < p.q_dim + p.kv_dim) { kind = 1; col0 = head_base - p.q_dim; }
      else { kind = 2; col0 = head_base - p.q_dim - p.kv_dim; }
    } else {
      proj = head_base / (2 * p.kv_dim);
      const int within = head_base % (2 * p.kv_dim);
      kind = within < p.kv_dim ? 1 : 2;
      col0 = within % p.kv_dim;
    }
    const int blk_stride = hd == 128 ? 64 : 32;        // real columns between block 0 and block 1
    constexpr int RS = 64 * 2 + 16;
    float amax_h = 0.f;
    // Destination of this wave's columns, selected once (uniform over the wave): base pointer of the
    // head's first column and the row stride in elements; rows of the paged cache go through p.slots.
    // (Selecting per store, through a table indexed by `kind`, cost a private-memory lookup, a full
    // vmcnt wait and a flat store for each of the 32 stores of a wave tile.)
    bf16_t *obase;
    int64_t ostride;
    bool paged = false;
    if constexpr (EPI == EPI_QKV) {
      obase = p.q_out; ostride = p.q_dim;
      if (kind == 1) { obase = p.k_out; ostride = p.kv_dim; }
      if (kind == 2) { obase = p.v_out; ostride = p.kv_dim; }
    } else {
      obase = p.stage + (int64_t)proj * 2 * p.kv_dim + (kind == 2 ? p.kv_dim : 0); ostride = p.N;
      if (!p.stage) {
        obase = p.cache + (int64_t)(p.first_cache_layer + proj) * p.cache_layer_stride + (kind == 2 ? p.cache_kv_stride : 0);
        ostride = p.kv_dim; paged = true;
      }
    }
    obase += col0 + s * 32;
    // 1/rms of this lane's rows, all requested before the first use (one latency, not one per 32 rows)
    float rsv[FM];
#pragma unroll
    for (int bm = 0; bm < FM; ++bm) {
      const int m = m_base + bm * 32 + l32;
      rsv[bm] = p.rstd ? p.rstd[m < p.M ? m : p.M - 1] : 1.f;
    }
    // Two passes, so that no load follows a store: loads and stores share one counter, and with both
    // kinds pending every wait for a load becomes a wait for everything, stores included (which made
    // each 32-row block of the epilogue wait for the previous block's stores to reach memory).
    // Pass 1: per 32-row block the cos/sin pieces (requested CSD - 1 blocks ahead: they are 32-row gathers
    // that mostly miss L2, and one block of arithmetic covers only a third of their latency) and, for the
    // paged cache, the rows' slots; rotation, rounding, bf16 rows into the wave's LDS slab (FM blocks of 32 rows).
    // Pass 2: the slab leaves as 16-byte stores in which consecutive lanes cover a contiguous row piece.
    constexpr int SLAB_BM = 32 * RS;   // bytes per 32-row block
    constexpr int CSD = (EPI == EPI_QKV) ? 4 : 2;   // the paged variant keeps 64 registers of slots instead
    float4 csb[CSD][8];
    auto load_cs = [&](int bm) {
      const int m = m_base + bm * 32 + l32;
      const float2 *cs = p.cos_sin + (int64_t)(m < p.M ? m : p.M - 1) * (hd / 2) + s * 32 + 4 * g;
#pragma unroll
      for (int jg = 0; jg < 4; ++jg) {
        csb[bm % CSD][2 * jg] = *(const float4 *)(cs + 8 * jg);
        csb[bm % CSD][2 * jg + 1] = *(const float4 *)(cs + 8 * jg + 2);
      }
    };
    if (kind != 2) {
#pragma unroll
      for (int b = 0; b < CSD - 1 && b < FM; ++b) load_cs(b);
    }
    uint32_t orow[FM][4];   // output rows of this lane's stores (the paged cache: their slots; 2^31 slots would not fit the memory)
#pragma unroll
    for (int bm = 0; bm < FM; ++bm)
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int mm = m_base + bm * 32 + it * 8 + (lane >> 3);
        orow[bm][it] = mm;
        if constexpr (EPI == EPI_KV) { if (paged) orow[bm][it] = (uint32_t)p.slots[mm < p.M ? mm : p.M - 1]; }
      }
#pragma unroll
    for (int bm = 0; bm < FM; ++bm) {
      const int m = m_base + bm * 32 + l32;
      const float rs = rsv[bm];
      unsigned char *srow = slab + bm * SLAB_BM + l32 * RS;
      if (kind != 2 && bm + CSD - 1 < FM) load_cs(bm + CSD - 1);
#pragma unroll
      for (int jg = 0; jg < 4; ++jg) {
        float y1[4], y2[4];
        const int i0 = 8 * jg + 4 * g;
        float cv[4] = {1.f, 1.f, 1.f, 1.f}, sv[4] = {0.f, 0.f, 0.f, 0.f};
        if (kind != 2) {
          const float4 c01 = csb[bm % CSD][2 * jg], c23 = csb[bm % CSD][2 * jg + 1];
          cv[0] = c01.x; cv[1] = c01.z; cv[2] = c23.x; cv[3] = c23.z;
          sv[0] = c01.y; sv[1] = c01.w; sv[2] = c23.y; sv[3] = c23.w;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          y1[e] = acc[0][bm][4 * jg + e] * rs;
          y2[e] = acc[1][bm][4 * jg + e] * rs;
          rotate_pair(y1[e], y2[e], cv[e], sv[e]);
        }
        const uint2 p1 = make_uint2(pack_bf16x2(y1[0], y1[1]), pack_bf16x2(y1[2], y1[3]));
        const uint2 p2 = make_uint2(pack_bf16x2(y2[0], y2[1]), pack_bf16x2(y2[2], y2[3]));
        *(uint2 *)(srow + i0 * 2) = p1;
        *(uint2 *)(srow + (32 + i0) * 2) = p2;
        if (p.amax && kind != 0 && m < p.M) {   // absmax of the values as stored (bf16-rounded)
          const float a1 = fmaxf(fmaxf(fabsf(bf16lo(p1.x)), fabsf(bf16hi(p1.x))), fmaxf(fabsf(bf16lo(p1.y)), fabsf(bf16hi(p1.y))));
          const float a2 = fmaxf(fmaxf(fabsf(bf16lo(p2.x)), fabsf(bf16hi(p2.x))), fmaxf(fabsf(bf16lo(p2.y)), fabsf(bf16hi(p2.y))));
          amax_h = fmaxf(amax_h, fmaxf(a1, a2));
        }
      }
    }
    // a wave's LDS operations execute in order: the reads below see the writes above
#pragma unroll
    for (int bm = 0; bm < FM; ++bm)
#pragma unroll
      for (int it = 0; it < 4; ++it) {   // 8 rows per instruction, chunk ch = 8 local columns; local block ch/4
        const int row = it * 8 + (lane >> 3), ch = lane & 7;
        const int mm = m_base + bm * 32 + row;
        const uint4 val = *(const uint4 *)(slab + bm * SLAB_BM + row * RS + ch * 16);
        if (mm < p.M) *(uint4 *)(obase + (int64_t)orow[bm][it] * ostride + (ch >> 2) * blk_stride + (ch & 3) * 8) = val;
      }
    if (p.amax && kind != 0) {
      const float a = wave_max(amax_h);
      if (lane == 0)
        atomicMax(p.amax + ((int64_t)(p.first_cache_layer + proj) * 2 + (kind == 2 ? 1 : 0)) * (p.kv_dim / hd) + col0 / hd, __float_as_uint(a));
    }
  } else {
    static_assert(EPI == EPI_STORE_BF16 || EPI == EPI_SWIGLU, "epilogues of the 64-column wave tile");
    constexpr int NC = (EPI == EPI_SWIGLU) ? 32 : 64;   // output columns of the wave tile
    constexpr int RS = NC * 2 + 16;                      // bf16 row stride in bytes
    constexpr int CPR = NC / 8, RPI = 64 / CPR;          // 16-byte chunks per row, rows per store instruction
    float rsv[FM];
    if constexpr (EPI == EPI_SWIGLU) {   // 1/rms of this lane's rows, all requested before the first use
#pragma unroll
      for (int bm = 0; bm < FM; ++bm) {
        const int m = m_base + bm * 32 + l32;
        rsv[bm] = p.rstd ? p.rstd[m < p.M ? m : p.M - 1] : 1.f;
      }
    }
#pragma unroll
    for (int bm = 0; bm < FM; ++bm) {
      unsigned char *srow = slab + l32 * RS;
      if constexpr (EPI == EPI_SWIGLU) {
        const float rs = rsv[bm];
#pragma unroll
        for (int bn = 0; bn < 2; ++bn)
#pragma unroll
          for (int jg = 0; jg < 2; ++jg) {
            float o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float gt = acc[bn][bm][4 * jg + e] * rs, up = acc[bn][bm][4 * (jg + 2) + e] * rs;
              o[e] = gt * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * gt)) * up;   // silu(gate) * up
            }
            *(uint2 *)(srow + (bn * 16 + 8 * jg + 4 * g) * 2) = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
          }
      } else {
#pragma unroll
        for (int bn = 0; bn < 2; ++bn)
#pragma unroll
          for (int jg = 0; jg < 4; ++jg)
            *(uint2 *)(srow + (bn * 32 + 8 * jg + 4 * g) * 2) =
                make_uint2(pack_bf16x2(acc[bn][bm][4 * jg], acc[bn][bm][4 * jg + 1]), pack_bf16x2(acc[bn][bm][4 * jg + 2], acc[bn][bm][4 * jg + 3]));
      }
      const int ch = lane % CPR;
#pragma unroll
      for (int it = 0; it < 32 / RPI; ++it) {
        const int row = it * RPI + lane / CPR;
        const int m = m_base + bm * 32 + row;
        const uint4 val = *(const uint4 *)(slab + row * RS + ch * 16);
        if (m >= p.M) continue;
        bf16_t *dst = (bf16_t *)p.C + (int64_t)m * p.ldc + (EPI == EPI_SWIGLU ? n_base / 2 : n_base);
        *(uint4 *)(dst + ch * 8) = val;
      }
    }
  }
}

}  // namespace
