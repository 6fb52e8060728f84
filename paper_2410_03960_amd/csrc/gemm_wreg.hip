// Packed-weight main loop of the GEMM (weights in matrix-instruction fragment order, see launch_pack_w).
#include "gemm_epilogue.h"
#include <type_traits>

namespace {

// ---------------------------------------------------------------------------
// Main loop that keeps the weight operand out of LDS.  The weights are static, so
// they can be stored once in MFMA fragment order (`wpack`: for every block of 32
// output rows and 16 k values, the 1 KB that the 64 lanes hold as first operand,
// lane i at byte 16*i).  A wave then fetches its weight fragments with fully
// coalesced 16-byte-per-lane loads straight into registers, four 64-wide k steps
// ahead, and LDS carries the activations only: five stages of 32 FM rows x 128
// bytes, filled by LDS-DMA in whole 128-byte row pieces, three steps ahead.
// The four waves sit side by side along N (wave tile 32 FM x 64), so no weight byte
// is loaded twice; every wave reads all of the activation tile from LDS (the same
// LDS read volume as a 2 x 2 arrangement of 128 x 128 wave tiles, half the LDS
// writes, half the LDS-DMA requests).  One barrier per 64-wide step, placed
// before the last 16-wide sub-step, where the next step's activations are first
// read.  Needs K % 256 == 0 (four register slots, statically indexed) and
// N % 256 == 0.
// The tile height FM and the K splits come from plan_gemm_mid.  What a step costs is the bytes a CU fetches
// for it, through L2 and with a bounded number of requests in flight, against the MFMAs it hides them under:
// 0.89 us at FM = 4 (48 KB, 128 rows), 1.12 at 6, 1.46 at 8 (64 KB, 256 rows) with all CUs busy, so a taller
// tile is cheaper per row and a shorter one is taken where it fills a last round or leaves room for K splits.
// The four waves run in step, so their fragment reads are spread over all products of a sub-step (in a burst behind the
// first half of them they took every LDS cycle of that half; gate and up of 16384 rows, K 4096, 2714 -> 2706 us, of 1300 and 6000 level,
// down 0.3 to 0.6 %).  The uniform bases of the requests are worth more: with a pointer per lane 2739, 6000 rows 1040 -> 1028,
// 1300 252 -> 249, down of 16384 1439 -> 1424.  No gain, measured on this loop: six to ten stages where they fit, weights four steps ahead (the wait
// for a stage then leaves 22 instead of 14 requests in flight), 32 KB of a step's weights in one piece, each wave's requests
// a product later than its neighbour's; eight waves of 128 x 64, two to a SIMD: 3 % slower, as every wave's wait is stricter.
template <int EPI, int FM, bool NORM_OUT>
__device__ __forceinline__ void wreg_tile(const GemmParams &p, unsigned char *smem, const int block, const int first_n, const int tiles_n) {
  constexpr int BM = 32 * FM, BN = 256;
  constexpr int NSA = 5, STAGE = BM * 128;   // activation stages: BM rows x 128 bytes (one 64-wide k step)

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g = lane >> 5;

  const int tiles_m = (p.M + BM - 1) / BM;
  const int per_split = tiles_m * tiles_n, total = per_split * p.n_splits;
  const int per_xcd = (total + 7) / 8;
  const int logical = (block % 8) * per_xcd + block / 8;
  if (logical >= total) return;
  const int split = logical / per_split, tile = logical % per_split;
  constexpr int GM = 8;   // m tiles per rasterisation group
  const int group = tile / (GM * tiles_n);
  const int first_m = group * GM;
  const int gsz = (tiles_m - first_m) < GM ? (tiles_m - first_m) : GM;
  const int in_group = tile % (GM * tiles_n);
  const int tm = first_m + in_group % gsz, tn = first_n + in_group / gsz;
  const int m0 = tm * BM, n0 = tn * BN + wave * 64;   // n0: first column of this wave
  const int all_steps = p.K / 64, s_begin = split * p.split_steps;
  const int nk = (all_steps - s_begin) < p.split_steps ? (all_steps - s_begin) : p.split_steps;   // >= 1 by the plan

  // LDS-DMA sources: request i of this wave covers rows (wave*FM + i)*8 .. +7 of the tile, 128 bytes each;
  // this lane fetches row +(lane>>3), the 16-byte chunk that lands at physical chunk lane&7.  Addresses are a uniform base
  // plus a 32-bit offset per lane: with whole pointers per lane every request cost two vector adds between the MFMAs.
  unsigned a_off[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int r = (wave * FM + i) * 8 + (lane >> 3);
    const int in_tile = m0 + r < p.M ? r : p.M - 1 - m0;
    a_off[i] = (unsigned)in_tile * (unsigned)(p.lda * 2) + (((lane & 7) ^ ((r >> 1) & 7)) * 16);
  }
  const unsigned char *a_base = (const unsigned char *)(p.A + (int64_t)m0 * p.lda + (int64_t)s_begin * 64);
  // packed weight fragments of the wave's two 32-row blocks: (block, k16) at ((block * K/16) + k16) * 512 elements
  const unsigned char *w_base[2];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb) w_base[nb] = (const unsigned char *)(p.wpack + ((int64_t)(n0 / 32 + nb) * (p.K / 16) + (int64_t)s_begin * 4) * 512);
  const unsigned w_off = lane * 16;

  typedef __attribute__((address_space(3))) void *lds_ptr_t;
  const unsigned lds_base = (unsigned)(size_t)(lds_ptr_t)smem;

  floatx16 acc[2][FM];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int bm = 0; bm < FM; ++bm)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[nb][bm][v] = 0.f;

  // activation fragment of m block bm, sub-step kk: row bm*32 + l32, chunk (2*kk + g) ^ swizzle(row);
  // the swizzle of a 128-byte row is (row >> 1) & 7, the same for every m block, and kk enters as an XOR with 32*kk
  const unsigned a_lane = l32 * 128 + ((g ^ ((l32 >> 1) & 7)) << 4);

  bf16x8 wf[4][8];   // [slot of the step][2*kk + nb]
  bf16x8 af[2][FM];

  auto issue_a = [&](int i, int stage, int step) {
    lds_dma16_at(a_base + (int64_t)step * 128, a_off[i], lds_base + stage * STAGE + (wave * FM + i) * 1024);
  };
  // Plain loads: the compiler places their vmcnt waits.  It counts only these loads, not the LDS-DMA
  // requests issued from inline assembly in between, so its waits are stricter than necessary, never
  // weaker.  (Hand-placed waits that relied on register loads and LDS-DMA completing in one common
  // order gave results that changed from run to run: the two kinds do not complete in issue order
  // relative to each other.)
  auto load_w = [&](bf16x8 &dst, int nb, int kk, int step) {
    dst = *(const bf16x8 *)(w_base[nb] + ((int64_t)step * 4 + kk) * 1024 + (uint64_t)w_off);
  };

  // prologue: steps 0, 1, 2 requested (FM + 8 requests per wave and step, activations and weights alternating)
#pragma unroll
  for (int s0 = 0; s0 < 3; ++s0) {
    const int step = s0 < nk ? s0 : nk - 1;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i < FM) issue_a(i, s0, step);
      load_w(wf[s0][i], i & 1, i >> 1, step);
    }
  }
  constexpr int V0 = 2 * FM;            // step 0 has landed (this wave's part; at most the 2 FM LDS-DMA requests of steps 1, 2 remain)
  __builtin_amdgcn_s_waitcnt(0x0F70 | (V0 & 15) | ((V0 >> 4) << 14));
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int bm = 0; bm < FM; ++bm) af[0][bm] = *(const bf16x8 *)(smem + a_lane + bm * 4096);

  int sa = 0;   // stage of the current step
  auto step_fn = [&](auto slot_c, const int it) {
    constexpr int slot = decltype(slot_c)::value;
    constexpr int lslot = (slot + 3) & 3;                 // the slot freed by the previous step takes the weights of step it+3
    const int sn = sa == NSA - 1 ? 0 : sa + 1;            // stage of step it+1
    const int sld = sa >= 2 ? sa - 2 : sa + 3;            // stage of step it+3 = stage of step it-2 (free)
    const int kl = it + 3 < nk ? it + 3 : nk - 1;         // clamped: the request count per step stays constant
    const unsigned char *st = smem + sa * STAGE, *stn = smem + sn * STAGE;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      if (kk == 3) {
        // Step it+1 (requested during step it-2) must be resident before its first fragments are read.
        // V1 LDS-DMA requests are younger than it (FM of step it-1, 3 FM / 4 of this step: 7, 8, 10, 12, 14 at FM = 4 .. 8).  Register
        // loads and LDS-DMA do not complete in one common order, so all V1 requests that may stay in flight
        // could be LDS-DMA ones: the wait is for V1 in total, not for V1 + the younger weight loads.
        constexpr int V1 = FM + 3 * FM / 4;
        __builtin_amdgcn_s_waitcnt(0x0F70 | (V1 & 15) | ((V1 >> 4) << 14));
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 0; i < 2 * FM; ++i) {
        const int nb = i / FM, bm = i % FM;
        acc[nb][bm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[slot][kk * 2 + nb], af[kk & 1][bm], acc[nb][bm], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (i % 2 == 0) af[(kk + 1) & 1][i / 2] = *(const bf16x8 *)((kk < 3 ? st : stn) + (a_lane ^ (unsigned)(((kk + 1) & 3) * 32)) + (i / 2) * 4096);
        const int a_req = kk * FM / 4 + i / FM;   // one or two activation requests per sub-step, FM per step
        if (i % FM == (FM - 1) / 2 && a_req < (kk + 1) * FM / 4) issue_a(a_req, sld, kl);
        if (i % FM == FM - 1) load_w(wf[lslot][kk * 2 + i / FM], i / FM, kk, kl);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    sa = sn;
  };
  for (int it = 0; it < nk; it += 4) {   // nk is a multiple of 4
    step_fn(std::integral_constant<int, 0>{}, it);
    step_fn(std::integral_constant<int, 1>{}, it + 1);
    step_fn(std::integral_constant<int, 2>{}, it + 2);
    step_fn(std::integral_constant<int, 3>{}, it + 3);
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);   // drain the clamped extra requests ...
  __builtin_amdgcn_s_barrier();         // ... of every wave, before LDS is reused by the epilogue
  // per-wave slab: one 32-row block of fp32 (272-byte rows), or, for the rotating epilogues, all FM blocks of bf16 (144-byte rows)
  unsigned char *slab = smem + wave * ((EPI == EPI_QKV || EPI == EPI_KV) ? FM * 32 * (64 * 2 + 16) : 32 * (64 * 4 + 16));
  gemm_epilogue_n64<EPI, FM, NORM_OUT>(p, acc, m0, n0, lane, slab, EPI == EPI_PARTIAL ? (int64_t)split * p.M * p.N : 0);
}

// FL > 0: two tile heights in a launch, 32 FM rows over the first columns of tiles and 32 FL over the last p.low_tiles_n (the rule and
// what it gives: plan_gemm_mid).  The tall tiles have the lower block ids, so the low ones start as CUs run out of tall ones.
template <int EPI, int FM, bool NORM_OUT, int FL>
__global__ __launch_bounds__(256) void gemm_wreg_kernel(GemmParams p) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int tiles_n = p.N / 256, block = blockIdx.x;
  if constexpr (FL > 0) {
    const int tall_n = tiles_n - p.low_tiles_n, tall = ((p.M + 32 * FM - 1) / (32 * FM) * tall_n + 7) / 8 * 8;
    if (block >= tall) {
      wreg_tile<EPI, FL, NORM_OUT>(p, smem, block - tall, tall_n, p.low_tiles_n);
      return;
    }
    wreg_tile<EPI, FM, NORM_OUT>(p, smem, block, 0, tall_n);
  } else {
    wreg_tile<EPI, FM, NORM_OUT>(p, smem, block, 0, tiles_n);
  }
}

template <int EPI, int FM, bool NORM_OUT, int FL = 0>
int launch_wreg_k(const GemmParams &p, hipStream_t st) {
  constexpr int SLAB = 4 * ((EPI == EPI_QKV || EPI == EPI_KV) ? FM * 32 * (64 * 2 + 16) : 32 * (64 * 4 + 16));
  constexpr int SMEM = 5 * FM * 32 * 128 > SLAB ? 5 * FM * 32 * 128 : SLAB;
  auto kern = gemm_wreg_kernel<EPI, FM, NORM_OUT, FL>;
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
    if (e != hipSuccess) return (int)e;
    attr_set = true;
  }
  const int tiles = ((p.M + 32 * FM - 1) / (32 * FM)) * (p.N / 256 - p.low_tiles_n) * p.n_splits;
  const int low = FL > 0 ? ((p.M + 32 * FL - 1) / (32 * FL)) * p.low_tiles_n : 0;
  hipLaunchKernelGGL(kern, dim3(((tiles + 7) / 8 + (low + 7) / 8) * 8), dim3(256), SMEM, st, p);
  return 0;
}
template <int EPI, bool NORM_OUT>
int launch_fm(const GemmParams &p, int fm, hipStream_t st) {
  switch (fm) {
    case 4: return launch_wreg_k<EPI, 4, NORM_OUT>(p, st);
    case 5: return launch_wreg_k<EPI, 5, NORM_OUT>(p, st);
    case 6: return launch_wreg_k<EPI, 6, NORM_OUT>(p, st);
    case 7: return launch_wreg_k<EPI, 7, NORM_OUT>(p, st);
    case 8: return launch_wreg_k<EPI, 8, NORM_OUT>(p, st);
  }
  return -1;
}

}  // namespace

// tile height 32 * fm (the last p.low_tiles_n columns of tiles: 32 * fm_low), p.n_splits ranges of p.split_steps (a multiple of 4) 64-wide steps
int launch_gemm_wreg(const GemmParams &p, int epi, int fm, int fm_low, hipStream_t st) {
  if (fm_low) {
    if (epi != EPI_SWIGLU || fm != 8 || p.n_splits != 1) return -1;
    return fm_low == 6 ? launch_wreg_k<EPI_SWIGLU, 8, false, 6>(p, st) : fm_low == 4 ? launch_wreg_k<EPI_SWIGLU, 8, false, 4>(p, st) : -1;
  }
  switch (epi) {
    case EPI_STORE_BF16: return launch_fm<EPI_STORE_BF16, false>(p, fm, st);
    case EPI_RESID: return p.hb && p.ssq ? launch_fm<EPI_RESID, true>(p, fm, st) : launch_fm<EPI_RESID, false>(p, fm, st);
    case EPI_SWIGLU: return launch_fm<EPI_SWIGLU, false>(p, fm, st);
    case EPI_QKV: return launch_fm<EPI_QKV, false>(p, fm, st);
    case EPI_KV: return launch_fm<EPI_KV, false>(p, fm, st);
    case EPI_PARTIAL: return launch_fm<EPI_PARTIAL, false>(p, fm, st);
  }
  return -1;
}
