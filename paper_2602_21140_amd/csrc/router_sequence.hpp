// Router logits in bf16: x [T, H] times w [E, H]^T, fp32 sums, with K summed in one sequence of 16x16x32 MFMAs (or in
// slices that are added in their order).
//
// A token's logits must not depend on how many others are in the call, so both kernels here give the same bits.
#pragma once

#include <hip/hip_runtime.h>

#include "gemm_bf16.hpp"

namespace revive {

__device__ __forceinline__ f32x4 mfma_16x16x32(u32x4 a, u32x4 b, f32x4 acc) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

// Few tokens: XR tokens and WR experts per workgroup (8 or 16; the MFMA's other rows repeat them).  Eight wavefronts
// fetch eight steps of 64 K-elements at a time, D rounds ahead, and the first one multiplies them in order.
// Bound by latency: the chain of 224 dependent MFMAs at H = 7168 and the LDS reads in front of them, which a condition
// per step kept from running ahead.  E = 256, H = 7168, us back to back and with cold caches: 1 token 11.8 and 14.4 ->
// 9.2 and 12.3 without that condition, 7.6 and 11.1 with 8 x 8 tiles; 24 tokens 11.8 and 15.2 -> 7.9 and 12.2; 192
// tokens (16 x 16 tiles) 12.2 and 15.5 -> 9.7 and 14.7.  More rounds ahead are slower (8 x 8 tiles, 6 rounds 8.4).
template <int XR, int WR, int D>
__global__ __launch_bounds__(512, 2) void router_sequence_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ w,
                                                                 float* __restrict__ logits, int T, int E, int H, int n_exp) {
  constexpr int KS = 8, NX = XR / 8, NL = NX + WR / 8;
  static_assert(D % 2 == 0, "the LDS buffer of a round is its position in the register ring modulo 2");
  __shared__ __attribute__((aligned(16))) unsigned char lds[2][KS][NL * 8 * 128];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t0 = blockIdx.x / n_exp * XR, e0 = blockIdx.x % n_exp * WR;
  const int64_t row_bytes = static_cast<int64_t>(H) * 2;
  const unsigned char* xb = reinterpret_cast<const unsigned char*>(x) + t0 * row_bytes;
  const unsigned char* wb = reinterpret_cast<const unsigned char*>(w) + e0 * row_bytes;
  const int steps = H >> 6;  // H is a multiple of 64
  uint32_t off[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {  // rows past the last token or expert: the last one again, not stored
    const int r = (i < NX ? i : i - NX) * 8 + (lane >> 3);
    off[i] = static_cast<uint32_t>((i < NX ? min(r, T - 1 - t0) : min(r, E - 1 - e0)) * row_bytes + (lane & 7) * 16);
  }
  u32x4 buf[D][NL];
  auto load = [&](int round, int d) {
    const int64_t k = static_cast<int64_t>(min(round * KS + wave, steps - 1)) * 128;
#pragma unroll
    for (int i = 0; i < NL; ++i) buf[d][i] = load_global_16B((i < NX ? xb : wb) + off[i] + k);
  };
  const int r16 = lane & 15, quad = lane >> 4;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  const int rx = r16 % XR, rw = XR + r16 % WR;
  auto multiply = [&](int b, int n) {
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      if (q < n) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const u32x4 fw = *reinterpret_cast<const u32x4*>(lds[b][q] + rw * 128 + (((h * 4 + quad) ^ swz(rw)) << 4));
          const u32x4 fx = *reinterpret_cast<const u32x4*>(lds[b][q] + rx * 128 + (((h * 4 + quad) ^ swz(rx)) << 4));
          acc = mfma_16x16x32(fw, fx, acc);
        }
      }
    }
  };
#pragma unroll
  for (int d = 0; d < D; ++d) load(d, d);
  for (int r0 = 0;; r0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if ((r0 + d) * KS >= steps) goto done;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int r = i * 8 + (lane >> 3);
        *reinterpret_cast<u32x4*>(lds[d & 1][wave] + r * 128 + (((lane & 7) ^ swz(r)) << 4)) = buf[d][i];
      }
      load(r0 + d + D, d);
      // A buffer is written again two barriers later: the first wavefront has then read it.
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      if (wave == 0) {
        // A whole round without a condition inside: its fragment reads run ahead of the chain of MFMAs.
        const int left = steps - (r0 + d) * KS;
        if (left >= KS) multiply(d & 1, KS);
        else multiply(d & 1, left);
      }
    }
  }
done:
  if (wave == 0 && r16 < XR && t0 + r16 < T) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = quad * 4 + i;
      if (e < WR && e0 + e < E) logits[static_cast<int64_t>(t0 + r16) * E + e0 + e] = acc[i];
    }
  }
}

// More tokens: BM tokens and BN experts per workgroup of WM x WN wavefronts; K in steps of BK through a ring of S
// stages filled by asynchronous global->LDS copies.  What bounds it is how fast a CU pulls its rows of x and w in out
// of L2, or with a short K the start and end of a tile (router_form has the rule and the figures).
//
// LDS layout of a stage: row r (tokens, then experts) at r * BK * 2 bytes, its 16-byte chunks stored at chunk ^ swizzle,
// so that the 16 rows of a fragment read fall on 16 different 16-byte bank groups.
//
// SLICES > 1: K is summed in SLICES parts, [H/64 * q / SLICES, H/64 * (q+1) / SLICES) steps of 64 elements, and the
// partial sums are added in their order: the bits of router_kernel, whose wavefronts share K that way.
template <int BM, int BN, int WM, int WN, int BK, int S, int SLICES = 1>
__global__ __launch_bounds__(64 * WM * WN) void router_tile_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ w,
                                                                   float* __restrict__ logits, int T, int E, int H, int n_tok, int n_exp) {
  constexpr int NW = WM * WN, TM = BM / WM / 16, TN = BN / WN / 16;
  constexpr int ROWB = BK * 2, CH = ROWB / 16, RPC = 64 / CH;  // bytes and chunks of a row, rows of one copy instruction
  constexpr int CP = (BM + BN) / RPC / NW, STAGE = (BM + BN) * ROWB;
  static_assert(BK == 64 || (BK == 128 && SLICES == 1), "swizzles and slices below");
  static_assert(BM % (WM * 16) == 0 && BN % (WN * 16) == 0 && BM % RPC == 0 && (BM + BN) % (RPC * NW) == 0, "tile shape");
  typedef __attribute__((address_space(3))) void* lptr;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  auto swizzle = [](int row) { return BK == 64 ? (row >> 1) & 7 : row & 15; };
  // Workgroup i runs on XCD i % 8: a token tile's workgroups share its rows of x in one XCD's L2.
  const int local = blockIdx.x >> 3, tok = local / n_exp * 8 + (blockIdx.x & 7), ex = local % n_exp;
  if (tok >= n_tok) return;
  const int t0 = tok * BM, e0 = ex * BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const uint32_t row_bytes = static_cast<uint32_t>(H) * 2;
  // copy i of this wavefront fills rows [(i * NW + wave) * RPC, + RPC) of a stage
  uint32_t cp_off[CP];
#pragma unroll
  for (int i = 0; i < CP; ++i) {  // rows past the last token or expert: the last one again, not stored
    const int r = (i * NW + wave) * RPC + lane / CH, chunk = (lane % CH) ^ swizzle(r);
    cp_off[i] = (r < BM ? min(r, T - 1 - t0) : min(r - BM, E - 1 - e0)) * row_bytes + chunk * 16;
  }
  const uint32_t smem_lds = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lptr)smem));
  const uint64_t base_x = reinterpret_cast<uint64_t>(x) + static_cast<uint64_t>(t0) * row_bytes;
  const uint64_t base_w = reinterpret_cast<uint64_t>(w) + static_cast<uint64_t>(e0) * row_bytes;
  // H is a multiple of 64 and not below BK.  A last step that K does not fill takes K's last BK elements, of which
  // only the second half is new.
  const int KT = (H + BK - 1) / BK;
  // Past the last step the last one is copied again (not multiplied), so that the count of copies in flight stays exact.
  auto issue_copy = [&](int kt) {
    const uint32_t stage = smem_lds + kt % S * STAGE;
    const uint64_t k = min(static_cast<uint32_t>(kt) * ROWB, row_bytes - ROWB);
#pragma unroll
    for (int i = 0; i < CP; ++i) {
      const int blk = i * NW + wave;
      const uint64_t src = (blk * RPC < BM ? base_x : base_w) + k;
      const uint32_t dst = __builtin_amdgcn_readfirstlane(stage + blk * 1024);
      copy_to_lds_16B(dst, src, cp_off[i]);
    }
  };
  f32x4 acc[TM][TN], sum[TM][TN];  // sum: the finished slices
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = sum[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  int slice = 1, slice_end = KT / SLICES;  // empty slices (KT < SLICES) are passed over
  if (SLICES > 1)
    while (slice_end == 0) slice_end = KT * ++slice / SLICES;
  const int r16 = lane & 15, quad = lane >> 4, sw = swizzle(r16);  // the swizzles have period 16
  auto step = [&](int kt, int h0) {
    // this wavefront's copies of step kt have landed; after the barrier everybody's have, and stage kt - 1 is free
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((S - 2) * CP));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    issue_copy(kt + S - 1);
    const unsigned char* cur = smem + kt % S * STAGE + r16 * ROWB;
#pragma unroll
    for (int h = 0; h < BK / 32; ++h) {
      if (h < h0) continue;
      const int c = ((h * 4 + quad) ^ sw) << 4;
      u32x4 a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = *reinterpret_cast<const u32x4*>(cur + (wm * TM + i) * (16 * ROWB) + c);
#pragma unroll
      for (int j = 0; j < TN; ++j) b[j] = *reinterpret_cast<const u32x4*>(cur + (BM / 16 + wn * TN + j) * (16 * ROWB) + c);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma_16x16x32(b[j], a[i], acc[i][j]);
    }
    if (SLICES > 1 && kt + 1 == slice_end) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          sum[i][j] += acc[i][j];
          acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      while (slice < SLICES && slice_end == kt + 1) slice_end = KT * ++slice / SLICES;
    }
  };
#pragma unroll
  for (int s = 0; s < S - 1; ++s) issue_copy(s);
  for (int kt = 0; kt + 1 < KT; ++kt) step(kt, 0);
  step(KT - 1, (KT * BK - H) / 32);
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));  // no copy lands in LDS after this workgroup
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int t = t0 + (wm * TM + i) * 16 + r16;
    if (t >= T) continue;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const f32x4 v = SLICES > 1 ? sum[i][j] : acc[i][j];
      const int e = e0 + (wn * TN + j) * 16 + quad * 4;
      float* dst = logits + static_cast<int64_t>(t) * E + e;
      if (e + 3 < E && (E & 3) == 0) {
        *reinterpret_cast<f32x4*>(dst) = v;
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (e + r < E) dst[r] = v[r];
      }
    }
  }
}

}  // namespace revive
