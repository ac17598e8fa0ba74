// Grouped fp32 GEMM of the fp32 layer on the bf16 matrix cores.
//
// Same contract as the bf16 kernels: C[row, n] = sum_k A[row, k] * B_group[n, k], with row-tiles that each
// belong to one group, and an optional fused SwiGLU (B holds gate rows then up rows).
//
// An fp32 number is the sum of three bf16 numbers (8 + 8 + 8 bits, each the rounded rest of the one before), and
// products of bf16 numbers are exact in fp32.  Six of the nine partial products are taken; two of those left out may reach
// 2^-25 of the product each.  The leading one is summed on its own, the other five, a hundredth of it, beside it, so that
// what they lose to rounding does not show.  Against 64 bits (2-norm) sums of 1024 products then FFN: 3.2e-7, where
// v_mfma_f32_16x16x4_f32 gives 9.6e-7; of 256: 1.6e-7 and 4.8e-7 (with all six in one sum 8.2e-7 and 3.8e-7).  A K-step
// of 32 takes 6 x 16 cycles of the matrix cores for 16 x 16 outputs, instead of 8 x 32.
// The parts of numbers below 2^-110 are denormal (the matrix cores keep those) and lose up to 2^-134 of them: a sum of K
// products up to K 2^-134 times the largest numbers of its two rows together.  Sums that are not 2^22 times as large, and
// not of zeros, are worked out again in fp32 (redo); so are those that are not finite, since a number that rounds to no
// finite bf16, or is not finite itself, makes its sums NaN.  With numbers in ordinary ranges neither occurs.  To know the
// largest numbers costs 2 % (layer of 1001 tokens, H = 1024, I = 512, 32 experts: 171.6 -> 174.5 us).  us of the FFN, H =
// 1024, I = 512, 36 slots and a shared expert, 5 and 110 rows per slot: 58 and 240; one row of NaN 59 and 220, one infinity
// 79 and 220, all NaN 69 and 267, all x of 2^-115 159 and 608 (v_mfma_f32_16x16x4_f32 throughout: 70 and 260 to 290).  The
// sums in fp32 read their operands a row per lane, which is what they wait for; loads two groups ahead gained nothing.
//
// 64 x 64 outputs per workgroup of four wavefronts, each with all the tile's rows and 16 output columns (SwiGLU: 16 gate
// and 16 up), so that a tile of few rows keeps every wavefront equally busy and skips the 16-row sub-tiles it has not
// got.  K is walked in steps of 32 through two LDS buffers, one barrier per step; loads are two steps ahead.  The words of
// the next step are taken apart between the MFMAs of this one (scheduling groups), which is what the time goes into.  Layer of
// 1001 tokens, gate/up and down: vector instructions 37 and 43 % of the cycles, LDS 33 and 44, MFMAs 26 and 23.
// us of the FFN, H = 1024, I = 512, 36 slots and a shared expert, against v_mfma_f32_16x16x4_f32: 5 rows per slot 72 and
// 57, 25 rows 100 and 83, 110 rows 259 and 198; H = 360, I = 180, 8 rows 26 and 20; H = 1024, I = 64, 800 rows 107 and 78.
// Taken apart ahead of the MFMAs instead: 63, 88, 216.  As fast or slower: one LDS buffer and three workgroups per CU (63
// to 67, 84 to 87, 209), eight wavefronts per workgroup (68, 83, 205), loads four steps ahead (63, 84, 204).
#pragma once

#include <hip/hip_runtime.h>

#include <cfloat>
#include <cmath>
#include <type_traits>

#include "gemm_bf16.hpp"
#include "gemm_f32.hpp"
#include "row_tiles.hpp"

namespace revive {

// Off: bytes between the first of a tile's 64 rows and any element of them.
template <bool SWIGLU, typename Off>
__global__ __launch_bounds__(256, SWIGLU ? 2 : 3) void gemm_f32_split_kernel(GemmF32Args a) {
  // Known to address HBM: global loads.  A pointer out of the weight table made flat ones, which every LDS wait drains.
  typedef const __attribute__((address_space(1))) unsigned char* gptr;
  typedef const __attribute__((address_space(1))) f32x4* gptr_f32x4;
  constexpr int BM = kTileM_f32, BN = kTileN_f32, W = SWIGLU ? 2 : 1, D = 2;
  constexpr int NB = W * BN * 8 / 256;           // 16-byte words of weights per thread and K-step
  constexpr int PLANE = (BM + W * BN) * 64;      // bytes of one of the three parts of a step: rows of 32 bf16
  __shared__ __attribute__((aligned(16))) unsigned char lds[2][3 * PLANE];
  __shared__ __attribute__((aligned(16))) float largest[BM + W * BN];  // magnitude in each row of the tile and of the weights
  const bool dense = blockIdx.x < static_cast<unsigned>(a.dense.blocks);
  const GemmF32Problem g = dense ? a.dense : a.grouped;
  const int b = dense ? blockIdx.x : blockIdx.x - a.dense.blocks;
  int row_begin, row_end, n_idx;
  const float* B;
  if (dense) {
    const int m_idx = b / g.n_col_tiles;
    n_idx = b - m_idx * g.n_col_tiles;
    row_begin = m_idx * BM;
    row_end = min(g.M, row_begin + BM);
    B = g.B_one;
  } else {
    const GridTile t = grid_tile(a.slot_offsets, a.P, BM, g.n_col_tiles, b, g.B_tab);
    if (t.group < 0) return;
    n_idx = t.n_idx;
    row_begin = t.row_begin;
    row_end = t.row_end;
    B = static_cast<const float*>(t.w);
  }
  const int n0 = n_idx * BN, rows = row_end - row_begin;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  auto publish = [&]() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  const int KT = (g.K + 31) >> 5;
  const int r16 = lane & 15, quad = lane >> 4;
  const int get = r16 * 64 + ((quad ^ swz32(r16)) << 4);  // 16 rows further on the swizzle is the same
  auto base = [](const float* p) { return reinterpret_cast<gptr>(reinterpret_cast<uintptr_t>(p)); };
  const gptr a_base = base(g.A + static_cast<int64_t>(row_begin) * g.lda);
  const gptr b_base[2] = {base(B + n0 * g.ldb), base(B + (static_cast<int64_t>(n0) + g.n_out) * g.ldb)};
  auto run = [&](auto tm_tag) {
    constexpr int TM = decltype(tm_tag)::value;
    // keeps the four forms' beginnings apart: shared, they would stay in registers through the first form's loop (40 spilled)
    asm volatile("; %0 sub-tiles" ::"n"(TM) : "memory");
    // copy plan: 16-byte word w of a step is K-chunk w % 8 of row w / 8
    constexpr int NA = (TM + 1) / 2;  // words of activations per thread and K-step: no more rows than the tile's sub-tiles hold
    constexpr int WORDS = NA + NB;
    const int c = tid & 7, r0 = tid >> 3, put = r0 * 64 + (((c >> 1) ^ swz32(r0)) << 4) + (c & 1) * 8;
    Off a_off[NA], b_off[BN / 32];  // bytes from the uniform bases
#pragma unroll
    for (int i = 0; i < NA; ++i) a_off[i] = static_cast<Off>(min(i * 32 + r0, rows - 1)) * static_cast<Off>(g.lda * 4);  // rows past the tile read its last row again
#pragma unroll
    for (int i = 0; i < BN / 32; ++i) b_off[i] = static_cast<Off>(min(i * 32 + r0, g.n_out - 1 - n0)) * static_cast<Off>(g.ldb * 4);
    f32x4 word[D][WORDS];  // of the activations, then of the weights
    float top[WORDS];      // largest magnitude of the row's words that this thread has staged
#pragma unroll
    for (int u = 0; u < WORDS; ++u) top[u] = 0.f;
    auto load = [&](int kt, int d) {  // past the last K-element: the last four again
      const Off k = static_cast<Off>(min(kt * 32 + c * 4, g.K - 4)) * 4;
#pragma unroll
      for (int i = 0; i < NA; ++i) word[d][i] = *reinterpret_cast<gptr_f32x4>(a_base + (a_off[i] + k));
#pragma unroll
      for (int i = 0; i < NB; ++i) word[d][NA + i] = *reinterpret_cast<gptr_f32x4>(b_base[i / (BN / 32)] + (b_off[i % (BN / 32)] + k));
    };
    auto stage = [&](int kt, int d, int buf, int u) {
      f32x4 v = word[d][u];
      if (u < NA) {  // K-elements past the last one count as zero; of one operand is enough
        const bool in = kt * 32 + c * 4 < g.K;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = in ? v[j] : 0.f;
      }
      // not fmaxf(), which would first quieten its operands
#pragma unroll
      for (int j = 0; j < 4; ++j) top[u] = __builtin_elementwise_maximum(top[u], fabsf(v[j]));
      unsigned char* dst = lds[buf] + put + (u < NA ? u * (32 * 64) : BM * 64 + (u - NA) * (32 * 64));
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const u32x2 part = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        *reinterpret_cast<u32x2*>(dst + p * PLANE) = part;
        if (p < 2) {  // what the part leaves over, exactly
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] -= __uint_as_float(j & 1 ? part[j >> 1] & 0xffff0000u : part[j >> 1] << 16);
        }
      }
    };
    f32x4 acc[W][TM], low[W][TM];
#pragma unroll
    for (int s = 0; s < W; ++s)
#pragma unroll
      for (int i = 0; i < TM; ++i) acc[s][i] = low[s][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    // The products of step kt, in buffer `buf`; between them (STAGE) the next step's words, d_next of the ring, go into
    // the other buffer.
    auto step = [&](int kt, int d_next, int buf, auto stage_tag) {
      constexpr bool STAGE = decltype(stage_tag)::value;
      bf16x8 x[3][TM], w[3][W];
      auto read = [&](int pw, int px) {
#pragma unroll
        for (int s = 0; s < W; ++s) w[pw][s] = *reinterpret_cast<const bf16x8*>(lds[buf] + pw * PLANE + get + (BM + wave * 16 + s * BN) * 64);
#pragma unroll
        for (int i = 0; i < TM; ++i) x[px][i] = *reinterpret_cast<const bf16x8*>(lds[buf] + px * PLANE + get + i * (16 * 64));
      };
      read(0, 2);
      read(2, 0);
      __builtin_amdgcn_sched_barrier(0);
      constexpr int PW[6] = {0, 2, 1, 0, 1, 0}, PX[6] = {2, 0, 1, 1, 0, 0};  // parts that are multiplied, the smallest products first
#pragma unroll
      for (int q = 0; q < 6; ++q) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int s = 0; s < W; ++s) {
            f32x4& sum = q < 5 ? low[s][i] : acc[s][i];
            sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[PW[q]][s], x[PX[q]][i], sum, 0, 0, 0);
          }
        if (q == 0) read(1, 1);
        if (!STAGE) continue;
#pragma unroll
        for (int u = 0; u < WORDS; ++u)
          if (u * 6 / WORDS == q) stage(kt + 1, d_next, buf ^ 1, u);
        // an MFMA (0x008) and three vector instructions (0x002) in turn, then the LDS writes (0x200) and reads (0x100)
#pragma unroll
        for (int m = 0; m < TM * W; ++m) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x200, 3, 0);
        if (q == 0) __builtin_amdgcn_sched_group_barrier(0x100, TM + W, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    using Y = std::true_type;
    using F = std::false_type;
    // every load is unconditional, so that the compiler's count of loads in flight stays exact; surplus ones
    // fetch the last step again and are not multiplied
#pragma unroll
    for (int d = 0; d < D; ++d) load(min(d, KT - 1), d);
#pragma unroll
    for (int u = 0; u < WORDS; ++u) stage(0, 0, 0, u);
    publish();
    int kt = 0;
    for (; kt + D < KT; kt += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        load(min(kt + D + d, KT - 1), d);  // the place of this step's words, which are in LDS
        __builtin_amdgcn_sched_barrier(0);
        step(kt + d, d ^ 1, d, Y{});
        publish();
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // Once the last words are staged.  The lane's numbers are worked out here and not ahead of the loop, where they would
    // take registers; likewise below.
    auto late = [&]() {
      int t = tid;
      asm volatile("" : "+v"(t));
      return t;
    };
    auto share_largest = [&]() {
      int m[WORDS];  // not negative: in the order of the numbers
#pragma unroll
      for (int u = 0; u < WORDS; ++u) m[u] = __float_as_int(top[u]);
      // the eight threads of a row: lanes ^ 1, ^ 2 and 7 - lane
#pragma unroll
      for (int u = 0; u < WORDS; ++u) m[u] = max(m[u], dpp_or_zero<0xB1, 0xF>(m[u]));
#pragma unroll
      for (int u = 0; u < WORDS; ++u) m[u] = max(m[u], dpp_or_zero<0x4E, 0xF>(m[u]));
#pragma unroll
      for (int u = 0; u < WORDS; ++u) m[u] = max(m[u], dpp_or_zero<0x141, 0xF>(m[u]));
      const int t = late();
      if ((t & 7) == 0) {
#pragma unroll
        for (int u = 0; u < WORDS; ++u) largest[(u < NA ? u * 32 : BM + (u - NA) * 32) + (t >> 3)] = __int_as_float(m[u]);
      }
    };
    if (kt + 1 < KT) {
      step(kt, 1, 0, Y{});
      share_largest();
      publish();
      step(kt + 1, 0, 1, F{});
    } else {
      share_largest();
      step(kt, 0, 0, F{});
      publish();
    }
    const int t = late(), r16 = t & 15, quad = t >> 4 & 3;
    // the size from which on a sum has lost nothing that counts, in two terms; none where a row has only zeros
    const float share = static_cast<float>(g.K) * 0x1p-112f;
    auto term = [&](float top) { return top > 0.f ? top * share : -INFINITY; };
    f32x4 w_term[W];
    float w_most = -INFINITY;
#pragma unroll
    for (int s = 0; s < W; ++s) {
      w_term[s] = *reinterpret_cast<const f32x4*>(&largest[BM + s * BN + wave * 16 + quad * 4]);
#pragma unroll
      for (int r = 0; r < 4; ++r) w_most = fmaxf(w_most, w_term[s][r] = term(w_term[s][r]));
    }
    // a lane holds four consecutive output columns of activation row lane % 16
    const int col = n0 + wave * 16 + quad * 4;
    bool suspect = false;  // a sum of the lane's may not be what the parts give
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      float least = FLT_MAX, total = 0.f;
#pragma unroll
      for (int s = 0; s < W; ++s) {
        acc[s][i] += low[s][i];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float size = fabsf(acc[s][i][r]);
          least = fminf(least, size);
          total += size;
        }
      }
      suspect |= !((total <= FLT_MAX) & (least >= term(largest[i * 16 + r16]) + w_most));
      const int row = row_begin + i * 16 + r16;
      if (row >= row_end || col >= g.n_out) continue;
      f32x4 v = acc[0][i];
      if (SWIGLU) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = v[r] / (1.0f + expf(-v[r])) * acc[W - 1][i][r];
      }
      *reinterpret_cast<f32x4*>(g.C + static_cast<int64_t>(row) * g.ldc + col) = v;  // n_out is a multiple of 4
    }
    if (__ballot(suspect) == 0) return;
    uint32_t redo = 0;  // outputs i * 4 + r with a sum that the parts do not give
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const float x_term = term(largest[i * 16 + r16]);
      uint32_t fine = 15;
#pragma unroll
      for (int s = 0; s < W; ++s)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float size = fabsf(acc[s][i][r]);
          if (!((size <= FLT_MAX) & (size >= x_term + w_term[s][r]))) fine &= ~(1u << r);
        }
      if (row_begin + i * 16 + r16 < row_end && col < g.n_out) redo |= (fine ^ 15) << (i * 4);
    }
    // In fp32 then, 16 rows at a time where one of the wavefront's lanes asks for it: operands from memory, 16x16x4 MFMAs.
    // Both operands permute K alike, as a lane's 16 bytes are four consecutive K-elements that feed four MFMAs.  A sum that
    // is NaN stays it, and one row of NaN makes its sums NaN throughout: no further where nothing else is left.
    const gptr w_row = base(B + min(n0 + wave * 16 + r16, g.n_out - 1) * g.ldb);
#pragma unroll 1
    for (int i = 0; i < TM; ++i) {
      const uint32_t mine = redo >> (i * 4) & 15;
      if (__ballot(mine != 0) == 0) continue;
      const int row = row_begin + i * 16 + r16;
      const gptr x_row = base(g.A + static_cast<int64_t>(min(row, row_end - 1)) * g.lda);
      constexpr int U = 4;  // groups of 16 K-elements that are loaded together, each with sums of its own
      f32x4 sum[U][W], all[W];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int s = 0; s < W; ++s) sum[u][s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int k0 = 0; k0 < g.K; k0 += U * 16) {
        f32x4 x[U], w[U][W];
#pragma unroll
        for (int u = 0; u < U; ++u) {  // past the last K-element: zeros, not the last four again
          const int64_t k = min(k0 + u * 16 + quad * 4, g.K - 4) * 4ll;
          x[u] = *reinterpret_cast<gptr_f32x4>(x_row + k);
#pragma unroll
          for (int s = 0; s < W; ++s) w[u][s] = *reinterpret_cast<gptr_f32x4>(w_row + s * g.n_out * g.ldb * 4 + k);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bool in = k0 + u * 16 + quad * 4 < g.K;
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int s = 0; s < W; ++s) sum[u][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? w[u][s][j] : 0.f, in ? x[u][j] : 0.f, sum[u][s], 0, 0, 0);
        }
        bool open = false;
#pragma unroll
        for (int s = 0; s < W; ++s) all[s] = (sum[0][s] + sum[1][s]) + (sum[2][s] + sum[3][s]);
#pragma unroll
        for (int r = 0; r < 4; ++r) open |= (mine >> r & 1) && !(isnan(all[0][r]) || isnan(all[W - 1][r]));
        if (__ballot(open) == 0) break;
      }
      f32x4 v = all[0];
      if (SWIGLU) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = v[r] / (1.0f + expf(-v[r])) * all[W - 1][r];
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (mine >> r & 1) g.C[static_cast<int64_t>(row) * g.ldc + col + r] = v[r];
    }
  };
  if (rows <= 16) run(std::integral_constant<int, 1>{});
  else if (rows <= 32) run(std::integral_constant<int, 2>{});
  else if (rows <= 48) run(std::integral_constant<int, 3>{});
  else run(std::integral_constant<int, 4>{});
}

// Either problem may be absent (blocks == 0).
template <bool SWIGLU>
int launch_gemm_f32_split(revive_ctx* ctx, const GemmF32Args& args, hipStream_t stream) {
  const int grid = args.dense.blocks + args.grouped.blocks;
  if (grid <= 0) return REVIVE_OK;
  const bool narrow = args.dense.lda < kNarrowRows_f32 && args.grouped.lda < kNarrowRows_f32;  // ldb = lda
  const auto kernel = narrow ? gemm_f32_split_kernel<SWIGLU, uint32_t> : gemm_f32_split_kernel<SWIGLU, uint64_t>;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, stream, args);
  return check_hip(ctx, hipGetLastError(), "gemm_f32_split launch");
}

}  // namespace revive
