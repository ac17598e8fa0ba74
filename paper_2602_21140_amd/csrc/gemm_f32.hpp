// Grouped fp32 GEMM of the fp32 layer on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 products and sums).
//
// Same contract as the bf16 kernels: C[row, n] = sum_k A[row, k] * B_group[n, k], with row-tiles that each
// belong to one group, and an optional fused SwiGLU (B holds gate rows then up rows).
//
// 64 x 64 outputs per workgroup of four wavefronts, each with all the tile's rows and 16 output columns
// (SwiGLU: 16 gate and 16 up), so that a tile of few rows keeps every wavefront equally busy and skips the
// 16-row sub-tiles it has not got.  K is walked in steps of 32 through two LDS buffers, one barrier per
// step, with the loads of D steps in flight in registers.  A lane's 16 LDS bytes are four consecutive
// K-elements of its row and feed four MFMAs (both operands permute K alike).  The matrix cores are what
// bounds a full tile (16 MFMAs of 32 cycles per 16 K-elements and wavefront against 160 to 192 cycles of
// LDS for the whole workgroup); a tile of few rows is bound by latency.  D = 4 takes 216 registers with SwiGLU, one
// workgroup per CU less, and is 1 to 19 % slower there (2181 tokens, H = 88, I = 1288, 256 experts, k = 4: 211 -> 250 us;
// 3952 tokens, H = 312, I = 168: 113 -> 129); tiles of up to 16 rows gain where a CU has several of them (7 tokens, H =
// 296, I = 1188, 128 experts, k = 8: 68 -> 52 us; 10 tokens, H = 368, I = 1928: 66 -> 54) and nothing where it has one
// (5 tokens, H = 1144, I = 80: 28).  D = 2 throughout.  Loads issued a step earlier gained nothing.
// Vector instructions between the MFMAs cost as well: a thread keeps 32-bit offsets from wavefront-uniform bases and
// LDS addresses that are the same in every step, and copies only as many rows as the tile has sub-tiles.  Routed and
// shared expert, H = 1024, I = 512, 32 experts, k = 4: 200 tokens 91 -> 82 us, 1001 tokens 199 -> 184, 4000 tokens
// 580 -> 557 (113 TFLOP/s).  What is left at 1001 tokens is balance: of gate/up's 800 workgroups, of one to four sub-tiles
// each, 768 fit at once (48 KiB of LDS, three to a CU), and CUs end between 81 and 132 us.
// Narrower workgroups spread better and lose more by reading the activations twice as often (1001 tokens 195 us; of
// two wavefronts, 239, since they load the SIMDs unevenly).
//
// Against the vector-FMA kernel that stood here (64 x 64 tiles, no load ahead of its use): the same
// layer, 1 token 288 -> 45 us, 1001 tokens 408 -> 204 us, 4000 tokens 920 -> 589 us.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "ctx.hpp"
#include "row_tiles.hpp"

namespace revive {

struct GemmF32Problem {
  const float* A;
  int64_t lda;
  const void* const* B_tab;  // slot -> weights (grouped), or
  const float* B_one;        // the one weight matrix (dense)
  int64_t ldb;
  float* C;
  int64_t ldc;
  int n_out;
  int K;  // multiple of 4
  int n_col_tiles;
  int blocks;  // workgroups of the grid that belong to this problem
  int M;       // rows (dense)
};

struct GemmF32Args {
  GemmF32Problem dense;    // served by the first dense.blocks workgroups
  GemmF32Problem grouped;  // served by the others
  const int32_t* slot_offsets;
  int P;
};

constexpr int kTileN_f32 = 64;

// SLICES > 1: the K-steps are summed in SLICES parts that are added in their order (see router_tile_kernel).
// Off: bytes between the first of a tile's 64 rows and any element of them.
template <bool SWIGLU, int D, int SLICES, typename Off>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmF32Args a) {
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  // Known to address HBM: global loads.  A pointer out of the weight table made flat ones, which every LDS wait drains.
  typedef const __attribute__((address_space(1))) unsigned char* gptr;
  typedef const __attribute__((address_space(1))) f32x4* gptr_f32x4;
  constexpr int BM = kTileM_f32, BN = kTileN_f32, W = SWIGLU ? 2 : 1;
  constexpr int NB = W * BN * 8 / 256;  // 16-byte words of weights per thread and K-step
  static_assert(D % 2 == 0, "the LDS buffer of a step is its position in the register ring modulo 2");
  __shared__ __attribute__((aligned(16))) unsigned char lds[2][(BM + W * BN) * 128];
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
    const GridTile t = grid_tile(a.slot_offsets, a.P, BM, g.n_col_tiles, b);
    if (t.group < 0) return;
    n_idx = t.n_idx;
    row_begin = t.row_begin;
    row_end = t.row_end;
    B = static_cast<const float*>(g.B_tab[t.group]);
  }
  const int n0 = n_idx * BN, rows = row_end - row_begin;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // 16 rows further on the swizzle is the same
  auto swizzle = [](int row, int c) { return row * 128 + ((c ^ ((row >> 1) & 7)) << 4); };

  auto publish = [&]() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  const int KT = (g.K + 31) >> 5;
  const int r16 = lane & 15, quad = lane >> 4;
  const int get[2] = {swizzle(r16, quad), swizzle(r16, 4 + quad)};
  auto base = [](const float* p) { return reinterpret_cast<gptr>(reinterpret_cast<uintptr_t>(p)); };
  const gptr a_base = base(g.A + static_cast<int64_t>(row_begin) * g.lda);
  const gptr b_base[2] = {base(B + n0 * g.ldb), base(B + (static_cast<int64_t>(n0) + g.n_out) * g.ldb)};
  auto run = [&](auto tm_tag) {
    constexpr int TM = decltype(tm_tag)::value;
    // copy plan: 16-byte word w of a step is K-chunk w % 8 of row w / 8
    constexpr int NA = (TM + 1) / 2;  // words of activations per thread and K-step: no more rows than the tile's sub-tiles hold
    const int c = tid & 7, r0 = tid >> 3, put = swizzle(r0, c);
    Off a_off[NA], b_off[BN / 32];  // bytes from the uniform bases
#pragma unroll
    for (int i = 0; i < NA; ++i) a_off[i] = static_cast<Off>(min(i * 32 + r0, rows - 1)) * static_cast<Off>(g.lda * 4);  // rows past the tile read its last row again
#pragma unroll
    for (int i = 0; i < BN / 32; ++i) b_off[i] = static_cast<Off>(min(i * 32 + r0, g.n_out - 1 - n0)) * static_cast<Off>(g.ldb * 4);
    f32x4 af[D][NA], bf[D][NB];
    auto load = [&](int kt, int d) {  // past the last K-element: the last four again, zeroed when staged
      const Off k = static_cast<Off>(min(kt * 32 + c * 4, g.K - 4)) * 4;
#pragma unroll
      for (int i = 0; i < NA; ++i) af[d][i] = *reinterpret_cast<gptr_f32x4>(a_base + (a_off[i] + k));
#pragma unroll
      for (int i = 0; i < NB; ++i) bf[d][i] = *reinterpret_cast<gptr_f32x4>(b_base[i / (BN / 32)] + (b_off[i % (BN / 32)] + k));
    };
    auto stage = [&](int kt, int d, int buf) {
      const bool in = kt * 32 + c * 4 < g.K;
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < NA; ++i) *reinterpret_cast<f32x4*>(lds[buf] + put + i * (32 * 128)) = in ? af[d][i] : zero;
#pragma unroll
      for (int i = 0; i < NB; ++i) *reinterpret_cast<f32x4*>(lds[buf] + BM * 128 + put + i * (32 * 128)) = in ? bf[d][i] : zero;
    };
    f32x4 acc[W][TM];
#pragma unroll
    for (int s = 0; s < W; ++s)
#pragma unroll
      for (int i = 0; i < TM; ++i) acc[s][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 sum[W][TM];  // SLICES > 1: the finished slices
    int slice = 1, slice_end = KT / SLICES;  // empty slices (KT < SLICES) are passed over
    if (SLICES > 1) {
#pragma unroll
      for (int s = 0; s < W; ++s)
#pragma unroll
        for (int i = 0; i < TM; ++i) sum[s][i] = acc[s][i];
      while (slice_end == 0) slice_end = KT * ++slice / SLICES;
    }
    auto end_step = [&](int kt) {
      if (SLICES > 1 && kt + 1 == slice_end) {
#pragma unroll
        for (int s = 0; s < W; ++s)
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            sum[s][i] += acc[s][i];
            acc[s][i] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
        while (slice < SLICES && slice_end == kt + 1) slice_end = KT * ++slice / SLICES;
      }
    };
    auto mac = [&](int buf) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        f32x4 x[TM], w[W];
#pragma unroll
        for (int s = 0; s < W; ++s) w[s] = *reinterpret_cast<const f32x4*>(lds[buf] + BM * 128 + get[h] + (wave * 16 + s * BN) * 128);
#pragma unroll
        for (int i = 0; i < TM; ++i) x[i] = *reinterpret_cast<const f32x4*>(lds[buf] + get[h] + i * (16 * 128));
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int s = 0; s < W; ++s) acc[s][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s][j], x[i][j], acc[s][i], 0, 0, 0);
      }
    };
    // every load is unconditional, so that the compiler's count of loads in flight stays exact; surplus ones
    // fetch the last step again and are not multiplied
#pragma unroll
    for (int d = 0; d < D; ++d) load(min(d, KT - 1), d);
    stage(0, 0, 0);
    publish();
    int kt = 0;
    for (; kt + D < KT; kt += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        stage(kt + d + 1, (d + 1) % D, (d + 1) & 1);
        mac(d & 1);
        end_step(kt + d);
        load(min(kt + D + d, KT - 1), d);
        publish();
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (d + 1 < D) stage(kt + d + 1, d + 1, (d + 1) & 1);
      if (kt + d < KT) {
        mac(d & 1);
        end_step(kt + d);
      }
      if (d + 1 < D) publish();
    }
    if (SLICES > 1) {
#pragma unroll
      for (int s = 0; s < W; ++s)
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[s][i] = sum[s][i];
    }
    // a lane holds four consecutive output columns of activation row lane % 16
    const int col = n0 + wave * 16 + quad * 4;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = row_begin + i * 16 + r16;
      if (row >= row_end || col >= g.n_out) continue;
      f32x4 v = acc[0][i];
      if (SWIGLU) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = v[r] / (1.0f + expf(-v[r])) * acc[W - 1][i][r];
      }
      *reinterpret_cast<f32x4*>(g.C + static_cast<int64_t>(row) * g.ldc + col) = v;  // n_out is a multiple of 4
    }
  };
  if (rows <= 16) run(std::integral_constant<int, 1>{});
  else if (rows <= 32) run(std::integral_constant<int, 2>{});
  else if (rows <= 48) run(std::integral_constant<int, 3>{});
  else run(std::integral_constant<int, 4>{});
}

// Either problem may be absent (blocks == 0).
template <bool SWIGLU, int SLICES = 1>
int launch_gemm_f32(revive_ctx* ctx, const GemmF32Args& args, hipStream_t stream) {
  const int grid = args.dense.blocks + args.grouped.blocks;
  if (grid <= 0) return REVIVE_OK;
  constexpr int64_t kNarrow = 1 << 24;  // 64 rows of as many floats are 4 GiB
  const bool narrow = args.dense.lda < kNarrow && args.grouped.lda < kNarrow;  // ldb = lda
  const auto kernel = narrow ? gemm_f32_kernel<SWIGLU, 2, SLICES, uint32_t> : gemm_f32_kernel<SWIGLU, 2, SLICES, uint64_t>;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, stream, args);
  return check_hip(ctx, hipGetLastError(), "gemm_f32 launch");
}

}  // namespace revive
