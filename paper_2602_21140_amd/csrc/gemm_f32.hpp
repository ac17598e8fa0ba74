// fp32 GEMM of large routers on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 products and sums), and what the fp32
// GEMMs are told.
//
// C[row, n] = sum_k A[row, k] * B[n, k], 64 x 64 outputs per workgroup of four wavefronts, each with all the tile's rows
// and 16 output columns.  K is walked in steps of 32 through two LDS buffers, one barrier per step, with the loads of D
// steps in flight in registers.  A lane's 16 LDS bytes are four consecutive K-elements of its row and feed four MFMAs
// (both operands permute K alike).  The matrix cores are what bounds it (16 MFMAs of 32 cycles per 16 K-elements and
// wavefront against 160 cycles of LDS for the whole workgroup).  Vector instructions between the MFMAs cost as well: a
// thread keeps 32-bit offsets from wavefront-uniform bases and LDS addresses that are the same in every step.
#pragma once

#include <hip/hip_runtime.h>

#include "ctx.hpp"

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
constexpr int64_t kNarrowRows_f32 = 1 << 24;  // elements of a row from which on 64 rows do not lie within 4 GiB

// The K-steps are summed in SLICES parts that are added in their order (see router_tile_kernel).
// Off: bytes between the first of a tile's 64 rows and any element of them.
template <int D, int SLICES, typename Off>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmF32Problem g) {
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  typedef const __attribute__((address_space(1))) unsigned char* gptr;
  typedef const __attribute__((address_space(1))) f32x4* gptr_f32x4;
  constexpr int BM = kTileM_f32, BN = kTileN_f32, TM = BM / 16;
  constexpr int NA = BM / 32, NB = BN / 32;  // 16-byte words of activations and weights per thread and K-step
  static_assert(D % 2 == 0, "the LDS buffer of a step is its position in the register ring modulo 2");
  __shared__ __attribute__((aligned(16))) unsigned char lds[2][(BM + BN) * 128];
  const int m_idx = blockIdx.x / g.n_col_tiles, n_idx = blockIdx.x - m_idx * g.n_col_tiles;
  const int row_begin = m_idx * BM, row_end = min(g.M, row_begin + BM);
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
  const gptr a_base = base(g.A + static_cast<int64_t>(row_begin) * g.lda), b_base = base(g.B_one + n0 * g.ldb);
  // copy plan: 16-byte word w of a step is K-chunk w % 8 of row w / 8
  const int c = tid & 7, r0 = tid >> 3, put = swizzle(r0, c);
  Off a_off[NA], b_off[NB];  // bytes from the uniform bases
#pragma unroll
  for (int i = 0; i < NA; ++i) a_off[i] = static_cast<Off>(min(i * 32 + r0, rows - 1)) * static_cast<Off>(g.lda * 4);  // rows past the tile read its last row again
#pragma unroll
  for (int i = 0; i < NB; ++i) b_off[i] = static_cast<Off>(min(i * 32 + r0, g.n_out - 1 - n0)) * static_cast<Off>(g.ldb * 4);
  f32x4 af[D][NA], bf[D][NB];
  auto load = [&](int kt, int d) {  // past the last K-element: the last four again, zeroed when staged
    const Off k = static_cast<Off>(min(kt * 32 + c * 4, g.K - 4)) * 4;
#pragma unroll
    for (int i = 0; i < NA; ++i) af[d][i] = *reinterpret_cast<gptr_f32x4>(a_base + (a_off[i] + k));
#pragma unroll
    for (int i = 0; i < NB; ++i) bf[d][i] = *reinterpret_cast<gptr_f32x4>(b_base + (b_off[i] + k));
  };
  auto stage = [&](int kt, int d, int buf) {
    const bool in = kt * 32 + c * 4 < g.K;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NA; ++i) *reinterpret_cast<f32x4*>(lds[buf] + put + i * (32 * 128)) = in ? af[d][i] : zero;
#pragma unroll
    for (int i = 0; i < NB; ++i) *reinterpret_cast<f32x4*>(lds[buf] + BM * 128 + put + i * (32 * 128)) = in ? bf[d][i] : zero;
  };
  f32x4 acc[TM], sum[TM];  // sum: the finished slices
#pragma unroll
  for (int i = 0; i < TM; ++i) acc[i] = sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  int slice = 1, slice_end = KT / SLICES;  // empty slices (KT < SLICES) are passed over
  while (slice_end == 0) slice_end = KT * ++slice / SLICES;
  auto end_step = [&](int kt) {
    if (kt + 1 == slice_end) {
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        sum[i] += acc[i];
        acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      while (slice < SLICES && slice_end == kt + 1) slice_end = KT * ++slice / SLICES;
    }
  };
  auto mac = [&](int buf) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      f32x4 x[TM];
      const f32x4 w = *reinterpret_cast<const f32x4*>(lds[buf] + BM * 128 + get[h] + wave * (16 * 128));
#pragma unroll
      for (int i = 0; i < TM; ++i) x[i] = *reinterpret_cast<const f32x4*>(lds[buf] + get[h] + i * (16 * 128));
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[j], x[i][j], acc[i], 0, 0, 0);
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
  // a lane holds four consecutive output columns of activation row lane % 16
  const int col = n0 + wave * 16 + quad * 4;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int row = row_begin + i * 16 + r16;
    if (row < row_end && col < g.n_out) *reinterpret_cast<f32x4*>(g.C + static_cast<int64_t>(row) * g.ldc + col) = sum[i];  // n_out is a multiple of 4
  }
}

template <int SLICES>
int launch_gemm_f32(revive_ctx* ctx, const GemmF32Problem& g, hipStream_t stream) {
  const auto kernel = g.lda < kNarrowRows_f32 ? gemm_f32_kernel<2, SLICES, uint32_t> : gemm_f32_kernel<2, SLICES, uint64_t>;  // ldb = lda
  hipLaunchKernelGGL(kernel, dim3(g.blocks), dim3(256), 0, stream, g);
  return check_hip(ctx, hipGetLastError(), "gemm_f32 launch");
}

}  // namespace revive
