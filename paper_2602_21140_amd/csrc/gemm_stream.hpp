// Grouped bf16 GEMM for few rows per expert: the weights are streamed once, straight into registers.
//
// Same contract and the same results (bit for bit) as gemm_bf16_dma_kernel (gemm_bf16.hpp).  With a few
// rows per slot the layer reads 6 H I bytes of weights per slot and multiplies next to nothing: what counts
// is how fast HBM is read.  Measured on this chip, reading 12 GiB once: 6.3-6.4 TB/s with plain loads
// whatever the number in flight, 7.2 TB/s with non-temporal ones.
//
// Weights: non-temporal 16-byte loads into registers, in MFMA operand order (lane l: row l % 16, K-chunk
//   l / 16 of a 16 x 32 block, which the tiled layout keeps in one contiguous KiB).  Four neighbouring
//   lanes then touch two 128-byte lines, so a CU takes in 75 GB/s of them (132 GB/s with lanes in address
//   order), well above its share of HBM (28 GB/s).
// Activations: rows of x are H apart, and read in operand order they come in at 38 GB/s per CU, which
//   made the loads of two to four 16-row sub-tiles dearer than the weights (gate/up at 60 rows per slot
//   6.1 ms).  They are fetched in address order (130 GB/s), once per workgroup, and pass through two LDS
//   buffers of 64 K-elements with one barrier each (2.8 ms).
// Both run D groups of 64 K-elements ahead in a ring of registers.
#pragma once

#include "gemm_bf16.hpp"
#include "row_tiles.hpp"

namespace revive {

struct StreamProblem {
  const void* A;             // [rows, K] bf16, or K-panel-major [K/32][a_rows][32] when a_rows > 0
  int64_t lda;
  int a_rows;
  const void* const* B_tab;  // device table slot -> tiled weight matrix (grouped), or
  const void* B_one;         // the one weight matrix (dense)
  void* C;                   // bf16 [rows, n_out], or K-panel-major [n_out/32][c_rows][32] when c_rows > 0
  int64_t ldc;
  int c_rows;
  int n_out;                 // output columns, a multiple of 64
  int K;                     // multiple of 64
  int b_rows_pad;            // rows of B (of each half for SwiGLU) padded to whole 128-row panels
  int n_col_tiles;
  int blocks;                // workgroups of the grid that belong to this problem
  int M;                     // rows (dense)
};

struct StreamArgs {
  StreamProblem dense;          // served by the first dense.blocks workgroups
  StreamProblem grouped;        // served by the others
  const int32_t* slot_offsets;  // [P + 1]: rows of every slot (grouped)
  int P;
};

// TMX: 16-row sub-tiles a workgroup covers at most; W: 16-row sets of weight rows per wavefront
// (SwiGLU: half of them gate, half up); D: groups of 64 K-elements in flight; NW: wavefronts.
template <int TMX, int W, int D, int NW, int EPI, int KID>
__global__ __launch_bounds__(64 * NW, 2) void gemm_bf16_stream_kernel(StreamArgs a) {
  constexpr int WOUT = EPI == EPI_SWIGLU ? W / 2 : W;  // 16-column output sets per wavefront
  constexpr int NT = 64 * NW;
  static_assert(D % 2 == 0, "the LDS buffer of a group is its position in the register ring modulo 2");
  __shared__ __attribute__((aligned(16))) unsigned char lds[2][TMX * 16 * 128];
  const bool dense = blockIdx.x < static_cast<unsigned>(a.dense.blocks);
  const StreamProblem g = dense ? a.dense : a.grouped;
  const int b = dense ? blockIdx.x : blockIdx.x - a.dense.blocks;
  int n_idx, row_begin, row_end;
  const unsigned char* B;
  bool once = true;  // nobody else reads these weights
  if (dense) {
    const int m_idx = b / g.n_col_tiles;
    n_idx = b - m_idx * g.n_col_tiles;
    row_begin = m_idx * (16 * TMX);
    row_end = min(g.M, row_begin + 16 * TMX);
    B = static_cast<const unsigned char*>(g.B_one);
    once = g.M <= 16 * TMX;
  } else {
    const GridTile t = grid_tile(a.slot_offsets, a.P, 16 * TMX, g.n_col_tiles, b, g.B_tab);
    if (t.group < 0) return;
    n_idx = t.n_idx;
    row_begin = t.row_begin;
    row_end = t.row_end;
    B = static_cast<const unsigned char*>(t.w);
    once = t.in_group == 1;
  }
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int own_col0 = (n_idx * NW + wave) * (WOUT * 16);  // first output column of this wavefront
  const int col0 = min(own_col0, g.n_out - WOUT * 16);  // past the last column: another wavefront's columns, not stored

  const int rows = row_end - row_begin;

  const int r16 = lane & 15, chunk = lane >> 4;
  // weights: a lane takes the 16 bytes (row lane % 16, K-chunk lane / 16) of a 16 x 32 block of the panel
  uint32_t w_off[W];
#pragma unroll
  for (int s = 0; s < W; ++s) {
    const int R = EPI == EPI_SWIGLU ? (s >= WOUT ? g.b_rows_pad : 0) + col0 + (s % WOUT) * 16 : col0 + s * 16;
    w_off[s] = static_cast<uint32_t>((static_cast<int64_t>(R / kWeightTileRows) * (g.K / kWeightTileK) * kWeightTileRows + R % kWeightTileRows + r16) * 64 + chunk * 16);
  }
  const unsigned char* a_base = static_cast<const unsigned char*>(g.A) + static_cast<int64_t>(row_begin) * (g.a_rows > 0 ? 32 : g.lda) * 2;
  const int64_t a_step = g.a_rows > 0 ? static_cast<int64_t>(g.a_rows) * 128 : 128;  // bytes between groups of 64 K-elements
  const int NG = g.K >> 6;

  auto run = [&](auto tm_tag, auto once_tag) {
    constexpr int TM = decltype(tm_tag)::value;
    constexpr bool ONCE = decltype(once_tag)::value;  // streamed past the caches' retention (non-temporal)
    constexpr int WORDS = TM * 16 * 8;                       // 16-byte words of one group of activations
    constexpr int NA = (WORDS + NT - 1) / NT;                // per thread
    uint32_t a_off[NA], a_dst[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int w = (i * NT + tid) % WORDS;                  // fewer words than threads: some are fetched twice
      const int row = w >> 3, c = w & 7;
      const int rrow = min(row, rows - 1);                   // rows past the tile read its last row again
      a_off[i] = g.a_rows > 0 ? static_cast<uint32_t>(static_cast<int64_t>(c >> 2) * g.a_rows * 64 + rrow * 64 + (c & 3) * 16)
                              : static_cast<uint32_t>(rrow * g.lda * 2 + c * 16);
      a_dst[i] = row * 128 + ((c ^ swz(row)) << 4);
    }
    f32x4 acc[W][TM];
#pragma unroll
    for (int s = 0; s < W; ++s)
#pragma unroll
      for (int i = 0; i < TM; ++i) acc[s][i] = f32x4{0.f, 0.f, 0.f, 0.f};

    u32x4 wf[D][2][W], af[D][NA];
    auto load = [&](int q, int d) {
      const unsigned char* wp = B + static_cast<int64_t>(q) * (2 * kWeightTileRows * kWeightTileK * 2);
      const unsigned char* ap = a_base + q * a_step;
#pragma unroll
      for (int i = 0; i < NA; ++i) af[d][i] = load_global_16B(ap + a_off[i]);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int s = 0; s < W; ++s) {
          const gptr_u32x4 p = reinterpret_cast<gptr_u32x4>(reinterpret_cast<uintptr_t>(wp + h * (kWeightTileRows * kWeightTileK * 2) + w_off[s]));
          wf[d][h][s] = ONCE ? __builtin_nontemporal_load(p) : *p;
        }
    };
    auto stage = [&](int d, int buf) {
#pragma unroll
      for (int i = 0; i < NA; ++i) *reinterpret_cast<u32x4*>(lds[buf] + a_dst[i]) = af[d][i];
    };
    auto mac = [&](int d, int buf) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const unsigned char* base = lds[buf] + r16 * 128 + (((h * 4 + chunk) ^ swz(r16)) << 4);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const bf16x8 x = *reinterpret_cast<const bf16x8*>(base + i * (16 * 128));
#pragma unroll
          for (int s = 0; s < W; ++s)
            acc[s][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf[d][h][s]), x, acc[s][i], 0, 0, 0);
        }
      }
    };
    auto publish = [&]() {  // this wavefront's LDS accesses are done; then everybody's are
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
    // The compiler counts the loads in flight to place its waits, and a load under a condition would make
    // it assume the fewest: every load is unconditional.  A number of groups that is no multiple of D is
    // rounded up, the surplus loads fetch the last group again and are not multiplied.
#pragma unroll
    for (int d = 0; d < D; ++d) load(min(d, NG - 1), d);
    stage(0, 0);
    publish();
    int q = 0;
    for (; q + D < NG; q += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        stage((d + 1) % D, (d + 1) & 1);
        mac(d, d & 1);
        load(min(q + D + d, NG - 1), d);
        publish();
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (d + 1 < D) stage(d + 1, (d + 1) & 1);
      if (q + d < NG) mac(d, d & 1);
      if (d + 1 < D) publish();
    }

    if (own_col0 >= g.n_out) return;
    // a lane holds four consecutive output columns (lane / 16) * 4 + {0..3} of activation row lane % 16
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = row_begin + i * 16 + r16;
      if (row >= row_end) continue;
#pragma unroll
      for (int s = 0; s < WOUT; ++s) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = EPI == EPI_SWIGLU ? silu_f32(acc[s][i][r]) * acc[s + W - WOUT][i][r] : acc[s][i][r];
        const u32x2 o = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        const int col = col0 + s * 16 + chunk * 4;
        uint16_t* dst = static_cast<uint16_t*>(g.C);
        if (g.c_rows > 0) dst += (static_cast<int64_t>(col / kWeightTileK) * g.c_rows + row) * kWeightTileK + col % kWeightTileK;
        else dst += static_cast<int64_t>(row) * g.ldc + col;
        *reinterpret_cast<u32x2*>(dst) = o;
      }
    }
  };
  using Y = std::true_type;
  if (!once) run(std::integral_constant<int, TMX>{}, std::false_type{});
  else if (TMX == 1 || rows <= 16) run(std::integral_constant<int, 1>{}, Y{});
  else if (TMX == 2 || rows <= 32) run(std::integral_constant<int, (TMX < 2 ? TMX : 2)>{}, Y{});
  else if (TMX == 4 || rows <= 64) run(std::integral_constant<int, (TMX < 4 ? TMX : 4)>{}, Y{});
  else run(std::integral_constant<int, TMX>{}, Y{});
}

// Output columns and rows of a workgroup.
template <int W, int NW, int EPI> constexpr int stream_tile_n = NW * 16 * (EPI == EPI_SWIGLU ? W / 2 : W);

// Either problem may be absent (blocks == 0).
template <int TMX, int W, int D, int NW, int EPI, int KID>
int launch_gemm_bf16_stream(revive_ctx* ctx, const StreamArgs& args, hipStream_t stream) {
  const int grid = args.dense.blocks + args.grouped.blocks;
  if (grid <= 0) return REVIVE_OK;
  hipLaunchKernelGGL((gemm_bf16_stream_kernel<TMX, W, D, NW, EPI, KID>), dim3(grid), dim3(64 * NW), 0, stream, args);
  return check_hip(ctx, hipGetLastError(), "gemm_bf16_stream launch");
}

}  // namespace revive
