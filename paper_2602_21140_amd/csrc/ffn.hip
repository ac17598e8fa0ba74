// Grouped SwiGLU expert FFN of the failure-remapped MoE layer.
//
// Paper: Sec. 2.1 (each expert acts as an FFN).  Every physical slot p that received rows
// [slot_offsets[p], slot_offsets[p+1]) of the permuted activations applies its own weights:
// h = silu(X G_p) * (X U_p), y = h D_p.  Slots without rows (in particular every slot of a failed
// rank, Sec. 3.5) produce no tile, so their weight pointers are never dereferenced.
//
// The row counts exist only on the device, so the launch is shaped by an upper bound: the GEMM grids
// cover floor(N / tile) + P row-tiles, and workgroups beyond the last one exit at once.  Which rows a
// workgroup owns comes from a list that a small kernel makes of slot_offsets (bf16, many rows per
// slot), or the workgroup works it out from slot_offsets itself (row_tiles.hpp).
#include "ffn_rules.hpp"
#include "gemm_bf16.hpp"
#include "gemm_f32_split.hpp"
#include "gemm_stream.hpp"

namespace revive {

namespace {

__global__ __launch_bounds__(kMaxP) void ffn_tiles_kernel(const int32_t* __restrict__ slot_offsets, int P, int tile_m, int tall_m,
                                                          const void* const* __restrict__ w_gate_up,
                                                          const void* const* __restrict__ w_down,
                                                          MTile* __restrict__ tiles, int32_t* __restrict__ tile_count) {
  __shared__ int wave_sums[kMaxP / 64];
  __shared__ int tile_base[kMaxP + 1];  // first row-tile of every slot (exclusive prefix sum), [P] = total
  const int p = threadIdx.x;
  int first = 0, end = 0;
  if (p < P) {
    first = slot_offsets[p];
    end = slot_offsets[p + 1];
  }
  const int mine = tiles_of(end - first, tile_m, tall_m);
  const int lane = p & 63, wave = p >> 6;
  int incl = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(incl, o);
    if (lane >= o) incl += v;
  }
  if (lane == 63) wave_sums[wave] = incl;
  __syncthreads();
  if (wave == 0) {
    const int w = lane < kMaxP / 64 ? wave_sums[lane] : 0;
    int wi = w;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      const int v = __shfl_up(wi, o);
      if (lane >= o) wi += v;
    }
    if (lane < kMaxP / 64) wave_sums[lane] = wi - w;
    if (lane == kMaxP / 64 - 1) tile_count[0] = wi;
  }
  __syncthreads();
  const int base = wave_sums[wave] + incl - mine;
  if (p < P) tile_base[p] = base;
  if (p == P - 1) tile_base[P] = base + mine;
  __syncthreads();
  // One record per row-tile, the records dealt to the threads in order (a slot that holds most of the
  // rows, e.g. when every token picks the same experts, does not leave its thousands of records to one
  // thread).  The slot of record i is the last one whose first record is <= i: a binary search over the
  // prefix sums.  Only slots that received rows have their weight pointers read.
  const int total = tile_base[P];
  for (int i = p; i < total; i += kMaxP) {
    int lo = 0, hi = P - 1;  // invariant: tile_base[lo] <= i, and the answer is in [lo, hi]
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (tile_base[mid] <= i) lo = mid; else hi = mid - 1;
    }
    const int g = lo;  // among slots with equal base (empty ones) the last, which is the one that holds tiles
    MTile t;
    t.group_begin = slot_offsets[g];
    t.group_end = slot_offsets[g + 1];
    t.pad = ((tile_base[g + 1] - tile_base[g]) << 16) | (i - tile_base[g]);
    t.w[0] = w_gate_up[g];
    t.w[1] = w_down[g];
    tiles[i] = t;
  }
}

// Tile shapes of the bf16 GEMMs: 256 x 256 outputs per workgroup of 8 wavefronts (2 x 4), K in
// steps of 32 through a four-stage ring of asynchronous global->LDS copies.  Problems too small
// to give every CU a 256 x 256 tile use 256 x 128 tiles on 4 wavefronts (two workgroups per CU).
//
// A slot of 257 to 320 rows is one tall tile instead of two: a second tile with few rows costs half a full one
// and reads the weights again.  H = 7168, I = 2048, 8192 tokens over 261 live slots (half of them hold more than
// 256 rows): gate/up 4.83 -> 4.40 ms, down 2.43 -> 2.25; 3000 tokens of the smaller layer (286 rows): 0.34 ->
// 0.32 and 0.18 -> 0.165.  All tiles 320 rows high were slower where 256 does as well: 8192 tokens the same,
// but 170 rows +4 %, 341 rows +4 %, 607 rows +2.5 % (more rows copied than there are; two tiles of 300 rows
// against three of 200: +5 %).
// Below 128 rows per slot on average hardly a slot is that full, and the kernel without tall tiles starts sooner
// (a layer of 84 us: 45 rows per slot, 2 us).  And where a tile per slot leaves half of the CUs without work, two
// tiles side by side end sooner than a tall one: 10 slots, H = 3328, I = 768, 261 rows per slot (60 workgroups of
// gate/up) 74 us against 104.  1000 random layers of 190 to 340 rows per slot, tall against not: under 64 workgroups
// of the smaller launch 10 % slower on average, 64 to 127 3 %, 128 to 255 7 % faster, from 512 on 5 % faster and
// never slower by more than 3 %.
constexpr int kBN = 256, kWM = 2, kWN = 4;
constexpr int kTallM_bf16 = 320, kTallRowsPerSlot = 128, kTallWorkgroups = 128;

struct Bf16Ffn {  // one SwiGLU FFN: rows of A -> h -> y
  const void* A;
  const void* gu; const void* dn;  // weights (dense; the slots' are in the tile records)
  void* h; void* y;
  int I;
  const MTile* tiles; const int32_t* tile_count; int M;
  int max_m_tiles;
  int h_rows;  // rows of the intermediate h, which is kept K-panel-major: [I/32][h_rows][32]
};

GemmArgs gate_up_args(const revive_ctx* ctx, const Bf16Ffn& f, int bn_out) {
  GemmArgs a{};
  a.A = f.A; a.lda = ctx->cfg.H;
  a.B = f.gu;
  a.C = f.h; a.ldc = f.I; a.c_rows = f.h_rows;
  a.n_out = f.I; a.K = ctx->cfg.H;
  a.tiles = f.tiles; a.tile_count = f.tile_count; a.M = f.M;
  a.n_col_tiles = ceil_div(f.I, bn_out);
  a.b_sel = 0;
  a.b_rows_pad = ceil_div(f.I, kWeightTileRows) * kWeightTileRows;
  return a;
}

GemmArgs down_args(const revive_ctx* ctx, const Bf16Ffn& f, int bn_out) {
  GemmArgs d{};
  d.A = f.h; d.lda = f.I; d.a_rows = f.h_rows;
  d.B = f.dn;
  d.C = f.y; d.ldc = ctx->cfg.H;
  d.n_out = ctx->cfg.H; d.K = f.I;
  d.tiles = f.tiles; d.tile_count = f.tile_count; d.M = f.M;
  d.n_col_tiles = ceil_div(ctx->cfg.H, bn_out);
  d.b_sel = 1;
  d.b_rows_pad = ceil_div(ctx->cfg.H, kWeightTileRows) * kWeightTileRows;
  return d;
}

// Runs one FFN, or two in the same pair of launches (their tiles share the grid, which shortens
// the partially filled last round of workgroups).  K_GATE_UP / K_DOWN name the launches.
template <int BM, int K_GATE_UP, int K_DOWN>
int bf16_ffn(revive_ctx* ctx, const Bf16Ffn& f0, const Bf16Ffn* f1, hipStream_t stream) {
  const int H = ctx->cfg.H;
  const int64_t tiles_big_down = static_cast<int64_t>(f0.max_m_tiles) * ceil_div(H, kBN) +
                                 (f1 ? static_cast<int64_t>(f1->max_m_tiles) * ceil_div(H, kBN) : 0);
  const bool small = !f1 && f0.tiles == nullptr && tiles_big_down < 2 * 256;  // dense and under two tiles per CU
  {
    KernelTimer timer(ctx, K_GATE_UP, stream);
    int rc;
    if (small) {
      GemmArgs a0 = gate_up_args(ctx, f0, 64);
      rc = launch_gemm_bf16_dma<kTileM_bf16, 128, 2, 2, EPI_SWIGLU, K_GATE_UP>(ctx, a0, f0.max_m_tiles, nullptr, 0, stream);
    } else {
      GemmArgs a0 = gate_up_args(ctx, f0, kBN / 2), a1{};
      if (f1) a1 = gate_up_args(ctx, *f1, kBN / 2);
      rc = launch_gemm_bf16_dma<BM, kBN, kWM, kWN, EPI_SWIGLU, K_GATE_UP>(ctx, a0, f0.max_m_tiles, f1 ? &a1 : nullptr,
                                                                           f1 ? f1->max_m_tiles : 0, stream);
    }
    if (rc != REVIVE_OK) return rc;
  }
  KernelTimer timer(ctx, K_DOWN, stream);
  if (small) {
    GemmArgs d0 = down_args(ctx, f0, 128);
    return launch_gemm_bf16_dma<kTileM_bf16, 128, 2, 2, EPI_BF16, K_DOWN>(ctx, d0, f0.max_m_tiles, nullptr, 0, stream);
  }
  GemmArgs d0 = down_args(ctx, f0, kBN), d1{};
  if (f1) d1 = down_args(ctx, *f1, kBN);
  return launch_gemm_bf16_dma<BM, kBN, kWM, kWN, EPI_BF16, K_DOWN>(ctx, d0, f0.max_m_tiles, f1 ? &d1 : nullptr,
                                                                    f1 ? f1->max_m_tiles : 0, stream);
}

// Alone, the shared expert streams up to 128 tokens (H = 7168, I_shared = 2048, 1 token 76 -> 29 us, 128 tokens 98 ->
// 56; more have not been compared).
constexpr int kStreamDenseRows = 128;

// One FFN call: routed experts, shared expert, or both.
struct FfnArgs {
  const void* x_perm; const int32_t* slot_offsets; const void* const* w_gate_up; const void* const* w_down; void* h; void* y_perm;
  int N;  // routed rows; 0 = no routed experts
  const void* x; const void* w_sh_gate_up; const void* w_sh_down; void* h_shared; void* y_shared;
  int T;  // tokens of the shared expert; 0 = none
};

// The FFN of few rows per slot: two launches of the streaming kernel.
template <int TMX, int W, int D, int NW, int EPI, int KID>
int stream_gemm(revive_ctx* ctx, const FfnArgs& f, hipStream_t stream) {
  constexpr int tile_n = stream_tile_n<W, NW, EPI>, tile_m = 16 * TMX;
  constexpr bool gu = EPI == EPI_SWIGLU;
  const revive_config& c = ctx->cfg;
  auto problem = [&](const void* x, void* h, void* y, int rows, int I, int m_tiles) {
    StreamProblem p{};
    p.A = gu ? x : h; p.lda = gu ? c.H : I; p.a_rows = gu ? 0 : rows;
    p.C = gu ? h : y; p.ldc = gu ? I : c.H; p.c_rows = gu ? rows : 0;
    p.n_out = gu ? I : c.H; p.K = gu ? c.H : I;
    p.b_rows_pad = ceil_div(p.n_out, kWeightTileRows) * kWeightTileRows;
    p.n_col_tiles = ceil_div(p.n_out, tile_n);
    p.blocks = m_tiles * p.n_col_tiles;
    p.M = rows;
    return p;
  };
  StreamArgs a{};
  a.slot_offsets = f.slot_offsets;
  a.P = ctx->P;
  if (f.T > 0) {
    a.dense = problem(f.x, f.h_shared, f.y_shared, f.T, c.I_shared, ceil_div(f.T, tile_m));
    a.dense.B_one = gu ? f.w_sh_gate_up : f.w_sh_down;
  }
  if (f.N > 0) {
    const int used = f.N < ctx->P ? f.N : ctx->P;  // slots that can hold a row
    a.grouped = problem(f.x_perm, f.h, f.y_perm, f.N, c.I, f.N / tile_m + used);
    a.grouped.blocks = ceil_div(a.grouped.blocks, 8) * 8;
    a.grouped.B_tab = gu ? f.w_gate_up : f.w_down;
  }
  KernelTimer timer(ctx, KID, stream);
  return launch_gemm_bf16_stream<TMX, W, D, NW, EPI, KID>(ctx, a, stream);
}

template <int TMX, int W, int D, int NW, int K_GATE_UP, int K_DOWN>
int stream_ffn_as(revive_ctx* ctx, const FfnArgs& f, hipStream_t stream) {
  const int rc = stream_gemm<TMX, W, D, NW, EPI_SWIGLU, K_GATE_UP>(ctx, f, stream);
  return rc != REVIVE_OK ? rc : stream_gemm<TMX, W, D, NW, EPI_BF16, K_DOWN>(ctx, f, stream);
}

// Routed experts, with the shared expert or without.
template <int K_GATE_UP, int K_DOWN>
int stream_ffn(revive_ctx* ctx, const FfnArgs& f, const FfnSizes& sizes, hipStream_t stream) {
  static_assert(stream_tile_n<4, 4, EPI_SWIGLU> == 128 && stream_tile_n<4, 4, EPI_BF16> == 256 && stream_tile_n<2, 4, EPI_SWIGLU> == 64 &&
                stream_tile_n<2, 2, EPI_SWIGLU> == 32, "the columns that stream_form() counts");
  switch (stream_form(sizes)) {
    case k128x128: return stream_ffn_as<8, 4, 2, 4, K_GATE_UP, K_DOWN>(ctx, f, stream);
    case k64x64: return stream_ffn_as<4, 2, 4, 4, K_GATE_UP, K_DOWN>(ctx, f, stream);
    case k64x32: break;
  }
  return stream_ffn_as<4, 2, 4, 2, K_GATE_UP, K_DOWN>(ctx, f, stream);
}

// fp32: the routed and the shared experts in the same two launches.
template <bool SWIGLU, int KID>
int f32_gemm(revive_ctx* ctx, const FfnArgs& f, hipStream_t stream) {
  constexpr bool gu = SWIGLU;
  const revive_config& c = ctx->cfg;
  auto problem = [&](const void* x, void* h, void* y, int rows, int I, int m_tiles) {
    GemmF32Problem p{};
    p.A = static_cast<const float*>(gu ? x : h); p.lda = gu ? c.H : I; p.ldb = p.lda;
    p.C = static_cast<float*>(gu ? h : y); p.ldc = gu ? I : c.H;
    p.n_out = gu ? I : c.H; p.K = gu ? c.H : I;
    p.n_col_tiles = ceil_div(p.n_out, kTileN_f32);
    p.blocks = m_tiles * p.n_col_tiles;
    p.M = rows;
    return p;
  };
  GemmF32Args a{};
  a.slot_offsets = f.slot_offsets;
  a.P = ctx->P;
  if (f.T > 0) {
    a.dense = problem(f.x, f.h_shared, f.y_shared, f.T, c.I_shared, ceil_div(f.T, kTileM_f32));
    a.dense.B_one = static_cast<const float*>(gu ? f.w_sh_gate_up : f.w_sh_down);
  }
  if (f.N > 0) {
    a.grouped = problem(f.x_perm, f.h, f.y_perm, f.N, c.I, f.N / kTileM_f32 + (f.N < ctx->P ? f.N : ctx->P));
    a.grouped.blocks = ceil_div(a.grouped.blocks, 8) * 8;
    a.grouped.B_tab = gu ? f.w_gate_up : f.w_down;
  }
  KernelTimer timer(ctx, KID, stream);
  return launch_gemm_f32_split<SWIGLU>(ctx, a, stream);
}

template <int K_GATE_UP, int K_DOWN>
int f32_ffn(revive_ctx* ctx, const FfnArgs& f, hipStream_t stream) {
  const int rc = f32_gemm<true, K_GATE_UP>(ctx, f, stream);
  return rc != REVIVE_OK ? rc : f32_gemm<false, K_DOWN>(ctx, f, stream);
}

}  // namespace

int launch_expert_ffn(revive_ctx* ctx, const void* x_perm, const int32_t* slot_offsets, const void* const* w_gate_up,
                      const void* const* w_down, void* y_perm, const void* x, const void* w_sh_gate_up, const void* w_sh_down,
                      void* y_shared, int T, hipStream_t stream) {
  const revive_config& c = ctx->cfg;
  const int64_t N = static_cast<int64_t>(T) * c.k;
  constexpr int GU = REVIVE_K_FFN_GATE_UP, DN = REVIVE_K_FFN_DOWN;
  const FfnArgs f{x_perm, slot_offsets, w_gate_up, w_down, ctx->d_ws + ctx->ws.off_h, y_perm, static_cast<int>(N),
                  x, w_sh_gate_up, w_sh_down, ctx->d_ws + ctx->ws.off_h_shared, y_shared, y_shared ? T : 0};
  if (c.dtype != REVIVE_DTYPE_BF16) return f32_ffn<GU, DN>(ctx, f, stream);
  const FfnSizes sizes{ctx->P, c.H, c.I, c.I_shared, N, f.T};
  if (takes_stream(sizes)) return stream_ffn<GU, DN>(ctx, f, sizes, stream);
  MTile* tiles = reinterpret_cast<MTile*>(ctx->d_ws + ctx->ws.off_tiles);
  int32_t* tile_count = reinterpret_cast<int32_t*>(ctx->d_ws + ctx->ws.off_tile_count);
  // a row-tile per slot and 256 rows of the shared expert, times the column tiles of each launch
  const int64_t dense = ceil_div(f.T, kTileM_bf16);
  const int64_t gate_up = ctx->P * ceil_div(c.I, kBN / 2) + dense * ceil_div(c.I_shared, kBN / 2);
  const int64_t down = (ctx->P + dense) * ceil_div(c.H, kBN);
  const bool tall = N >= static_cast<int64_t>(kTallRowsPerSlot) * ctx->P && gate_up >= kTallWorkgroups && down >= kTallWorkgroups;
  {
    KernelTimer timer(ctx, REVIVE_K_FFN_TILES, stream);
    hipLaunchKernelGGL(ffn_tiles_kernel, dim3(1), dim3(kMaxP), 0, stream, slot_offsets, ctx->P, kTileM_bf16,
                       tall ? kTallM_bf16 : kTileM_bf16, w_gate_up, w_down, tiles, tile_count);
    REVIVE_HIP(ctx, hipGetLastError());
  }
  Bf16Ffn routed{x_perm, nullptr, nullptr, f.h, y_perm, c.I, tiles, tile_count, 0,
                 max_tiles(N, ctx->P, kTileM_bf16), f.N};
  // routed and shared experts in the same two launches
  Bf16Ffn shared{x, w_sh_gate_up, w_sh_down, f.h_shared, y_shared, c.I_shared,
                 nullptr, nullptr, T, ceil_div(T, kTileM_bf16), T};
  const Bf16Ffn* second = y_shared ? &shared : nullptr;
  return tall ? bf16_ffn<kTallM_bf16, GU, DN>(ctx, routed, second, stream) : bf16_ffn<kTileM_bf16, GU, DN>(ctx, routed, second, stream);
}

int launch_shared_ffn(revive_ctx* ctx, const void* x, const void* w_sh_gate_up, const void* w_sh_down, void* y_shared, int T,
                      hipStream_t stream) {
  const revive_config& c = ctx->cfg;
  void* h_shared = ctx->d_ws + ctx->ws.off_h_shared;
  constexpr int SGU = REVIVE_K_FFN_SHARED_GATE_UP, SDN = REVIVE_K_FFN_SHARED_DOWN;
  const FfnArgs f{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0, x, w_sh_gate_up, w_sh_down, h_shared, y_shared, T};
  if (c.dtype != REVIVE_DTYPE_BF16) return f32_ffn<SGU, SDN>(ctx, f, stream);
  // Always the small workgroups: the down projection has few output columns however wide the shared expert is
  // (H = 1024, 1 token, I_shared = 32 000: 107 us against 173, 65 536: 217 against 351).
  if (T <= kStreamDenseRows) return stream_ffn_as<4, 2, 4, 2, SGU, SDN>(ctx, f, stream);
  Bf16Ffn shared{x, w_sh_gate_up, w_sh_down, h_shared, y_shared, c.I_shared, nullptr, nullptr, T, ceil_div(T, kTileM_bf16), T};
  return bf16_ffn<kTileM_bf16, SGU, SDN>(ctx, shared, nullptr, stream);
}

}  // namespace revive
