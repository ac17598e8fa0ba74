// Grouped bf16 GEMM on the gfx950 matrix cores, fp32 accumulate.
//
//   C[rows of tile, n] = sum_k A[row, k] * B_group[n, k]        ("NT": both operands K-contiguous)
//
// A is one tall activation matrix whose rows are split into row-tiles that each belong to one
// group (physical expert slot); B is that group's output-major weight matrix.  Two epilogues:
//   EPI_BF16    round to bf16 and store            (down projection)
//   EPI_SWIGLU  B holds gate rows [0, n_out) and up rows [n_out, 2 n_out); store
//               bf16(silu(gate) * up)              (gate/up projection of a SwiGLU expert)
//
// Work decomposition: one workgroup computes a BM x BN tile with WAVES_M x WAVES_N wavefronts of
// 64 lanes; each wavefront owns (BM/WAVES_M) x (BN/WAVES_N) outputs as 16x16 MFMA tiles.  The
// weights go in as the MFMA's first operand so that each lane ends up with four consecutive output
// columns of one activation row.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "ctx.hpp"

namespace revive {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
// Pointers that are known to address HBM: lets the compiler emit global_load/global_store
// instead of flat accesses (which also tick the LDS counter and so serialise with LDS waits).
typedef const __attribute__((address_space(1))) u32x4* gptr_u32x4;

__device__ __forceinline__ u32x4 load_global_16B(const unsigned char* p) {
  return *reinterpret_cast<gptr_u32x4>(reinterpret_cast<uintptr_t>(p));
}

// Asynchronous copy of 16 bytes per lane to LDS: lane l's from src + off to dst + 16 l (dst and src wavefront-uniform).
// Inline assembly on purpose: the compiler's wait-count bookkeeping treats a global_load_lds it knows about as "may touch
// both memory and LDS" and from then on turns every LDS wait into a full drain, which would undo a software pipeline.
// Issued this way the copies are invisible to that bookkeeping and have to be waited for explicitly before the barrier
// that publishes them.  So is the wait state that the hardware needs between a write of M0 and the copy that uses it.
__device__ __forceinline__ void copy_to_lds_16B(uint32_t dst, uint64_t src, uint32_t off) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(src), "s"(dst) : "memory", "m0");
}

enum { EPI_BF16 = 1, EPI_SWIGLU = 2 };

// Tiled weight layout: a [rows, K] output-major matrix is stored as [rows/128][K/32][128][32]
// (rows zero-padded to a multiple of 128), so the 128 x 32 block a workgroup fetches per K-step is
// 8 KiB contiguous and a whole 128-row panel is one contiguous stream over K.
constexpr int kWeightTileRows = 128;
constexpr int kWeightTileK = 32;

struct GemmArgs {
  const void* A;             // [rows, K] bf16
  int64_t lda;               // elements between rows of A
  const void* B;             // dense: [n_rows_B, K] bf16 in the tiled weight layout (see kWeightTileRows); grouped: the tile records have it
  void* C;                   // [rows, n_out] bf16
  int64_t ldc;
  int n_out;                 // output columns (SwiGLU: I, with B holding 2*I rows)
  int K;                     // multiple of 64
  const MTile* tiles;        // device row-tile list, or null for a dense [0, M) matrix
  const int32_t* tile_count; // device count of valid entries in `tiles`
  int M;                     // dense case: number of rows
  int n_col_tiles;
  int b_sel;                 // grouped: which of the tile record's two matrices
  int b_rows_pad;            // rows of B (of each half for SwiGLU) padded to whole tiles
  int a_rows;                // > 0: A is stored K-panel-major, [K/32][a_rows][32]: the 32 K-elements of a row that one
                             // K-step needs are 64 contiguous bytes and consecutive rows follow each other, so the
                             // copies of a row-tile read one contiguous run per K-step (used for the intermediate h)
  int c_rows;                // > 0: C is written in the same layout, [n_out/32][c_rows][32]
};

// Up to two independent problems served by one launch (e.g. the routed experts' grouped GEMM and
// the shared expert's dense GEMM): their tiles are numbered one after the other.
struct GemmArgs2 {
  GemmArgs p0, p1;
  int two;  // 0: only p0 is valid
};

// Two fp32 -> one word of two bf16 (round-to-nearest-even), one v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// LDS swizzle.  The gfx950 LDS has 64 four-byte banks (256 B per clock) and serves a 16-byte
// per-lane access in groups of 16 lanes.  Tile rows are 128 bytes, so rows r and r+2 start on the
// same bank; XOR-ing the 16-byte chunk index with (row >> 1) & 7 makes the 16 rows a lane group
// touches (same logical chunk) fall on 16 distinct 16-byte bank groups.
__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

// silu(z) = z / (1 + exp(-z)) with the hardware reciprocal (1 ulp) instead of an IEEE division: the
// result is rounded to bf16 right after, and the division sequence is ten instructions per output.
// exp overflows to +inf for z < -88, where the product is the correct -0.
__device__ __forceinline__ float silu_f32(float z) { return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

// Operands reach LDS by asynchronous copies (global_load_lds_dwordx4) through a four-stage ring.
//
// KID (the library's kernel id) only gives each use of the kernel its own symbol name in profiles.
//
// K is walked in steps of 32; a stage holds
// a BM x 32 tile of A and a BN x 32 tile of B (64-byte rows).  The copy of K-step t+3 is issued
// while step t is being multiplied, so three steps (about 1.3 us of MFMA work at full rate) are
// in flight to cover HBM latency, and no register is spent on staging.  Per K-step there is one
// workgroup barrier, placed before the second half of the row sub-tiles' MFMAs so that the first
// fragment reads of the next stage overlap them.
//
// What bounds it on large problems is power: the clock falls to 1.5 to 1.7 GHz under it.  Hence the
// MFMA that costs least for a product, 16x16x32 (it reads and writes half the accumulators of
// 32x32x16 per multiplication; the sums are the same bits), and an order in which each MFMA shares
// an operand with the one before.  And sub-tiles of 16 rows pad a ragged row-tile less.  TFLOP/s of
// 32x32x16, of 16x16x32, of that to and fro, and with sub-tiles of 16 rows and slots cut evenly:
// dense 8192 x 7168 x 4096 with SwiGLU 1289, 1400, 1429 (1318 and 1476 in another run); gate/up of
// 414 slots of 640 to 740 rows, K = 7168, 1111, 1124, 1162, 1196, down 1068, 1095, 1130, 1154; of 261
// slots of 230 to 290 rows 986 and 1025, 964 and 1000; of 63 slots of 350 to 430 rows, K = 2048 and
// 1408, 865 and 887, 800 and 838.  By counters, 414 slots of 293 to 830 rows, K = 7168, gate/up with 32x32x16 and as it is:
// 1.37 and 1.55 GHz, matrix cores busy in 79 and 73 % of the cycles, 15.7 and 14.7 ms.
// 4 x 2 wavefronts (64 x 128 each) are 1 % faster on the dense shape and 2 to 4 % slower on slots; 2 x 2 wavefronts 10 % slower; weights kept over the row sub-tiles
// beat activations kept over the column tiles by 1 %.
//
// LDS layout of a stage: row r at r*64 bytes, its four 16-byte chunks stored at chunk ^ ((r>>2)&3):
// a copy instruction writes lane l's 16 bytes to (its 1 KiB window) + 16*l, i.e. 16 rows per
// wavefront instruction, and each lane fetches the chunk that belongs in its slot; the fragment
// reads (16 lanes = 16 consecutive rows, same logical chunk) then cover all 64 banks once.
// s_waitcnt immediate (gfx9 encoding) for "vmcnt(vm) lgkmcnt(0)", export counter ignored.
__host__ __device__ constexpr int waitcnt_vm_lgkm0(int vm) { return (vm & 0xF) | ((vm >> 4) << 14) | (0x7 << 4) | (0 << 8); }

// Row sub-tiles of 16 rows whose outputs all wavefronts can hold in LDS at a time.
constexpr int epilogue_pass(int tm, int waves, int row_bytes) {
  int pass = tm;
  while (waves * pass * 16 * row_bytes > 160 * 1024) pass = (pass + 1) / 2;
  return pass;
}

__device__ __forceinline__ int swz32(int row) { return (row >> 2) & 3; }

constexpr int kStages = 4;

template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int KID>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_bf16_dma_kernel(GemmArgs2 a2) {
  constexpr int NT = 64 * WAVES_M * WAVES_N, NW = WAVES_M * WAVES_N;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  constexpr int TM = WM / 16, TN = WN / 16;
  constexpr int BN_OUT = EPI == EPI_SWIGLU ? BN / 2 : BN;
  constexpr int D = kStages - 1;  // copies run D K-steps ahead of the MFMAs
  constexpr int STAGE = (BM + BN) * 64;       // bytes
  // Row-tiles are BM0 rows high; BM may be higher by a quarter, for a slot that overflows one row-tile by less
  // than that (see tiles_of).  Copy instructions per wavefront and stage: CP_B + CP_A, and in such a tall tile
  // the first half of the wavefronts (which then issues CPT) takes one block of A more each.
  constexpr int BM0 = BM > kTileM_bf16 ? kTileM_bf16 : BM;
  constexpr int CP_B = BN / 16 / NW, CP_A = BM0 / 16 / NW, CP = CP_A + CP_B, CPT = CP + (BM > BM0);
  static_assert(BM0 % (16 * NW) == 0 && BN % (16 * NW) == 0 && (BM == BM0 || BM - BM0 == NW / 2 * 16), "copy split");
  constexpr int TM0 = BM0 / WAVES_M / 16;
  static_assert(TM0 == 8 && (BM == BM0 || TM == TM0 + 2), "row sub-tile dispatch below");
  static_assert(EPI != EPI_SWIGLU || TN % 2 == 0, "SwiGLU needs gate and up tiles in one wave");
  typedef __attribute__((address_space(3))) void* lptr;

  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  auto stage_of = [](int kt) { return kt & (kStages - 1); };

  // Tile -> workgroup map.  Workgroup i runs on XCD i % 8; each XCD takes a contiguous eighth of
  // every problem's tiles (neighbouring tiles share activations / weights in that XCD's L2), and
  // works through the problem with the longer K first so that the cheap tiles fill the last round.
  // A dense problem (no tile list) is split by whole row-tiles instead: XCD x owns n_m / 8 of them
  // (the first n_m % 8 XCDs one more), so that the order below can walk its own block of the
  // output; its workgroup budget per XCD is that of the XCDs with one more.
  const int nm0 = a2.p0.tiles ? *a2.p0.tile_count : (a2.p0.M + BM0 - 1) / BM0;
  const int nm1 = a2.two ? (a2.p1.tiles ? *a2.p1.tile_count : (a2.p1.M + BM0 - 1) / BM0) : 0;
  const int t0 = nm0 * a2.p0.n_col_tiles, t1 = nm1 * a2.p1.n_col_tiles;
  const int px0 = a2.p0.tiles ? (t0 + 7) >> 3 : ((nm0 + 7) >> 3) * a2.p0.n_col_tiles;
  const int px1 = !a2.two ? 0 : a2.p1.tiles ? (t1 + 7) >> 3 : ((nm1 + 7) >> 3) * a2.p1.n_col_tiles;
  const int xcd = blockIdx.x & 7;
  int local = blockIdx.x >> 3;
  const bool p1_first = a2.two && a2.p1.K > a2.p0.K;
  bool second;  // uniform: this workgroup serves the second problem
  if (p1_first) {
    second = local < px1;
    if (!second) local -= px1;
  } else {
    second = local >= px0;
    if (second) local -= px0;
  }
  if (local >= (second ? px1 : px0)) return;
  const GemmArgs g = second ? a2.p1 : a2.p0;
  int m_idx, n_idx, logical = 0;
  if (g.tiles) {
    logical = xcd * (second ? px1 : px0) + local;
    if (logical >= (second ? t1 : t0)) return;
    m_idx = logical / g.n_col_tiles;
    n_idx = logical - m_idx * g.n_col_tiles;
  } else {
    // The XCD's G row-tiles times all column tiles, column tiles taken in pairs and inside a pair
    // the row-tile slower than the column: a row-tile's activations are needed again by the very
    // next workgroup and a column tile's weights by the one after that, down the whole block,
    // instead of the weights coming back only after a full row of column tiles.
    const int nm = second ? nm1 : nm0;
    const int G = (nm >> 3) + (xcd < (nm & 7));
    if (local >= G * g.n_col_tiles) return;
    const int blk = local / (2 * G), within = local - blk * 2 * G;
    int j;
    if (blk * 2 + 1 < g.n_col_tiles) { j = within >> 1; n_idx = blk * 2 + (within & 1); }
    else { j = within; n_idx = blk * 2; }
    m_idx = xcd * (nm >> 3) + min(xcd, nm & 7) + j;
  }

  int row_begin, row_end;
  const unsigned char* Bbase;
  if (g.tiles) {
    // One read of any record of the group tells everything.  Inside one group's block of tiles
    // the column index runs slowest: the row-tiles of a slot that use the same weight columns are
    // neighbours in launch order and meet in L2 (up to two row-tiles; see below for more).
    const MTile t = g.tiles[m_idx];
    const int in_group = t.pad >> 16;
    int j = t.pad & 0xFFFF;
    if (in_group > 1) {
      const int r = logical - (m_idx - j) * g.n_col_tiles;
      if (in_group >= 3) {
        // three or more row-tiles: column tiles are taken in pairs and inside a pair the row-tile
        // runs slower than the column, so that a row-tile's activations are needed again by the
        // very next workgroup instead of in_group workgroups later (by then L2 has dropped them)
        const int blk = r / (2 * in_group), within = r - blk * 2 * in_group;
        if (blk * 2 + 1 < g.n_col_tiles) { j = within >> 1; n_idx = blk * 2 + (within & 1); }
        else { j = within; n_idx = blk * 2; }
      } else {
        n_idx = r / in_group;
        j = r - n_idx * in_group;
      }
    }
    tile_span(t.group_begin, t.group_end, in_group, j, row_begin, row_end);
    Bbase = static_cast<const unsigned char*>(g.b_sel ? t.w[1] : t.w[0]);  // indexed, the record would go through private scratch
  } else {
    row_begin = m_idx * BM0;
    row_end = min(g.M, row_begin + BM0);
    Bbase = static_cast<const unsigned char*>(g.B);
  }
  const unsigned char* Abase = static_cast<const unsigned char*>(g.A);
  const int n0 = n_idx * BN_OUT;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wavefront-uniform: keeps per-wavefront offsets in SGPRs
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;

  // ---- copy plan: instruction i of this wavefront fills rows [(wave*CP_x + i)*16, +16) of the A
  // (then B) part of a stage; lane l owns row l/4 of those, physical chunk l%4.
  // The source address of a copy is a wavefront-uniform 64-bit base (the tile's first row of A, the
  // weight matrix) kept in scalar registers plus a 32-bit per-lane byte offset that never changes:
  // walking K only advances the two scalar bases, no vector arithmetic.
  uint32_t cp_off[CPT];
  int cp_dst[CPT];  // wavefront-uniform LDS offset of the 1 KiB window inside a stage
#pragma unroll
  for (int i = 0; i < CPT; ++i) {  // the B blocks first, a tall tile's additional block last
    const bool isA = i >= CP_B;
    const int blk = !isA ? wave * CP_B + i : i < CP ? wave * CP_A + (i - CP_B) : BM0 / 16 + wave;
    const int row = blk * 16 + (lane >> 2);
    const int chunk = (lane & 3) ^ swz32(row);
    if (isA) {
      const int rrow = min(row, row_end - row_begin - 1);  // rows past the tile re-read its last row
      cp_off[i] = g.a_rows > 0 ? static_cast<uint32_t>((rrow * 32 + chunk * 8) * 2)
                               : static_cast<uint32_t>((static_cast<int64_t>(rrow) * g.lda + chunk * 8) * 2);
      cp_dst[i] = blk * 1024;
    } else {
      // padded row index of this LDS row in the tiled matrix (gate half first, then up half)
      int R;
      if (EPI == EPI_SWIGLU) {
        const int half = row >= BN / 2;
        R = min(n0 + row - half * (BN / 2), g.b_rows_pad - 1) + half * g.b_rows_pad;
      } else {
        R = min(n0 + row, g.b_rows_pad - 1);
      }
      const int64_t panel = static_cast<int64_t>(R / kWeightTileRows) * (g.K / kWeightTileK) * kWeightTileRows;
      cp_off[i] = static_cast<uint32_t>(((panel + (R % kWeightTileRows)) * kWeightTileK + chunk * 8) * 2);
      cp_dst[i] = BM * 64 + blk * 1024;
    }
  }
  const uint32_t smem_lds = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lptr)smem));
  auto uniform64 = [](uint64_t v) {
    // the builtin returns a signed int: widen both halves as unsigned
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v >> 32)));
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
    return (static_cast<uint64_t>(hi) << 32) | lo;
  };
  uint64_t base_a = uniform64(reinterpret_cast<uint64_t>(Abase) + static_cast<uint64_t>(row_begin) * (g.a_rows > 0 ? 32 : g.lda) * 2);
  const uint64_t kstep_a = g.a_rows > 0 ? static_cast<uint64_t>(g.a_rows) * 64 : 64;
  uint64_t base_b = uniform64(reinterpret_cast<uint64_t>(Bbase));
  // Five wait states before a copy may read a scalar register that a vector instruction wrote.
  asm volatile("s_nop 4" : "+s"(base_a), "+s"(base_b));
  constexpr uint32_t kstep_b = kWeightTileRows * kWeightTileK * 2;  // bytes between K-steps of B
  auto issue_copy = [&](int kt, auto cp_tag) {
    const uint32_t stage = smem_lds + stage_of(kt) * STAGE;
    const uint64_t src_a = base_a + static_cast<uint64_t>(kt) * kstep_a;
    const uint64_t src_b = base_b + static_cast<uint64_t>(kt) * kstep_b;
#pragma unroll
    for (int i = 0; i < decltype(cp_tag)::value; ++i) {
      const uint32_t dst = __builtin_amdgcn_readfirstlane(stage + cp_dst[i]);
      copy_to_lds_16B(dst, i < CP_B ? src_b : src_a, cp_off[i]);
    }
  };

  // The same with the ring position PH of the destination stage known at compile time.
  auto issue_copy_at = [&](int kt, auto ph_tag, auto cp_tag) {
    constexpr int PH = decltype(ph_tag)::value;
    const uint64_t src_a = base_a + static_cast<uint64_t>(kt) * kstep_a;
    const uint64_t src_b = base_b + static_cast<uint64_t>(kt) * kstep_b;
#pragma unroll
    for (int i = 0; i < decltype(cp_tag)::value; ++i) {
      const uint32_t dst = __builtin_amdgcn_readfirstlane(smem_lds + cp_dst[i] + PH * STAGE);
      copy_to_lds_16B(dst, i < CP_B ? src_b : src_a, cp_off[i]);
    }
  };
  using Cp = std::integral_constant<int, CP>;
  using CpTall = std::integral_constant<int, CPT>;

  // ---- per-lane fragment addresses.  16-row sub-tiles are dealt round-robin to the wavefront
  // rows (sub-tile tm*WAVES_M + wm), so a ragged row-tile keeps every wavefront equally busy.
  // Every fragment row of a lane is (a multiple of 16) + lane % 16, so the swizzle term depends on
  // the lane only: the lane keeps one loop-invariant byte offset per operand, and the individual
  // fragments are reached with immediate offsets from it.
  const int lrow = lane & 15;
  const int sw = ((lane >> 4) ^ swz32(lrow)) << 4;
  const int a_off = (wm * 16 + lrow) * 64 + sw;
  const int b_off = (BM + (EPI == EPI_SWIGLU ? wn * (WN / 2) : wn * WN) + lrow) * 64 + sw;
  // The same bases two stages further on: with the ring position known at compile time every
  // fragment of every stage is an immediate offset below 64 KiB away from one of the two.
  const int a_off2 = a_off + 2 * STAGE, b_off2 = b_off + 2 * STAGE;
  constexpr int A_STEP = WAVES_M * 16 * 64;  // bytes between a wavefront's successive row sub-tiles
  auto b_imm = [](int tn) {                   // byte offset of column tile tn from the lane's base
    if (EPI == EPI_SWIGLU) return ((tn >= TN / 2 ? BN / 2 : 0) + (tn % (TN / 2)) * 16) * 64;
    return tn * 16 * 64;
  };
  auto frag = [](const unsigned char* p) { return *reinterpret_cast<const bf16x8*>(p); };
  f32x4 acc[TM][TN];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) acc[tm][tn] = f32x4{0.f, 0.f, 0.f, 0.f};

  // A ragged row-tile leaves some 16-row sub-tiles of a wavefront without any valid row; the
  // main loop is instantiated for each count of valid sub-tiles so that those MFMAs (and their
  // fragment reads) are not issued at all.  The wavefront still takes part in copies and barriers.
  const int KT = g.K >> 5;
  const int n_sub = (row_end - row_begin + 15) >> 4;  // sub-tiles holding at least one valid row
  const int tm_valid = min(TM, max(0, (n_sub - wm + WAVES_M - 1) / WAVES_M));

  // early_tag: copies per stage of the first half of the wavefronts.
  auto run = [&](auto tmv_tag, auto early_tag) {
    constexpr int TMV = decltype(tmv_tag)::value, CPE = decltype(early_tag)::value;
    // A K-step has two phases: the first half of the row sub-tiles (H0 of them) times all column tiles, then the
    // rest (H1).  The fragments that a phase does not have yet are read while the phase before it multiplies: phase
    // 0 reads the second half's activations; phase 1, which comes after the barrier, reads the next stage's first
    // half and its weights, each weight fragment in the place of the one whose last MFMA has just been issued.
    constexpr int H0 = (TMV + 1) / 2, H1 = TMV / 2;
    bf16x8 af0[TM], af1[TM], bf[TN];
    // MFMA idx of a phase of HM row sub-tiles: to and fro over the sub-tiles, so that each MFMA shares one operand
    // with the one before it.
    auto mfma = [&](int idx, int HM, const bf16x8* a, int base) {
      const int tn = idx / HM, tm = (tn & 1) ? HM - 1 - idx % HM : idx % HM;
      acc[base + tm][tn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[tn], a[tm], acc[base + tm][tn], 0, 0, 0);
    };
    // The reads are dealt between the MFMAs and their order is pinned with scheduling groups (0x008: MFMA, 0x100:
    // LDS read): they then issue in the shadow of the matrix pipe instead of in a block ahead of it.
    auto phase0 = [&](const unsigned char* pa) {
      if (TMV == 0) return;
#pragma unroll
      for (int idx = 0; idx < H0 * TN; ++idx) {
        mfma(idx, H0, af0, 0);
        if (idx < H1) af1[idx] = frag(pa + (H0 + idx) * A_STEP);
      }
#pragma unroll
      for (int i = 0; i < H1; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, H0 * TN - H1, 0);
    };
    auto phase1 = [&](const unsigned char* pa, const unsigned char* pb, auto last_tag) {
      constexpr bool LAST = decltype(last_tag)::value;  // no next stage
      if (TMV == 0) return;
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) {
#pragma unroll
        for (int tm = 0; tm < H1; ++tm) {
          mfma(tn * H1 + tm, H1, af1, H0);
          if (!LAST && tn == 0) af0[tm] = frag(pa + tm * A_STEP);
        }
        if (!LAST && tn == 0 && H0 > H1) af0[H0 - 1] = frag(pa + (H0 - 1) * A_STEP);
        if (!LAST) bf[tn] = frag(pb + b_imm(tn));
      }
      if (!LAST) {
#pragma unroll
        for (int i = 0; i < H1; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        if (H0 > H1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
#pragma unroll
        for (int i = 1; i < TN; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          if (H1 > 0) __builtin_amdgcn_sched_group_barrier(0x008, H1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
    };
    auto load_first = [&]() {
      if (TMV == 0) return;
#pragma unroll
      for (int tm = 0; tm < H0; ++tm) af0[tm] = frag(smem + a_off + tm * A_STEP);
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) bf[tn] = frag(smem + b_off + b_imm(tn));
    };
    // This wavefront's copies of the next step have landed once only vm newer ones are pending; all its fragment
    // reads of the current stage have returned (lgkmcnt 0).
    auto wait_barrier = [&](auto vm_tag) {
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(decltype(vm_tag)::value));
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
    // One K-step.  COPY: issue the copy of step kt + D, into the stage that held step kt - 1 (every wavefront
    // finished reading it before the last barrier).  vm: copies that may stay pending at the barrier (those of the
    // steps after kt + 1).  LAST: no next stage to publish.
    auto step = [&](int kt, auto copy_tag, auto vm_tag, auto last_tag) {
      if (decltype(copy_tag)::value) issue_copy(kt + D, early_tag);
      __builtin_amdgcn_sched_barrier(0);
      phase0(smem + stage_of(kt) * STAGE + a_off);
      __builtin_amdgcn_sched_barrier(0);
      if (!decltype(last_tag)::value) wait_barrier(vm_tag);
      const unsigned char* next = smem + stage_of(kt + 1) * STAGE;
      phase1(next + a_off, next + b_off, last_tag);
      __builtin_amdgcn_sched_barrier(0);
    };
    // Skewed schedule.  Both wavefronts of a SIMD (w and w + NW/2) would otherwise leave the
    // barrier in lockstep and do their non-MFMA work (copy issue, address arithmetic) at the same
    // time, leaving the matrix pipe idle.  The late group issues its copy right after the barrier
    // (one step further ahead, into this step's own stage: all its reads ended before the barrier)
    // instead of after the second phase, so one group's overhead always runs under the other
    // group's MFMAs.
    auto step_late = [&](int kt, auto copy_tag, auto vm_tag, auto last_tag) {
      phase0(smem + stage_of(kt) * STAGE + a_off);
      __builtin_amdgcn_sched_barrier(0);
      if (!decltype(last_tag)::value) {
        wait_barrier(vm_tag);
        if (decltype(copy_tag)::value) issue_copy(kt + D + 1, Cp{});
        __builtin_amdgcn_sched_barrier(0);
      }
      const unsigned char* next = smem + stage_of(kt + 1) * STAGE;
      phase1(next + a_off, next + b_off, last_tag);
      __builtin_amdgcn_sched_barrier(0);
    };
    // Steady-state forms of the two with the ring position PH = kt % 4 known at compile time: stage
    // addresses fold into immediates and the K loop, unrolled by four, carries no vector ALU
    // instruction at all.
    auto a_at = [&](auto ph_tag) { constexpr int PH = decltype(ph_tag)::value; return smem + (PH >= 2 ? a_off2 : a_off) + (PH & 1) * STAGE; };
    auto b_at = [&](auto ph_tag) { constexpr int PH = decltype(ph_tag)::value; return smem + (PH >= 2 ? b_off2 : b_off) + (PH & 1) * STAGE; };
    auto step_at = [&](int kt, auto ph_tag) {
      constexpr int PH = decltype(ph_tag)::value;
      using Next = std::integral_constant<int, (PH + 1) & 3>;
      issue_copy_at(kt + D, std::integral_constant<int, (PH + D) & 3>{}, early_tag);
      __builtin_amdgcn_sched_barrier(0);
      phase0(a_at(ph_tag));
      __builtin_amdgcn_sched_barrier(0);
      wait_barrier(std::integral_constant<int, (D - 1) * CPE>{});
      phase1(a_at(Next{}), b_at(Next{}), std::false_type{});
      __builtin_amdgcn_sched_barrier(0);
    };
    auto step_late_at = [&](int kt, auto ph_tag) {
      constexpr int PH = decltype(ph_tag)::value;
      using Next = std::integral_constant<int, (PH + 1) & 3>;
      phase0(a_at(ph_tag));
      __builtin_amdgcn_sched_barrier(0);
      wait_barrier(std::integral_constant<int, (D - 1) * CP>{});
      issue_copy_at(kt + D + 1, ph_tag, Cp{});  // (PH + 4) % 4
      __builtin_amdgcn_sched_barrier(0);
      phase1(a_at(Next{}), b_at(Next{}), std::false_type{});
      __builtin_amdgcn_sched_barrier(0);
    };
    using T = std::true_type;
    using F = std::false_type;
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    using P2 = std::integral_constant<int, 2>;
    using P3 = std::integral_constant<int, 3>;
    int kt = 0;  // a multiple of four in the unrolled loops: ring position = unrolled position
    if (wave < NW / 2) {
      load_first();
      for (; kt + D + 3 < KT; kt += 4) { step_at(kt, P0{}); step_at(kt + 1, P1{}); step_at(kt + 2, P2{}); step_at(kt + 3, P3{}); }
      for (; kt + D < KT; ++kt) step(kt, T{}, std::integral_constant<int, (D - 1) * CPE>{}, F{});
      // here kt + D >= KT: the copies of every remaining step are already issued
      if (kt + 2 < KT) { step(kt, F{}, std::integral_constant<int, CPE>{}, F{}); ++kt; }
      if (kt + 1 < KT) { step(kt, F{}, std::integral_constant<int, 0>{}, F{}); ++kt; }
      step(kt, F{}, std::integral_constant<int, 0>{}, T{});
    } else {
      if (KT > D) issue_copy(D, Cp{});
      load_first();
      for (; kt + D + 4 < KT; kt += 4) { step_late_at(kt, P0{}); step_late_at(kt + 1, P1{}); step_late_at(kt + 2, P2{}); step_late_at(kt + 3, P3{}); }
      for (; kt + D + 1 < KT; ++kt) step_late(kt, T{}, std::integral_constant<int, (D - 1) * CP>{}, F{});
      // with j steps of copies ahead left, (j - 1) * CP copies may stay pending at the barrier
      if (kt + 3 < KT) { step_late(kt, F{}, std::integral_constant<int, 2 * CP>{}, F{}); ++kt; }
      if (kt + 2 < KT) { step_late(kt, F{}, std::integral_constant<int, CP>{}, F{}); ++kt; }
      if (kt + 1 < KT) { step_late(kt, F{}, std::integral_constant<int, 0>{}, F{}); ++kt; }
      step_late(kt, F{}, std::integral_constant<int, 0>{}, T{});
    }
  };

  // prologue: copies of the first D steps, then publish step 0
  auto prologue = [&](auto cp_tag) {
    constexpr int CP = decltype(cp_tag)::value;
    issue_copy(0, cp_tag);
    if (KT > 1) issue_copy(1, cp_tag);
    if (KT > 2) issue_copy(2, cp_tag);
    asm volatile("" ::: "memory");
    if (KT > 2) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(2 * CP));
    else if (KT > 1) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(CP));
    else __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
  };
  const bool tall = BM > BM0 && row_end - row_begin > BM0;
  if (tall && wave < NW / 2) prologue(CpTall{});
  else prologue(Cp{});
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  if (tall) {  // more than BM0 rows: at least TM0 sub-tiles
    if (tm_valid == TM) run(std::integral_constant<int, TM>{}, CpTall{});
    else if (tm_valid == TM - 1) run(std::integral_constant<int, TM - 1>{}, CpTall{});
    else run(std::integral_constant<int, TM0>{}, CpTall{});
  } else {
    switch (tm_valid) {
      case 0: run(std::integral_constant<int, 0>{}, Cp{}); break;
      case 1: run(std::integral_constant<int, 1>{}, Cp{}); break;
      case 2: run(std::integral_constant<int, 2>{}, Cp{}); break;
      case 3: run(std::integral_constant<int, 3>{}, Cp{}); break;
      case 4: run(std::integral_constant<int, 4>{}, Cp{}); break;
      case 5: run(std::integral_constant<int, 5>{}, Cp{}); break;
      case 6: run(std::integral_constant<int, 6>{}, Cp{}); break;
      case 7: run(std::integral_constant<int, 7>{}, Cp{}); break;
      default: run(std::integral_constant<int, TM0>{}, Cp{}); break;
    }
  }

  // ---- epilogue.  Per 16x16 tile a lane holds the four columns (lane/16)*4 + {0..3} of activation
  // row lane % 16.  Each wavefront transposes its outputs through its own slice of LDS (padded rows)
  // and stores them to global memory as full 16-byte words, a whole row segment per group of lanes.
  constexpr int TN_OUT = EPI == EPI_SWIGLU ? TN / 2 : TN;
  constexpr int WN_OUT = EPI == EPI_SWIGLU ? WN / 2 : WN;
  constexpr int ROWB = WN_OUT * 2 + 8;          // bytes between rows of the wavefront's LDS slice
  constexpr int PASS = epilogue_pass(TM, NW, ROWB);  // row sub-tiles that fit the LDS at a time
  constexpr int SLICE = PASS * 16 * ROWB;
  constexpr int LPR = WN_OUT * 2 / 16;          // lanes per row when reading back
  constexpr int RPI = 64 / LPR;                 // rows per read-back instruction, inside one sub-tile
  static_assert(RPI <= 16, "read-back");
  __syncthreads();                              // every wavefront is done with the copy stages
  unsigned char* slice = smem + wave * SLICE;
  const int rcol = (lane % LPR) * 8;
  const int col = n0 + wn * WN_OUT + rcol;
#pragma unroll
  for (int p0 = 0; p0 < TM; p0 += PASS) {
#pragma unroll
    for (int tm = p0; tm < (p0 + PASS < TM ? p0 + PASS : TM); ++tm) {
      if (tm >= tm_valid) continue;
#pragma unroll
      for (int tn = 0; tn < TN_OUT; ++tn) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (EPI == EPI_SWIGLU) v[r] = silu_f32(acc[tm][tn][r]) * acc[tm][tn + TN / 2][r];
          else v[r] = acc[tm][tn][r];
        }
        u32x2 o = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        *reinterpret_cast<u32x2*>(slice + ((tm - p0) * 16 + (lane & 15)) * ROWB + (tn * 16 + (lane >> 4) * 4) * 2) = o;
      }
    }
    // read back: lane l takes 16 bytes (8 columns) of row l / LPR of each group of RPI rows
    if (col >= g.n_out) continue;  // n_out is a multiple of 8: a word is entirely inside or outside
#pragma unroll
    for (int it = 0; it < PASS * 16 / RPI; ++it) {
      const int lrow = it * RPI + lane / LPR;     // row inside the wavefront's slice
      const int tm = p0 + (it * RPI >> 4);
      if (tm >= tm_valid) break;
      const int row = row_begin + (tm * WAVES_M + wm) * 16 + (lrow & 15);
      if (row < row_end) {
        const u32x4 o = *reinterpret_cast<const u32x4*>(slice + lrow * ROWB + rcol * 2);
        uint16_t* dst = static_cast<uint16_t*>(g.C);
        // a 16-byte word is 8 columns inside one 32-column panel
        if (g.c_rows > 0) dst += (static_cast<int64_t>(col / kWeightTileK) * g.c_rows + row) * kWeightTileK + col % kWeightTileK;
        else dst += static_cast<int64_t>(row) * g.ldc + col;
        *reinterpret_cast<u32x4*>(dst) = o;
      }
    }
  }
}

// Launch helpers: grids cover `max_m_tiles` row-tiles per problem (upper bounds; surplus
// workgroups exit at once).
template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int KID>
int launch_gemm_bf16_dma(revive_ctx* ctx, const GemmArgs& p0, int max_m_tiles0, const GemmArgs* p1, int max_m_tiles1,
                         hipStream_t stream) {
  constexpr int NT = 64 * WAVES_M * WAVES_N;
  constexpr int WN_OUT_ = (EPI == EPI_SWIGLU ? BN / 2 : BN) / WAVES_N;
  constexpr int rowb = WN_OUT_ * 2 + 8;
  constexpr size_t lds_epi = static_cast<size_t>(WAVES_M * WAVES_N) * epilogue_pass(BM / WAVES_M / 16, WAVES_M * WAVES_N, rowb) * 16 * rowb;
  constexpr size_t lds_ring = kStages * (BM + BN) * 64;
  constexpr size_t lds = lds_ring > lds_epi ? lds_ring : lds_epi;
  auto kern = gemm_bf16_dma_kernel<BM, BN, WAVES_M, WAVES_N, EPI, KID>;
  REVIVE_HIP(ctx, allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds));
  GemmArgs2 a{};
  a.p0 = p0;
  a.two = p1 != nullptr;
  if (p1) a.p1 = *p1;
  auto budget = [](const GemmArgs& p, int max_m_tiles) -> int64_t {  // workgroups per XCD, as the kernel splits the problem
    return p.tiles ? (static_cast<int64_t>(max_m_tiles) * p.n_col_tiles + 7) / 8 : static_cast<int64_t>((max_m_tiles + 7) / 8) * p.n_col_tiles;
  };
  const int64_t per_xcd = budget(p0, max_m_tiles0) + (p1 ? budget(*p1, max_m_tiles1) : 0);
  if (per_xcd <= 0) return REVIVE_OK;
  const int grid = static_cast<int>(per_xcd * 8);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(NT), lds, stream, a);
  return check_hip(ctx, hipGetLastError(), "gemm_bf16_dma launch");
}

}  // namespace revive
