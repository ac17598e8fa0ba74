// Which kernels serve the bf16 expert FFN: rules on sizes, with both sides of each line measured.  Host code without HIP.
#pragma once

#include <algorithm>
#include <cstdint>

namespace revive {

// One call of the FFN: P slots, N routed rows (0: no routed experts), T tokens of the shared expert (0: none).
struct FfnSizes { int P, H, I, I_shared; int64_t N; int T; };

// Which problems take the streaming kernel (gemm_stream.hpp).  Up to 96 routed rows per slot on average the
// weights dominate and it wins whatever the load's shape: against the 256-row-tile kernel, H = 7168, I = 2048,
// 288 slots, whole layer: 5 rows 4.31 -> 3.80 ms, 28 uneven rows 4.38 -> 3.99, 42 rows 4.71 -> 4.44, 89 rows
// 5.17 -> 4.87; at 114 rows a slot often needs a second row-tile of 128 and it loses (5.70 -> 5.89).  The
// shared expert's rows go along in the same launches (k = 1, 8192 tokens: 5.16 -> 4.85) unless they are many and
// weigh more than the slots (takes_stream).
// Weights that the 256 MB last-level cache holds come in faster than HBM streams; above 16 rows per slot the
// streaming kernel's set-up then costs more than it saves (141 MB, 61 rows: 84 -> 88 us; 27 MB, 20 rows: 58 ->
// 59; 226 MB, 40 rows: 108 -> 104; 113 MB, 14 rows: 71 -> 65).
constexpr int kStreamRowsPerSlot = 96, kStreamRowsPerSlotCached = 16;
constexpr int64_t kCachedWeights = 192ll << 20;

// A streaming workgroup looks its row-tile up in all slots' offsets; the 256-row kernel has a list.
constexpr int kStreamSlotsCached = 640, kStreamSlots = 768;

inline bool weights_cached(const FfnSizes& f) { return static_cast<int64_t>(f.P) * 6 * f.H * f.I <= kCachedWeights; }

inline bool takes_stream(const FfnSizes& f) {
  const bool cached = weights_cached(f);
  if (f.N > static_cast<int64_t>(cached ? kStreamRowsPerSlotCached : kStreamRowsPerSlot) * f.P) return false;
  // With many slots a search that took twice as long cost more than it saved where a workgroup has little to stream, and
  // the lines were drawn for it.  Today's costs less than the lines allow for; they have not been moved.  Time of the 256-row
  // kernel over time streamed, other data in the caches, 400 random layers: cached, 513 to 768 slots 1.45, beyond 1.37 (at
  // least 1.06); larger weights beyond 768 slots, up to 256 rows in all and products of up to 640 columns 1.47, more than 64
  // rows and up to 128 K-elements in one of the products 1.14 (least 0.87: P = 1000, H = 128, I = 320, 921 rows 66 and 76 us).
  if (cached && (f.P > kStreamSlots || (f.P > kStreamSlotsCached && f.N <= 256))) return false;
  if (f.P > kStreamSlots && f.N <= 256 && std::max(f.H, f.I) <= 640) return false;
  if (f.P > kStreamSlots && f.N > 64 && std::min(f.H, f.I) <= 128 && f.I > 64) return false;
  // Every 128 rows of the shared expert read its weights once more.  That loses against the 256-row kernel once they
  // are many rows and what is read that way outweighs the slots' weights, sooner where the cache does not hold the
  // shared expert.  288 slots, H = 7168, I = 2048, one row per token, ms of the 256-row kernel and streamed:
  // I_shared = 9 I, 2048 tokens 5.60 and 5.40, 4096 (as much as the slots) 6.65 and 7.17, 27 648 21.8 and 30.5;
  // 2 I (cached), 27 648 tokens (1.5 times the slots) 8.70 and 8.71.  Share of 1500 random layers that lose: up to
  // 1024 tokens none; above, uncached, from the slots' weights on 66 %; cached, up to 4096 tokens 9 %, above 3 % up to
  // twice the slots' weights and 54 % from there on.
  const bool shared_cached = 6ll * f.H * f.I_shared <= kCachedWeights;
  if (f.T <= (shared_cached ? 4096 : 1024)) return true;
  return static_cast<int64_t>((f.T + 127) / 128) * f.I_shared < static_cast<int64_t>(shared_cached ? 2 : 1) * f.P * f.I;
}

// Forms of the streaming kernel: rows x columns of a workgroup of gate/up; those of the down projection have as many rows
// and twice the columns.
enum StreamForm { k128x128, k64x64, k64x32 };

// Times are us of the FFN with other data in the caches, of the forms in the order of their names, on the same weights in one
// process in turn (from one process to the next they differ by 4 %).  Ratios are geometric means over 1760 random layers near
// the lines, each form timed on each.  Rows are rows per slot; blocks count gate/up's workgroups of 64 columns.
//
// Row-tiles of 128 read the weights of a slot with more than 64 rows once, at one workgroup less per CU.  Time with tiles
// of 64 over time with tiles of 128, where these are many (three and more of gate/up per CU, two of down): even rows 0.99 at 8
// to 12, 1.00 at 12 to 16, 1.03 at 16 to 30, uneven rows 1.02, 1.05, 1.06.  P = 144, H = 2624, I = 1152, 17.3 uneven rows 515,
// 577, 611; P = 240, H = 3456, I = 512, 15.2 uneven 406, 453, 470.  Fewer leave CUs without work: 0.90 at 8 to 20 rows, 0.95
// at 20 to 30, 0.99 beyond; P = 18, H = 4736, I = 704, 16.8 rows 112, 73, 84 (but P = 40, H = 1728, I = 1600, 17.8 uneven rows
// 142, 158, 163).  Up to three tiles of 128 columns cover a narrow expert exactly and read its activations half as often:
// I = 128, 8 to 14 rows 1.02 (P = 384, H = 640, 13.8 rows 68, 77, 78), I = 384, many, 1.03, but few of I = 256 and 384 0.95.
// Many rows of the shared expert take the tall tiles too, where they would read its weights a quarter as often as the slots
// read theirs.  Where all that leaves a quarter of the CUs without work and the cache holds the weights, which may then be
// read again, the small tiles are better: 0.67 over 131 such layers; P = 72, H = 512, I = 384, 12.2 rows (144 workgroups of
// down) 35, 33, 32; P = 20, H = 768, I = 1856, 10.8 rows beside a shared expert of 2 I (66) 102, 61, 62.
//
// Half the columns where fewer than two workgroups of 64 columns fall to a CU: that spreads the streams evenly, and a CU
// alone does not pull more than about 38 GB/s from HBM (one token, 288 -> 576 workgroups: 110 -> 95 us).  Up to four where
// the products are long: time with 64 columns over time with half 1.03 at 512 to 768 blocks, 1.02 to 1024, cached 1.06 and
// 1.05; P = 20, H = 512, I = 2048, 2.1 rows (672) 68, 47, 38; but H = 3840, I = 768, 0.7 rows (672) 98 and 102, H = 1920, I =
// 192 (648) 63.5 and 65.3.  How full the last round is moves either by 5 %: P = 36, H = 3776, I = 1600, 0.7 uneven rows (625)
// 111 and 117.  The row-tiles of the shared expert count: P = 24, H = 640, I = 1728, 11.2 rows, 270 tokens beside I_shared =
// 4 I (1188) 149, 91, 99.
inline StreamForm stream_form(const FfnSizes& f) {
  auto tiles = [](int64_t n, int of) { return (n + of - 1) / of; };
  const int64_t used = std::min<int64_t>(f.N, f.P);  // slots that can hold a row
  const int64_t dense = tiles(f.T, 128);
  const int64_t gate_up = used * tiles(f.I, 128) + dense * tiles(f.I_shared, 128), down = (used + dense) * tiles(f.H, 256);  // of 128 rows
  const bool cached = weights_cached(f), narrow = f.I % 128 == 0 && f.I < 512, many = !cached && gate_up >= 3 * 256 && down >= 2 * 256;
  if (f.N > static_cast<int64_t>(narrow ? 8 : many ? 12 : 20) * f.P || (f.T > 128 && 8 * dense * f.I_shared > used * f.I)) {
    if (!cached || (gate_up >= 192 && down >= 192)) return k128x128;
  }
  if ((used + (f.T > 0)) * tiles(f.I, 64) < 2 * 256) return k64x32;
  const int64_t blocks = used * tiles(f.I, 64) + tiles(f.T, 64) * tiles(f.I_shared, 64);
  return blocks < 4 * 256 && std::min(f.H, f.I) >= 512 && f.H <= 4 * f.I ? k64x32 : k64x64;
}

}  // namespace revive
