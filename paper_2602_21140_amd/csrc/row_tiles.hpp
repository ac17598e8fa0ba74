// Row-tiles of a grouped GEMM, worked out by the workgroup that needs one.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace revive {

// Inclusive prefix sum over the wavefront, by cross-lane operands of the additions (through LDS, as a shuffle goes, each of
// the six steps takes ten times as long): four steps inside the rows of 16 lanes, two between rows.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_or_zero(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false); }
__device__ __forceinline__ int wave_scan(int v) {
  v += dpp_or_zero<0x111, 0xF>(v);  // lanes 1, 2, 4, 8 below, in the row
  v += dpp_or_zero<0x112, 0xF>(v);
  v += dpp_or_zero<0x114, 0xF>(v);
  v += dpp_or_zero<0x118, 0xF>(v);
  v += dpp_or_zero<0x142, 0xA>(v);  // the last lane of the row below
  v += dpp_or_zero<0x143, 0xC>(v);  // lane 31
  return v;
}

// The tile of workgroup b in a grid of (an upper bound on) all slots' row-tiles times n_col column tiles: rows [row_begin,
// row_end) of `group`, whose weights `tab` has, and column tile n_idx; group = -1: nothing to do.  Slots' rows are cut into
// ceil(rows / tile_m) row-tiles each, evenly, slots in order.
//
// Workgroup i runs on XCD i % 8.  Each XCD takes a contiguous eighth of the tiles (a row-tile's column
// tiles share its activations in that XCD's L2); inside a slot the column tile runs slower than the
// row-tile, so that the row-tiles that read the same weights are neighbours.
//
// Every wavefront works out by itself which tile is its own, which saves the launch of 5 us that would build a list; where
// workgroups are short the list is the better way.  It is a chain of three loads in front of the first weights, so the
// rest is kept short: a lane adds up ceil(P / 64) slots in a row, one prefix sum over the lanes gives the number of tiles
// and the lane that has the wanted one, and its slots, one per lane, come with their weights' addresses.  us of the FFN
// back to back, against two passes over the slots with shuffles and the address behind them: bf16, H = 256, I = 128, 64
// rows, 20 slots 7.8 and 6.6, 640 slots 14.8 and 7.3; H = 512, I = 256, 40 rows, 288 slots 12.2 and 8.9; H = 704, I = 192,
// 400 rows, 1024 slots 73 and 58; fp32, H = 64, I = 32, 64 rows, 1024 slots 20.8 and 10.6.
struct GridTile { int group, row_begin, row_end, n_idx, in_group; const void* w; };
__device__ __forceinline__ GridTile grid_tile(const int32_t* __restrict__ slot_offsets, int P, int tile_m, int n_col, int b, const void* const* __restrict__ tab) {
  GridTile g{-1, 0, 0, 0, 0, nullptr};
  const int lane = threadIdx.x & 63;
  const int per = (P + 63) >> 6;  // slots of a lane, 16 at most
  int n = 0;
#pragma unroll
  for (int c = 0; c < 16; c += 4) {
    if (c >= per) break;
    int end[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) end[i] = slot_offsets[min(lane * per + min(c + i, per), P)];  // past the lane's slots: no rows
#pragma unroll
    for (int i = 0; i < 4; ++i) n += max(0, (end[i + 1] - end[i] + tile_m - 1) / tile_m);
  }
  const int incl = wave_scan(n);
  const int total = __builtin_amdgcn_readlane(incl, 63) * n_col;
  const int per_xcd = (total + 7) >> 3, local = b >> 3;
  const int pos = (b & 7) * per_xcd + local;
  if (local >= per_xcd || pos >= total) return g;
  const int m = pos / n_col;
  const int src = __builtin_ctzll(__ballot(incl > m));  // the first lane whose slots' tiles reach beyond m
  const int before = __builtin_amdgcn_readlane(incl - n, src);
  const int p = min(src * per + min(lane, per), P);
  const int first = slot_offsets[p], end = slot_offsets[min(p + 1, P)];
  const uint64_t w = reinterpret_cast<uint64_t>(tab[min(p, P - 1)]);
  const int mine = lane < per ? max(0, (end - first + tile_m - 1) / tile_m) : 0;
  const int reach = before + wave_scan(mine);
  const int at = __builtin_ctzll(__ballot(reach > m));
  const int tiles = __builtin_amdgcn_readlane(mine, at), base = __builtin_amdgcn_readlane(reach, at) - tiles;  // first row-tile of the slot
  const int row0 = __builtin_amdgcn_readlane(first, at), row1 = __builtin_amdgcn_readlane(end, at);
  const int r = pos - base * n_col;
  g.n_idx = r / tiles;
  const int rows_each = ((row1 - row0 + tiles - 1) / tiles + 15) & ~15;
  g.row_begin = row0 + (r - g.n_idx * tiles) * rows_each;
  g.row_end = min(row1, g.row_begin + rows_each);
  g.in_group = tiles;
  g.w = reinterpret_cast<const void*>(static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(w >> 32), at))) << 32 |
                                      static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(w), at)));
  if (g.row_begin < g.row_end) g.group = src * per + at;
  return g;
}

}  // namespace revive
