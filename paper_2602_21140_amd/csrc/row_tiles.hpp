// Row-tiles of a grouped GEMM, worked out by the workgroup that needs one.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace revive {

// Slots' rows are cut into ceil(rows / tile_m) row-tiles each, slots in order.  Every wavefront works out
// by itself which tile is its own (64 slots at a time, a prefix sum over the lanes), which saves the
// launch of 5 us that would build a list; where workgroups are short the list is the better way.

// Number of row-tiles of all slots.
__device__ __forceinline__ int count_row_tiles(const int32_t* __restrict__ slot_offsets, int P, int tile_m) {
  int n = 0;
  for (int p0 = 0; p0 < P; p0 += 256) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int p = p0 + c * 64 + (threadIdx.x & 63);
      if (p < P) n += max(0, (slot_offsets[p + 1] - slot_offsets[p] + tile_m - 1) / tile_m);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
  return __builtin_amdgcn_readfirstlane(n);
}

// The slot that holds row-tile m, 0 <= m < count_row_tiles().
struct SlotTiles { int group, first, end, base, n; };  // rows [first, end) in n tiles, the first of them tile `base`
__device__ __forceinline__ SlotTiles find_slot(const int32_t* __restrict__ slot_offsets, int P, int tile_m, int m) {
  const int lane = threadIdx.x & 63;
  SlotTiles t{0, 0, 0, 0, 0};
  int before = 0;  // tiles of the slots in front
  for (int p0 = 0; p0 < P; p0 += 256) {
    int first[4], end[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {  // the loads of 256 slots go out together
      const int p = p0 + c * 64 + lane;
      first[c] = p < P ? slot_offsets[p] : 0;
      end[c] = p < P ? slot_offsets[p + 1] : 0;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int n = max(0, (end[c] - first[c] + tile_m - 1) / tile_m);
      int incl = n;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
      }
      const int total = __builtin_amdgcn_readlane(incl, 63);
      if (m < before + total) {
        const int src = __builtin_ctzll(__ballot(before + incl > m));  // first slot whose tiles reach beyond m
        t.group = p0 + c * 64 + src;
        t.first = __builtin_amdgcn_readlane(first[c], src);
        t.end = __builtin_amdgcn_readlane(end[c], src);
        t.n = __builtin_amdgcn_readlane(n, src);
        t.base = before + __builtin_amdgcn_readlane(incl, src) - t.n;
        return t;
      }
      before += total;
    }
  }
  return t;
}

// The tile of workgroup b in a grid of (an upper bound on) all slots' row-tiles times n_col column tiles:
// rows [row_begin, row_end) of `group` and column tile n_idx; group = -1: nothing to do.
//
// Workgroup i runs on XCD i % 8.  Each XCD takes a contiguous eighth of the tiles (a row-tile's column
// tiles share its activations in that XCD's L2); inside a slot the column tile runs slower than the
// row-tile, so that the row-tiles that read the same weights are neighbours.  A slot's rows are cut evenly.
struct GridTile { int group, row_begin, row_end, n_idx, in_group; };
__device__ __forceinline__ GridTile grid_tile(const int32_t* __restrict__ slot_offsets, int P, int tile_m, int n_col, int b) {
  GridTile g{-1, 0, 0, 0, 0};
  const int total = count_row_tiles(slot_offsets, P, tile_m) * n_col;
  const int per_xcd = (total + 7) >> 3, local = b >> 3;
  const int pos = (b & 7) * per_xcd + local;
  if (local >= per_xcd || pos >= total) return g;
  const SlotTiles t = find_slot(slot_offsets, P, tile_m, pos / n_col);
  const int r = pos - t.base * n_col;
  g.n_idx = r / t.n;
  const int j = r - g.n_idx * t.n;
  const int rows_each = ((t.end - t.first + t.n - 1) / t.n + 15) & ~15;
  g.row_begin = t.first + j * rows_each;
  g.row_end = min(t.end, g.row_begin + rows_each);
  g.in_group = t.n;
  if (g.row_begin < g.row_end) g.group = t.group;
  return g;
}

}  // namespace revive
