// Which kernel serves a call of the gate: rules on sizes, with both sides of each line measured.  Host code without HIP.
#pragma once

#include <cstdint>

namespace revive {

// The bf16 router with K in one sequence: router_sequence_kernel with 8 x 8 or 16 x 16 tiles of tokens and experts, or
// router_tile_kernel.  The names give tokens x experts x K-elements of a step and the stages of the ring.
enum RouterForm { kSeq8x8, kSeq16x16, k32x32x64s2, k128x64x64s2, k128x64x64s3, k32x32x128s4, k32x64x128s4, k64x64x128s4, k64x128x64s3, k128x128x64s4, k128x192x64s3, k128x256x64s3 };

// The smallest tiles of which at most 256, one per CU, cover the logits.  us with cold caches, E = 256, H = 7168, of a 128 x
// 64 register-staged GEMM and of the tile taken: 512 tokens 73 and 19 (16 x 16 in sequence: 20), 1003 tokens 74 and 21 (32
// x 64 tiles 25), 2048 74 and 26 (32 x 32 tiles 32, 64 x 64 36), 4096 77 and 36 (32 x 64 49, 64 x 128 50), 8192 81 and 54
// (64 x 64 68, 128 x 128 73), 16 384 95 and 79 (64 x 128 102), 32 768 163 and 129 (128 x 128 156); 32 768 tokens and
// E = 384 247 and 187 (128 x 128 219).  Just past a line the next tile leaves CUs without work, but the smaller ones would
// take a second round: back to back, 257 tokens (72 tiles of 32 x 32) 18.8 (16 x 16 in sequence 16.5), 1025 tokens (132 of
// 32 x 64) 23.4 (32 x 32 22.2), 2049 (132 of 64 x 64) 27.4 (32 x 64 41), 4097 (130 of 64 x 128) 41.1 (64 x 64 51).
//
// A short K does not fill a deep ring of large steps: what a tile costs is its first copies and its stores, which need
// several workgroups on a CU to hide one another.  us of route() back to back, of the GEMM, of the rule above (which sent
// all of H = 64 to 16 x 16 in sequence) and of the short forms: H = 64, E = 256: 1003 tokens 6.9, 9.3, 6.0, 8192 14.1, 40,
// 11.8, 65 536 36, 252, 37; H = 64, E = 40, 16 384 tokens 9.9, 19.0, 8.7; H = 128, E = 256, 32 768 tokens 28, 34, 27; H =
// 320, the same 28, 30, 28.  At H = 704 the two are equal (E = 192, 65 536 tokens 42 and 43).
//
// Many tokens: one round of tiles as long as any form makes one; beyond it the widest.  Few experts do not fill a wide tile:
// E = 40, H = 704, 32 769 tokens 128 x 64 16.4, 128 x 128 22.0, 128 x 192 25.2 (the GEMM 20.2); E = 64, H = 2112 33, 44, 51
// (37); E = 100, of which 257 tiles of 128 x 128 would start a second round, 39, 45, 54 (47), but E = 128, 65 536 tokens 86,
// 71, 76 (79).  E = 192, 16 385 tokens, H = 7168: 258 tiles of 128 x 128 113, 129 of 128 x 192 79 (the GEMM 88); E = 512,
// 12 000 tokens, H = 2112: 376 of 128 x 128 48, 188 of 128 x 256 43 (50).
inline RouterForm router_form(int T, int E, int H) {
  auto tiles = [&](int bm, int bn) { return static_cast<int64_t>((T + bm - 1) / bm) * ((E + bn - 1) / bn); };
  auto fits = [&](int bm, int bn) { return tiles(bm, bn) <= 256; };
  if (fits(8, 8)) return kSeq8x8;
  if (H < 128) return tiles(32, 32) <= 1024 ? k32x32x64s2 : k128x64x64s2;
  if (fits(16, 16)) return kSeq16x16;
  if (fits(32, 32)) return k32x32x128s4;
  if (fits(32, 64)) return k32x64x128s4;
  if (fits(64, 64)) return k64x64x128s4;
  if (fits(64, 128)) return k64x128x64s3;
  if (H < 512) return k128x64x64s2;
  if (E <= 64) return k128x64x64s3;
  if (fits(128, 128)) return k128x128x64s4;
  if (E <= 128) return tiles(128, 128) <= 384 ? k128x64x64s3 : k128x128x64s4;
  const int wide = (E + 255) / 256, each = (E + wide - 1) / wide;  // column tiles of up to 256 experts, and their experts
  return each <= 192 ? k128x192x64s3 : k128x256x64s3;
}

// The bf16 router of few experts, K in the slices of router_kernel: that kernel, or router_tile_kernel in those slices.
enum RouterSlicedForm { kSlicedRouter, kSliced128x64s4, kSliced128x64s3, kSliced128x128s4 };

// router_kernel reads x once per 32 experts; with many tokens the tiles, which read it once.  us of route() back to back,
// router_kernel, 128 x 64 tiles with a ring of four stages and of three, 128 x 128 tiles: E = 64, H = 4096: 8192 tokens
// 24, 28, 29, 39, 16 384 39, 30, 30, 41, 32 768 71, 47, 48, 49; E = 128, H = 7168: 4097 tokens 40, 42, -, 63, 16 384 102,
// 51, 54, 66; H = 4096, 32 768 tokens (256 tiles of 128 x 128) 124, 71, 68, 60.  A ring of three lets two tiles onto a CU:
// past 256 tiles of 128 x 64 (E = 40, H = 2048, 32 769 tokens) 37 with four and 31 with three; E = 128, where 257 tiles of
// 128 x 128 would start a second round, 47, 42 and with those 49.
inline RouterSlicedForm router_sliced_form(int T, int E, int H) {
  if (static_cast<int64_t>((T + 31) / 32) * E * H * 2 <= (128ll << 20)) return kSlicedRouter;
  const int tall = (T + 127) / 128;  // tiles of 128 tokens
  if (tall * ((E + 63) / 64) <= 256) return kSliced128x64s4;
  return E <= 64 || (tall > 256 && tall <= 384) ? kSliced128x64s3 : kSliced128x128s4;
}

// The selection with a row of 16 lanes per token (route_topk_rows_kernel) instead of a wavefront (route_topk_kernel).
//
// A row does a quarter of the work per token, but its lanes have four times as many experts to go through one after the
// other: it wins with many tokens, which keep the ALUs busy, and where the experts are few.  us of route() with the
// product, H = 256, back to back, a wavefront per token and a row per token (E experts, g groups, k choices):
//   no groups   E = 64: k = 6, 37 tokens 6.7 and 6.5, 4096 9.4 and 8.0; k = 16, 17 tokens 7.9 and 8.2, 2049 10.2 and 10.1;
//               E = 128: k = 8, 64 tokens 7.4 and 7.8, 300 7.5 and 7.5; k = 16, 1003 9.6 and 10.4, 2560 12.9 and 12.5;
//               E = 192, k = 8: 2049 9.2 and 10.2, 3584 11.5 and 11.0; E = 384, k = 8: 2560 12.5 and 13.6, 3584 14.6 and
//               14.9; on given logits, 65 536 tokens: E = 384, k = 8 69 and 42, E = 512, k = 1 26.6 and 26.7
//   groups      a row finds all groups' scores at once.  E = 128, g = 4, k = 2, 64 tokens 7.6 and 7.2; E = 192: g = 8, k =
//               2, 64 tokens 8.8 and 7.5, g = 2, k = 8, 1003 9.1 and 10.1; E = 256, g = 8, k = 8: 1003 9.8 and 10.5, 2049
//               12.3 and 11.8, 8192 24.3 and 18.4; E = 512, g = 2, k = 8: 3000 17.1 and 17.7, 3584 19.5 and 18.1; E = 64, g =
//               4, k = 16: 129 tokens 8.7 and 8.9, 2048 10.5 and 10.1; E = 400
//               (no multiple of 64: 4-byte loads), g = 2, k = 4, given logits: 3072 8.0 and 9.0, 4096 9.6 and 9.0
inline bool selects_by_rows(int T, int E, int n_group, int k) {
  if (k > 16 || T <= 16) return false;
  if (n_group == 1) {
    if (E > 128) return T >= 3584;
    return T >= (E > 64 ? (k > 8 ? 2560 : 129) : (k > 8 ? 2049 : 17));
  }
  if (E % 16 != 0 || (n_group != 2 && n_group != 4 && n_group != 8)) return false;
  if (k <= (E <= 128 ? 8 : E > 192 ? 0 : n_group == 2 ? 2 : n_group == 4 ? 6 : 8)) return true;
  if (E % 64 != 0 && E > 384) return T >= 4096;
  if (E > 128 * n_group) return T > 3072;
  return T >= (k <= 8 ? 2049 : E < 128 ? 1500 : n_group == 8 ? 2049 : 2560);
}

// Of the calls that are left, those that route_topk_kernel serves with four tokens to a wavefront: less work in all, but
// longer one by one.  us on given logits, one token and four: 120 experts in 5 groups, k = 2: 8193 tokens 13.7 and 14.1,
// 12 288 17.7 and 14.9, 65 536 71 and 56; 200 experts in 8, k = 16: 8193 28 and 37, 16 384 45 and 46, 65 536 157 and 145.
inline bool selects_four_tokens(int T, int n_group, int k) { return n_group <= 8 && k <= 16 && T > (k <= 8 ? 10240 : 16384); }

}  // namespace revive
