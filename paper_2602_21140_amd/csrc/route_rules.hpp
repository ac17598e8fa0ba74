// Which kernel serves a call of the gate: rules on sizes, with both sides of each line measured.  Host code without HIP.
#pragma once

namespace revive {

// The selection with a row of 16 lanes per token (route_topk_rows_kernel) instead of a wavefront (route_topk_kernel).
//
// A row does a quarter of the work per token, but its lanes have four times as many experts to go through one after the
// other: it wins where there are tokens enough to keep the ALUs busy.  us of route() on given logits, back to back, a
// wavefront per token and a row per token (E experts, g groups, k choices):
//   no groups   E = 64, k = 6: 64 tokens 3.4 and 3.6, 2049 3.9 and 3.8, 8192 8.6 and 5.6; E = 192, k = 8, 64 tokens 4.7
//               and 5.6; E = 112, k = 16, 1003 tokens 5.5 and 6.7; E = 384, k = 8: 2049 6.4 and 7.2, 3072 6.9 and 7.1,
//               4096 7.9 and 7.3, 65 536 69 and 42; E = 512, k = 1, 65 536 26.6 and 26.7; E = 500, the same 26.5 and 23
//   groups      E = 256, g = 8, k = 8: 1003 6.6 and 7.2, 2049 7.9 and 7.3, 8192 16.8 and 10.1, 65 536 77 and 39; E = 512,
//               g = 2, k = 16: 2049 13.9 and 14.5, 4096 17.7 and 14.7; E = 400 (no multiple of 64: 4-byte loads), g = 2,
//               k = 4: 3072 8.0 and 9.0, 4096 9.6 and 9.0.  Few experts and choices win from a few tokens on, since a row
//               finds all groups' scores at once: E = 128, g = 4, k = 2, 64 tokens 4.3 and 4.0, E = 192, g = 8, k = 2, 64
//               tokens 6.0 and 4.8 (k = 8: 1003 tokens, g = 2, 6.0 and 6.7).
inline bool selects_by_rows(int T, int E, int n_group, int k) {
  if (k > 16 || T <= 16) return false;
  if (n_group > 1 && (E % 16 != 0 || (n_group != 2 && n_group != 4 && n_group != 8))) return false;
  if (n_group == 1) return T >= (E <= 128 ? 2560 : 3584);
  if (k <= (E <= 128 ? 6 : E <= 192 ? 2 : 0)) return true;
  if (E % 64 != 0 && E > 384) return T >= 4096;
  return T > (k <= 8 ? 2048 : 3072);
}

}  // namespace revive
