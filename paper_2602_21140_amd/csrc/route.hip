// Gate of the failure-remapped MoE layer: router logits, failure-masked (group-limited) top-k,
// renormalised weights and the logical->physical replica remap.
//
// Paper: Sec. 2.1 (gating scores, top-k), Sec. 3.4 "Missing experts" and Sec. 4.2 (experts with
// no replica left are masked to -inf immediately before the top-k), Sec. 3.4 "Redundant experts"
// (the logical-to-physical map decides which replica serves a token).
#include <algorithm>

#include "gemm_f32.hpp"
#include "route_rules.hpp"
#include "router_sequence.hpp"

namespace revive {

namespace {

struct RouteParams {
  const float* logits;
  const int32_t* l2p_count;
  const int32_t* l2p_table;
  int32_t* topk_logical;
  float* topk_weight;
  int32_t* topk_phys;
  int T, E, k, max_replicas, score_fn, n_group, topk_group;
  int none;            // expert that route_topk_kernel gives a row of NaN, which holds no best key
  long long t_offset;  // index of token 0 within the whole batch
  float route_scale;
};

// Reductions over the wavefront without LDS: four steps inside the rows of 16 lanes, two between rows, all
// of them cross-lane operands of an ALU instruction (a shuffle through LDS takes ten times as long).
// Step 0..3 combine halves of 2, 4, 8 and 16 lanes, after which every lane of a row has the row's result;
// steps 4 and 5 bring the rows' results to lanes 31 and 63, and then to lane 63.  Lanes that a step has
// nothing for get `other`.
template <int STEP>
__device__ __forceinline__ float dpp_step(float v, float other) {
  constexpr int ctrl = STEP == 0 ? 0xB1 : STEP == 1 ? 0x4E : STEP == 2 ? 0x141 : STEP == 3 ? 0x140 : STEP == 4 ? 0x142 : 0x143;
  constexpr int rows = STEP == 4 ? 0xA : STEP == 5 ? 0xC : 0xF;
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(other), __float_as_int(v), ctrl, rows, 0xF, false));
}
__device__ __forceinline__ float wave_max(float v) {
  const float NEG = -__builtin_inff();
  v = fmaxf(v, dpp_step<0>(v, NEG));
  v = fmaxf(v, dpp_step<1>(v, NEG));
  v = fmaxf(v, dpp_step<2>(v, NEG));
  v = fmaxf(v, dpp_step<3>(v, NEG));
  v = fmaxf(v, dpp_step<4>(v, NEG));
  v = fmaxf(v, dpp_step<5>(v, NEG));
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
// The two largest of two disjoint sets, each given by its two largest.
template <int STEP>
__device__ __forceinline__ void top2_step(float& m1, float& m2) {
  const float NEG = -__builtin_inff();
  const float o1 = dpp_step<STEP>(m1, NEG), o2 = dpp_step<STEP>(m2, NEG);
  const float lo = fmaxf(fminf(m1, o1), fmaxf(m2, o2));
  m1 = fmaxf(m1, o1);
  m2 = lo;
}

template <int CTRL>
__device__ __forceinline__ int dpp_int(int v) { return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, false); }  // v of another lane

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = dpp_int<CTRL>(static_cast<int>(b)), hi = dpp_int<CTRL>(static_cast<int>(b >> 32));
  return __longlong_as_double(static_cast<long long>(hi) << 32 | static_cast<uint32_t>(lo));
}

// Slot of token t's expert e, which has `count` copies: the (batch index of t mod count)-th surviving one, ascending slot id.
__device__ __forceinline__ int replica(const RouteParams& p, int t, int e, int count) {
  if (count <= 0) return -1;
  const unsigned long long b = static_cast<unsigned long long>(p.t_offset) + t;
  const int r = p.t_offset + p.T <= 0x7fffffffll ? static_cast<int>(static_cast<uint32_t>(b) % static_cast<uint32_t>(count)) : static_cast<int>(b % count);
  return p.l2p_table[e * p.max_replicas + r];
}

// A wavefront selects for TPW tokens.  Lane l holds the logits of experts l, l+64, l+128, ... (VALS of them)
// of each; a masked or excluded expert's key is -inf.  Expert order is decided on the fp32 logits themselves
// (softmax and sigmoid are increasing, so this is the order of the scores); group scores, which add two
// scores, and the output weights are evaluated in fp64.
//
// The fp64 work (an exponential per group and per chosen expert) keeps few lanes busy and is what a token
// costs most, so each token has LPT = 64 / TPW lanes of its own for it: lane g of them takes the best score
// of group g, lane LPT/2 + g the second best, lane j the j-th chosen expert's weight.
template <int VALS, int TPW, bool GROUPED>
__global__ __launch_bounds__(256) void route_topk_kernel(RouteParams p) {
  constexpr int LPT = 64 / TPW, HALF = LPT / 2;
  const int lane = threadIdx.x & 63;
  const int t0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * TPW;
  if (t0 >= p.T) return;  // whole wavefront leaves together
  const float NEG = -__builtin_inff();
  const int my_q = lane / LPT, li = lane % LPT;  // the token whose fp64 work this lane shares, and its place in it

  int cnt[VALS];
  float key[TPW][VALS];
#pragma unroll
  for (int i = 0; i < VALS; ++i) {
    const int e = lane + 64 * i;
    cnt[i] = e < p.E ? p.l2p_count[e] : 0;
#pragma unroll
    for (int q = 0; q < TPW; ++q)
      key[q][i] = e < p.E ? p.logits[static_cast<int64_t>(min(t0 + q, p.T - 1)) * p.E + e] : NEG;
  }
  float my_max = NEG;  // largest live logit of my token: common shift of the exponentials (the best chosen score is exactly 1)
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    float m = NEG;
#pragma unroll
    for (int i = 0; i < VALS; ++i) {
      if (cnt[i] <= 0) key[q][i] = NEG;  // failure mask
      m = fmaxf(m, key[q][i]);
    }
    m = wave_max(m);
    if (my_q == q) my_max = m;
  }
  const double shift = static_cast<double>(my_max);
  auto score64 = [&](float z) -> double {  // unnormalised gating score of a live expert of my token
    const double zd = static_cast<double>(z);
    return p.score_fn == REVIVE_SCORE_SIGMOID ? 1.0 / (1.0 + exp(-zd)) : exp(zd - shift);
  };

  if (GROUPED) {
    // Group score = sum of the two best live scores of the group (one if only one is live, -inf if none).
    // A NaN must not enter the pairs: the smaller of a key and a NaN is the key, which would then count twice.
    auto number = [NEG](float z) { return z > NEG ? z : NEG; };
    const int gsz = p.E / p.n_group;
    float top = NEG;  // li < HALF: best key of group li; else second best of group li - HALF
    if (gsz >= 8 && (gsz & (gsz - 1)) == 0 && gsz <= 64) {
      // groups are aligned runs of lanes: all groups at once
      const int per_block = 64 / gsz, g = li % HALF;
      const int src = (g % per_block) * gsz + gsz - 1, block = g / per_block;
#pragma unroll
      for (int q = 0; q < TPW; ++q) {
#pragma unroll
        for (int i = 0; i < VALS; ++i) {
          float m1 = number(key[q][i]), m2 = NEG;
          top2_step<0>(m1, m2);
          top2_step<1>(m1, m2);
          top2_step<2>(m1, m2);
          if (gsz >= 16) top2_step<3>(m1, m2);
          if (gsz >= 32) top2_step<4>(m1, m2);
          if (gsz >= 64) top2_step<5>(m1, m2);
          const float a = __shfl(m1, src), b = __shfl(m2, src);
          if (my_q == q && block == i) top = li < HALF ? a : b;
        }
      }
    } else {
#pragma unroll 1
      for (int g = 0; g < p.n_group; ++g) {
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
          float m1 = NEG, m2 = NEG;
#pragma unroll
          for (int i = 0; i < VALS; ++i) {
            const int e = lane + 64 * i;
            const float z = e >= g * gsz && e < (g + 1) * gsz ? number(key[q][i]) : NEG;
            m2 = fmaxf(m2, fminf(m1, z));
            m1 = fmaxf(m1, z);
          }
          top2_step<0>(m1, m2);
          top2_step<1>(m1, m2);
          top2_step<2>(m1, m2);
          top2_step<3>(m1, m2);
          top2_step<4>(m1, m2);
          top2_step<5>(m1, m2);
          const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(m1), 63));
          const float b = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(m2), 63));
          if (my_q == q && li % HALF == g) top = li < HALF ? a : b;
        }
      }
    }
    const double s = top > NEG ? score64(top) : 0.0;
    const double second = __shfl(s, lane + HALF);
    const double gs = li < p.n_group && top > NEG ? s + second : -__builtin_inf();
    // rank of my group among all groups of the token (better score first, ties to the lower group id)
    int rank = 0;
#pragma unroll 4
    for (int h = 0; h < p.n_group; ++h) {
      const double o = __shfl(gs, my_q * LPT + h);
      rank += (o > gs) || (o == gs && h < li);
    }
    const unsigned long long kept = __ballot(li < p.n_group && rank < p.topk_group);
#pragma unroll
    for (int i = 0; i < VALS; ++i) {
      // e / gsz: exact, e + 1/2 is never within 2^-11 of a multiple of gsz
      const int g = static_cast<int>((static_cast<float>(lane + 64 * i) + 0.5f) / static_cast<float>(gsz));
#pragma unroll
      for (int q = 0; q < TPW; ++q)
        if (!((static_cast<uint32_t>(kept >> (q * LPT)) >> (g & 31)) & 1u)) key[q][i] = NEG;  // expert of a dropped group
    }
  }

  // k rounds of wave-wide arg-max (largest key, ties to the lower expert id); the winner of token q's round j
  // lands in lane q * LPT + j
  int my_e = 0;
  float my_z = 0.f;
#pragma unroll 1
  for (int j = 0; j < p.k; ++j) {
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
      float m = key[q][0];
#pragma unroll
      for (int i = 1; i < VALS; ++i) m = fmaxf(m, key[q][i]);
      const float best = wave_max(m);
      int wi = 0;
      unsigned long long holders = 1ull;
#pragma unroll
      for (int i = VALS - 1; i >= 0; --i) {
        const unsigned long long b = __ballot(key[q][i] == best);
        if (b) { holders = b; wi = i; }
      }
      const int w = __builtin_ctzll(holders);
#pragma unroll
      for (int i = 0; i < VALS; ++i)
        if (wi == i && lane == w) key[q][i] = NEG;
      if (lane == q * LPT + j) { my_e = wi * 64 + w; my_z = best; }
    }
  }

  my_e = min(my_e, p.E - 1);  // a row of NaN holds no best key but the -inf of lanes without an expert (RouteParams::none)

  // weights: score of the chosen expert over the sum of the chosen scores
  const int t = t0 + my_q;
  const double s = li < p.k ? score64(my_z) : 0.0;
  double sum = s;
#pragma unroll
  for (int o = HALF; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  int c = 0;  // replicas of my expert, held by lane my_e % 64
#pragma unroll
  for (int i = 0; i < VALS; ++i) {
    const int v = __shfl(cnt[i], my_e & 63);
    if (my_e >> 6 == i) c = v;
  }
  if (li < p.k && t < p.T) {
    const int64_t o = static_cast<int64_t>(t) * p.k + li;
    const int phys = replica(p, t, my_e, c);
    p.topk_logical[o] = my_e;
    p.topk_weight[o] = static_cast<float>(s / sum * static_cast<double>(p.route_scale));
    p.topk_phys[o] = phys;
  }
}

// The same selection with 16 lanes, one DPP row, per token: four tokens to a wavefront, every instruction for all four.
// A group of experts (all of them in a layer without groups) is a run of lg = 16 / n_group lanes (n_group a power of two
// up to 8, E a multiple of 16), and a lane holds n = ceil(E / 16) <= V of its experts, dealt so that the run's loads are
// contiguous: lane j of the run holds the group's experts j, j + lg, ..., or with WIDE (E a multiple of 64, 16-byte loads)
// its words of four j, j + lg, ...  A reduction is four steps instead of six, and ties go to the lowest expert id.  The
// kernel above gives a token 64 lanes and works on one after the other; it is bound by the ALU from a few thousand
// tokens on (selects_by_rows has the figures).  With a lane's experts side by side instead each load touched four times
// as many lines and more: 65 536 tokens, one choice, 512 experts 52 us (27 as it is), 500 experts 320 (23).
template <int V, bool GROUPED, bool WIDE>
__global__ __launch_bounds__(256) void route_topk_rows_kernel(RouteParams p) {
  static_assert(!WIDE || V % 4 == 0, "16-byte loads");
  struct Choice { int e; float z; };
  __shared__ Choice chosen[4][4][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = lane >> 4, li = lane & 15;
  const int t0 = (blockIdx.x * 4 + wave) * 4, t = t0 + row;
  if (t0 >= p.T) return;  // whole wavefront leaves together
  const float NEG = -__builtin_inff(), NONE = __builtin_nanf("");  // NONE: no expert in this place, equal to no key
  const int n = (p.E + 15) >> 4;
  const int lg = GROUPED ? 16 / p.n_group : 16, lj = li & (lg - 1);  // lanes of a group, this one's place among them
  const int e0 = GROUPED ? li / lg * (p.E / p.n_group) : 0;          // the group's first expert
  auto expert = [&](int i) { return e0 + (WIDE ? (i >> 2) * 4 * lg + lj * 4 + (i & 3) : i * lg + lj); };  // place i
  const float* z = p.logits + static_cast<int64_t>(min(t, p.T - 1)) * p.E;

  float key[V];
  if (WIDE) {
#pragma unroll
    for (int i = 0; i < V; i += 4) {
      if (i < n) {  // n is a multiple of 4
        const f32x4 v = *reinterpret_cast<const f32x4*>(z + expert(i));
        const int4 c = *reinterpret_cast<const int4*>(p.l2p_count + expert(i));
        key[i] = c.x > 0 ? v[0] : NEG; key[i + 1] = c.y > 0 ? v[1] : NEG;  // failure mask
        key[i + 2] = c.z > 0 ? v[2] : NEG; key[i + 3] = c.w > 0 ? v[3] : NEG;
      } else {
        key[i] = key[i + 1] = key[i + 2] = key[i + 3] = NONE;
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const int e = min(expert(i), p.E - 1);
      const float v = z[e];
      const int c = p.l2p_count[e];
      key[i] = i < n && expert(i) < p.E ? c > 0 ? v : NEG : NONE;
    }
  }
  auto lane_max = [&]() {
    float m = NEG;
#pragma unroll
    for (int i = 0; i < V; ++i) m = fmaxf(m, key[i]);
    return m;
  };
  auto row_max = [&](float m) {
    m = fmaxf(m, dpp_step<0>(m, NEG));
    m = fmaxf(m, dpp_step<1>(m, NEG));
    m = fmaxf(m, dpp_step<2>(m, NEG));
    return fmaxf(m, dpp_step<3>(m, NEG));
  };
  // largest live logit of the token: common shift of the exponentials (the best chosen score is exactly 1)
  const double shift = p.score_fn == REVIVE_SCORE_SIGMOID ? 0.0 : static_cast<double>(row_max(lane_max()));
  auto score64 = [&](float v) -> double {  // unnormalised gating score of a live expert
    const double d = static_cast<double>(v);
    return p.score_fn == REVIVE_SCORE_SIGMOID ? 1.0 / (1.0 + exp(-d)) : exp(d - shift);
  };

  if (GROUPED) {
    // Group score = sum of the two best live scores of the group (one if only one is live, -inf if none).  A NaN does
    // not enter the pairs (see above).
    float m1 = NEG, m2 = NEG;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const float v = key[i] > NEG ? key[i] : NEG;
      m2 = fmaxf(m2, fminf(m1, v));
      m1 = fmaxf(m1, v);
    }
    top2_step<0>(m1, m2);
    if (lg >= 4) top2_step<1>(m1, m2);
    if (lg >= 8) top2_step<2>(m1, m2);
    const float mine = li & 1 ? m2 : m1;  // an even lane evaluates the group's best score, its neighbour the second
    const double s = mine > NEG ? score64(mine) : 0.0;
    const double both = s + dpp_f64<0xB1>(s);
    const double gs = m1 > NEG ? both : -__builtin_inf();
    // rank of my group among all groups of the token (better score first, ties to the lower group id)
    int rank = 0;
    double o = gs;
    int h = li;
    for (int r = 1; r < p.n_group; ++r) {
      if (lg == 2) { o = dpp_f64<0x122>(o); h = dpp_int<0x122>(h); }       // rotate the row by a group
      else if (lg == 4) { o = dpp_f64<0x124>(o); h = dpp_int<0x124>(h); }
      else { o = dpp_f64<0x128>(o); h = dpp_int<0x128>(h); }
      rank += (o > gs) || (o == gs && h < li);
    }
    const bool kept = rank < p.topk_group;
#pragma unroll
    for (int i = 0; i < V; ++i) key[i] = kept ? key[i] : NEG;
  }

  // k rounds of arg-max (largest key, ties to the lower expert id)
  constexpr int kNone = 1 << 16;
  auto row_min = [&](int v) {
    v = min(v, dpp_int<0xB1>(v));   // lanes 1 apart
    v = min(v, dpp_int<0x4E>(v));   // 2 apart
    v = min(v, dpp_int<0x124>(v));  // 4 apart: lanes of four are equal by now
    return min(v, dpp_int<0x128>(v));
  };
#pragma unroll 1
  for (int j = 0; j < p.k; ++j) {
    const float best = row_max(lane_max());
    int at = V;  // the lowest place of the key in this lane; four short chains of minima
    {
      int part[4] = {V, V, V, V};
#pragma unroll
      for (int i = 0; i < V; ++i) part[i & 3] = min(part[i & 3], key[i] == best ? i : V);
      at = min(min(part[0], part[1]), min(part[2], part[3]));
    }
    const int mine = at < V ? expert(at) : kNone, e = row_min(mine);
    if (mine == e) chosen[wave][row][j] = {e == kNone ? p.none : e, best};  // kNone: no key is the best one in a row of NaN
    at = mine == e ? at : V;
#pragma unroll
    for (int i = 0; i < V; ++i) key[i] = i == at ? NEG : key[i];
  }
  __builtin_amdgcn_wave_barrier();  // the wavefront's own LDS accesses are in order

  // weights: score of the chosen expert over the sum of the chosen scores, added as in the kernel above
  Choice c = {0, 0.f};
  if (li < p.k) c = chosen[wave][row][li];
  const int count = p.l2p_count[c.e];
  const double s = li < p.k ? score64(c.z) : 0.0;
  double sum = s + dpp_f64<0x128>(s);  // lanes 8 apart
  sum += dpp_f64<0x124>(sum);          // 4 apart: lanes 8 apart are equal by now
  sum += dpp_f64<0x4E>(sum);
  sum += dpp_f64<0xB1>(sum);
  if (li < p.k && t < p.T) {
    const int64_t o = static_cast<int64_t>(t) * p.k + li;
    const int phys = replica(p, t, c.e, count);
    p.topk_logical[o] = c.e;
    p.topk_weight[o] = static_cast<float>(s / sum * static_cast<double>(p.route_scale));
    p.topk_phys[o] = phys;
  }
}

// Router logits: x [T, H] times w [E, H]^T, fp32 sums.
//
// A workgroup owns TM*16 tokens and TN*16 experts; its KS wavefronts each multiply a slice of the hidden
// dimension on their own (no barrier) and the KS partial sums are added in wavefront order through LDS (a
// fixed order: the result is deterministic).  What bounds it is how fast one CU pulls its rows of x and w in
// out of L2, and, with few workgroups, the latency of doing so: the K split keeps KS * D * (TM + TN) * 2 KiB
// in flight, and the loads are in address order (eight lanes take a row's 128 bytes, 130 GB/s per CU, against
// 38 GB/s for loads in MFMA operand order), each wavefront turning its rows over to operand order in LDS of
// its own.  A lane's 16 LDS bytes are consecutive K-elements of its row.
//
// Against the kernels that stood here, us between events: bf16, H = 2048, E = 64, 37 tokens 12 -> 6, 4096 tokens
// 13 -> 10; fp32, H = 1024, E = 32, 1001 tokens 59 -> 7.
template <typename T> struct RouterMath;
template <> struct RouterMath<uint16_t> {
  static __device__ __forceinline__ f32x4 mac(u32x4 w, u32x4 x, f32x4 acc) {
    return mfma_16x16x32(w, x, acc);
  }
};
template <> struct RouterMath<float> {
  static __device__ __forceinline__ f32x4 mac(u32x4 w, u32x4 x, f32x4 acc) {
    const f32x4 a = __builtin_bit_cast(f32x4, w), b = __builtin_bit_cast(f32x4, x);
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], acc, 0, 0, 0);
    return acc;
  }
};

template <typename El, int TM, int TN, int KS, int D>
__global__ __launch_bounds__(64 * KS, 2) void router_kernel(const El* __restrict__ x, const El* __restrict__ w, float* __restrict__ logits,
                                                         int T, int E, int H, int n_tok, int n_exp) {
  constexpr int ROWS = (TM + TN) * 16, NL = ROWS / 8;  // rows of both operands, 16-byte loads per lane and step
  __shared__ __attribute__((aligned(16))) unsigned char lds[KS][ROWS * 128];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Workgroup i runs on XCD i % 8.  With at least eight token tiles a tile's workgroups share its rows of x in
  // one XCD's L2; with fewer the experts are dealt over the XCDs.
  int tok, ex;
  if (n_tok >= 8) {
    const int local = blockIdx.x >> 3;
    tok = local / n_exp * 8 + (blockIdx.x & 7);
    ex = local % n_exp;
  } else {
    tok = blockIdx.x / n_exp;
    ex = blockIdx.x % n_exp;
  }
  if (tok >= n_tok) return;
  const int t0 = tok * (TM * 16), e0 = ex * (TN * 16);
  const int64_t row_bytes = static_cast<int64_t>(H) * sizeof(El);
  const unsigned char* xb = reinterpret_cast<const unsigned char*>(x) + t0 * row_bytes;
  const unsigned char* wb = reinterpret_cast<const unsigned char*>(w) + e0 * row_bytes;
  const int steps = static_cast<int>((row_bytes + 127) >> 7);  // of 128 bytes of K
  const int s0 = steps * wave / KS, n = steps * (wave + 1) / KS - s0;
  const int c16 = (lane & 7) * 16;
  uint32_t off[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {  // rows past the last token or expert: the last one again, not stored
    const int r = i * 8 + (lane >> 3);
    off[i] = static_cast<uint32_t>((r < TM * 16 ? min(r, T - 1 - t0) : min(r - TM * 16, E - 1 - e0)) * row_bytes);
  }
  unsigned char* mine = lds[wave];
  u32x4 buf[D][NL];
  auto load = [&](int s, int d) {
    const int64_t k = min(static_cast<int64_t>(s0 + max(0, min(s, n - 1))) * 128 + c16, row_bytes - 16);
#pragma unroll
    for (int i = 0; i < NL; ++i) buf[d][i] = load_global_16B((i < TM * 2 ? xb : wb) + off[i] + k);
  };
  const int r16 = lane & 15, quad = lane >> 4;
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto mac = [&](int s, int d) {
    const bool in = static_cast<int64_t>(s0 + s) * 128 + c16 < row_bytes;  // K-elements past the last one count as zero
    const u32x4 zero = {0u, 0u, 0u, 0u};
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int r = i * 8 + (lane >> 3);
      *reinterpret_cast<u32x4*>(mine + r * 128 + (((lane & 7) ^ swz(r)) << 4)) = in ? buf[d][i] : zero;
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const unsigned char* p = mine + r16 * 128 + (((h * 4 + quad) ^ swz(r16)) << 4);  // swz has period 16
      u32x4 a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = *reinterpret_cast<const u32x4*>(p + i * (16 * 128));
#pragma unroll
      for (int j = 0; j < TN; ++j) b[j] = *reinterpret_cast<const u32x4*>(p + (TM + j) * (16 * 128));
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = RouterMath<El>::mac(b[j], a[i], acc[i][j]);
    }
  };
  // unconditional loads, so that the compiler's count of loads in flight stays exact
#pragma unroll
  for (int d = 0; d < D; ++d) load(d, d);
  int s = 0;
  for (; s + D < n; s += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      mac(s + d, d);
      load(s + D + d, d);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (s + d < n) mac(s + d, d);

  // partial sums into this wavefront's LDS as [token][expert], then all threads add them up
  static_assert(TM * TN * 16 * 16 * 4 <= ROWS * 128, "the partial sums fit the wavefront's rows");
  constexpr int NE = TN * 16;
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
      *reinterpret_cast<f32x4*>(mine + ((i * 16 + r16) * NE + j * 16 + quad * 4) * 4) = acc[i][j];
  __syncthreads();
  for (int i = threadIdx.x; i < TM * 16 * NE; i += 64 * KS) {
    float v = 0.f;
#pragma unroll
    for (int q = 0; q < KS; ++q) v += *reinterpret_cast<const float*>(lds[q] + i * 4);
    const int t = t0 + i / NE, e = e0 + i % NE;
    if (t < T && e < E) logits[static_cast<int64_t>(t) * E + e] = v;
  }
}

template <typename El, int TM, int TN, int KS, int D>
int launch_router(revive_ctx* ctx, const void* x, const void* w, float* logits, int T, hipStream_t stream) {
  const int E = ctx->cfg.E, n_tok = ceil_div(T, TM * 16), n_exp = ceil_div(E, TN * 16);
  const int grid = (n_tok >= 8 ? ceil_div(n_tok, 8) * 8 : n_tok) * n_exp;
  hipLaunchKernelGGL((router_kernel<El, TM, TN, KS, D>), dim3(grid), dim3(64 * KS), 0, stream, static_cast<const El*>(x),
                     static_cast<const El*>(w), logits, T, E, ctx->cfg.H, n_tok, n_exp);
  return check_hip(ctx, hipGetLastError(), "router launch");
}

// The larger tile once it gives every CU a workgroup: it reads x and w half as often.  us between events, bf16,
// 16 x 16 against 32 x 32 tiles: E = 64, H = 2048, 2000 tokens (126 workgroups of the larger tile) 8.5 and 8.8, 4096
// (256) 13.0 and 10.1; E = 128, H = 7168, 1000 tokens (128) 16.6 and 16.9, 2000 (252) 27.3 and 18.6, 4096 (512) 49
// and 29; E = 32, H = 4096, 4096 tokens (128) 11.8 and 13.2, 8192 (256) 18.7 and 18.9.  Both split K alike.
constexpr int kRouterSlices = 8;
template <typename El>
int router(revive_ctx* ctx, const void* x, const void* w, float* logits, int T, hipStream_t stream) {
  const int E = ctx->cfg.E;
  if (E > 16 && static_cast<int64_t>(ceil_div(T, 32)) * ceil_div(E, 32) >= 256)
    return launch_router<El, 2, 2, kRouterSlices, 2>(ctx, x, w, logits, T, stream);
  return launch_router<El, 1, 1, kRouterSlices, 4>(ctx, x, w, logits, T, stream);
}

template <int XR, int WR>
int router_sequence(revive_ctx* ctx, const void* x, const void* w, float* logits, int T, hipStream_t stream) {
  const int E = ctx->cfg.E, n_exp = ceil_div(E, WR);
  hipLaunchKernelGGL((router_sequence_kernel<XR, WR, 2>), dim3(ceil_div(T, XR) * n_exp), dim3(512), 0, stream,
                     static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(w), logits, T, E, ctx->cfg.H, n_exp);
  return check_hip(ctx, hipGetLastError(), "router_sequence launch");
}

template <int BM, int BN, int WM, int WN, int BK, int S, int SLICES = 1>
int router_tile(revive_ctx* ctx, const void* x, const void* w, float* logits, int T, hipStream_t stream) {
  constexpr size_t lds = static_cast<size_t>(S) * (BM + BN) * BK * 2;
  auto kern = router_tile_kernel<BM, BN, WM, WN, BK, S, SLICES>;
  REVIVE_HIP(ctx, allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds));
  const int E = ctx->cfg.E, n_tok = ceil_div(T, BM), n_exp = ceil_div(E, BN);
  hipLaunchKernelGGL(kern, dim3(ceil_div(n_tok, 8) * 8 * n_exp), dim3(64 * WM * WN), lds, stream, static_cast<const uint16_t*>(x),
                     static_cast<const uint16_t*>(w), logits, T, E, ctx->cfg.H, n_tok, n_exp);
  return check_hip(ctx, hipGetLastError(), "router_tile launch");
}

// K in one sequence.
int router_one_sequence(revive_ctx* ctx, const void* x, const void* w, float* logits, int T, hipStream_t stream) {
  switch (router_form(T, ctx->cfg.E, ctx->cfg.H)) {
    case kSeq8x8: return router_sequence<8, 8>(ctx, x, w, logits, T, stream);
    case kSeq16x16: return router_sequence<16, 16>(ctx, x, w, logits, T, stream);
    case k32x32x64s2: return router_tile<32, 32, 2, 2, 64, 2>(ctx, x, w, logits, T, stream);
    case k128x64x64s2: return router_tile<128, 64, 4, 2, 64, 2>(ctx, x, w, logits, T, stream);
    case k128x64x64s3: return router_tile<128, 64, 4, 2, 64, 3>(ctx, x, w, logits, T, stream);
    case k32x32x128s4: return router_tile<32, 32, 2, 2, 128, 4>(ctx, x, w, logits, T, stream);
    case k32x64x128s4: return router_tile<32, 64, 2, 2, 128, 4>(ctx, x, w, logits, T, stream);
    case k64x64x128s4: return router_tile<64, 64, 4, 2, 128, 4>(ctx, x, w, logits, T, stream);
    case k64x128x64s3: return router_tile<64, 128, 2, 4, 64, 3>(ctx, x, w, logits, T, stream);
    case k128x128x64s4: return router_tile<128, 128, 2, 4, 64, 4>(ctx, x, w, logits, T, stream);
    case k128x192x64s3: return router_tile<128, 192, 2, 4, 64, 3>(ctx, x, w, logits, T, stream);
    case k128x256x64s3: return router_tile<128, 256, 2, 4, 64, 3>(ctx, x, w, logits, T, stream);
  }
  return fail(ctx, REVIVE_EINVAL, "router: no kernel");
}

// Many tokens in fp32, K in the router kernel's slices.  The number of experts is a multiple of 4.
int router_gemm_f32(revive_ctx* ctx, const void* x, const void* w, float* logits, int T, hipStream_t stream) {
  const revive_config& c = ctx->cfg;
  GemmF32Problem p{};
  p.A = static_cast<const float*>(x); p.lda = c.H;
  p.B_one = static_cast<const float*>(w); p.ldb = c.H;
  p.C = logits; p.ldc = c.E;
  p.n_out = c.E; p.K = c.H;
  p.n_col_tiles = ceil_div(c.E, kTileN_f32);
  p.blocks = ceil_div(T, kTileM_f32) * p.n_col_tiles;
  p.M = T;
  return launch_gemm_f32<kRouterSlices>(ctx, p, stream);
}

}  // namespace

int launch_router_gemm(revive_ctx* ctx, const void* x, const void* w, float* logits, int T, hipStream_t stream) {
  const revive_config& c = ctx->cfg;
  KernelTimer timer(ctx, REVIVE_K_ROUTER_GEMM, stream);
  if (c.dtype != REVIVE_DTYPE_BF16) {
    // Beyond one or two rounds of the router kernel's workgroups the GEMM's larger tiles win, later for a longer K, which
    // its one workgroup per tile walks alone.  us between events, router kernel and GEMM: 512 experts, H = 128, 8192
    // tokens 58 and 20; 64 experts, H = 128 (the line: 512 workgroups), 4096 tokens (256) 8.2 and 10.0, 8192 (512) 11.1
    // and 9.6; 192 experts, H = 256 (768), 2048 tokens (384) 11.1 and 13.2, 4096 (768) 15.8 and 14.1; 192 experts,
    // H = 1536 (2048), 8192 tokens (1536) 69 and 73, 16 384 (3072) 137 and 109.
    const int64_t workgroups = static_cast<int64_t>(ceil_div(T, 32)) * ceil_div(c.E, 32);
    if (c.E % 4 == 0 && workgroups >= 256 + c.H + std::min(c.H, 256)) return router_gemm_f32(ctx, x, w, logits, T, stream);
    return router<float>(ctx, x, w, logits, T, stream);
  }
  // The order in which K is summed follows from E and H alone, so that a token's logits do not depend on how many
  // others are in the call.  Small routers: K in slices.
  if (c.E <= 128 && c.H % 256 == 0) {
    switch (router_sliced_form(T, c.E, c.H)) {
      case kSlicedRouter: return router<uint16_t>(ctx, x, w, logits, T, stream);
      case kSliced128x64s4: return router_tile<128, 64, 4, 2, 64, 4, kRouterSlices>(ctx, x, w, logits, T, stream);
      case kSliced128x64s3: return router_tile<128, 64, 4, 2, 64, 3, kRouterSlices>(ctx, x, w, logits, T, stream);
      case kSliced128x128s4: return router_tile<128, 128, 2, 4, 64, 4, kRouterSlices>(ctx, x, w, logits, T, stream);
    }
  }
  // Many experts, or an odd K: K is summed in one sequence.  A K split is faster for a middling number of tokens (1003
  // tokens, E = 256, H = 7168: 19 us) but another order moves one of 8192 x 256 logits across a near tie in every few
  // calls.  (The small routers' sums are three times nearer the exact ones.)
  return router_one_sequence(ctx, x, w, logits, T, stream);
}

int launch_route_topk(revive_ctx* ctx, const float* logits, int T, int32_t* topk_logical, float* topk_weight,
                      int32_t* topk_phys, hipStream_t stream) {
  const revive_config& c = ctx->cfg;
  RouteParams p{};
  p.logits = logits;
  p.l2p_count = ctx->d_l2p_count();
  p.l2p_table = ctx->d_l2p_table();
  p.topk_logical = topk_logical;
  p.topk_weight = topk_weight;
  p.topk_phys = topk_phys;
  p.T = T; p.E = c.E; p.k = c.k; p.max_replicas = c.max_replicas;
  p.score_fn = c.score_fn; p.n_group = c.n_group; p.topk_group = c.topk_group;
  p.route_scale = c.route_scale;
  p.t_offset = ctx->token_offset;
  const int vals = ceil_div(c.E, 64), held = vals <= 2 ? vals : vals <= 4 ? 4 : vals <= 6 ? 6 : 8;  // experts per lane of route_topk_kernel
  p.none = c.E == held * 64 ? 0 : c.E - 1;
  KernelTimer timer(ctx, REVIVE_K_ROUTE_TOPK, stream);
  if (selects_by_rows(T, c.E, c.n_group, c.k)) {
    const int n = ceil_div(c.E, 16);
    const dim3 grid(ceil_div(T, 16)), block(256);
    const bool wide = c.E % 64 == 0;
#define REVIVE_ROUTE_LAUNCH(V)                                                                                                      \
  do {                                                                                                                              \
    if (c.n_group > 1 && wide) hipLaunchKernelGGL((route_topk_rows_kernel<V, true, true>), grid, block, 0, stream, p);              \
    else if (c.n_group > 1) hipLaunchKernelGGL((route_topk_rows_kernel<V, true, false>), grid, block, 0, stream, p);                \
    else if (wide) hipLaunchKernelGGL((route_topk_rows_kernel<V, false, true>), grid, block, 0, stream, p);                         \
    else hipLaunchKernelGGL((route_topk_rows_kernel<V, false, false>), grid, block, 0, stream, p);                                  \
  } while (0)
    if (n <= 4) REVIVE_ROUTE_LAUNCH(4);
    else if (n <= 8) REVIVE_ROUTE_LAUNCH(8);
    else if (n <= 16) REVIVE_ROUTE_LAUNCH(16);
    else if (n <= 24) REVIVE_ROUTE_LAUNCH(24);
    else REVIVE_ROUTE_LAUNCH(32);
#undef REVIVE_ROUTE_LAUNCH
    return check_hip(ctx, hipGetLastError(), "route_topk launch");
  }
  // Few tokens, other groups, more choices.
  const bool four = selects_four_tokens(T, c.n_group, c.k);
  const dim3 grid(ceil_div(T, four ? 16 : 4)), block(256);
#define REVIVE_ROUTE_LAUNCH(V)                                                                                       \
  do {                                                                                                               \
    if (four) hipLaunchKernelGGL((route_topk_kernel<V, 4, true>), grid, block, 0, stream, p);                        \
    else if (c.n_group > 1) hipLaunchKernelGGL((route_topk_kernel<V, 1, true>), grid, block, 0, stream, p);          \
    else hipLaunchKernelGGL((route_topk_kernel<V, 1, false>), grid, block, 0, stream, p);                            \
  } while (0)
  if (held == 1) REVIVE_ROUTE_LAUNCH(1);
  else if (held == 2) REVIVE_ROUTE_LAUNCH(2);
  else if (held == 4) REVIVE_ROUTE_LAUNCH(4);
  else if (held == 6) REVIVE_ROUTE_LAUNCH(6);
  else REVIVE_ROUTE_LAUNCH(8);
#undef REVIVE_ROUTE_LAUNCH
  return check_hip(ctx, hipGetLastError(), "route_topk launch");
}

}  // namespace revive
