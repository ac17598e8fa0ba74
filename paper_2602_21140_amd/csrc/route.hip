// Gate of the failure-remapped MoE layer: router logits, failure-masked (group-limited) top-k,
// renormalised weights and the logical->physical replica remap.
//
// Paper: Sec. 2.1 (gating scores, top-k), Sec. 3.4 "Missing experts" and Sec. 4.2 (experts with
// no replica left are masked to -inf immediately before the top-k), Sec. 3.4 "Redundant experts"
// (the logical-to-physical map decides which replica serves a token).
#include "gemm_bf16.hpp"

namespace revive {

namespace {

// Ordering of candidates: larger key first, equal keys by lower expert id.
__device__ __forceinline__ bool better(float ka, int ea, float kb, int eb) { return ka > kb || (ka == kb && ea < eb); }

struct RouteParams {
  const float* logits;
  const int32_t* l2p_count;
  const int32_t* l2p_table;
  int32_t* topk_logical;
  float* topk_weight;
  int32_t* topk_phys;
  int T, E, k, max_replicas, score_fn, n_group, topk_group;
  long long t_offset;  // index of token 0 within the whole batch
  float route_scale;
};

// One wavefront per token.  Lane l holds the logits of experts l, l+64, l+128, ... (VALS of them);
// a masked or excluded expert's key is -inf.  Expert order is decided on the fp32 logits
// themselves (softmax and sigmoid are increasing, so this is the order of the scores); group
// scores, which add two scores, and the output weights are evaluated in fp64.
// GROUPED variants hold the group scores in registers (n_group <= 8 or <= 32).
template <int VALS, int MAXG>
__global__ __launch_bounds__(256) void route_topk_kernel(RouteParams p) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= p.T) return;  // whole wavefront leaves together
  const float NEG = -__builtin_inff();

  float key[VALS];
  const float* row = p.logits + static_cast<int64_t>(t) * p.E;
  float vmax = NEG;  // largest live logit of the row: common shift of the exponentials (the best chosen score is exactly 1)
#pragma unroll
  for (int i = 0; i < VALS; ++i) {
    const int e = lane + 64 * i;
    float z = NEG;
    if (e < p.E) {
      z = row[e];
      if (p.l2p_count[e] <= 0) z = NEG;  // failure mask
      vmax = fmaxf(vmax, z);
    }
    key[i] = z;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) vmax = fmaxf(vmax, __shfl_xor(vmax, o));
  const double shift = static_cast<double>(vmax);

  auto score64 = [&](float z) -> double {  // unnormalised gating score of a live expert
    const double zd = static_cast<double>(z);
    return p.score_fn == REVIVE_SCORE_SIGMOID ? 1.0 / (1.0 + exp(-zd)) : exp(zd - shift);
  };

  if (MAXG > 1) {
    // Group score = sum of the two best live scores of the group (one if only one is live, -inf
    // if none).  A wave-wide top-2 per group finds the two logits; lane g then evaluates group
    // g's score in fp64 and every lane ranks it against the others through shuffles.
    const int gsz = p.E / p.n_group;
    float top1 = NEG, top2 = NEG;  // lane g keeps group g's two best keys
#pragma unroll 1
    for (int g = 0; g < p.n_group; ++g) {
      float m1 = NEG, m2 = NEG;
#pragma unroll
      for (int i = 0; i < VALS; ++i) {
        const int e = lane + 64 * i;
        const float z = (e < p.E && e / gsz == g) ? key[i] : NEG;
        if (z > m1) { m2 = m1; m1 = z; } else if (z > m2) { m2 = z; }
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const float o1 = __shfl_xor(m1, o), o2 = __shfl_xor(m2, o);
        const float hi = fmaxf(m1, o1);
        const float lo = fmaxf(fminf(m1, o1), fmaxf(m2, o2));
        m1 = hi;
        m2 = lo;
      }
      if (lane == g) { top1 = m1; top2 = m2; }
    }
    double gs = -__builtin_inf();
    if (lane < p.n_group && top1 > NEG) {
      gs = score64(top1);
      if (top2 > NEG) gs += score64(top2);
    }
    // rank of my group among all groups (better score first, ties to the lower group id)
    int rank = 0;
#pragma unroll
    for (int h = 0; h < MAXG; ++h) {
      const double o = __shfl(gs, h);
      if (h < p.n_group) rank += (o > gs) || (o == gs && h < lane);
    }
    const unsigned long long kept = __ballot(lane < p.n_group && rank < p.topk_group);
#pragma unroll
    for (int i = 0; i < VALS; ++i) {
      const int e = lane + 64 * i;
      if (e < p.E && !((kept >> (e / gsz)) & 1ull)) key[i] = NEG;  // expert of a dropped group
    }
  }

  // k rounds of wave-wide arg-max; the winner of round j lands in lane j.
  int my_e = -1;
  float my_z = 0.f;
  for (int j = 0; j < p.k; ++j) {
    float bk = NEG;
    int be = 0x7fffffff;
#pragma unroll
    for (int i = 0; i < VALS; ++i) {
      const int e = lane + 64 * i;
      if (e < p.E && better(key[i], e, bk, be)) { bk = key[i]; be = e; }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const float ok = __shfl_xor(bk, o);
      const int oe = __shfl_xor(be, o);
      if (better(ok, oe, bk, be)) { bk = ok; be = oe; }
    }
    if ((be & 63) == lane) {
#pragma unroll
      for (int i = 0; i < VALS; ++i)
        if (i == (be >> 6)) key[i] = NEG;
    }
    if (lane == j) { my_e = be; my_z = bk; }
  }

  // weights: score of the chosen expert over the sum of the chosen scores
  double s = (lane < p.k) ? score64(my_z) : 0.0;
  double sum = s;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  if (lane < p.k) {
    const int64_t o = static_cast<int64_t>(t) * p.k + lane;
    const int c = p.l2p_count[my_e];
    p.topk_logical[o] = my_e;
    p.topk_weight[o] = static_cast<float>(s / sum * static_cast<double>(p.route_scale));
    // replica of this token: the (batch index of t mod count)-th surviving slot, ascending slot id
    p.topk_phys[o] = c > 0 ? p.l2p_table[my_e * p.max_replicas + static_cast<int>((p.t_offset + t) % c)] : -1;
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
// Against the kernels that stood here (us): bf16, H = 7168, E = 256, T = 1: 53 -> 10, 192: 53 -> 11, 1003:
// 55 -> 19, 4096: 59 -> 40; H = 2048, E = 64, T = 37: 12 -> 6, 4096: 13 -> 10; fp32, H = 1024, E = 32, T = 1001:
// 59 -> 7.  The shorter sums are also nearer the exact ones (H = 7168: 5.3e-7 -> 1.8e-7).
template <typename T> struct RouterMath;
template <> struct RouterMath<uint16_t> {
  static __device__ __forceinline__ f32x4 mac(u32x4 w, u32x4 x, f32x4 acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), acc, 0, 0, 0);
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

// The largest tile that still gives every CU a workgroup: larger tiles read x and w fewer times.  us, all
// sizes of tile tried: T = 512, E = 256, H = 7168: 17 (16 x 16), 17 (32 x 32); T = 1003: 28, 19; T = 2000:
// 49, 29, 37 (64 x 64); T = 4096: 95, 52, 40.
template <typename El>
int router(revive_ctx* ctx, const void* x, const void* w, float* logits, int T, hipStream_t stream) {
  const int E = ctx->cfg.E;
  auto blocks = [&](int m, int n) { return static_cast<int64_t>(ceil_div(T, m)) * ceil_div(E, n); };
  if (E > 32 && blocks(64, 64) >= 256) return launch_router<El, 4, 4, 4, 2>(ctx, x, w, logits, T, stream);
  if (E > 16 && blocks(32, 32) >= 256) return launch_router<El, 2, 2, 8, 2>(ctx, x, w, logits, T, stream);
  return launch_router<El, 1, 1, 8, 4>(ctx, x, w, logits, T, stream);
}

}  // namespace

int launch_router_gemm(revive_ctx* ctx, const void* x, const void* w, float* logits, int T, hipStream_t stream) {
  const revive_config& c = ctx->cfg;
  KernelTimer timer(ctx, REVIVE_K_ROUTER_GEMM, stream);
  if (c.dtype != REVIVE_DTYPE_BF16) return router<float>(ctx, x, w, logits, T, stream);
  const int64_t wide = static_cast<int64_t>(ceil_div(T, 128)) * ceil_div(c.E, 128);
  if (wide >= 512) {
    // 128 x 128 tiles fill the chip twice over and read x and w half as often (T = 32768, E = 384: 267 us
    // against 380; T = 8192, E = 256, 128 tiles: 64 against 64)
    GemmArgs a{};
    a.A = x; a.lda = c.H;
    a.B_one = w; a.ldb = c.H;
    a.C = logits; a.ldc = c.E;
    a.n_out = c.E; a.K = c.H;
    a.M = T;
    a.n_col_tiles = ceil_div(c.E, 128);
    return launch_gemm_bf16<128, 128, 2, 2, EPI_F32, REVIVE_K_ROUTER_GEMM>(ctx, a, ceil_div(T, 128), stream);
  }
  return router<uint16_t>(ctx, x, w, logits, T, stream);
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
  KernelTimer timer(ctx, REVIVE_K_ROUTE_TOPK, stream);
  const dim3 grid(ceil_div(T, 4)), block(256);
  const int vals = ceil_div(c.E, 64);
#define REVIVE_ROUTE_LAUNCH(V)                                                                               \
  do {                                                                                                       \
    if (c.n_group <= 1) hipLaunchKernelGGL((route_topk_kernel<V, 1>), grid, block, 0, stream, p);            \
    else if (c.n_group <= 8) hipLaunchKernelGGL((route_topk_kernel<V, 8>), grid, block, 0, stream, p);       \
    else hipLaunchKernelGGL((route_topk_kernel<V, 32>), grid, block, 0, stream, p);                          \
  } while (0)
  if (vals <= 1) REVIVE_ROUTE_LAUNCH(1);
  else if (vals <= 2) REVIVE_ROUTE_LAUNCH(2);
  else if (vals <= 4) REVIVE_ROUTE_LAUNCH(4);
  else if (vals <= 6) REVIVE_ROUTE_LAUNCH(6);
  else REVIVE_ROUTE_LAUNCH(8);
#undef REVIVE_ROUTE_LAUNCH
  return check_hip(ctx, hipGetLastError(), "route_topk launch");
}

}  // namespace revive
