// Activation counting for the lost-expert study (paper Sec. 4.2: experts are ranked by how
// often they are activated, per layer and aggregated, to choose which ones to fail).
#include <algorithm>

#include "ctx.hpp"

namespace revive {

namespace {

// Per-workgroup LDS histogram of the selected expert ids, then one 64-bit atomic add per expert
// and workgroup.  Integer addition: the result does not depend on the order of the adds.
// Bound by the latency of the loads, which go out together, and by the adds of all workgroups to the same words.  us,
// 65 536 ids of 256 experts and 262 144: 1024 ids of a workgroup, one load after the other 3.6 and 7.7, together 3.4 and
// 7.4, 512 4.6 and 12.8, 2048 2.9 and 4.9, 4096 3.0 and 4.0; but 16 800 ids 2.7, 2.4, 2.6, 2.5 and 2.9.
constexpr int kIds = 2048;  // ids of a workgroup at a time
__global__ __launch_bounds__(256) void expert_counts_kernel(const int32_t* __restrict__ topk_logical, int n, int E,
                                                            unsigned long long* __restrict__ counts) {
  __shared__ int hist[kMaxE];
  for (int e = threadIdx.x; e < E; e += 256) hist[e] = 0;
  __syncthreads();
  for (int i = blockIdx.x * kIds + threadIdx.x; i < n; i += gridDim.x * kIds) {
    int e[kIds / 256];  // the loads go out together
#pragma unroll
    for (int j = 0; j < kIds / 256; ++j) e[j] = i + j * 256 < n ? topk_logical[i + j * 256] : -1;
#pragma unroll
    for (int j = 0; j < kIds / 256; ++j)
      if (e[j] >= 0 && e[j] < E) atomicAdd(&hist[e[j]], 1);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < E; e += 256)
    if (hist[e]) atomicAdd(&counts[e], static_cast<unsigned long long>(hist[e]));
}

}  // namespace

int launch_expert_counts(revive_ctx* ctx, const int32_t* topk_logical, int T, int64_t* counts, hipStream_t stream) {
  const int n = T * ctx->cfg.k;
  const int grid = std::min(1024, ceil_div(n, kIds));
  KernelTimer timer(ctx, REVIVE_K_EXPERT_COUNTS, stream);
  hipLaunchKernelGGL(expert_counts_kernel, dim3(std::max(1, grid)), dim3(256), 0, stream, topk_logical, n, ctx->cfg.E,
                     reinterpret_cast<unsigned long long*>(counts));
  return check_hip(ctx, hipGetLastError(), "expert_counts launch");
}

}  // namespace revive
