// What ends a graph step after its solve: the sum of the edge costs and the update of the poses, used by launches of their
// own and by the launch that ends a plain step.
#pragma once

#include "common.hpp"
#include "internal.hpp"
#include "sim3.hpp"

namespace ds3 {

// Deterministic sum of per-edge costs and counts over one block of 256 threads (fixed strided split + fixed
// tree); thread 0 writes them. With ctr, the sum and *status are also appended to a history (slot *ctr,
// then ctr advances; slots past hist_len are dropped).
__device__ inline void sum_costs_block(const double* __restrict__ cost_e, const int64_t* __restrict__ count_e,
                                       int n_edges, double* __restrict__ cost_out, int64_t* __restrict__ count_out,
                                       const int32_t* __restrict__ status, unsigned* __restrict__ ctr,
                                       double* __restrict__ cost_hist, int32_t* __restrict__ status_hist,
                                       int hist_len) {
  __shared__ double sc[256];
  __shared__ long long sn[256];
  double c = 0.0;
  long long m = 0;
  for (int e = threadIdx.x; e < n_edges; e += 256) {
    c += cost_e[e];
    m += count_e[e];
  }
  sc[threadIdx.x] = c;
  sn[threadIdx.x] = m;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w) {
      sc[threadIdx.x] += sc[threadIdx.x + w];
      sn[threadIdx.x] += sn[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    if (cost_out) *cost_out = sc[0];
    if (count_out) *count_out = sn[0];
    if (ctr) {
      const unsigned k = *ctr;
      if (k < unsigned(hist_len)) {
        cost_hist[k] = sc[0];
        status_hist[k] = *status;
      }
      *ctr = k + 1;
    }
  }
}

// Over a grid of at least two blocks of 256 threads: the last block sums the costs, the others apply T <- Exp(tau) T
// (Sec. III-D), fixed poses untouched.
__device__ inline void step_tail(const StepTail& t) {
  if (blockIdx.x == gridDim.x - 1) {
    sum_costs_block(t.cost_e, t.count_e, t.n_edges, t.cost_out, nullptr, nullptr, nullptr, nullptr, nullptr, 0);
    return;
  }
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < t.n_kf; k += (gridDim.x - 1) * blockDim.x) {
    if (t.fixed && t.fixed[k]) continue;
    Sim3 E = sim3_exp(t.tau + 7 * int64_t(k));
    Sim3 T = sim3_load(t.poses + 8 * int64_t(k));
    sim3_store(sim3_mul(E, T), t.poses + 8 * int64_t(k));
  }
}

}  // namespace ds3
