// Internal: the flip bookkeeping of one sequence (Section 4.3.4), shared by lsp_flip_update and lsp_commit_step.
#pragma once
#include "lsp_common.h"

namespace lsp {

struct FlipArgs {
  const int32_t *base_prefix_len;
  int32_t *last_id;
  unsigned long long *counters;
  int G, window_lo, window_hi;
  int32_t *step_counts;
};

// One workgroup per sequence; a position counts
// when it already had a prediction at the previous step.  The sequence's counts
// also go to the mid-generation window when the number of its positions already
// committed lies in [window_lo, window_hi].  P, N: the sequence's lengths before this step's commit.
// THREADS: of the workgroup (asked of the hardware, it would be an implicit argument, and 256 bytes more to fetch).
template <int THREADS>
__device__ __forceinline__ void count_flips(const FlipArgs &f, int b, const int32_t *__restrict__ top1_id, int S, int P, int N) {
  __shared__ int total[2];
  const int done = P - f.base_prefix_len[b];
  if (threadIdx.x < 2) total[threadIdx.x] = 0;
  __syncthreads();
  int flips = 0, seen = 0;
  for (int u = threadIdx.x; u < N; u += THREADS) {
    const int j = done + u;
    if (j < 0 || j >= f.G) continue;
    const int32_t cur = top1_id[int64_t(b) * S + u];
    const int32_t old = f.last_id[int64_t(b) * f.G + j];
    if (old >= 0) {
      ++seen;
      flips += (old != cur);
    }
    f.last_id[int64_t(b) * f.G + j] = cur;
  }
#pragma unroll
  for (int m = 1; m < kWave; m <<= 1) {
    flips += __shfl_xor(flips, m);
    seen += __shfl_xor(seen, m);
  }
  if ((threadIdx.x & (kWave - 1)) == 0 && seen > 0) {
    atomicAdd(&total[0], flips);
    atomicAdd(&total[1], seen);
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  if (f.step_counts != nullptr) {
    f.step_counts[2 * b] = total[0];
    f.step_counts[2 * b + 1] = total[1];
  }
  if (total[1] > 0) {
    atomicAdd(&f.counters[0], (unsigned long long)total[0]);
    atomicAdd(&f.counters[1], (unsigned long long)total[1]);
    if (done >= f.window_lo && done <= f.window_hi) {
      atomicAdd(&f.counters[2], (unsigned long long)total[0]);
      atomicAdd(&f.counters[3], (unsigned long long)total[1]);
    }
  }
}

}  // namespace lsp
