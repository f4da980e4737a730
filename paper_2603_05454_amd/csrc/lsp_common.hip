// Library-wide pieces of liblsp: error text, version, flip bookkeeping.
#include <limits.h>
#include <stdarg.h>

#include "lsp_flips.h"

namespace lsp {

static thread_local char g_error[512] = "";

void set_error(const char *fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_error, sizeof(g_error), fmt, ap);
  va_end(ap);
}

namespace {

constexpr int kFlipThreads = 256;
__global__ __launch_bounds__(kFlipThreads) void flip_kernel(FlipArgs f, const int32_t *__restrict__ top1_id, int S,
                                                   const int32_t *__restrict__ prefix_len,
                                                   const int32_t *__restrict__ suffix_len) {
  const int b = blockIdx.x;
  count_flips<kFlipThreads>(f, b, top1_id, S, prefix_len[b], min(max(suffix_len[b], 0), S));
}

// What a decode loop asks between two steps, in one launch and written straight to host memory: the host reads the flag
// without a copy or a synchronisation behind it.  (As seven small torch operations and a transfer it stood 60-80 us
// between a step's append and the next step's attention; now about 20.)
constexpr int kPollThreads = 256;
__global__ __launch_bounds__(kPollThreads) void poll_kernel(const int32_t *__restrict__ suffix_len,
                                                   const int32_t *__restrict__ commit_len, int B, int32_t *host) {
  __shared__ int s_left, s_stalled;
  if (threadIdx.x == 0) {
    s_left = INT_MIN;
    s_stalled = 0;
  }
  __syncthreads();
  int left = INT_MIN;
  bool stalled = false;
  for (int b = threadIdx.x; b < B; b += kPollThreads) {
    const int n = suffix_len[b];
    left = max(left, n);
    stalled |= commit_len != nullptr && n > 0 && commit_len[b] == 0;
  }
  atomicMax(&s_left, left);
  if (stalled) s_stalled = 1;
  __syncthreads();
  if (threadIdx.x != 0) return;
  __hip_atomic_store(host, s_left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __hip_atomic_store(host + 1, s_stalled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __hip_atomic_store(host + 2, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The same for a host that has other things to do meanwhile: one wave, no barrier, and every word in one store with the call's
// number beside it, where values and a flag after them were two trips to host memory.
constexpr int kProgressWords = 12;
__global__ __launch_bounds__(kWave) void progress_kernel(const int32_t *__restrict__ suffix_len, const int32_t *__restrict__ commit_len,
                                                         const int32_t *__restrict__ prefix_len, const int32_t *__restrict__ base,
                                                         const uint32_t *__restrict__ counters, int B, uint32_t call, uint64_t *host) {
  const int lane = threadIdx.x;
  const uint32_t count = lane >= 4 && lane < kProgressWords ? counters[lane - 4] : 0;
  int left = INT_MIN, stalled = 0;
  int64_t committed = 0;
  for (int b = lane; b < B; b += kWave) {
    const int n = suffix_len[b];
    left = max(left, n);
    stalled |= commit_len != nullptr && n > 0 && commit_len[b] == 0;
    committed += prefix_len[b] - base[b];
  }
#pragma unroll
  for (int m = 1; m < kWave; m <<= 1) {
    left = max(left, __shfl_xor(left, m));
    stalled |= __shfl_xor(stalled, m);
    committed += __shfl_xor(committed, m);
  }
  const uint32_t word = lane == 0 ? uint32_t(left) : lane == 1 ? uint32_t(stalled) : lane == 2 ? uint32_t(committed) : lane == 3 ? uint32_t(uint64_t(committed) >> 32) : count;
  if (lane < kProgressWords) __hip_atomic_store(host + lane, uint64_t(call) << 32 | word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Measurement helper: a bare streaming read.  Workgroup w reads segment w of the buffer
// with 16-byte non-temporal loads, four in flight per lane, and folds them with XOR; one
// word per workgroup is written.  This is the floor under any kernel that has to read a
// buffer of that size once (launch, first loads, drain included).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(512) void read_kernel(const u32x4 *__restrict__ p, int64_t vec_per_wg,
                                                   uint32_t *__restrict__ out) {
  const u32x4 *q = p + int64_t(blockIdx.x) * vec_per_wg;
  u32x4 acc = {0, 0, 0, 0};
  int64_t i = threadIdx.x;
  for (; i + 3 * 512 < vec_per_wg; i += 4 * 512) {
    const u32x4 a = __builtin_nontemporal_load(q + i), b = __builtin_nontemporal_load(q + i + 512);
    const u32x4 c = __builtin_nontemporal_load(q + i + 1024), d = __builtin_nontemporal_load(q + i + 1536);
    acc ^= a ^ b ^ c ^ d;
  }
  for (; i < vec_per_wg; i += 512) acc ^= __builtin_nontemporal_load(q + i);
  uint32_t v = acc.x ^ acc.y ^ acc.z ^ acc.w;
#pragma unroll
  for (int m = 1; m < kWave; m <<= 1) v ^= __shfl_xor(v, m);
  if ((threadIdx.x & (kWave - 1)) == 0) atomicXor(&out[blockIdx.x], v);
}

// Measurement helper: a bare matrix-instruction loop (no memory traffic inside the loop).
// Every lane loads 8 A and 8 B fragments (16 bytes each) once, then issues
// v_mfma_f32_32x32x16_bf16 over them round robin into four accumulators.  What it sustains
// depends on the operand VALUES: with random operands the chip lowers its clock to stay inside
// its power limit, so this is the matrix ceiling a kernel working on such data can be held to.
typedef float f32x16 __attribute__((ext_vector_type(16)));
__global__ __launch_bounds__(512) void mfma_kernel(const u32x4 *__restrict__ operands, int32_t iters,
                                                   float *__restrict__ out) {
  u32x4 A[8], B[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    A[s] = operands[s * 512 + threadIdx.x];
    B[s] = operands[(8 + s) * 512 + threadIdx.x];
  }
  f32x16 acc[4];
#pragma unroll
  for (int n = 0; n < 4; ++n)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[n][r] = 0.f;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int s = 0; s < 8; ++s)
      asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc[s & 3]) : "v"(A[s]), "v"(B[(s * 3 + 1) & 7]));
  }
  float t = 0.f;
#pragma unroll
  for (int n = 0; n < 4; ++n)
#pragma unroll
    for (int r = 0; r < 16; ++r) t += acc[n][r];
  out[blockIdx.x * 512 + threadIdx.x] = t;
}

}  // namespace
}  // namespace lsp

extern "C" int32_t lsp_bench_mfma(const void *operands, int32_t iters, int32_t workgroups, float *out, void *stream) {
  using namespace lsp;
  LSP_CHECK_ARG(operands && out && iters > 0 && workgroups > 0, "lsp_bench_mfma: bad argument");
  LSP_CHECK_ARG(aligned16(operands), "lsp_bench_mfma: operands must be 16-byte aligned");
  mfma_kernel<<<workgroups, 512, 0, static_cast<hipStream_t>(stream)>>>(static_cast<const u32x4 *>(operands), iters, out);
  LSP_CHECK_LAUNCH("lsp_bench_mfma: launch");
  return LSP_OK;
}

extern "C" int32_t lsp_bench_read(const void *buffer, int64_t bytes, int32_t workgroups, uint32_t *out, void *stream) {
  using namespace lsp;
  LSP_CHECK_ARG(buffer && out && bytes > 0 && workgroups > 0, "lsp_bench_read: bad argument");
  LSP_CHECK_ARG(aligned16(buffer) && bytes % (int64_t(workgroups) * 16) == 0,
                "lsp_bench_read: buffer must be 16-byte aligned and split evenly into 16-byte vectors per workgroup");
  read_kernel<<<workgroups, 512, 0, static_cast<hipStream_t>(stream)>>>(static_cast<const u32x4 *>(buffer),
                                                                         bytes / (int64_t(workgroups) * 16), out);
  LSP_CHECK_LAUNCH("lsp_bench_read: launch");
  return LSP_OK;
}

extern "C" int32_t lsp_poll_lengths(const int32_t *suffix_len, const int32_t *commit_len, int32_t B, int32_t *host, void *stream) {
  using namespace lsp;
  LSP_CHECK_ARG(suffix_len && host && B > 0, "lsp_poll_lengths: bad argument");
  poll_kernel<<<1, kPollThreads, 0, static_cast<hipStream_t>(stream)>>>(suffix_len, commit_len, B, host);
  LSP_CHECK_LAUNCH("lsp_poll_lengths: launch");
  return LSP_OK;
}

extern "C" int32_t lsp_poll_progress(const int32_t *suffix_len, const int32_t *commit_len, const int32_t *prefix_len,
                                     const int32_t *base_prefix_len, const int64_t *counters, int32_t B, uint32_t call,
                                     uint64_t *host, void *stream) {
  using namespace lsp;
  LSP_CHECK_ARG(suffix_len && prefix_len && base_prefix_len && counters && host && B > 0, "lsp_poll_progress: bad argument");
  progress_kernel<<<1, kWave, 0, static_cast<hipStream_t>(stream)>>>(suffix_len, commit_len, prefix_len, base_prefix_len,
                                                                     reinterpret_cast<const uint32_t *>(counters), B, call, host);
  LSP_CHECK_LAUNCH("lsp_poll_progress: launch");
  return LSP_OK;
}

extern "C" const char *lsp_version(void) { return "liblsp 0.1 (gfx950)"; }
extern "C" const char *lsp_last_error(void) { return lsp::g_error; }

extern "C" int32_t lsp_flip_update(const int32_t *top1_id, int32_t B, int32_t S, int32_t G,
                                   const int32_t *prefix_len, const int32_t *suffix_len,
                                   const int32_t *base_prefix_len, int32_t *last_id,
                                   int64_t *counters, int32_t window_lo, int32_t window_hi,
                                   int32_t *step_counts, void *stream) {
  using namespace lsp;
  LSP_CHECK_ARG(top1_id && prefix_len && suffix_len && base_prefix_len && last_id && counters,
                "lsp_flip_update: null pointer");
  LSP_CHECK_ARG(B > 0 && S > 0 && G > 0, "lsp_flip_update: bad B/S/G");
  const FlipArgs f = {base_prefix_len, last_id, reinterpret_cast<unsigned long long *>(counters), G, window_lo, window_hi, step_counts};
  flip_kernel<<<B, kFlipThreads, 0, static_cast<hipStream_t>(stream)>>>(f, top1_id, S, prefix_len, suffix_len);
  LSP_CHECK_LAUNCH("lsp_flip_update: launch");
  return LSP_OK;
}
