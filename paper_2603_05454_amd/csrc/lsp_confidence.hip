// lsp_confidence: per-position top-1 id, logit margin (Eq. 1 of the paper;
// Algorithm 1 line 5) and top-1 soft-max probability, as one streaming pass
// over the logits.
//
// The kernel is bound by HBM reads (V * sizeof(elem) bytes per active row, each
// byte read once), so the design goal is: 16-byte coalesced loads with several
// in flight per lane, and few enough VALU operations per element that the
// arithmetic hides under the stream:
//   - top-2 tracking costs two operations per element: m2 = med3(m1, x, m2),
//     m1 = max(m1, x) (valid because m2 <= m1 always);
//   - the arg-max index is not tracked per element.  A lane only remembers in
//     which group of its 16-byte vectors its running maximum last rose
//     strictly; since a lane visits its elements in increasing index order,
//     that group holds the lane's first occurrence of its maximum; the lane keeps a
//     copy of it in registers, which is scanned once at the end;
//   - the soft-max sum uses one exp2 per element against a lagging per-lane
//     reference r (log2 domain) which is only moved when the lane maximum has
//     run more than 32 octaves ahead of it, so the rescale branch is cold.  A
//     group's top-2 pass runs before its sum pass, so the reference always
//     covers the values being exponentiated.
// Lane results are merged in two steps: the maximum first (DPP reduction), then
// each lane rescales its sum to it and the runner-up, the sum and the lowest
// index among the lanes holding the maximum are plain max / add / min
// reductions.  The same merge runs across the waves of a workgroup through
// LDS and - when one row is split over several workgroups because there are
// too few rows to fill the chip - in the last of these workgroups.
#include <float.h>
#include <limits.h>

#include <chrono>
#include <mutex>
#include <type_traits>

#include "lsp_common.h"

namespace lsp {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLagOctaves = 32.0f;  // the reference may lag the maximum by this much

struct Top {
  float m1, m2;  // largest and second largest value seen (duplicates count)
  float s;       // sum of exp2(x*log2e - r)
  float r;       // reference exponent (log2 domain): some earlier maximum times log2e, ROUNDED
  int idx;       // >= 0: element index of the first maximum; < 0: ~(first element of the lane's group holding it)
};

__device__ __forceinline__ void top_init(Top &t) {
  t.m1 = -INFINITY;
  t.m2 = -INFINITY;
  t.s = 0.f;
  t.r = -FLT_MAX;
  t.idx = INT_MAX;
}

// max as exactly one v_max_f32.  fmaxf() costs two here: the kernel runs in IEEE
// mode, where the compiler first quiets a possible signalling NaN in each
// operand; the precondition excludes NaN, so the bare instruction is enough.
__device__ __forceinline__ float fmax_raw(float a, float b) {
  float d;
  asm("v_max_f32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}

// Top-2 update over N values; `tag` is recorded when the maximum rose strictly.
template <int N>
__device__ __forceinline__ void absorb_top2(Top &t, const float (&x)[N]) {
#pragma unroll
  for (int j = 0; j < N; ++j) {
    t.m2 = __builtin_amdgcn_fmed3f(t.m1, x[j], t.m2);
    t.m1 = fmax_raw(t.m1, x[j]);
  }
}

// Move the reference up when the maximum has run ahead of it (cold branch).
__device__ __forceinline__ void settle_reference(Top &t) {
  const float mc = t.m1 * kLog2e;
  if (mc - t.r > kLagOctaves) {
    t.s *= __builtin_amdgcn_exp2f(t.r - mc);
    t.r = mc;
  }
}

// Soft-max sum over N values that are already covered by t.m1 / t.r.
template <int N>
__device__ __forceinline__ void absorb_sum(Top &t, const float (&x)[N]) {
  // One fma + exp2 per element.  r is a ROUNDED product, so every term is off by
  // the same factor 2^(m*log2e - r) (up to 2e-5 for logits around 500); the fold
  // in wave_combine takes the sum off this reference with an fma of its own,
  // which removes that factor exactly.
  const float nr = -t.r;
#pragma unroll
  for (int j = 0; j < N; ++j) t.s += __builtin_amdgcn_exp2f(__builtin_fmaf(x[j], kLog2e, nr));
}

template <int N>
__device__ __forceinline__ void absorb(Top &t, const float (&x)[N], int tag) {
  const float old = t.m1;
  absorb_top2<N>(t, x);
  t.idx = t.m1 > old ? tag : t.idx;
  settle_reference(t);
  absorb_sum<N>(t, x);
}

template <typename T>
struct Vec;
template <>
struct Vec<float> {
  static constexpr int N = 4;
  static __device__ __forceinline__ void unpack(const u32x4 &w, float (&x)[4]) {
    x[0] = __uint_as_float(w.x);
    x[1] = __uint_as_float(w.y);
    x[2] = __uint_as_float(w.z);
    x[3] = __uint_as_float(w.w);
  }
  static __device__ __forceinline__ float scalar(const float *p) { return *p; }
};
template <>
struct Vec<uint16_t> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void unpack(const u32x4 &w, float (&x)[8]) {
    x[0] = bf16_lo(w.x); x[1] = bf16_hi(w.x);
    x[2] = bf16_lo(w.y); x[3] = bf16_hi(w.y);
    x[4] = bf16_lo(w.z); x[5] = bf16_hi(w.z);
    x[6] = bf16_lo(w.w); x[7] = bf16_hi(w.w);
  }
  static __device__ __forceinline__ float scalar(const uint16_t *p) { return bf16_to_f32(*p); }
};

// ---- cross-lane reductions on the DPP network (no LDS traffic) ---------------
// Classic GCN reduction: two quad permutes, row shifts by 4 and 8, then the row
// broadcasts 15 and 31; lane 63 ends up holding the reduction of all 64 lanes.
// Lanes without a source keep op(v, v), which never feeds lane 63.
template <typename Op>
__device__ __forceinline__ float wave_reduce(float v, Op op) {
#define LSP_DPP_STEP(ctrl)                                                                    \
  v = op(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), \
                                                       ctrl, 0xf, 0xf, false)))
  LSP_DPP_STEP(0xb1);   // quad_perm [1,0,3,2]
  LSP_DPP_STEP(0x4e);   // quad_perm [2,3,0,1]
  LSP_DPP_STEP(0x114);  // row_shr:4
  LSP_DPP_STEP(0x118);  // row_shr:8
  LSP_DPP_STEP(0x142);  // row_bcast:15
  LSP_DPP_STEP(0x143);  // row_bcast:31
#undef LSP_DPP_STEP
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
struct OpMax { __device__ __forceinline__ float operator()(float a, float b) const { return fmax_raw(a, b); } };
struct OpAdd { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };
// min over non-negative ints: their float bit patterns order the same way
struct OpMinI {
  __device__ __forceinline__ float operator()(float a, float b) const {
    return __int_as_float(min(__float_as_int(a), __float_as_int(b)));
  }
};

struct RowStat {  // wave-uniform: maximum, second, sum of exp(x - m1), first index of the maximum
  float m1, m2, s;
  int idx;
};

// Combine the 64 lane states of a wave, given the maximum over the lanes and the
// factor w that takes this lane's sum from its own reference to that maximum.
// The remaining reductions are plain max/add/min.  A lane's idx is only read
// when the lane holds the maximum.
__device__ __forceinline__ RowStat wave_combine(const Top &t, float wave_max, float w) {
  RowStat o;
  o.m1 = wave_max;
  const bool top = t.m1 == o.m1;
  const int ntop = __popcll(__ballot(top));
  const float second = wave_reduce(top ? t.m2 : t.m1, OpMax());
  o.m2 = ntop >= 2 ? o.m1 : second;  // the maximum held by two lanes is its own runner-up
  o.idx = __float_as_int(wave_reduce(__int_as_float(top ? t.idx : INT_MAX), OpMinI()));
  const float sum = wave_reduce(t.s * w, OpAdd());
  o.s = o.m1 == -INFINITY ? 0.f : sum;  // an all -inf segment has an empty sum
  return o;
}

// Merge of up to 64 parts of a row, one a lane (idle lanes: top_init), each sum relative to its part's own maximum.
__device__ __forceinline__ RowStat merge_stats(const Top &t) {
  const float all_max = wave_reduce(t.m1, OpMax());
  return wave_combine(t, all_max, __builtin_amdgcn_exp2f((t.m1 - all_max) * kLog2e));  // exp(m1 - max); 0 for the idle lanes
}

// One workgroup reduces elements [c0, c1) of one row.  NT threads; U vectors per
// lane per group; two groups of loads in flight (ping-pong register buffers).
// The result is valid in wave 0; the other waves only take part.
template <typename T, int NT, int U>
__device__ __forceinline__ RowStat segment_stat(const T *row, int c0, int c1) {
  constexpr int N = Vec<T>::N;
  const int tid = threadIdx.x;

  Top t;
  top_init(t);

  // split [c0,c1) into an unaligned head, 16-byte vectors, and a tail
  const int len = c1 - c0;
  int head = int(((16u - (unsigned(reinterpret_cast<uintptr_t>(row + c0)) & 15u)) & 15u) / sizeof(T));
  head = min(head, len);
  const int nvec = (len - head) / N;
  const int tail0 = c0 + head + nvec * N;

  if (tid < head) {
    float x[1] = {Vec<T>::scalar(row + c0 + tid)};
    absorb<1>(t, x, c0 + tid);
  }

  const u32x4 *vp = reinterpret_cast<const u32x4 *>(row + c0 + head);
  const int vbase = c0 + head;  // element index of vector 0
  constexpr int G = NT * U;     // vectors per group
  const int ngroups = (nvec + G - 1) / G;  // the last one may be partial

  // Lanes past the end of the last, partial group re-read the row's last vector
  // (their values are replaced by -inf below), so that group is one burst of
  // loads like every other.
  auto load_group = [&](u32x4 (&buf)[U], int g, auto last) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = g * G + u * NT + tid;
      buf[u] = __builtin_nontemporal_load(vp + (decltype(last)::value ? min(v, nvec - 1) : v));
    }
  };
  // phase 1: top-2 over the whole group, one index tag and one reference check per
  // group; phase 2: the soft-max sum.  (The tag names the lane's first vector of the
  // group; the lane keeps a copy of its U vectors of that group, eight selects per
  // group, and scans the copy at the end.  Re-reading them from memory instead put
  // a dependent round trip at the end of every row.)
  u32x4 kept[U];
#pragma unroll
  for (int u = 0; u < U; ++u) kept[u] = u32x4{0, 0, 0, 0};
  auto process_group = [&](const u32x4 (&buf)[U], int g, auto last) {
    float x[U][N];
    const float old = t.m1;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      Vec<T>::unpack(buf[u], x[u]);
      if (decltype(last)::value && g * G + u * NT + tid >= nvec) {
#pragma unroll
        for (int k = 0; k < N; ++k) x[u][k] = -INFINITY;  // never the maximum, adds 0 to the sum
      }
      absorb_top2<N>(t, x[u]);
    }
    const bool rose = t.m1 > old;
    t.idx = rose ? ~(vbase + (g * G + tid) * N) : t.idx;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      kept[u].x = rose ? buf[u].x : kept[u].x;
      kept[u].y = rose ? buf[u].y : kept[u].y;
      kept[u].z = rose ? buf[u].z : kept[u].z;
      kept[u].w = rose ? buf[u].w : kept[u].w;
    }
    settle_reference(t);
#pragma unroll
    for (int u = 0; u < U; ++u) absorb_sum<N>(t, x[u]);
  };
  if (ngroups > 0) {
    const std::false_type full;
    const std::true_type maybe_partial;
    u32x4 ping[U], pong[U];
    if (ngroups == 1) load_group(ping, 0, maybe_partial); else load_group(ping, 0, full);
    int g = 0;
    for (; g + 3 < ngroups; g += 2) {  // groups g+1 and g+2 are full
      load_group(pong, g + 1, full);
      process_group(ping, g, full);
      load_group(ping, g + 2, full);
      process_group(pong, g + 1, full);
    }
    // one to three groups left; only the very last may be partial
    if (g + 2 < ngroups) {
      load_group(pong, g + 1, full);
      process_group(ping, g, full);
      load_group(ping, g + 2, maybe_partial);
      process_group(pong, g + 1, full);
      process_group(ping, g + 2, maybe_partial);
    } else if (g + 1 < ngroups) {
      load_group(pong, g + 1, maybe_partial);
      process_group(ping, g, full);
      process_group(pong, g + 1, maybe_partial);
    } else {
      process_group(ping, g, maybe_partial);
    }
  }
  if (tid < c1 - tail0) {
    float x[1] = {Vec<T>::scalar(row + tail0 + tid)};
    absorb<1>(t, x, tail0 + tid);
  }

  // A lane whose maximum came from a group scans its copy of that group, from the
  // last vector to the first so that the lowest index wins.
  const float wave_max = wave_reduce(t.m1, OpMax());
  if (t.idx < 0) {
    const int e0 = ~t.idx;
    int found = INT_MAX;
#pragma unroll
    for (int u = U - 1; u >= 0; --u) {
      const int eb = e0 + u * NT * N;
      if (eb >= tail0) continue;  // past the end of a partial group (the copy holds a repeat of the last vector)
      float x[N];
      Vec<T>::unpack(kept[u], x);
#pragma unroll
      for (int k = N - 1; k >= 0; --k) found = (x[k] == t.m1) ? eb + k : found;
    }
    t.idx = found;
  }

  // exp2(r - max*log2e) with the product unrounded inside the fma; 0 for an empty lane (r = -FLT_MAX)
  RowStat r = wave_combine(t, wave_max, __builtin_amdgcn_exp2f(__builtin_fmaf(-wave_max, kLog2e, t.r)));
  constexpr int NW = NT / kWave;
  if (NW > 1) {
    __shared__ RowStat lds[NW];
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    if (lane == 0) lds[wave] = r;
    __syncthreads();
    if (wave != 0) return r;
    top_init(t);
    if (lane < NW) {
      const RowStat w = lds[lane];
      t.m1 = w.m1; t.m2 = w.m2; t.s = w.s; t.idx = w.idx;
    }
    r = merge_stats(t);
  }
  return r;
}

__device__ __forceinline__ void store_row(const RowStat &r, int64_t o, int32_t *__restrict__ top1_id,
                                          float *__restrict__ top1_prob, float *__restrict__ margin) {
  top1_id[o] = r.idx;
  margin[o] = r.m1 - r.m2;
  top1_prob[o] = 1.0f / r.s;
}

// One workgroup per row of the buffer.  (Registers as in confidence_split_kernel; fp32 rows take 68 and get another order of loads where
// something is asked for: 5 x 600 rows of 30 000 with 360 active 31.7 us, 33.5 so.)
template <typename T, int NT, int U>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 2 ? 4 : 1))) void confidence_kernel(
    const T *__restrict__ logits, int S, int V, int64_t row_stride, int64_t batch_stride,
    const int32_t *__restrict__ suffix_len, int32_t *__restrict__ top1_id, float *__restrict__ top1_prob,
    float *__restrict__ margin) {
  const int i = blockIdx.x, b = blockIdx.y;
  fetch_now(logits, S, V, row_stride, batch_stride, top1_id, top1_prob, margin);
  if (suffix_len != nullptr && i >= suffix_len[b]) return;
  const RowStat r = segment_stat<T, NT, U>(logits + int64_t(b) * batch_stride + int64_t(i) * row_stride, 0, V);
  if (threadIdx.x == 0) store_row(r, int64_t(b) * S + i, top1_id, top1_prob, margin);
}

// The same where rows may be cut into 2^k segments, one workgroup each: k follows the number of ACTIVE rows,
// which only the device knows (in a decode loop few are left of a large buffer).  Workgroup w takes segment
// w % 2^k of active row w / 2^k, counted over all sequences.  What a segment leaves in the workspace is its
// statistics and, beside each of the four numbers, this call's tag; a workgroup then reads the row's other
// segments and, where it finds all of them, merges and stores the row.  The last one to write does find them; if
// another one does too, both store the same.  Nobody waits for anybody, and the workspace need not be
// cleared before (it would have to hold the tag four times over by chance); whoever merged clears the
// tags, so that a graph replayed with the same tag finds nothing of the replay before.
// Numbers and tags pass between workgroups as device-scope atomic stores and loads of 8 bytes, which go past the
// XCD's own L2: waiting for the stores is all the order they need.  A release fence writes that L2 back instead,
// once per workgroup, and a counter of arrivals is one address that they queue for (20 rows in 16 segments each:
// 22 us with a fence, 19 with a counter, 6.4 so; 103 rows in 8: 28, 18, 12).
// What it saves: a row is 7.4 us of arithmetic for one compute unit, so that 3 rows took as long as 100.  One sequence
// of 256 rows of 126 464 entries, per call before -> now: 3 rows active 11.5 -> 5.6 us, 20: 11.8 -> 6.3, 103: 12.6 ->
// 9.9; all 256 stay whole (13.5 -> 13.8, the price of the count); 8 x 1024 rows with 220 active 29.3 -> 15.6, all of
// 8 x 1024 x 152 064 367 -> 361 (no workgroups without a row between the others).
// Rows are cut as long as that makes no more workgroups of 256 threads than this, or half as many of 512: a wave's own
// reductions cost as much as 80 of its vectors, so that shorter segments lose more than the fuller chip gives (100 rows with 512
// threads whole 12.3 us, in 2 segments 9.9, 4 10.1, 8 12.5; with 256 threads 16.4, 11.9, 9.8, 10.1; 505 rows with 256 threads
// whole 23.2, halved 25.5).
constexpr int kSplitTarget = 512;
constexpr int kMaxLog2 = 4;         // 16 segments' numbers fill a wave
constexpr int kMinSegment = 4096;   // elements; a segment is a few groups of loads
constexpr int kMinCut = 16384;      // rows of at most this many are not cut (100 rows of 9000: 4.8 us whole, 5.6 cut)
// fp32 rows are twice the bytes for the same arithmetic and are cut once more, down to segments of this many elements (65 rows of
// 126 464 in 2 segments 13.6 us, in 4 10.4; 40 in 4 9.2, in 8 8.3; 100 rows of 20 000 in 2 5.9, in 4 6.4).
constexpr int kMinSegmentF32 = 7168;
// bf16 rows up to this long are not merely halved: half a row is a group and a quarter of loads (100 rows of 20 000 whole 5.3 us, halved 5.9,
// 40 in 4 segments 5.0 for 5.1; 100 of 30 000 whole 6.1, halved 6.1).
constexpr int kMinHalved = 24576;
// Buffers of fewer rows than this: short rows are cut as well, and all with 512 threads (400 rows of 30 000 in fp32 10.5 us, 12.4
// with 256; 130 of them of 126 464 in bf16 12.7 and 13.2; 505 rows 23.4 and 23.2).
constexpr int kSplitRows = 512;
// FEW: buffers of up to this many sequences, and more rows than run at once: lengths through the scalar cache, where all workgroups but
// the first find them (6 x 189 rows of 126 464 54.4 -> 53.0 us; 2 x 200, which run at once, 24.1 -> 24.7).
// Not with three workgroups to a compute unit: 8 x 1024 rows with 204 active 49.6 -> 53.4, all of 152 064 359 -> 365.
constexpr int kFewSequences = 8;
constexpr int kFewRows = 768;
constexpr int kMaxScannedBatch = 256;  // sequences: every workgroup reads all their lengths, 64 at a time
constexpr int64_t kMaxSplitGrid = int64_t(1) << 22;  // workgroups; more rows than this need no cutting
// OCC: waves per SIMD that registers are allotted for.  bf16 rows are 129 registers where nothing is asked for, which leaves three
// workgroups of 256 threads to a compute unit: a little faster over many rounds of them (8192 rows of 126 464: 299 us,
// 305 with four), slower where the rows just do not fit one or two (900 rows of 152 064: 55.6 and 48.8).
constexpr int kManyRows = 4096;  // of the buffer
// (with 256 threads it would be more segments than the workspace holds)
template <typename T>
__host__ __device__ constexpr bool cut_once_more(int threads) { return sizeof(T) == 4 && threads == 512; }
template <typename T, int NT, int U, int OCC, bool FEW>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 2 ? OCC : 1))) void confidence_split_kernel(
    const T *__restrict__ logits, int B, int S, int V, int64_t row_stride, int64_t batch_stride,
    const int32_t *__restrict__ suffix_len, int max_log2, uint32_t tag, int32_t *__restrict__ top1_id,
    float *__restrict__ top1_prob, float *__restrict__ margin, unsigned long long *segments) {
  const int lane = threadIdx.x & (kWave - 1);
  fetch_now(logits, row_stride, batch_stride, V, max_log2, top1_id, top1_prob, margin, segments, tag);
  // active rows, and for batches of up to 64 the rows up to and including this lane's sequence
  int rows = 0, upto = 0, n = 0, lens[kFewSequences];
  auto scan = [&](int b0) {
    const int b = b0 + lane;
    n = b < B ? min(max(suffix_len[b], 0), S) : 0;
    upto = n;
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x111, 0xf, 0xf, false);  // row_shr:1
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x112, 0xf, 0xf, false);  // row_shr:2
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x114, 0xf, 0xf, false);  // row_shr:4
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x118, 0xf, 0xf, false);  // row_shr:8
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
    return __builtin_amdgcn_readlane(upto, kWave - 1);
  };
  if (suffix_len == nullptr) {
    rows = B * S;
  } else if (FEW) {
#pragma unroll
    for (int j = 0; j < kFewSequences; ++j) lens[j] = suffix_len[min(j, B - 1)];
#pragma unroll
    for (int j = 0; j < kFewSequences; ++j) rows += lens[j] = j < B ? min(max(lens[j], 0), S) : 0;
  } else if (B == 1) {
    rows = upto = n = min(max(suffix_len[0], 0), S);
  } else {
    for (int b0 = 0; b0 < B; b0 += kWave) rows += scan(b0);
  }
  int k = 0;
  if (rows <= kSplitTarget * 128 / NT) {
    while (k < max_log2 && rows << (k + 1) <= kSplitTarget * 256 / NT) ++k;
    if (cut_once_more<T>(NT) && k > 0 && k < max_log2 && V >> (k + 1) >= kMinSegmentF32) ++k;
    if (sizeof(T) == 2 && k == 1 && V <= kMinHalved) k = 0;
  }
  const int row = int(blockIdx.x >> k), seg = int(blockIdx.x) & ((1 << k) - 1);
  if (row >= rows) return;
  int b = 0, i = row;  // sequence and position of that row
  if (suffix_len == nullptr) {
    b = row / S;
    i = row - b * S;
  } else if (FEW) {
    bool beyond = true;
#pragma unroll
    for (int j = 0; j < kFewSequences - 1; ++j) {
      beyond = beyond && i >= lens[j];
      if (beyond) {
        i -= lens[j];
        ++b;
      }
    }
  } else {
    if (B > kWave)
      for (;; b += kWave) {
        const int t = scan(b);
        if (i < t) break;
        i -= t;
      }
    const int s = __popcll(__ballot(upto <= i));
    i -= __builtin_amdgcn_readlane(upto, s) - __builtin_amdgcn_readlane(n, s);
    b += s;
  }

  const int len = (((V + (1 << k) - 1) >> k) + 63) & ~63;
  RowStat r = segment_stat<T, NT, U>(logits + int64_t(b) * batch_stride + int64_t(i) * row_stride, seg * len,
                                     min(V, (seg + 1) * len));
  if (threadIdx.x >= kWave) return;
  if (k > 0) {
    const int own = lane & 3;  // lane 4j + i: number i of segment j
    unsigned long long *w = segments + (int64_t(row) << (k + 2));
    const uint32_t mine = own == 0   ? __float_as_uint(r.m1)
                          : own == 1 ? __float_as_uint(r.m2)
                          : own == 2 ? __float_as_uint(r.s)
                                     : uint32_t(r.idx);
    if (lane < 4)
      __hip_atomic_store(w + 4 * seg + lane, uint64_t(mine) << 32 | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the four are where every workgroup sees them
    const bool used = lane < 4 << k;
    const unsigned long long x = used ? __hip_atomic_load(w + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    if (__any(used && uint32_t(x) != tag)) return;
    if (used) __hip_atomic_store(w + lane, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    Top t;
    top_init(t);
    const int v = int(x >> 32);
    const int m1 = __builtin_amdgcn_update_dpp(v, v, 0x00, 0xf, 0xf, false);  // quad_perm: number 0, 1, 2, 3 of the four lanes
    const int m2 = __builtin_amdgcn_update_dpp(v, v, 0x55, 0xf, 0xf, false);
    const int sum = __builtin_amdgcn_update_dpp(v, v, 0xaa, 0xf, 0xf, false);
    const int idx = __builtin_amdgcn_update_dpp(v, v, 0xff, 0xf, 0xf, false);
    if (used && own == 0) {
      t.m1 = __int_as_float(m1); t.m2 = __int_as_float(m2); t.s = __int_as_float(sum); t.idx = idx;
    }
    r = merge_stats(t);
  }
  if (lane == 0) store_row(r, int64_t(b) * S + i, top1_id, top1_prob, margin);
}

// Launch shape (measured on MI355X).  A workgroup takes a row; it is as wide as
// leaves each lane about 64 vectors of 16 bytes (one wave for rows of a few
// thousand entries, four waves for a 126 464-entry bf16 row: 2-7 % faster there
// than one wave per row, and a 512-thread workgroup is 3x slower on 4 096-entry
// rows); with few rows it widens further so that at least 2048 waves are in
// flight.  Per element the kernel issues about nine VALU cycles (the
// exponential counts four), which at these sizes is as long as the memory time
// itself.  Where rows are long or few, confidence_split_kernel counts the active
// rows and cuts them further.
struct Plan {
  int nt;
  int max_log2;    // rows may be cut into up to 2^max_log2 segments, if there is a workspace
  bool required;   // the call is not made without one
};
inline Plan plan(int64_t rows, int V, int elem_bytes) {
  Plan p;
  int nt = 64;
  const int64_t nvec = int64_t(V) * elem_bytes / 16;
  while (nt < 512 && nvec / nt >= 96) nt *= 2;
  p.max_log2 = 0;
  if (nt >= 256 || rows < kSplitRows)
    while (V > kMinCut && p.max_log2 < kMaxLog2 && (V >> (p.max_log2 + 1)) >= kMinSegment) ++p.max_log2;
  p.required = p.max_log2 > 0 && rows < 128;
  if (p.max_log2 > 0 && nt < 256) nt = 256;
  if (p.max_log2 > 0 && rows < kSplitRows) nt = 512;
  p.nt = nt;
  return p;
}
// without a workspace
inline int unsplit_threads(int64_t rows, int nt) {
  while (nt < 512 && rows * (nt / 64) < 2048) nt *= 2;
  return nt;
}

// what a call writes into its workspace: four numbers of each segment, each beside the tag
constexpr size_t kSplitBytes = size_t(kSplitTarget) * 4 * sizeof(unsigned long long);

// The tag of one call: another one for the next four thousand million calls of the process, not 0, and scrambled so that
// memory is not likely to hold it.
inline uint32_t call_tag() {
  static std::atomic<uint32_t> count{uint32_t(std::chrono::steady_clock::now().time_since_epoch().count() >> 10)};
  uint32_t x;
  do {
    x = count.fetch_add(1, std::memory_order_relaxed) * 0x9e3779b1u;  // odd factors and shifted copies of itself: a permutation
    x = (x ^ x >> 15) * 0x85ebca6bu;
    x ^= x >> 13;
  } while (x == 0);
  return x;
}

template <typename T>
void launch_rows(int nt, hipStream_t st, const T *z, int B, int S, int V, int64_t row_stride, int64_t batch_stride,
                 const int32_t *suffix_len, int32_t *top1_id, float *top1_prob, float *margin) {
  const dim3 grid(S, B);
#define LSP_CONF_CASE(NT_) \
  if (nt == NT_)           \
    return confidence_kernel<T, NT_, 2><<<grid, NT_, 0, st>>>(z, S, V, row_stride, batch_stride, suffix_len, top1_id, top1_prob, margin)
  LSP_CONF_CASE(64);
  LSP_CONF_CASE(128);
  LSP_CONF_CASE(256);
  LSP_CONF_CASE(512);
#undef LSP_CONF_CASE
}

template <typename T>
void launch_split(const Plan &p, hipStream_t st, const T *z, int B, int S, int V, int64_t row_stride, int64_t batch_stride,
                  const int32_t *suffix_len, int32_t *top1_id, float *top1_prob, float *margin, void *workspace) {
  const int64_t rows = int64_t(B) * S, most = rows << p.max_log2;
  const int64_t target = cut_once_more<T>(p.nt) ? kSplitTarget : kSplitTarget * 256 / p.nt;
  const int64_t grid = rows > target ? rows : most < target ? most : target;
  const bool few = B > 1 && B <= kFewSequences && rows >= kFewRows;
  auto kern = p.nt == 512        ? (few ? confidence_split_kernel<T, 512, 2, 4, true> : confidence_split_kernel<T, 512, 2, 4, false>)
              : rows >= kManyRows ? confidence_split_kernel<T, 256, 2, 3, false>
                                  : (few ? confidence_split_kernel<T, 256, 2, 4, true> : confidence_split_kernel<T, 256, 2, 4, false>);
  kern<<<unsigned(grid), p.nt, 0, st>>>(z, B, S, V, row_stride, batch_stride, suffix_len, p.max_log2, call_tag(), top1_id,
                                        top1_prob, margin, static_cast<unsigned long long *>(workspace));
}

}  // namespace
}  // namespace lsp

extern "C" size_t lsp_confidence_workspace_bytes(int32_t B, int32_t S, int32_t V) {
  if (B <= 0 || S <= 0 || V <= 0) return 0;
  // the dtype is not an argument here: enough for either
  const int64_t rows = int64_t(B) * S;
  return lsp::plan(rows, V, 2).max_log2 > 0 || lsp::plan(rows, V, 4).max_log2 > 0 ? lsp::kSplitBytes : 0;
}

namespace lsp {
namespace {

int32_t scratch_address(void **out);  // device address of the library's own scratch buffer (defined below)

// Host side shared by both entry points: validation, launch plan, launch.
// `own_scratch`: the call has no workspace and may use the library's buffer where it needs one.
int32_t confidence_run(const char *who, bool own_scratch, int32_t dtype, const void *logits, int32_t B,
                       int32_t S, int32_t V, int64_t row_stride, int64_t batch_stride,
                       const int32_t *suffix_len, int32_t *top1_id, float *top1_prob, float *margin,
                       void *workspace, size_t workspace_bytes, void *stream) {
  LSP_CHECK_ARG(dtype == LSP_F32 || dtype == LSP_BF16, "%s: unknown dtype %d", who, dtype);
  LSP_CHECK_ARG(logits && top1_id && top1_prob && margin, "%s: null pointer", who);
  LSP_CHECK_ARG(B > 0 && S > 0 && V >= 2, "%s: need B>0, S>0, V>=2 (got %d %d %d)", who, B, S, V);
  LSP_CHECK_ARG(B <= 65535 && S <= 65535, "%s: B and S must be <= 65535", who);
  if (row_stride == 0) row_stride = V;
  if (batch_stride == 0) batch_stride = int64_t(S) * row_stride;
  LSP_CHECK_ARG(row_stride >= V && batch_stride >= 0, "%s: bad strides", who);
  const size_t es = elem_size(dtype);
  LSP_CHECK_ARG((reinterpret_cast<uintptr_t>(logits) & (es - 1)) == 0, "%s: logits misaligned", who);
  const int64_t rows = int64_t(B) * S;
  const Plan p = plan(rows, V, int(es));
  if (own_scratch && p.required) {
    const int32_t rc = scratch_address(&workspace);
    if (rc != LSP_OK) return rc;
    workspace_bytes = kSplitBytes;
  }
  const bool room = workspace != nullptr && workspace_bytes >= kSplitBytes && (reinterpret_cast<uintptr_t>(workspace) & 15u) == 0;
  const bool split = p.max_log2 > 0 && (suffix_len == nullptr || B <= kMaxScannedBatch) && rows <= kMaxSplitGrid && room;
  if (p.required && !split) {
    set_error("%s: workspace of %zu bytes (16-byte aligned) required, got %zu", who, kSplitBytes, workspace_bytes);
    return LSP_ERR_WORKSPACE;
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  const auto *zb = static_cast<const uint16_t *>(logits);
  const auto *zf = static_cast<const float *>(logits);
  if (split && dtype == LSP_BF16)
    launch_split(p, st, zb, B, S, V, row_stride, batch_stride, suffix_len, top1_id, top1_prob, margin, workspace);
  else if (split)
    launch_split(p, st, zf, B, S, V, row_stride, batch_stride, suffix_len, top1_id, top1_prob, margin, workspace);
  else if (dtype == LSP_BF16)
    launch_rows(unsplit_threads(rows, p.nt), st, zb, B, S, V, row_stride, batch_stride, suffix_len, top1_id, top1_prob, margin);
  else
    launch_rows(unsplit_threads(rows, p.nt), st, zf, B, S, V, row_stride, batch_stride, suffix_len, top1_id, top1_prob, margin);
  LSP_CHECK_LAUNCH("lsp_confidence: launch");
  return LSP_OK;
}

}  // namespace
}  // namespace lsp

extern "C" int32_t lsp_confidence(int32_t dtype, const void *logits, int32_t B, int32_t S, int32_t V,
                                  int64_t row_stride, int64_t batch_stride,
                                  const int32_t *suffix_len, int32_t *top1_id, float *top1_prob,
                                  float *margin, void *workspace, size_t workspace_bytes,
                                  void *stream) {
  return lsp::confidence_run("lsp_confidence", false, dtype, logits, B, S, V, row_stride, batch_stride,
                             suffix_len, top1_id, top1_prob, margin, workspace, workspace_bytes, stream);
}

// ---- the same call for callers that cannot allocate ----------------------------
// Where lsp_confidence needs a workspace (long rows, fewer than 128 of them), a
// buffer that is part of the library's device image takes its place.  With more
// rows this form has none and does not cut them, so that calls on several streams
// share nothing.
#define LSP_CONF_SCRATCH_BYTES 65536
static __device__ __align__(256) unsigned char scratch[LSP_CONF_SCRATCH_BYTES];
static_assert(lsp::kSplitBytes <= LSP_CONF_SCRATCH_BYTES, "a call's segments");

namespace lsp {
namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices];  // device address of `scratch` on each GPU (every GPU has its own copy)

// Device address of the scratch array on the current GPU, looked up once per GPU.
int32_t scratch_address(void **out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "lsp_confidence_static: hipGetDevice");
  if (dev < 0 || dev >= kMaxDevices) {
    set_error("lsp_confidence_static: device ordinal %d not supported (< %d)", dev, kMaxDevices);
    return LSP_ERR_UNSUPPORTED;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr) return hip_fail(e, "lsp_confidence_static: hipGetSymbolAddress");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return LSP_OK;
}
}  // namespace
}  // namespace lsp

extern "C" size_t lsp_confidence_static_scratch_bytes(void) { return LSP_CONF_SCRATCH_BYTES; }

extern "C" int32_t lsp_confidence_static(int32_t dtype, const void *logits, int32_t B, int32_t S, int32_t V,
                                         int64_t row_stride, int64_t batch_stride,
                                         const int32_t *suffix_len, int32_t *top1_id, float *top1_prob,
                                         float *margin, void *stream) {
  // Every segment result that is read was written by the same call, so nothing has to be cleared between calls.
  return lsp::confidence_run("lsp_confidence_static", true, dtype, logits, B, S, V, row_stride, batch_stride,
                             suffix_len, top1_id, top1_prob, margin, nullptr, 0, stream);
}
