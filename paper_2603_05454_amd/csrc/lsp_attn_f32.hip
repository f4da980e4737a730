// fp32 variant of the suffix attention (Algorithm 1 line 4; Section 3.2) for
// full-precision callers and checks: fp32 products and sums throughout, on
// v_mfma_f32_16x16x4_f32 (whose products and accumulation are IEEE fp32).
//
// A workgroup owns 16 queries and its waves split the key stream in tiles of 16
// keys, with the same transposed formulation as the bf16 kernels: S^T = K.Q^T
// leaves a lane with four scores of ONE query (keys 4*grp + r), and those four
// registers are, as they are, the B operands of the four matrix steps of
// O^T += V^T.P^T.  The order in which a contraction visits its index is free, so
// operands are loaded from global memory straight into fragment registers, 16
// bytes per lane, with no LDS:
//   K, Q  lane (row i, grp) holds d = 16c + 4 grp + e for every c (16 rows x 64 bytes per load);
//   V     lane (i, grp) holds d = 64c + 4i + e of key 4 grp + r (4 rows x 256 bytes per load),
//         which makes row i of output block (c, e) column d = 64c + 4i + e.
//
// What bounds it at the sizes it is used for (4 heads of 64, 64 queries, 192 keys)
// is latency: a launch, one trip to memory for the lengths, one for the operands,
// and the chain of dependent matrix steps.  Hence the narrow query tile and the keys
// of a tile split eight ways and merged through LDS.  (Q stands in the source before
// the lengths are known; the compiler requests it behind them.)  Measured, kernel
// alone: that size 5.4 us (137 us for one query per lane on plain FMAs with K/V
// broadcast from LDS, which leaves 4 waves in flight), 256 queries x 1280 keys x 4
// heads 13.7 us (903), 8 sequences of 1024 x 2048 x 8 heads 371 us (1589).  Tiles of 32 queries and a four-way split
// are 15 % faster at that last size and 30-60 % slower at the small ones; a
// sixteen-way split changes nothing, requesting the next tile ahead takes 8 % longer.
#include <chrono>
#include <type_traits>

#include "lsp_attn.h"

namespace lsp {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kTile = 16;  // queries per workgroup, keys per step of a wave
constexpr int kWaves = 8;  // way split of the keys
constexpr int kComputeUnits = 256;

// over the four lanes (grp = 0..3) that hold scores of the same query
__device__ __forceinline__ float group_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16));
  return fmaxf(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ float group_sum(float x) {
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}

// Keys of a tile divided between workgroups as well, in parts of kPart keys dealt out in turn: a part leaves its 16 rows of
// unnormalised output, maxima and sums in the workspace, then the call's tag.  A workgroup that finds the tags of all parts
// there merges them in order and stores the rows (the last one to write does; if another one does too, both store the same),
// and clears the tags for a replay.  Everything passes as device-scope atomics of 8 bytes, as in confidence_split_kernel.
// One compute unit's matrix pipe and load path were what a tile waited for, 1.1 us for 128 keys of 64, 2.9 of 128, while
// most of the others had none.  4 heads, 16 rows of 64: 400 keys 8.4 -> 6.9 us, 700 11.7 -> 7.3, 1280 19.1 -> 8.1; 128 rows
// on 1280 19.3 -> 10.3; of 128: 400 keys 14.8 -> 9.8, 1000 28.1 -> 10.7.  The exchange takes 1.5 to 2 us, hence kSavedKeys,
// the fewer keys that a part must have (16 rows of 64, 260 keys 6.97 us whole and 7.41 divided, 330 keys 7.79 and 6.84; of
// 128, 200 keys 10.6 and 11.9, 260 keys 11.7 and 9.7).  That is decided with the lengths, on the device: a launch with room for
// parts whose keys turn out too few takes 1 % longer for the workgroups that find nothing.  The merge requests all pieces of a
// thread at once, for up to 4, 8 and 16 parts (16 for every number: 16 rows of 64 on 700 keys 8.2 for 7.3).  The rms
// error against 64 bits is 0.68 to 0.99 of whole keys' (16 to 128 rows, 346 to 2016 keys, scores of deviation 1 and 4).
constexpr int kPart = kTile * kWaves;
constexpr int kMaxParts = 16;
template <int D>
constexpr int kSavedKeys = D == 64 ? 176 : 100;
template <int D>
constexpr size_t kPartBytes = kTile * D * 4 + kTile * 8;
template <int D>
__host__ __device__ __forceinline__ int parts_of(int keys, int most) {
  const int rounds = (keys + kPart - 1) / kPart, parts = rounds < most ? rounds : most;
  return parts > 1 && keys - (rounds + parts - 1) / parts * kPart >= kSavedKeys<D> ? parts : 1;
}

template <int D, bool SPLIT>
__global__ __launch_bounds__(64 * kWaves, 2) void attn_f32_kernel(AttnArgs a_in, int max_parts, uint64_t tag) {
  constexpr int CK = D / 16;  // 16-byte K (and Q) pieces per lane and row
  constexpr int CV = D / 64;  // 16-byte V pieces per lane and key
  constexpr int OP = D + 4;   // floats per merged O row
  AttnArgs a = a_in;
  a.layers = 1;
  fetch_operands(a);
  const Place pl = place<false>(a, kTile, SPLIT ? int(blockIdx.x) : workgroup_id());
  if (!pl.valid) return;
  const int b = pl.b, g = pl.g, h = pl.h, q0 = pl.q0;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, grp = lane >> 4;

  // rows up to S-1 exist whatever N turns out to be
  f32x4 qf[CK];
  const float *q = static_cast<const float *>(a.q) + b * a.qs[0] + min(q0 + i, a.S - 1) * a.qs[1] + h * a.qs[2] + 4 * grp;
#pragma unroll
  for (int c = 0; c < CK; ++c) qf[c] = *reinterpret_cast<const f32x4 *>(q + 16 * c);
  const auto [N, P] = lengths_of(a, b);
  if (q0 >= N) return;
  const int T = P + N;
  const int parts = SPLIT ? parts_of<D>(T, max_parts) : 1, part = SPLIT ? int(blockIdx.y) : 0;
  if (part >= parts) return;
  const float *kc = static_cast<const float *>(a.k_cache) + b * a.cs[0] + g * a.cs[2];
  const float *vc = static_cast<const float *>(a.v_cache) + b * a.cs[0] + g * a.cs[2];
  const float *ks = static_cast<const float *>(a.k_suf) + b * a.ks[0] + g * a.ks[2];
  const float *vs = static_cast<const float *>(a.v_suf) + b * a.ks[0] + g * a.ks[2];
  auto row_of = [&](const float *cache, const float *suf, int t) {  // row of key t; the last one beyond the end
    t = min(t, T - 1);
    if (t >= P) return suf + int64_t(t - P) * a.ks[1];
    return cache + int64_t(a.cache_rows ? cache_row<true>(a, b, t) : t) * a.cs[1];
  };

  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 o[CV][4];
#pragma unroll
  for (int c = 0; c < CV; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) o[c][e] = zero;
  float m = -INFINITY, l = 0.f;
  const float sc = a.scale * kLog2e;
  for (int t0 = kPart * part + kTile * wave; t0 < T; t0 += kPart * parts) {
    f32x4 kf[CK], vf[4][CV];
    const float *kp = row_of(kc, ks, t0 + i) + 4 * grp;
#pragma unroll
    for (int c = 0; c < CK; ++c) kf[c] = *reinterpret_cast<const f32x4 *>(kp + 16 * c);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float *vp = row_of(vc, vs, t0 + 4 * grp + r) + 4 * i;
#pragma unroll
      for (int c = 0; c < CV; ++c) vf[r][c] = *reinterpret_cast<const f32x4 *>(vp + 64 * c);
    }
    f32x4 s0 = zero, s1 = zero;  // two chains: a matrix instruction does not wait for the one before it
#pragma unroll
    for (int c = 0; c < CK; ++c)
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][e], qf[c][e], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][e + 1], qf[c][e + 1], s1, 0, 0, 0);
      }
    f32x4 s = s0 + s1;
    if (t0 + kTile > T) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const bool key = t0 + 4 * grp + r < T;
        s[r] = key ? s[r] : -INFINITY;
#pragma unroll
        for (int c = 0; c < CV; ++c) vf[r][c] = key ? vf[r][c] : zero;  // (0 x an infinite last row would be NaN)
      }
    }
    const float mo = m, bm = group_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))) * sc;
    m = fmaxf(mo, bm);
    const float mn = m == -INFINITY ? 0.f : m;  // only scores of -infinity so far: weights 0, not exp(-inf + inf)
    const float alpha = __builtin_amdgcn_exp2f(mo - mn);  // 0 on the first tile
    l *= alpha;
    f32x4 p;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], sc, -mn));
      l += p[r];
    }
#pragma unroll
    for (int c = 0; c < CV; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) o[c][e] *= alpha;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < CV; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[c][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][c][e], p[r], o[c][e], 0, 0, 0);
  }

  // merge: lane (query i, grp) holds O^T rows 4 grp + r of blocks (c, e), d = 64c + 16 grp + 4r + e
  __shared__ __attribute__((aligned(16))) float so[kWaves][kTile][OP];
  __shared__ float sm[kWaves][kTile], sl[kWaves][kTile];
  l = group_sum(l);
#pragma unroll
  for (int c = 0; c < CV; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const f32x4 v = {o[c][0][r], o[c][1][r], o[c][2][r], o[c][3][r]};
      *reinterpret_cast<f32x4 *>(&so[wave][i][64 * c + 16 * grp + 4 * r]) = v;
    }
  if (grp == 0) {
    sm[wave][i] = m;
    sl[wave][i] = l;
  }
  __syncthreads();
  unsigned long long *mine = nullptr, *flags = nullptr;
  if (SPLIT && parts > 1) {
    const int tile = blockIdx.x, tiles = gridDim.x;
    flags = static_cast<unsigned long long *>(a.workspace) + size_t(tile) * kMaxParts;
    mine = static_cast<unsigned long long *>(a.workspace) + size_t(tiles) * kMaxParts + size_t(tile) * max_parts * (kPartBytes<D> / 8);
  }
  auto pass = [](unsigned long long *p, float lo, float hi) {
    __hip_atomic_store(p, (unsigned long long)(__float_as_uint(hi)) << 32 | __float_as_uint(lo), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  for (int it = tid; it < kTile * (D / 4); it += 64 * kWaves) {
    const int qq = it / (D / 4), d = 4 * (it % (D / 4));
    if (q0 + qq >= N) continue;
    float M = sm[0][qq];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) M = fmaxf(M, sm[w][qq]);
    f32x4 acc = zero;
    float den = 0.f;
    const float own = SPLIT && parts > 1 && M == -INFINITY ? 0.f : M;  // (a part of such scores only adds nothing to the others)
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float wgt = __builtin_amdgcn_exp2f(sm[w][qq] - own);  // 0 for a wave that saw no key (or only scores of -infinity)
      den += sl[w][qq] * wgt;
      acc += *reinterpret_cast<const f32x4 *>(&so[w][qq][d]) * wgt;
    }
    if (SPLIT && parts > 1) {
      unsigned long long *o = mine + part * (kPartBytes<D> / 8);
      pass(o + (qq * D + d) / 2, acc.x, acc.y);
      pass(o + (qq * D + d) / 2 + 1, acc.z, acc.w);
      if (d == 0) pass(o + kTile * D / 2 + qq, M, den);
      continue;
    }
    float *out = static_cast<float *>(a.out) + b * a.os[0] + int64_t(q0 + qq) * a.os[1] + h * a.os[2] + d;
    *reinterpret_cast<f32x4 *>(out) = acc * (1.0f / den);
  }
  if (!SPLIT || parts == 1) return;

  __shared__ int s_all;
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): what this wave has passed on has arrived
  __syncthreads();
  if (wave == 0) {
    if (lane == 0) __hip_atomic_store(flags + part, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);
    asm volatile("" ::: "memory");
    const unsigned long long f = lane < parts ? __hip_atomic_load(flags + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : tag;
    const bool all = __all(f == tag);
    if (lane == 0) s_all = all;
  }
  __syncthreads();
  if (!s_all) return;
  auto low = [](unsigned long long x) { return __uint_as_float(uint32_t(x)); };
  auto high = [](unsigned long long x) { return __uint_as_float(uint32_t(x >> 32)); };
  auto merge = [&](auto most) {  // up to so many parts, all of a thread's pieces requested at once
    constexpr int U = decltype(most)::value;
    for (int it = tid; it < kTile * (D / 4); it += 64 * kWaves) {
      const int qq = it / (D / 4), d = 4 * (it % (D / 4));
      if (q0 + qq >= N) continue;
      unsigned long long ml[U], x[U], y[U];
#pragma unroll
      for (int p = 0; p < U; ++p) {
        unsigned long long *o = mine + min(p, parts - 1) * (kPartBytes<D> / 8);
        ml[p] = __hip_atomic_load(o + kTile * D / 2 + qq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x[p] = __hip_atomic_load(o + (qq * D + d) / 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        y[p] = __hip_atomic_load(o + (qq * D + d) / 2 + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      float M = low(ml[0]);
#pragma unroll
      for (int p = 1; p < U; ++p) M = fmaxf(M, low(ml[p]));
      f32x4 acc = zero;
      float den = 0.f;
#pragma unroll
      for (int p = 0; p < U; ++p)
        if (p < parts) {
          const float wgt = __builtin_amdgcn_exp2f(low(ml[p]) - M);
          den += high(ml[p]) * wgt;
          acc += f32x4{low(x[p]), high(x[p]), low(y[p]), high(y[p])} * wgt;
        }
      float *out = static_cast<float *>(a.out) + b * a.os[0] + int64_t(q0 + qq) * a.os[1] + h * a.os[2] + d;
      *reinterpret_cast<f32x4 *>(out) = acc * (1.0f / den);
    }
  };
  if (parts <= 4) merge(std::integral_constant<int, 4>{});
  else if (parts <= 8) merge(std::integral_constant<int, 8>{});
  else merge(std::integral_constant<int, kMaxParts>{});
  if (tid < parts) __hip_atomic_store(flags + tid, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Parts that a tile's keys may be divided into: as many as there are compute units for, and as the buffers hold keys for.
template <int D>
int most_parts(int64_t tiles, int64_t keys) {
  const int64_t fit = kComputeUnits / tiles, most = fit < kMaxParts ? fit : kMaxParts;
  return parts_of<D>(int(keys < (1 << 20) ? keys : 1 << 20), int(most));
}
// The tag of one call: another one for the next 2^64 calls of the process, not 0, scrambled by the first steps of SplitMix64's mixing
// function (Steele, Lea and Flood, Fast Splittable Pseudorandom Number Generators, 2014).
inline uint64_t call_tag() {
  static std::atomic<uint64_t> count{uint64_t(std::chrono::steady_clock::now().time_since_epoch().count())};
  uint64_t x;
  do {
    x = count.fetch_add(1, std::memory_order_relaxed) * 0x9e3779b97f4a7c15u;  // odd factors and shifted copies of itself: a permutation
    x = (x ^ x >> 30) * 0xbf58476d1ce4e5b9u;
    x ^= x >> 27;
  } while (x == 0);
  return x;
}

template <int D>
int32_t launch(AttnArgs a, hipStream_t st) {
  AttnLayers none;
  none.n = 0;
  // One unit after the other (taking the tiles of eight in turn costs a division, 0.1 of 6 us, and gains nothing), cut
  // into pieces only beyond 16 tiles per XCD (4 heads of 64: 64 queries x 192 keys 6.2 us whole and 6.5 in pieces, 256 x
  // 1280 19.5 and 19.9, three sequences of that 21.7 and 20.2, keys undivided).
  const int64_t nwg = place_grid(a, none, kTile, 0, 1, 16);
  if (nwg > kMaxGrid) {
    set_error("lsp_attn_step: launch of %lld workgroups is too large", (long long)nwg);
    return LSP_ERR_UNSUPPORTED;
  }
  const int parts = a.workspace != nullptr ? most_parts<D>(nwg, int64_t(a.C) + a.S) : 1;
  if (parts > 1)
    attn_f32_kernel<D, true><<<dim3(unsigned(nwg), unsigned(parts)), 64 * kWaves, 0, st>>>(a, parts, call_tag());
  else
    attn_f32_kernel<D, false><<<grid_of(nwg), 64 * kWaves, 0, st>>>(a, 1, 0);
  LSP_CHECK_LAUNCH("lsp_attn_step: fp32 launch");
  return LSP_OK;
}

}  // namespace

size_t attn_f32_workspace_bytes(int32_t B, int32_t S, int32_t Hq, int32_t Hkv, int32_t D, int32_t C) {
  // (asked on every call: most are answered without the placement, which has as many workgroups as tiles or more; and of any sizes)
  if (B > kComputeUnits || Hq > kComputeUnits || S > kComputeUnits * kTile) return 0;
  const int64_t keys = int64_t(C) + S, tiles = int64_t(B) * Hq * ((int64_t(S) + kTile - 1) / kTile);
  if ((D == 64 ? most_parts<64>(tiles, keys) : D == 128 ? most_parts<128>(tiles, keys) : 1) < 2) return 0;
  AttnArgs a = {};
  AttnLayers none;
  none.n = 0;
  a.B = B; a.S = S; a.Hq = Hq; a.Hkv = Hkv;
  const int64_t nwg = place_grid(a, none, kTile, 0, 1, 16);
  const int parts = D == 64 ? most_parts<64>(nwg, keys) : most_parts<128>(nwg, keys);
  return parts < 2 ? 0 : size_t(nwg) * (8 * kMaxParts + parts * (D == 64 ? kPartBytes<64> : kPartBytes<128>));
}

int32_t launch_attn_f32(const AttnArgs &a, hipStream_t st) {
  if (a.D == 64) return launch<64>(a, st);
  if (a.D == 128) return launch<128>(a, st);
  set_error("lsp_attn_step: fp32 head_dim %d not built (64, 128)", a.D);
  return LSP_ERR_UNSUPPORTED;
}

}  // namespace lsp
