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
// alone: that size 6.1 us (137 us for one query per lane on plain FMAs with K/V
// broadcast from LDS, which leaves 4 waves in flight), 256 queries x 1280 keys x 4
// heads 19.5 us (903), 8 sequences of 1024 x 2048 x 8 heads 371 us (1589).  Tiles of 32 queries and a four-way split
// are 15 % faster at that last size and 30-60 % slower at the small ones; a
// sixteen-way split and requesting the next tile ahead change nothing.
#include "lsp_attn.h"

namespace lsp {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kTile = 16;  // queries per workgroup, keys per step of a wave
constexpr int kWaves = 8;  // way split of the keys

// over the four lanes (grp = 0..3) that hold scores of the same query
__device__ __forceinline__ float group_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16));
  return fmaxf(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ float group_sum(float x) {
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}

template <int D>
__global__ __launch_bounds__(64 * kWaves, 2) void attn_f32_kernel(AttnArgs a_in) {
  constexpr int CK = D / 16;  // 16-byte K (and Q) pieces per lane and row
  constexpr int CV = D / 64;  // 16-byte V pieces per lane and key
  constexpr int OP = D + 4;   // floats per merged O row
  AttnArgs a = a_in;
  a.layers = 1;
  fetch_operands(a);
  const Place pl = place<false>(a, kTile);
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
  for (int t0 = kTile * wave; t0 < T; t0 += kTile * kWaves) {
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
  for (int it = tid; it < kTile * (D / 4); it += 64 * kWaves) {
    const int qq = it / (D / 4), d = 4 * (it % (D / 4));
    if (q0 + qq >= N) continue;
    float M = sm[0][qq];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) M = fmaxf(M, sm[w][qq]);
    f32x4 acc = zero;
    float den = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float wgt = __builtin_amdgcn_exp2f(sm[w][qq] - M);  // 0 for a wave that saw no key (or only scores of -infinity)
      den += sl[w][qq] * wgt;
      acc += *reinterpret_cast<const f32x4 *>(&so[w][qq][d]) * wgt;
    }
    float *out = static_cast<float *>(a.out) + b * a.os[0] + int64_t(q0 + qq) * a.os[1] + h * a.os[2] + d;
    *reinterpret_cast<f32x4 *>(out) = acc * (1.0f / den);
  }
}

template <int D>
int32_t launch(AttnArgs a, hipStream_t st) {
  AttnLayers none;
  none.n = 0;
  // One unit after the other (taking the tiles of eight in turn costs a division, 0.1 of 6 us, and gains nothing), cut
  // into pieces only beyond 16 tiles per XCD (4 heads of 64: 64 queries x 192 keys 6.2 us whole and 6.5 in pieces, 256 x
  // 1280 19.5 and 19.9, three sequences of that 21.7 and 20.2).
  const int64_t nwg = place_grid(a, none, kTile, 0, 1, 16);
  if (nwg > kMaxGrid) {
    set_error("lsp_attn_step: launch of %lld workgroups is too large", (long long)nwg);
    return LSP_ERR_UNSUPPORTED;
  }
  attn_f32_kernel<D><<<grid_of(nwg), 64 * kWaves, 0, st>>>(a);
  LSP_CHECK_LAUNCH("lsp_attn_step: fp32 launch");
  return LSP_OK;
}

}  // namespace

int32_t launch_attn_f32(const AttnArgs &a, hipStream_t st) {
  if (a.D == 64) return launch<64>(a, st);
  if (a.D == 128) return launch<128>(a, st);
  set_error("lsp_attn_step: fp32 head_dim %d not built (64, 128)", a.D);
  return LSP_ERR_UNSUPPORTED;
}

}  // namespace lsp
