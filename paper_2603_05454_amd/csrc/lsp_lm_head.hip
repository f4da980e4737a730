// Output head fused with the per-position confidence (Algorithm 1 lines 4-5):
// logits z = hidden . weight^T on the CDNA4 matrix cores, reduced inside the
// same kernel to top-1 id, logit margin (Eq. 1) and top-1 probability, so the
// [rows x V] logits never reach memory.
//
// Formulation.  A workgroup computes tiles of 256 vocabulary entries x 256, 128 or
// 64 rows of the TRANSPOSED logits
//   Z^T[v, row] = W[v, :] . H[row, :]      (A operand = weight, B = hidden)
// with v_mfma_f32_16x16x32_bf16, so that a lane's accumulator registers hold four
// vocabulary entries of ONE row per 16x16 block: the running (max, runner-up,
// arg-max, sum of exponentials) of Eq. 1 is per-lane state, updated in
// increasing vocabulary order, and only the last combine crosses lanes (the four
// quarter-columns of a block, then the waves that share the rows).  Every
// (row, vocabulary tile) leaves one 16-byte partial; a second, tiny kernel
// folds a row's partials.
//
// Only ACTIVE rows are computed: tiles are cut from the list of them, over all
// sequences (127 rows left in four buffers of 256 are one tile of 128, not four
// of 256: 195 against 1100 us at 126 464 entries and K = 4096).
//
// The K loop is generated (gen_lm_head.py: fragments read one slice ahead, one
// barrier per K step, loads that never drain); workgroups are persistent, one
// per compute unit, and request the next tile's first steps before they reduce
// the current tile.
//
// What bounds it.  Many rows: the board's power limit, as in the library's product
// (8192 rows x 126 464 x 4096: 5.97 ms = 1.42 PFLOP/s with Eq. 1, 4.69 on operands that
// do not toggle; the library's product alone 5.75 and 4.55; the compiler-scheduled
// loop this replaced 7.7 and 6.6).  Few rows: the weight stream from HBM (37 rows:
// 169 us = 6.1 TB/s; 128 rows: 182 us).
#include <float.h>

#include <type_traits>

#include "lsp_common.h"
#include "lsp_lm_head.h"

namespace lsp {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;

constexpr int TV = 256;          // vocabulary entries per tile

struct Partial {
  float m1, m2, s;
  int32_t idx;
};

struct LmArgs {
  const uint16_t *hidden, *weight;
  int32_t B, S, K, V;
  int64_t hrs, hbs, wrs;  // element strides
  const int32_t *suffix_len;
  Partial *partials;
  int32_t VT;
};

// what a lane fetches in place of elements beyond K (and beyond its last tile)
__device__ __attribute__((aligned(1024))) unsigned char g_zeros[1024];

__device__ __forceinline__ float fmax_raw(float a, float b) {
  float d;
  asm("v_max_f32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
__device__ __forceinline__ float fmin_raw(float a, float b) {
  float d;
  asm("v_min_f32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
__device__ __forceinline__ float fmed3_raw(float a, float b, float c) {
  float d;
  asm("v_med3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}

// Fold of two partial results of one row; ties on the maximum keep the lower index.
// Symmetric bit by bit: which of the two a lane holds depends on where the row lies in its tile.
__device__ __forceinline__ Partial fold(Partial a, Partial b) {
  const float am = a.m1, bm = b.m1;
  const int ai = a.idx, bi = b.idx;
  const float M = fmax_raw(am, bm), low = fmin_raw(am, bm);
  const float w = low == M ? 1.f : __builtin_amdgcn_exp2f((low - M) * kLog2e);
  const bool a_top = am == M;
  const bool take_b = bm > am || (bm == am && bi < ai);
  Partial r;
  r.m1 = M;
  r.m2 = fmax_raw(low, fmax_raw(a.m2, b.m2));
  r.s = __builtin_fmaf(a_top ? b.s : a.s, w, a_top ? a.s : b.s);
  r.idx = take_b ? bi : ai;
  return r;
}

// One wave-wide load from global memory straight into LDS: lane l fetches 16
// bytes at its own address g and they land at lds_base + 16 l (lds_base is
// wave-uniform; the counter to wait on is vmcnt).
template <bool STREAM = false>  // true: with the non-temporal hint
__device__ __forceinline__ void load_to_lds(const char *g, unsigned char *lds_base) {
  __builtin_amdgcn_global_load_lds(g, (__attribute__((address_space(3))) void *)lds_base, 16, 0, STREAM ? 2 : 0);
}

// ---- active rows ---------------------------------------------------------------
// Rows are numbered over the ACTIVE ones only: compact row c is row i of sequence b
// with sum(N_0 .. N_{b-1}) + i = c.  `pre` holds the first compact row of every
// group of G = ceil(B / 512) sequences (G = 1 in any ordinary batch).
struct RowMap {
  const int32_t *pre;
  int32_t G, n;  // sequences per group, groups
  int32_t R;     // active rows
};
constexpr int kThreads = 512;

__device__ __forceinline__ int active_of(const LmArgs &a, int b) { return min(max(a.suffix_len[b], 0), a.S); }

__device__ __forceinline__ RowMap map_rows(const LmArgs &a, int32_t *pre, int32_t *wave_sum) {
  RowMap m;
  m.pre = pre;
  if (a.suffix_len == nullptr) {
    m.G = 0; m.n = 0; m.R = a.B * a.S;
    return m;
  }
  m.G = (a.B + kThreads - 1) / kThreads;
  m.n = (a.B + m.G - 1) / m.G;
  const int tid = threadIdx.x, lane = tid & 63;
  int own = 0;
  for (int b = tid * m.G; b < min((tid + 1) * m.G, a.B); ++b) own += active_of(a, b);
  int x = own;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(x, d);
    x += lane >= d ? o : 0;
  }
  if (lane == 63) wave_sum[tid >> 6] = x;
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) {
    before += w < (tid >> 6) ? wave_sum[w] : 0;
    total += wave_sum[w];
  }
  pre[tid] = before + x - own;
  m.R = __builtin_amdgcn_readfirstlane(total);
  __syncthreads();
  return m;
}
// sequence and row of compact row c < R
__device__ __forceinline__ void row_at(const LmArgs &a, const RowMap &m, int c, int &b, int &i) {
  if (m.G == 0) {
    b = c / a.S;
    i = c - b * a.S;
    return;
  }
  int lo = 0, hi = m.n;  // the last group that starts at or before c
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (m.pre[mid] <= c) lo = mid; else hi = mid;
  }
  b = lo * m.G;
  i = c - m.pre[lo];
  if (m.G > 1) {
    for (int n = active_of(a, b); i >= n; n = active_of(a, b)) { i -= n; ++b; }
  }
}

// ---- tiles of a workgroup ---------------------------------------------------------
// Workgroups go to the 8 XCDs round-robin by id; an XCD owns a run of consecutive
// vocabulary tiles and its workgroups take them in turn (tiles dealt to the XCDs one by one
// put all eight at the same distance of few powers of two, see the start times in run_tiles:
// 37 rows x 126 464 entries x K = 4096 in step 236 us, in runs 177).  In that order, up to four
// row tiles of a group of vocabulary tiles come side by side: the 32 workgroups an XCD
// runs at a time read every weight slice four times and every hidden slice
// eight times out of one L2.
struct Tiles {
  int32_t *row;              // place b * S + i of the rows of two row tiles ...
  int64_t *off;              // ... and their byte offset in `hidden`; table k starts at k * cap
  int cap;
  RowMap map;
  int tr;                    // rows per row tile
  int first, nv, RT, VB, total;  // the XCD's vocabulary tiles, row tiles, vocabulary tiles per group, tiles
};
__device__ __forceinline__ void cut_rows(const LmArgs &a, Tiles &t) {
  const int R = t.map.R;
  t.tr = tile_rows(R, a.VT);
  t.RT = (R + t.tr - 1) / t.tr;
  const int xcd = blockIdx.x & 7, slots = gridDim.x >> 3;
  t.nv = a.VT / 8 + (xcd < a.VT % 8);
  t.first = xcd * (a.VT / 8) + min(xcd, a.VT % 8);
  t.VB = max(1, slots / max(1, min(t.RT, 4)));
  t.total = t.nv * t.RT;
}
struct Cursor {
  int m, vt, rt, buf;  // index in the list, tile, which of the two row tables holds its rows
};
__device__ __forceinline__ void tile_at(const Tiles &t, int m, int &vt, int &rt) {
  const int per = t.VB * t.RT, vg = m / per, q = m - vg * per;
  const int g = min(t.VB, t.nv - vg * t.VB);
  vt = t.first + vg * t.VB + q % g;
  rt = q / g;
}
__device__ __forceinline__ void fill_rows(const LmArgs &a, const Tiles &t, int buf, int rt) {
  const int i = threadIdx.x;
  if (i < t.cap) {
    int b, r;
    row_at(a, t.map, min(rt * t.tr + i, t.map.R - 1), b, r);  // rows beyond the last repeat it (never written)
    t.row[buf * t.cap + i] = b * a.S + r;
    t.off[buf * t.cap + i] = (int64_t(b) * a.hbs + int64_t(r) * a.hrs) * 2;
  }
  __syncthreads();
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));

// Eq. 1 on N logits of one row held by a lane: element e is vocabulary entry vbase + 16 (e/4) + e%4.
template <int N>
__device__ __forceinline__ Partial reduce(float (&x)[N], int vbase, int V, bool ragged) {
  if (ragged) {  // (a branch of its own, nothing of it formed ahead: two more instructions per logit otherwise)
    int left = V - vbase;
    asm volatile("" : "+v"(left));
#pragma unroll
    for (int e = 0; e < N; ++e) x[e] = 16 * (e >> 2) + (e & 3) >= left ? -INFINITY : x[e];
  }
  float m1 = -INFINITY, m2 = -INFINITY;
  int code = 0;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    code = x[e] > m1 ? e : code;
    m2 = fmed3_raw(m1, m2, x[e]);
    m1 = fmax_raw(m1, x[e]);
  }
  // sum of exp2(z*log2e - rc) against the ROUNDED product rc = m1*log2e (one fma +
  // exp2 per logit), then taken off that reference with an fma of its own, which
  // cancels the rounding of rc exactly
  const float ref = m1 == -INFINITY ? 0.f : m1;
  const float rc = ref * kLog2e;
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < N; ++e) s += __builtin_amdgcn_exp2f(__builtin_fmaf(x[e], kLog2e, -rc));
  s *= __builtin_amdgcn_exp2f(__builtin_fmaf(-ref, kLog2e, rc));
  Partial p;
  p.m1 = m1; p.m2 = m2; p.s = s;
  p.idx = vbase + 16 * (code >> 2) + (code & 3);
  return p;
}
// The four lanes of a row fold their results, each pair exchanging half of its row blocks: lanes 32
// apart first, then lanes 16 apart, so that no lane folds what another one folds as well.
// Which lane keeps which half: the upper of the two (in lane number) takes `hi`, the lower one `lo`; the swap leaves a lane with
// its own half and the other lane's, in an order that the fold does not see.
template <int D>
__device__ __forceinline__ void swap_halves(uint32_t &lo, uint32_t &hi) {
  const auto r = D == 32 ? __builtin_amdgcn_permlane32_swap(lo, hi, false, false) : __builtin_amdgcn_permlane16_swap(lo, hi, false, false);
  lo = r[0];
  hi = r[1];
}
template <int D>
__device__ __forceinline__ Partial exchange(const Partial &lo, const Partial &hi) {
  uint32_t a[4] = {__builtin_bit_cast(uint32_t, lo.m1), __builtin_bit_cast(uint32_t, lo.m2), __builtin_bit_cast(uint32_t, lo.s), uint32_t(lo.idx)};
  uint32_t b[4] = {__builtin_bit_cast(uint32_t, hi.m1), __builtin_bit_cast(uint32_t, hi.m2), __builtin_bit_cast(uint32_t, hi.s), uint32_t(hi.idx)};
#pragma unroll
  for (int k = 0; k < 4; ++k) swap_halves<D>(a[k], b[k]);
  auto part = [](const uint32_t (&x)[4]) {
    return Partial{__builtin_bit_cast(float, x[0]), __builtin_bit_cast(float, x[1]), __builtin_bit_cast(float, x[2]), int32_t(x[3])};
  };
  return fold(part(a), part(b));
}
// One thread per row folds the results of the tile's four groups of entries and leaves the tile's partial result.
__device__ __forceinline__ void finish_tile(const LmArgs &a, const Tiles &tb, const Partial *lds_part, const Cursor &cur, int vt) {
  const int t = threadIdx.x;
  if (t >= tb.tr || cur.rt * tb.tr + t >= tb.map.R) return;
  Partial p = lds_part[t * 4];
#pragma unroll
  for (int u = 1; u < 4; ++u) p = fold(p, lds_part[t * 4 + u]);
  a.partials[int64_t(tb.row[cur.buf * tb.cap + t]) * a.VT + vt] = p;
}

// ---- tiles -----------------------------------------------------------------------------
// Geometry by tile height (the same table as in gen_lm_head.py): waves along vocabulary and rows, LDS stages.
template <int H> struct Shape;
template <> struct Shape<256> { static constexpr int WV = 2, WR = 4, NS = 2; };
template <> struct Shape<128> { static constexpr int WV = 4, WR = 2, NS = 3; };
template <> struct Shape<64> { static constexpr int WV = 4, WR = 2, NS = 3; };
constexpr int KB = 64, TILE_W = TV * KB * 2;  // K step, bytes of a weight tile's step
template <int H> constexpr int stage_bytes() { return (TV + H) * KB * 2; }
// behind the stages: the next tile's hidden pointers (H = 256), then the partial results of four groups of entries per row
template <int H> constexpr int lds_bytes() { return Shape<H>::NS * stage_bytes<H>() + H * 4 * 16; }

template <int N> struct UVec;
template <> struct UVec<2> { typedef u32x2 T; };
template <> struct UVec<4> { typedef u32x4 T; };
template <> struct UVec<8> { typedef u32x8 T; };

// All tiles of a workgroup: K loop, Eq. 1, one partial result per row and tile.
// STREAM: weights that no cache can hold, read once (one row tile), are loaded with the non-temporal hint (37 rows x
// 126 464 entries: K = 3584 159 -> 141 us, 4096 in step 236 -> 212; 200 rows 262 -> 252).  With more row tiles a slice
// is read again out of L2, and the hint costs what it saves there (300 rows 386 -> 457).
template <int H, bool STREAM>
__device__ __forceinline__ void run_tiles(const LmArgs &a, unsigned char *smem, const Tiles &tb, Cursor cur) {
  constexpr int WV = Shape<H>::WV, WR = Shape<H>::WR, NS = Shape<H>::NS, STG = stage_bytes<H>();
  constexpr int MV = TV / WV / 16, MR = H / WR / 16, LH = H / 64;  // 16x16 blocks per wave, hidden loads per lane and step
  unsigned char *part = smem + NS * STG;
  const int KS_real = (a.K + KB - 1) / KB, KS = max(KS_real, NS);
  const int tail = (a.K % KB) / 8;
  const uint64_t zeros = reinterpret_cast<uint64_t>(g_zeros);
  int stage = 0;           // stage that holds step 0 of the current tile
  bool requested = false;  // its first steps have been requested by the previous tile's loop
  // Weight rows a multiple of 4 KB apart (K = 2048, 4096, 8192) keep workgroups that are at the same k on few memory
  // channels, so where the weight stream is the bound - one low row tile, every compute unit busy - the
  // workgroups of an XCD start a K step's time (3200 cycles) apart in 16 phases.  37 rows: K = 2048 115 -> 99 us
  // (126 464 entries) and 140 -> 125 (152 064), K = 4096 151 -> 138 (80 000) and 216 -> 217 (152 064), 8192 325 -> 315;
  // at 126 464 x 4096, where the runs of the XCDs happen to lie well, 157 -> 169.  It costs 5 % at other pitches,
  // 9 % at K = 1024 (16 steps per tile), 2 % where not every unit has a tile.
  if (H <= 128 && tb.RT == 1 && tb.nv >= kComputeUnits / 8 && KS_real >= 32 && a.wrs % 2048 == 0)
    for (int p = int(blockIdx.x >> 3) & 15; p > 0; --p) __builtin_amdgcn_s_sleep(50);
  for (;;) {
    // (opaque: what is derived from the thread id is formed again for every tile - kept across the loop it would spill)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wv = wave % WV, wr = wave / WV, l16 = lane & 15, grp = lane >> 4;
    // loader: this lane's row (of 8) and 16-byte chunk of it
    const int lrow = lane >> 3, chunk = (lane & 7) ^ (4 * (wave & 1) + (lane >> 4));
    const int vt = cur.vt, v0 = vt * TV;
    int vn = vt, rn = cur.rt, nbuf = cur.buf;
    const bool more = cur.m + int(gridDim.x >> 3) < tb.total;
    if (more) tile_at(tb, cur.m + (gridDim.x >> 3), vn, rn);
    if (rn != cur.rt) {
      nbuf = cur.buf ^ 1;
      fill_rows(a, tb, nbuf, rn);
    }
    auto hidden_at = [&](int buf, int i) {  // this lane's piece of load i of a hidden tile, at k = 0
      return reinterpret_cast<uint64_t>(a.hidden) + tb.off[buf * tb.cap + 8 * (wave + 8 * i) + lrow] + 16 * chunk;
    };
    uint64_t w[4], h[LH];  // this lane's pieces of a step: weight rows, hidden rows
#pragma unroll
    for (int i = 0; i < 4; ++i)
      w[i] = reinterpret_cast<uint64_t>(a.weight) + int64_t(min(v0 + 8 * (wave + 8 * i) + lrow, a.V - 1)) * a.wrs * 2 + 16 * chunk;
#pragma unroll
    for (int i = 0; i < LH; ++i) h[i] = hidden_at(cur.buf, i);
    if (!requested) {
      stage = 0;
#pragma unroll
      for (int p = 0; p < NS; ++p) {
        const bool in = p * KB + 8 * chunk < a.K;
        unsigned char *st = smem + p * STG + 1024 * wave;
#pragma unroll
        for (int i = 0; i < 4; ++i) load_to_lds<STREAM>(reinterpret_cast<const char *>(in ? w[i] + p * 2 * KB : zeros), st + 8192 * i);
#pragma unroll
        for (int i = 0; i < LH; ++i) load_to_lds(reinterpret_cast<const char *>(in ? h[i] + p * 2 * KB : zeros), st + TILE_W + 8192 * i);
      }
    }
    u32x8 wptr;  // of the next step to request
    typename UVec<2 * LH>::T hptr;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint64_t p = w[i] + NS * 2 * KB;
      wptr[2 * i] = uint32_t(p);
      wptr[2 * i + 1] = uint32_t(p >> 32);
    }
#pragma unroll
    for (int i = 0; i < LH; ++i) {
      const uint64_t p = h[i] + NS * 2 * KB;
      hptr[2 * i] = uint32_t(p);
      hptr[2 * i + 1] = uint32_t(p >> 32);
    }

    // The loads of a tile's last steps are followed by the first ones of the next tile where that is plain
    // pointer arithmetic: whole K steps, no vocabulary entry beyond V in either.
    const bool cross = more && tail == 0 && KS_real > NS && v0 + TV <= a.V && vn * TV + TV <= a.V;
    const uint64_t wstep = int64_t(vn - vt) * TV * a.wrs * 2 - int64_t(KS) * (2 * KB);

    f32x16 acc[MV * MR / 4];
#pragma unroll
    for (int k = 0; k < MV * MR / 4; ++k)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[k][r] = 0.f;
    {
      const uint32_t lds0 = uint32_t(uintptr_t((__attribute__((address_space(3))) unsigned char *)smem));
      u32x4 addr[NS];  // fragment addresses per stage: weight and hidden of k-slice 0, of k-slice 1
#pragma unroll
      for (int st = 0; st < NS; ++st)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          const uint32_t c = 16 * ((4 * kk + grp) ^ (l16 >> 1));
          addr[st][2 * kk] = lds0 + st * STG + (wv * (TV / WV) + l16) * (2 * KB) + c;
          addr[st][2 * kk + 1] = lds0 + st * STG + TILE_W + (wr * (H / WR) + l16) * (2 * KB) + c;
        }
      const uint32_t ldsw = lds0 + 1024 * wave, ks = KS, phase = stage, go_on = __builtin_amdgcn_readfirstlane(int(cross));
      const uint32_t event = min(KS, max(a.K / KB, NS));  // the first thing to happen to the pointers: the ragged end of K, or the next tile
      const uint32_t zlo = uint32_t(zeros), zhi = uint32_t(zeros >> 32);
      const uint64_t zmask = __ballot(chunk >= tail);
      if constexpr (H == 256) {
        // registers are full: the next tile's hidden pointers wait in LDS (a lane reads what it wrote)
#pragma unroll
        for (int i = 0; i < LH; i += 2) {
          const uint64_t h0 = hidden_at(nbuf, i), h1 = hidden_at(nbuf, i + 1);
          *reinterpret_cast<u32x4 *>(part + 4096 * i + 16 * tid) = u32x4{uint32_t(h0), uint32_t(h0 >> 32), uint32_t(h1), uint32_t(h1 >> 32)};
        }
        const uint32_t next = lds0 + NS * STG + 16 * tid;
        if constexpr (STREAM) {
#define LSP_WEIGHT_HINT " nt"
#include "lsp_lm_head_loop_256.inc"
#undef LSP_WEIGHT_HINT
        } else {
#define LSP_WEIGHT_HINT ""
#include "lsp_lm_head_loop_256.inc"
#undef LSP_WEIGHT_HINT
        }
      } else {
        typename UVec<2 * LH>::T next;
#pragma unroll
        for (int i = 0; i < LH; ++i) {
          const uint64_t h = hidden_at(nbuf, i);
          next[2 * i] = uint32_t(h);
          next[2 * i + 1] = uint32_t(h >> 32);
        }
        if constexpr (H == 128 && STREAM) {
#define LSP_WEIGHT_HINT " nt"
#include "lsp_lm_head_loop_128.inc"
#undef LSP_WEIGHT_HINT
        } else if constexpr (H == 128) {
#define LSP_WEIGHT_HINT ""
#include "lsp_lm_head_loop_128.inc"
#undef LSP_WEIGHT_HINT
        } else if constexpr (STREAM) {
#define LSP_WEIGHT_HINT " nt"
#include "lsp_lm_head_loop_64.inc"
#undef LSP_WEIGHT_HINT
        } else {
#define LSP_WEIGHT_HINT ""
#include "lsp_lm_head_loop_64.inc"
#undef LSP_WEIGHT_HINT
        }
      }
    }
    requested = cross;
    stage = (stage + KS) % NS;

    // element r of 16x16 block (i, j) is z[v][row], v = v0 + wv*(TV/WV) + 16 i + 4 grp + r (increasing in (i, r)),
    // row = wr*(H/WR) + 16 j + l16
    // Four groups of 64 entries per row and tile at every height, so that a row's sum of exponentials has one order
    // (a wave of the 256-row tile holds two of them; what reducing them apart costs, 0.6 us of a 100 us tile, the register
    // swaps of exchange() give back: 838 rows x 152 064 entries x K = 1024 304 us with LDS shuffles, 297 now).
    Partial *lds_part = reinterpret_cast<Partial *>(part);  // [H][4]
    const bool up32 = lane >= 32, up16 = (lane & 16) != 0;
#pragma unroll
    for (int u = 0; u < MV / 4; ++u) {
      Partial pj[MR];
#pragma unroll
      for (int j = 0; j < MR; ++j) {
        float x[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) x[e] = acc[(j * MV + 4 * u) / 4][e];
        pj[j] = reduce<16>(x, v0 + wv * (TV / WV) + 64 * u + 4 * grp, a.V, v0 + TV > a.V);
      }
      Partial p;
      int j;
      if constexpr (MR == 4) {
        p = exchange<16>(exchange<32>(pj[0], pj[2]), exchange<32>(pj[1], pj[3]));
        j = 2 * up32 + up16;
      } else {
        p = exchange<32>(pj[0], pj[1]);
        p = exchange<16>(p, p);
        j = up32;
      }
      lds_part[(wr * (H / WR) + 16 * j + l16) * 4 + wv * (MV / 4) + u] = p;
    }
    __syncthreads();
    finish_tile(a, tb, lds_part, cur, vt);
    __syncthreads();  // the partial results and the row tables may be overwritten
    cur.m += gridDim.x >> 3;
    cur.vt = vn; cur.rt = rn; cur.buf = nbuf;
    if (!more) break;
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): nothing is still on its way into LDS
}

// Weights (elements) from which they are streamed: 320 MB, a quarter more than the chip's last-level cache holds.  Smaller
// ones are partly or wholly still there from the step before, as long as they are loaded without the hint.  The same
// weights step after step, 37 rows, with and without it: 268 MB (65 536 x 2048) 68 and 52 us, 328 MB (40 000 x 4096)
// 70 and 70, 450 MB (110 000 x 2048) 93 and 102.
constexpr int64_t kStreamWeights = int64_t(320) << 19;

// Persistent kernel: one workgroup per compute unit walks its tiles.  How many rows are active, and with that the height of
// the tiles, is only known here (two kernels, one of which left at once, took 2 us more).  TALL: there may be tiles of 256
// rows; buffers of up to 128 never have any, and without their loop the kernel needs no scratch and starts sooner.
template <bool TALL>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void lm_head_kernel(LmArgs a) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  __shared__ int32_t s_pre[kThreads], s_wave[kThreads / 64];
  __shared__ int32_t s_row[2 * 128];
  __shared__ int64_t s_off[2 * 128];
  Tiles tb;
  tb.map = map_rows(a, s_pre, s_wave);
  cut_rows(a, tb);
  Cursor cur = {int(blockIdx.x >> 3), 0, 0, 0};
  if (cur.m >= tb.total) return;
  tile_at(tb, cur.m, cur.vt, cur.rt);
  auto run = [&](auto stream) {
    constexpr bool STREAM = decltype(stream)::value;
    tb.row = s_row; tb.off = s_off; tb.cap = 128;
    if constexpr (TALL)
      if (tb.tr == 256) {  // (the tables of taller tiles lie behind their two stages, where the lower ones have a third)
        tb.off = reinterpret_cast<int64_t *>(smem + lds_bytes<256>());
        tb.row = reinterpret_cast<int32_t *>(tb.off + 2 * 256);
        tb.cap = 256;
        fill_rows(a, tb, 0, cur.rt);
        run_tiles<256, STREAM>(a, smem, tb, cur);
        return;
      }
    fill_rows(a, tb, 0, cur.rt);
    if (min(tb.tr, tb.map.R) <= 64) run_tiles<64, STREAM>(a, smem, tb, cur);
    else run_tiles<128, STREAM>(a, smem, tb, cur);
  };
  if (tb.RT == 1 && int64_t(a.V) * a.wrs >= kStreamWeights) run(std::true_type{});
  else run(std::false_type{});
}

// One wave per row folds the row's VT partials and writes the three results.  (A grid dimension ends at 2^32 threads and a
// launch beyond loses its last workgroups without an error: more rows than kFinishGrid workgroups hold are taken in turn.)
constexpr int kFinishGrid = 1 << 20;
__global__ __launch_bounds__(256) void lm_head_finish_kernel(const Partial *__restrict__ partials, int rows, int S, int VT,
                                                             const int32_t *__restrict__ suffix_len,
                                                             int32_t *__restrict__ top1_id,
                                                             float *__restrict__ top1_prob,
                                                             float *__restrict__ margin) {
  const int lane = threadIdx.x & 63;
  for (int r = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); r < rows; r += gridDim.x * (blockDim.x >> 6)) {
    if (suffix_len != nullptr && (r % S) >= suffix_len[r / S]) continue;
    Partial p;
    p.m1 = -INFINITY; p.m2 = -INFINITY; p.s = 0.f; p.idx = 0x7fffffff;
    // eight loads in flight (one after the other they were most of this kernel)
    constexpr int U = 8;
    for (int t = lane; t < VT; t += 64 * U) {
      Partial q[U];
#pragma unroll
      for (int u = 0; u < U; ++u) q[u] = partials[int64_t(r) * VT + min(t + 64 * u, VT - 1)];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (t + 64 * u < VT) p = fold(p, q[u]);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
      Partial o;
      o.m1 = __shfl_xor(p.m1, d); o.m2 = __shfl_xor(p.m2, d); o.s = __shfl_xor(p.s, d); o.idx = __shfl_xor(p.idx, d);
      p = fold(p, o);
    }
    if (lane == 0) {
      top1_id[r] = p.idx;
      margin[r] = p.m1 - p.m2;
      top1_prob[r] = 1.0f / p.s;
    }
  }
}

template <bool TALL>
int32_t launch_lm_head(const LmArgs &a, hipStream_t st) {
  // at most one workgroup per compute unit, a multiple of 8 (the same number on every XCD)
  const int64_t rows = int64_t(a.B) * a.S;
  const int64_t per_xcd = (int64_t(a.VT) + 7) / 8 * ((rows + 63) / 64);
  const unsigned nwg = 8 * unsigned(per_xcd < kComputeUnits / 8 ? per_xcd : kComputeUnits / 8);
  constexpr size_t lds = lds_bytes<128>();
  static_assert(lds_bytes<256>() + 2 * 256 * 12 <= lds && lds_bytes<64>() <= lds, "");
  static std::atomic<uint64_t> configured{0};  // per instantiation, one bit per device
  if (const int32_t rc = ensure_dynamic_lds(reinterpret_cast<const void *>(lm_head_kernel<TALL>), lds, configured, "lsp_lm_head_confidence: hipFuncSetAttribute")) return rc;
  lm_head_kernel<TALL><<<dim3(nwg), kThreads, lds, st>>>(a);
  LSP_CHECK_LAUNCH("lsp_lm_head_confidence: launch");
  return LSP_OK;
}

}  // namespace
}  // namespace lsp

extern "C" size_t lsp_lm_head_confidence_workspace_bytes(int32_t B, int32_t S, int32_t V) {
  if (B <= 0 || S <= 0 || V <= 0) return 0;
  const size_t VT = (size_t(V) + lsp::TV - 1) / lsp::TV;
  return size_t(B) * S * VT * sizeof(lsp::Partial);
}

extern "C" int32_t lsp_lm_head_confidence(int32_t dtype, const void *hidden, const void *weight, int32_t B,
                                          int32_t S, int32_t K, int32_t V, int64_t hidden_row_stride,
                                          int64_t hidden_batch_stride, int64_t weight_row_stride,
                                          const int32_t *suffix_len, int32_t *top1_id, float *top1_prob,
                                          float *margin, void *workspace, size_t workspace_bytes,
                                          void *stream) {
  using namespace lsp;
  LSP_CHECK_ARG(dtype == LSP_F32 || dtype == LSP_BF16, "lsp_lm_head_confidence: unknown dtype %d", dtype);
  if (dtype != LSP_BF16) {
    set_error("lsp_lm_head_confidence: only bf16 operands are built");
    return LSP_ERR_UNSUPPORTED;
  }
  LSP_CHECK_ARG(hidden && weight && top1_id && top1_prob && margin, "lsp_lm_head_confidence: null pointer");
  LSP_CHECK_ARG(B > 0 && S > 0 && V >= 2 && K > 0, "lsp_lm_head_confidence: need B>0, S>0, K>0, V>=2 (got %d %d %d %d)", B, S, K, V);
  LSP_CHECK_ARG(K % 8 == 0, "lsp_lm_head_confidence: K must be a multiple of 8 (got %d)", K);
  LSP_CHECK_ARG(int64_t(B) * S <= 0x3fffffff, "lsp_lm_head_confidence: B*S too large");
  if (hidden_row_stride == 0) hidden_row_stride = K;
  if (hidden_batch_stride == 0) hidden_batch_stride = int64_t(S) * hidden_row_stride;
  if (weight_row_stride == 0) weight_row_stride = K;
  LSP_CHECK_ARG(hidden_row_stride >= K && weight_row_stride >= K && hidden_batch_stride >= 0 &&
                    hidden_row_stride % 8 == 0 && hidden_batch_stride % 8 == 0 && weight_row_stride % 8 == 0,
                "lsp_lm_head_confidence: strides must be >= K and multiples of 8 elements");
  LSP_CHECK_ARG(aligned16(hidden) && aligned16(weight), "lsp_lm_head_confidence: hidden and weight must be 16-byte aligned");
  const size_t need = lsp_lm_head_confidence_workspace_bytes(B, S, V);
  if (workspace == nullptr || workspace_bytes < need || !aligned16(workspace)) {
    set_error("lsp_lm_head_confidence: workspace of %zu bytes (16-byte aligned) required, got %zu", need, workspace_bytes);
    return LSP_ERR_WORKSPACE;
  }
  LmArgs a;
  a.hidden = static_cast<const uint16_t *>(hidden);
  a.weight = static_cast<const uint16_t *>(weight);
  a.B = B; a.S = S; a.K = K; a.V = V;
  a.hrs = hidden_row_stride; a.hbs = hidden_batch_stride; a.wrs = weight_row_stride;
  a.suffix_len = suffix_len;
  a.partials = static_cast<Partial *>(workspace);
  const int64_t rows = int64_t(B) * S;
  a.VT = (V + TV - 1) / TV;
  if (int64_t(a.VT) * ((rows + 63) / 64) > 0x7fffffff) {
    set_error("lsp_lm_head_confidence: %lld tiles are too many", (long long)(int64_t(a.VT) * ((rows + 63) / 64)));
    return LSP_ERR_UNSUPPORTED;
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int32_t rc = rows > 128 ? launch_lm_head<true>(a, st) : launch_lm_head<false>(a, st);
  if (rc != LSP_OK) return rc;
  const int64_t finish = (rows + 3) / 4;
  lm_head_finish_kernel<<<dim3(unsigned(finish < kFinishGrid ? finish : kFinishGrid)), 256, 0, st>>>(
      a.partials, int(rows), S, a.VT, suffix_len, top1_id, top1_prob, margin);
  LSP_CHECK_LAUNCH("lsp_lm_head_confidence: finish launch");
  return LSP_OK;
}
