// Internal: resolved arguments shared by the attention kernels.
#pragma once
#include "lsp_common.h"

namespace lsp {

// Division of 0 <= n < 2^31 by a number that the host knows: n / d = n m / 2^(31 + s) with m = ceil(2^(31 + s) / d),
// s = ceil(log2 d).  Exact: m d exceeds 2^(31 + s) by less than d <= 2^s, which adds less than 1 / d to a quotient of n < 2^31.
// Three scalar instructions instead of some forty dependent ones; a workgroup does four on the way to its first
// load (28/4 heads, 64 rows on 200: 8.60 -> 8.39 us).
struct Div {
  uint32_t m, s;
};
inline Div div_by(int64_t d) {
  Div v = {0, 0};
  while ((int64_t(1) << v.s) < d) ++v.s;
  v.m = uint32_t(((uint64_t(1) << (31 + v.s)) + d - 1) / d);
  return v;
}
__device__ __forceinline__ int quotient(int n, const Div &v) { return int(__umulhi(2u * uint32_t(n), v.m) >> v.s); }

struct AttnArgs {
  const void *q, *k_suf, *v_suf, *k_cache, *v_cache;
  void *out;
  const int32_t *prefix_len, *suffix_len;
  int32_t B, S, Hq, Hkv;
  int32_t rep, chunk, spread, layers, unit_group, per_unit;  // placement of the workgroups (place_grid); read first, with the line above
  int32_t table;  // operands from AttnLayers
  Div by_group, by_unit_group, by_units, by_heads, by_rep;  // its divisors: unit_group * chunk, unit_group, B * Hkv, Hkv, rep
  int32_t D, C;
  int32_t spread_blocks, units;  // head_dim 128, contiguous cache: blocks of a sequence that are still spread (spread_limit); units of the launch
  int32_t rounding;  // head_dim 128, contiguous cache: which reference short tiles' probabilities are rounded against (Reference)
  float scale;
  int64_t qs[3], ks[3], cs[3], os[3];  // element strides: batch, row, head
  void *workspace;
  const int32_t *cache_rows;  // gather form only: key t < P_b of sequence b is cache row cache_rows[b*C + t]; else null
};

// Operands of several layers for ONE launch (lsp_attn_step_layers): passed to the
// kernels by value, the layer is the slow index of the placement.  n = 0: single-layer call,
// the pointers in AttnArgs are used as they are.
constexpr int kMaxAttnLayers = 32;
struct AttnLayers {
  int32_t n;
  const void *q[kMaxAttnLayers], *k_suf[kMaxAttnLayers], *v_suf[kMaxAttnLayers];
  const void *k_cache[kMaxAttnLayers], *v_cache[kMaxAttnLayers];
  void *out[kMaxAttnLayers];
};
__device__ __forceinline__ void fetch_operands(const AttnArgs &a) {
  fetch_now(a.q, a.k_suf, a.v_suf, a.k_cache, a.v_cache, a.out, a.scale, a.C, a.qs[0], a.qs[1], a.qs[2], a.ks[0], a.ks[1], a.ks[2],
            a.cs[0], a.cs[1], a.cs[2], a.os[0], a.os[1], a.os[2]);
}
// Active and cached rows of a sequence, requested together:
//  * both through the scalar cache (as ordinary loads one trip followed the other, with the early exit between them: 32 layers, 2 x
//    724 rows of 32/32 heads with 10 active on 305 193 -> 181 us, 12 x 246 with 22 on 62 414 -> 393);
//  * the active ones only, where heads of a group share workgroups: none of those launches is then slower than with two ordinary loads,
//    which some are with both scalar (28/4 heads, 32 layers, 5 x 335 rows with 2 active on 1669 322 us ordinary, 327 scalar, 322 so; 7 x 168
//    with 1 on 2471 803, 783 to 834, 790; 2 x 455 with 11 on 404 64.0, 61.6, 63.0);
//  * neither, where every workgroup has rows (suffix buffers of one tile).  Their waves then wait for an issue slot less often: 3 x 71 rows of
//    32/32 heads with 20 active on 53, 32 layers, 59.5 -> 56.7 us; with the merge in pieces (merge_store) as well 55.3, and 11.9 of 54.0
//    million wave cycles are such waits, 16.9 of 61.9 before, for 4 to 6 % more vector and LDS instructions.
struct Lengths {
  int N, P;
};
enum LengthLoads { kScalarLengths, kScalarActive, kOrdinaryLengths };
template <LengthLoads HOW = kScalarLengths>
__device__ __forceinline__ Lengths lengths_of(const AttnArgs &a, int b) {
  typedef const __attribute__((address_space(4))) int32_t *Constant;
  int n, p;
  if constexpr (HOW == kScalarLengths) {
    n = reinterpret_cast<Constant>(reinterpret_cast<uint64_t>(a.suffix_len))[b];
    p = reinterpret_cast<Constant>(reinterpret_cast<uint64_t>(a.prefix_len))[b];
    fetch_now(n, p);
  } else {
    p = a.prefix_len[b];
    n = HOW == kOrdinaryLengths ? a.suffix_len[b] : reinterpret_cast<Constant>(reinterpret_cast<uint64_t>(a.suffix_len))[b];
  }
  return {min(max(n, 0), a.S), min(max(p, 0), a.C)};
}
// This workgroup's layer replaces the operand pointers.
__device__ __forceinline__ void for_layer(AttnArgs &a, const AttnLayers &L, int l) {
  if (a.table) {
    a.q = L.q[l]; a.k_suf = L.k_suf[l]; a.v_suf = L.v_suf[l];
    a.k_cache = L.k_cache[l]; a.v_cache = L.v_cache[l]; a.out = L.out[l];
  }
}

// A grid dimension is limited in THREADS to 2^32: launches of more workgroups than this go on in y.
// (The last row of such a grid may reach beyond the workgroups asked for: kernels check their id.)
constexpr int kGridBits = 20;
constexpr int64_t kMaxGrid = int64_t(0x7ff) << kGridBits;
inline dim3 grid_of(int64_t nwg) {
  const int64_t x = int64_t(1) << kGridBits;
  return nwg <= x ? dim3(unsigned(nwg)) : dim3(unsigned(x), unsigned((nwg + x - 1) / x));
}
__device__ __forceinline__ int workgroup_id() { return blockIdx.y << kGridBits | blockIdx.x; }

// Workgroup placement of all attention kernels.  Workgroups are handed to the 8
// XCDs round-robin by linear id, and each XCD has its own L2.  All workgroups
// that read the same K/V stream - the query tiles of every query head of one
// (sequence, KV head) unit - are therefore given ids that are congruent modulo
// 8, so the stream is fetched into one L2 instead of eight.
// Within an XCD the order is: groups of kUnitGroup units; inside a group the
// query tile is the slow index and the unit the fast one.  Tiles at or beyond
// the active length exit at once, and in a decode loop that is most tiles of
// every unit: with the tile as the fast index the surviving workgroups would sit
// at a fixed stride of the dispatch order, which the hardware maps onto a fixed
// subset of the compute units (measured: the time did not drop at all when the
// active length fell from 1024 to 256).  Runs of kUnitGroup live workgroups
// spread over all of them, and the tiles of one unit still run close enough
// together to share its K/V stream in L2.
// A launch of up to one and a half times the workgroups that run at once is one group: the tiles of a unit meet anyway,
// and the live workgroups, then first in the order, find a compute unit each before the hardware gives one a second
// (one layer, 32 heads, 4 x 128 rows with 50 active on 1000: 22.2 us in groups of 8 units, 16.9 in one; 3 x 700
// with 300 active on 500: 31.4, 27.5).  With two rounds the tiles of a unit would no longer meet (8 x 512 on 512: 82, 87).
// For the live ones' sake the tile is the slow index also among the heads of a unit.
constexpr int kUnitGroup = 8;
struct Place {
  int layer, b, g, h, q0;
  bool valid;
};
// Units are numbered over layers, sequences and KV heads.  When they are few, each is cut into
// 2^spread pieces so that every XCD gets as many: four KV heads of
// one sequence kept four of the eight XCDs idle (28 query heads, one layer, prefix 4096, suffix
// 1024: 234 us whole, 139 us in two pieces; fp32, 8 query heads of 64 on one KV head, same lengths:
// 905 us whole, 122 in eight).  A piece takes every 2^spread-th of the unit's (tile, head) list, so that the live tiles, which are
// the first ones, are shared evenly; as runs of that list the last pieces' XCDs had none (28/4 heads, 5 x 400 rows on 3500 with
// 128 active 80 -> 64 us, with 300 138 -> 90, all 156 -> 122).
struct UnitPlace {
  int layer, b, g, w;  // w: this workgroup's number among those of its unit
  bool valid;
};
template <bool GROUPS = true>  // false: groups of one unit
__device__ __forceinline__ UnitPlace place_in_unit(const AttnArgs &a, int n) {
  UnitPlace p;
  const int chunk = a.chunk;
  const int m8 = n >> 3;
  const int G = GROUPS ? a.unit_group : 1;
  const int grp = quotient(m8, a.by_group), r = m8 - grp * (G * chunk);
  int wu = GROUPS ? quotient(r, a.by_unit_group) : r, layer = 0;
  int unit = (grp * G + r - wu * G) * 8 + (n & 7);
  if (a.spread > 0) {
    wu = (wu << a.spread) + (unit & ((1 << a.spread) - 1));
    unit >>= a.spread;
  }
  const int units = a.B * a.Hkv;
  if (a.layers > 1) {
    layer = quotient(unit, a.by_units);
    unit -= layer * units;
  }
  p.valid = layer < a.layers && unit < units && wu < a.per_unit;
  p.layer = layer;
  p.b = quotient(unit, a.by_heads);
  p.g = unit - p.b * a.Hkv;
  p.w = wu;
  return p;
}
template <bool GROUPS = true>
__device__ __forceinline__ UnitPlace place_in_unit(const AttnArgs &a) {
  return place_in_unit<GROUPS>(a, workgroup_id());
}
template <bool GROUPS = true>
__device__ __forceinline__ Place place(const AttnArgs &a, int qtile, int n) {
  const UnitPlace u = place_in_unit<GROUPS>(a, n);
  const int tile = quotient(u.w, a.by_rep);
  return {u.layer, u.b, u.g, u.g * a.rep + u.w - tile * a.rep, tile * qtile, u.valid};
}
template <bool GROUPS = true>
__device__ __forceinline__ Place place(const AttnArgs &a, int qtile) {
  return place<GROUPS>(a, qtile, workgroup_id());
}
// Fields of that placement in `a`, and its number of workgroups.  Units are cut only where an XCD would get more than
// `enough` workgroups.  resident: workgroups that run at once on an XCD (0: groups as above whatever their number).  whole: whether
// the launch is one group for that reason.  pack: blocks of 32 rows that a workgroup takes from the unit's list of them (0: tiles of
// qtile rows of one head).  least: workgroups of a unit at least.
inline int64_t place_grid(AttnArgs &a, const AttnLayers &layers, int qtile, int resident = 0, int unit_group = kUnitGroup, int enough = 0,
                          bool *whole = nullptr, int pack = 0, int64_t least = 0) {
  const int64_t QT = (a.S + qtile - 1) / qtile, rep = a.Hq / a.Hkv;
  int64_t per_unit = pack > 0 ? ((a.S + int64_t(31)) / 32 * rep + pack - 1) / pack : rep * QT;
  if (per_unit < least) per_unit = least;
  a.per_unit = int32_t(per_unit);
  a.layers = layers.n > 0 ? layers.n : 1;
  a.table = layers.n > 0;
  const int64_t units = int64_t(a.layers) * a.B * a.Hkv;
  a.spread = 0;  // with 32 units or more an XCD has at most a quarter more than its share
  if (units < 32 && (units + 7) / 8 * per_unit > enough)
    while ((units << a.spread) % 8 != 0) ++a.spread;
  const int64_t chunk = (per_unit + (1 << a.spread) - 1) >> a.spread;
  a.rep = int32_t(rep);
  a.chunk = int32_t(chunk);
  const int64_t pieces8 = ((units << a.spread) + 7) / 8;  // pieces per XCD
  const bool one_group = 2 * pieces8 * chunk <= 3 * resident;
  const int64_t G = pieces8 < unit_group || one_group ? pieces8 : unit_group;
  if (whole != nullptr) *whole = one_group;
  a.unit_group = int32_t(G);
  a.by_group = div_by(G * chunk);
  a.by_unit_group = div_by(G);
  a.by_units = div_by(int64_t(a.B) * a.Hkv);
  a.by_heads = div_by(a.Hkv);
  a.by_rep = div_by(a.rep);
  return (pieces8 + G - 1) / G * G * chunk * 8;
}

// ---- which kernel: bf16, head_dim 128, contiguous cache --------------------------------
// A probability is rounded to bf16 relative to the running reference of its pass over the keys, so the last bits of a row follow
// how the keys are divided between references.  What the passes begin with is a matter of the launch's buffers for tiles of up to 32
// rows and the spread ones, whichever workgroups compute them:
enum Reference : int32_t {
  kEightParts,  // fewer than 512 tiles of 32 rows: key block j belongs to part j % 8
  kFourParts,   // fewer than 1024: j % 4
  kOnePass,     // suffix buffers of up to 128 rows: every wave begins with the reference of the first key block
  kTiles256,    // longer ones: with that of a ragged end, and for the last up to 32 rows behind a multiple of 256 eight parts
};
// (A wave moves its own reference on when a maximum exceeds it by 8 octaves, and taller tiles are one pass by all waves: there the last
// bits may follow the active lengths too.)
struct Contiguous128 {
  enum Kernel { kSplit8, kSplit4TwoParts, kSplit4, kTiles128Rows, kFineTiles128Rows, kTiles256Rows } kernel;
  Reference rounding;
  bool packed;  // tiles may hold blocks of several heads of a group (Blocks)
};
// The host knows the buffers (S rows, C cache rows; heads: of all sequences and layers; rep: of a KV head), not the active lengths.
// us per call, one layer of 32/32 or 28/4 heads unless said otherwise, B x S rows on P cached ones:
//  * more than 128 tiles of 128 rows: the hand-scheduled loop with four waves, two workgroups to a compute unit.  Before
//    it there were tiles of 256 rows, the shared-tile kernel for S <= 128 and the key split below 256 tiles of 128:
//    3 x 256 on 800 33.8 -> 21.6, 28/4 heads 1 x 1024 on 1024 64 -> 35, 8 x 128 on 2000 97 -> 61; 32 layers:
//    8 x 128 with 20 active on 4000 4333 -> 2994, 8 x 100 on 400 615 -> 524, 1 x 256 on 512 148 -> 139.
//    Not everywhere: 32 layers of 2 x 162 on 1430 447 when full and 425 with eight waves (353 and 363 with 113 active, 273
//    and 281 with 24), 3 x 140 on 1500 with 90 active 27 and 20 with the key split (28 and 32 with 128);
//  * of these, eight waves with 256-row tiles, which fetch every K/V block for twice as many rows: long caches and at
//    least four rounds of them (32 layers, 8 x 1024 on 4096: 19.9 ms, with four waves 20.6; 4 x 700 on 3000 5.4 and 5.6);
//    one round that is nearly full (28/4 heads, 4 x 497 on 1021: 47.3 and 48.6; 2 x 1024 on 1800: 87 and 89, but 61 and 43 with
//    256 active); and at least two rounds of up to 256
//    heads, where a compute unit is left with one workgroup when the sequences are down to their last rows (28/4
//    heads, 8 x 1024 on 1000: 239 and 228 when full, 20.5 and 28.3 with 30 rows left).  The same from one and a half rounds of the
//    smaller tiles on, where these are placed in groups (place_grid) and so two to a compute unit while others have none, if the
//    heads do not share K/V (5 x 640 on 800: 25 and 35 with 51 rows left, 39 and 44 with 224, 61 and 50 with 480, 86 and 87 full; 28/4
//    heads, 6 x 640 on 1800: 35 and 34 with 51, 54 and 45 with 160, 88 and 67 with 320).  Otherwise
//    what the smaller tiles save in part-filled ones and in rounds weighs more (3 x 1024 on 4000, one round and a
//    half: 254 and 231; 32 layers, 8 x 600 on 600, 28/4 heads: 3025 and 2903);
//  * fewer: the key split, eight ways while its workgroups are at most one to a compute unit, four ways beyond, where
//    two fit one (1 x 384 on 800: 18.9 four ways, 23.4 eight, 21.1 with 128-row tiles).
inline Contiguous128 contiguous128(int64_t heads, int32_t rep, int32_t S, int32_t C) {
  auto tiles = [&](int rows) { return heads * ((S + rows - 1) / rows); };
  const int64_t rows = heads * S;
  Contiguous128 r;
  r.rounding = rows >= 32768 ? (S > 128 ? kTiles256 : kOnePass) : rows >= 16384 ? kFourParts : kEightParts;
  if (tiles(128) > 128) {
    const int64_t wide = r.rounding == kTiles256 ? tiles(256) : 0;
    const bool rounds = heads <= 256 && (wide >= 512 || (wide > 0 && tiles(128) > 768 && rep == 1));
    if ((wide > 192 && wide <= 256) || rounds || (wide >= 1024 && C > 2048)) r.kernel = Contiguous128::kTiles256Rows;
    else r.kernel = r.rounding == kFourParts && S > 128 ? Contiguous128::kFineTiles128Rows : Contiguous128::kTiles128Rows;
  } else {
    r.kernel = tiles(32) <= 256            ? Contiguous128::kSplit8
               : r.rounding == kEightParts ? Contiguous128::kSplit4TwoParts
                                           : Contiguous128::kSplit4;
  }
  // (the choice between them on the device; more workgroups than run at once)
  r.packed = rep > 1 && (S > 32 || r.rounding == kOnePass) && (r.kernel == Contiguous128::kTiles256Rows ? tiles(256) > 256 : r.kernel == Contiguous128::kTiles128Rows && tiles(128) > 512);
  return r;
}
// Where few blocks of 32 rows are left in a whole launch, workgroups take one each and share its keys (one layer, 45 of 640 rows of
// 64 heads on 1000 cached ones: 25.6 -> 19.7 us).  That is up to about one to a compute unit.  Beyond, two share one, and each streams
// its head's whole K/V: 32/32 heads, 4 x 640 rows on 3500 with 128 active 59 us in tiles and 97 in blocks, 8 x 140 on 700
// with 50 active 22.5 and 31.7; 3 x 640 on 3500 with 90 active 55 and 38.  Up to two a compute unit it pays
//  * where the heads of a group stream the same K/V (28/4 heads, 6 x 400 on 1500 with 90 active 34.5 in tiles, 29.2 in blocks; 9 x
//    320 with 50 active 34.8 and 28.6), but not with a grid of blocks (FINE; 3 x 250 on 3500 with 200 active 54 and 62),
//  * where the launch is placed in groups, so that live tiles share a compute unit while others have none (5 x 640 on 1500 with
//    90 active 45 and 38).
// What it still takes: 3 x 400 rows of 32/32 heads on 100 with 128 active 15.2 in tiles, 13.4 in blocks; on longer caches the other way.
inline int32_t spread_limit(int rep, bool fine, bool one_group) { return fine || (rep == 1 && one_group) ? 288 : 512; }

// Blocks of 32 rows that the waves of a workgroup take (head_dim 128, contiguous cache).
//  * WM consecutive blocks of one head, or
//  * PACK, where that takes fewer rounds of workgroups: WM entries of the unit's list of all heads' blocks (entry e: block e / rep of its
//    head e % rep).  The heads of a group stream the same K/V, so whose rows a wave has is no matter to the others.  Otherwise seven heads
//    with a few rows left each are seven workgroups that stream it one by one, and 33 rows leave half the waves of seven idle.
//    28/4 heads, 32 layers: 16 x 100 rows with 10 active on 2968 2264 -> 796 us, 10 x 22 with 11 on 109 132 -> 55, 2 x 30 with 4 on 32
//    23.2 -> 11.7, 8 x 165 on 2971 2256 -> 2109.
//    Rounds are counted as a little less than one workgroup to a compute unit (the XCDs' shares are uneven): within one, tiles
//    of one head each find a compute unit of their own, and more rows to a workgroup take longer (6 x 33 on 3233, one layer, 168
//    tiles: 45.6 and 49.4 us packed; 9 x 954 with 61 active on 154, 252 tiles: 37.1 and 32.5); the same for a saving that ends in the same
//    round (32 layers, 1 x 208 on 87, 1792 and 1664: 59.2 and 63.0).  In launches that run at once (`packed` in contiguous128) even the
//    choice would cost (9 x 48 on 56 9.1 and 9.4).  Not a block whose keys belong to four or eight parts (Reference): a wave has one pass and
//    one reference.
//    Waves of taller tiles come out the same to the bit; a block that would be a tile of its own keeps the key split's 32-bit row sums
//    (attn_bf16_pipe_kernel, own_tile), with the same times.
//  * spread (spread_limit): one block, shared by all waves.
constexpr uint32_t kPackRound = 224;
// whether a sequence's last block (its only one, or the one behind a multiple of 256 rows) has its keys in several parts
__device__ __forceinline__ bool in_parts(const AttnArgs &a, int N) {
  return a.rounding == kTiles256 ? ((N - 1) & 255) < 32 : a.rounding != kOnePass && N <= 32;
}
template <int WM>
__host__ __device__ __forceinline__ bool saves_rounds(const AttnArgs &a, int blocks) {
  const uint32_t listed = uint32_t(a.rep * blocks + WM - 1) / WM, tiles = uint32_t(a.rep) * (uint32_t(blocks + WM - 1) / WM);
  return (listed * uint32_t(a.units) + kPackRound - 1) / kPackRound < (tiles * uint32_t(a.units) + kPackRound - 1) / kPackRound;
}
template <int WM, bool FINE, bool PACK>
inline int64_t place_blocks(AttnArgs &a, const AttnLayers &layers) {
  bool one_group;
  const int64_t nwg = place_grid(a, layers, FINE ? 32 : 32 * WM, FINE ? 1 << 20 : 32 * 8 / WM, kUnitGroup, 0, &one_group);  // FINE: always one
  const int64_t units = int64_t(a.B) * a.Hkv * a.layers;
  a.units = int32_t(units);
  a.spread_blocks = int32_t(spread_limit(a.rep, FINE, one_group) / (units * a.rep));
  if (!PACK || a.spread_blocks > 0 || !saves_rounds<WM>(a, (a.S + 31) / 32)) return nwg;
  // Packed as the longest suffix needs it, and room for what is never packed: a last block in parts, behind a multiple of 256
  // rows, or of a suffix of up to 32.
  const int64_t parts = a.rounding == kOnePass ? 0 : a.rounding == kTiles256 ? (a.S - 1) / 256 * (8 / WM) + 1 : 1;
  return place_grid(a, layers, 32 * WM, 32 * 8 / WM, kUnitGroup, 0, nullptr, WM, parts * a.rep);
}
struct Blocks {
  int w, first_head, rep, tile;  // tile: w / rep
  int first;                     // packed: this workgroup's first entry
  int count;                     // blocks in the list from this workgroup's first on: none or less, one, ...
  bool spread, packed;
};
template <int WM, bool FINE, bool PACK>
__device__ __forceinline__ Blocks blocks_of(const AttnArgs &a, const UnitPlace &p, int N) {
  Blocks k = {p.w, p.g * a.rep, a.rep, quotient(p.w, a.by_rep), WM * p.w, 0, false, false};
  const int blocks = (N + 31) >> 5;
  k.spread = WM == 4 && (FINE || blocks * a.rep <= a.per_unit) && blocks <= a.spread_blocks;
  if (PACK)
    k.packed = !k.spread && !in_parts(a, N) && (saves_rounds<WM>(a, blocks) || a.rep * ((blocks + WM - 1) / WM) > a.per_unit);
  k.count = k.spread ? blocks - k.tile : k.packed ? a.rep * blocks - k.first : blocks - WM * k.tile;
  // A single block at a list's end goes to the key split, which is where it would be as a tile of its own.  One that would be a wave of
  // a taller tile takes the entry before it along and stays one.
  if (PACK && k.packed && blocks % WM != 1) {
    if (k.count == WM + 1) k.count = WM - 1;
    if (k.count == 1) --k.first, k.count = 2;
  }
  return k;
}
// first row and head of wave v's block (v >= count: rows beyond the suffix, of some head of the group; up to two entries of a
// packed list are behind a workgroup's own)
template <int WM, bool PACK>
__device__ __forceinline__ void block_at(const AttnArgs &a, const Blocks &k, int v, int &row, int &h) {
  const int e = k.first + v + (v < k.count ? 0 : 2), r = PACK && k.packed ? quotient(e, a.by_rep) : k.tile;
  row = 32 * (k.packed || k.spread ? r : WM * k.tile + v);
  h = k.first_head + (k.packed ? e - r * k.rep : k.w - k.tile * k.rep);
}

// Cache row that holds key t (t < P_b) of sequence b.
template <bool GATHER>
__device__ __forceinline__ int cache_row(const AttnArgs &a, int b, int t) {
  if (!GATHER) return t;
  const int r = a.cache_rows[int64_t(b) * a.C + t];
  return min(max(r, 0), a.C - 1);  // a bad index must not leave the buffer
}

int32_t launch_attn_f32(const AttnArgs &a, hipStream_t st);
int32_t launch_attn_bf16(const AttnArgs &a, const AttnLayers &layers, hipStream_t st);
size_t attn_f32_workspace_bytes(int32_t B, int32_t S, int32_t Hq, int32_t Hkv, int32_t D, int32_t C);  // 0: of no use

}  // namespace lsp
