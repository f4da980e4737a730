"""Host-side check of the placement of the attention kernels' workgroups (csrc/lsp_attn.h): the header is compiled for the
CPU with a stub of the HIP runtime's header, and every workgroup of a launch is asked for its place."""
import os
import subprocess
from collections import Counter

import pytest

from paper_2603_05454_amd.build import CSRC, ROOT
from test_gpu_attention import MOVING, NEAR_THE_END, SPREAD, TILES

STUB = r"""
#pragma once
#include <stdint.h>
#include <algorithm>
#define __device__
#define __forceinline__ inline
#define __host__
typedef int hipError_t;
enum { hipSuccess, hipFuncAttributeMaxDynamicSharedMemorySize };
inline const char *hipGetErrorString(int) { return ""; }
inline int hipGetLastError() { return 0; }
inline int hipGetDevice(int *) { return 0; }
inline int hipFuncSetAttribute(const void *, int, int) { return 0; }
typedef void *hipStream_t;
struct dim3 { unsigned x, y, z; dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {} };
static dim3 blockIdx;
inline uint32_t __umulhi(uint32_t a, uint32_t b) { return uint32_t(uint64_t(a) * b >> 32); }
inline uint32_t __float_as_uint(float f) { uint32_t u; __builtin_memcpy(&u, &f, 4); return u; }
inline float __uint_as_float(uint32_t u) { float f; __builtin_memcpy(&f, &u, 4); return f; }
using std::min;
using std::max;
"""
MAIN = r"""
#include <stdio.h>
#include <stdlib.h>
#include "lsp_attn.h"
namespace lsp { void set_error(const char *, ...) {} }
int main(int argc, char **argv) {
  using namespace lsp;
  int L, B, S, Hq, Hkv, qtile, resident, group, enough;
  if (argc > 1) {  // heads, rep, S, C -> kernel, rounding
    const Contiguous128 r = contiguous128(atoll(argv[1]), atoi(argv[2]), atoi(argv[3]), atoi(argv[4]));
    return printf("%d %d\n", int(r.kernel), int(r.rounding)), 0;
  }
  while (scanf("%d %d %d %d %d %d %d %d %d", &L, &B, &S, &Hq, &Hkv, &qtile, &resident, &group, &enough) == 9) {
    AttnArgs a = {};
    AttnLayers layers = {};
    layers.n = L;
    a.B = B; a.S = S; a.Hq = Hq; a.Hkv = Hkv;
    const int64_t n = place_grid(a, layers, qtile, resident, group, enough);
    printf("%lld %d\n", (long long)n, a.spread);
    for (int64_t w = 0; w < n; ++w) {
      blockIdx.x = unsigned(w & ((1 << kGridBits) - 1));
      blockIdx.y = unsigned(w >> kGridBits);
      const Place p = group == 1 ? place<false>(a, qtile) : place(a, qtile);
      if (p.valid) printf("%lld %d %d %d %d %d\n", (long long)w, p.layer, p.b, p.g, p.h, p.q0);
    }
  }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("placement")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(STUB)
    (d / "main.cpp").write_text(MAIN)
    subprocess.run([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-fno-strict-aliasing", "-DNDEBUG", f"-I{d}", f"-I{CSRC}", f"-I{ROOT}/include",
                    str(d / "main.cpp"), "-o", str(d / "placement")], check=True)
    return str(d / "placement")


# layers (0: one), B, S, Hq, Hkv, rows a tile, workgroups at once on an XCD, units in a group, workgroups of an XCD not cut
FORMS = [(0, 1, 64, 4, 4, 16, 0, 1, 16), (0, 3, 257, 4, 1, 16, 0, 1, 16), (0, 2, 1000, 8, 2, 16, 0, 1, 16), (0, 1, 1024, 28, 4, 256, 32, 8, 0),
         (0, 5, 320, 28, 4, 128, 64, 8, 0), (0, 6, 640, 28, 4, 128, 64, 8, 0), (0, 5, 640, 32, 32, 128, 64, 8, 0), (0, 1, 33, 7, 7, 32, 64, 8, 0),
         (0, 3, 250, 28, 4, 32, 1 << 20, 8, 0), (0, 1, 545, 5, 1, 32, 32, 8, 0), (3, 2, 140, 28, 4, 128, 64, 8, 0), (32, 2, 300, 4, 2, 128, 64, 8, 0),
         (32, 1, 100, 28, 4, 128, 64, 8, 0), (0, 1, 2000, 3, 1, 128, 64, 8, 0), (0, 16, 400, 32, 32, 128, 64, 8, 0)]


@pytest.mark.parametrize("form", FORMS)
def test_every_tile_once_and_live_ones_on_all_xcds(program, form):
    L, B, S, Hq, Hkv, qtile, _, _, _ = form
    out = subprocess.run([program], input=" ".join(map(str, form)), capture_output=True, text=True, check=True).stdout.split("\n")
    n, spread = map(int, out[0].split())
    placed = [tuple(map(int, l.split())) for l in out[1:] if l]
    tiles = range(0, S, qtile)
    want = {(l, b, h, q) for l in range(max(L, 1)) for b in range(B) for h in range(Hq) for q in tiles}
    got = [(l, b, h, q) for _, l, b, _, h, q in placed]
    assert n % 8 == 0 and len(got) == len(want) and set(got) == want
    assert all(g == h // (Hq // Hkv) for _, _, _, g, h, _ in placed)
    # workgroup ids go round the XCDs: where a unit is cut, any number of live rows is shared by its pieces to within one
    # workgroup a piece, and every XCD has the same number of pieces
    units = max(L, 1) * B * Hkv
    if spread > 0:
        pieces = (units << spread) // 8
        for q in tiles:
            live = Counter(w % 8 for w, _, _, _, _, q0 in placed if q0 <= q)
            assert max(live.values()) - min(live[x] for x in range(8)) <= pieces, (q, live)


KERNELS = ["split8", "split4x2", "split4", "128", "128 fine", "256"]


def _kernel(program, *shape):
    return KERNELS[int(subprocess.run([program, *map(str, shape)], capture_output=True, text=True, check=True).stdout.split()[0])]


@pytest.mark.parametrize("rep", [1, 2])
@pytest.mark.parametrize("heads,S,C,kernel", [(layers * B * Hq, S, C, kernel) for layers, B, Hq, S, C, kernel in TILES + SPREAD + MOVING + NEAR_THE_END])
def test_shapes_of_the_gpu_tests_reach_the_kernel_they_name(program, heads, rep, S, C, kernel):
    assert _kernel(program, heads, rep, S, C) == kernel


@pytest.mark.parametrize("heads,rep,S,C,kernel", [(160, 1, 640, 1440, "256"), (160, 8, 640, 1440, "128"), (192, 1, 512, 1312, "128"), (224, 1, 512, 1312, "256"),
                                                 (384, 1, 384, 1000, "128"), (168, 7, 640, 2440, "128"), (768, 1, 128, 900, "128")])
def test_more_tiles_than_are_placed_at_once(program, heads, rep, S, C, kernel):
    assert _kernel(program, heads, rep, S, C) == kernel
