"""Output head: heights of row tiles by rounds (lsp_lm_head.h, tile_rows, which the kernel calls), every height with several tiles per workgroup."""
import os
import subprocess

import pytest
import torch

from paper_2603_05454_amd.build import CSRC, ROOT
from test_attn_placement import STUB
from test_gpu_lm_head import _compare, _run, lsp  # noqa: F401

MAIN = r"""
#include <stdio.h>
#include "lsp_lm_head.h"
namespace lsp { void set_error(const char *, ...) {} }
int main() {
  int R, VT;
  while (scanf("%d %d", &R, &VT) == 2) printf("%d\n", lsp::tile_rows(R, VT));
}
"""


@pytest.fixture(scope="module")
def heights(tmp_path_factory):
    """The kernel's own rule, compiled for the host: [(rows, vocabulary tiles)] -> rows per tile."""
    d = tmp_path_factory.mktemp("heights")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(STUB)
    (d / "main.cpp").write_text(MAIN)
    subprocess.run([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", f"-I{d}", f"-I{CSRC}", f"-I{ROOT}/include", str(d / "main.cpp"), "-o", str(d / "heights")], check=True)
    return lambda pairs: [int(x) for x in subprocess.run([str(d / "heights")], input="\n".join(f"{r} {v}" for r, v in pairs), capture_output=True,
                                                         text=True, check=True).stdout.split()]


def _plan(h, rows, vt):
    """Rows per tile, row tiles, tiles of the busiest workgroup."""
    return h, -(-rows // h), -(-(-(-vt // 8) * -(-rows // h)) // 32)


def test_height_takes_the_least_time_in_rounds(heights):
    pairs = [(r, v) for r in (1, 64, 65, 128, 129, 192, 256, 257, 300, 384, 450, 700, 1024, 8192, 1 << 26) for v in (1, 8, 36, 103, 128, 129, 157, 256, 257, 494, 594)
             if r * v < 1 << 31]
    for (rows, vt), h in zip(pairs, heights(pairs)):
        if rows <= 128:
            assert h == (64 if vt * (1 + (rows > 64)) <= 256 else 128)
        else:   # (of equals the tallest)
            cost = {c: {256: 17, 128: 10, 64: 7}[c] * _plan(c, rows, vt)[2] for c in (256, 128, 64)}
            assert h == min(cost, key=cost.get), (rows, vt)


@pytest.mark.gpu
@pytest.mark.parametrize("rows,vt,plan", [(250, 494, (256, 1, 2)), (700, 157, (256, 3, 2)), (300, 103, (256, 2, 1)), (208, 594, (128, 2, 5)),
                                          (580, 103, (128, 5, 3)), (140, 157, (64, 3, 2)), (129, 261, (64, 3, 4))])
@pytest.mark.parametrize("K", [64, 136, 320])
def test_heights_by_rounds(lsp, oracle, heights, rows, vt, plan, K):  # noqa: F811
    """Small integers: bit-exact on rows from all over the list; the last vocabulary tile is ragged, K has one step, a ragged end, or
    more steps than are in flight."""
    assert _plan(heights([(rows, vt)])[0], rows, vt) == plan
    g = torch.Generator(device="cuda").manual_seed(rows + K)
    h = torch.randint(-3, 4, (1, rows, K), generator=g, device="cuda").to(torch.bfloat16)
    w = torch.randint(-3, 4, (vt * 256 - 3, K), generator=g, device="cuda").to(torch.bfloat16)
    got = _run(lsp, h, w)
    pick = torch.unique(torch.linspace(0, rows - 1, 24).round().long())
    _compare(tuple(x[:, pick] for x in got), oracle.lm_head_confidence(h[:, pick].cpu(), w.cpu()), None, exact=True)
