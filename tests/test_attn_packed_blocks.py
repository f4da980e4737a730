"""Workgroups of several heads of a group (csrc/lsp_attn.h, Blocks): the division of blocks of 32 rows among workgroups and waves on
the CPU, and the kernels' outputs at its edges against the CPU oracle."""
import os
import subprocess

import pytest
import torch

import workloads as W
from paper_2603_05454_amd.build import CSRC, ROOT
from test_attn_placement import STUB

MAIN = r"""
#include <stdio.h>
#include "lsp_attn.h"
namespace lsp { void set_error(const char *, ...) {} }
using namespace lsp;
template <int WM, bool FINE, bool PACK>
void walk(AttnArgs &a, const AttnLayers &layers, const int *N) {
  const int64_t n = place_blocks<WM, FINE, PACK>(a, layers);
  for (int64_t w = 0; w < n; ++w) {
    blockIdx.x = unsigned(w & ((1 << kGridBits) - 1));
    blockIdx.y = unsigned(w >> kGridBits);
    const UnitPlace p = place_in_unit(a);
    if (!p.valid) continue;
    const Blocks k = blocks_of<WM, FINE, PACK>(a, p, N[p.b]);
    for (int v = 0; v < WM && (v < k.count || k.count > 0); ++v) {
      int row, h;
      block_at<WM, PACK>(a, k, v, row, h);
      const bool one = k.spread || k.count == 1;
      if (v == 0 || !one) printf("%d %d %d %d %d %d\n", p.layer, p.b, p.g, h, row, v < k.count);
    }
  }
}
int main() {
  int WM, pack, L, B, S, Hq, Hkv, N[64];
  while (scanf("%d %d %d %d %d %d %d", &WM, &pack, &L, &B, &S, &Hq, &Hkv) == 7) {
    for (int b = 0; b < B; ++b) if (scanf("%d", N + b) != 1) return 1;
    AttnArgs a = {};
    AttnLayers layers = {};
    layers.n = L;
    a.B = B; a.S = S; a.Hq = Hq; a.Hkv = Hkv;
    a.rounding = contiguous128(int64_t(L) * B * Hq, Hq / Hkv, S, 1000).rounding;
    if (WM == 8) pack ? walk<8, false, true>(a, layers, N) : walk<8, false, false>(a, layers, N);
    else if (pack == 2) walk<4, true, false>(a, layers, N);
    else pack ? walk<4, false, true>(a, layers, N) : walk<4, false, false>(a, layers, N);
  }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("blocks")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(STUB)
    (d / "main.cpp").write_text(MAIN)
    subprocess.run([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-fno-strict-aliasing", "-DNDEBUG", f"-I{d}", f"-I{CSRC}", f"-I{ROOT}/include",
                    str(d / "main.cpp"), "-o", str(d / "blocks")], check=True)
    return str(d / "blocks")


# waves, pack (2: a workgroup for every block), layers, S, query heads, KV heads, active rows
FORMS = [(4, 1, 32, 20, 28, 4, (1, 20, 0)), (4, 1, 32, 700, 7, 1, (700, 33, 32, 64, 65, 0, 129)), (4, 1, 16, 100, 40, 8, (97, 96, 31)),
         (4, 1, 1, 600, 28, 4, (600, 40, 3, 0, 300)), (4, 1, 3, 161, 12, 6, (161, 128, 127, 5)), (4, 1, 32, 300, 15, 5, (300, 161, 160, 17)),
         (8, 1, 32, 512, 8, 2, (512, 257, 256, 255, 33, 1)), (8, 1, 9, 1000, 28, 4, (1000, 31, 0)),
         (4, 1, 32, 18, 28, 4, (18, 2)), (4, 1, 32, 208, 28, 4, (208,)), (4, 1, 32, 75, 28, 4, (75,)), (4, 1, 32, 75, 28, 4, (33, 64)), (4, 1, 7, 1000, 28, 4, (70, 33, 130)), (4, 1, 32, 40, 28, 4, (40, 33, 32, 1)), (4, 1, 32, 290, 28, 4, (290, 257, 288, 289, 32, 1, 33)), (8, 1, 32, 600, 28, 4, (600, 513, 544, 20)),
         (4, 0, 1, 150, 28, 4, (150, 1, 64, 33)), (4, 2, 1, 250, 28, 4, (250, 100, 7)), (8, 0, 1, 600, 6, 2, (600, 290)), (4, 0, 2, 300, 5, 5, (300, 129))]


@pytest.mark.parametrize("form", FORMS)
def test_every_active_block_once(program, form):
    WM, pack, L, S, Hq, Hkv, N = form
    text = " ".join(map(str, (WM, pack, L, len(N), S, Hq, Hkv, *N)))
    out = subprocess.run([program], input=text, capture_output=True, text=True, check=True).stdout
    placed = [tuple(map(int, l.split())) for l in out.split("\n") if l]
    rep = Hq // Hkv
    want = sorted((l, b, h, r) for l in range(L) for b, n in enumerate(N) for h in range(Hq) for r in range(0, n, 32))
    assert sorted((l, b, h, r) for l, b, _, h, r, live in placed if live) == want
    assert all(g == h // rep for _, _, g, h, _, _ in placed)
    assert all(r >= N[b] for _, b, _, _, r, live in placed if not live)     # a wave without a block stores nothing


@pytest.fixture(scope="module")
def lsp():
    import paper_2603_05454_amd as m
    assert torch.cuda.is_available()
    return m


# layers, S, C, query heads, KV heads, active rows: lists whose last workgroup has one block, some, or all; lists that are cut by head
# instead (97 .. 128 rows); caches beyond 2048 rows and 512 heads, where a workgroup has eight waves
GPU = [(16, 100, 64, 35, 5, (100, 33, 1, 0)), (20, 40, 97, 28, 4, (40, 32, 20, 5, 33)), (16, 300, 70, 12, 4, (300, 161, 129, 64)),
       (6, 161, 40, 60, 2, (161, 96, 97, 40)), (32, 300, 2100, 8, 2, (300, 33)), (4, 520, 50, 14, 2, (520, 3, 0, 31, 65))]


@pytest.mark.gpu
@pytest.mark.parametrize("layers,S,C,Hq,Hkv,N", GPU)
def test_packed_workgroups_match_the_oracle(lsp, oracle, layers, S, C, Hq, Hkv, N):
    """The bound is the bf16 one of test_gpu_attention.py; rows beyond a suffix stay as they were."""
    w = W.scaled(W.C2, B=len(N), S=S, P=C, C=C, Hq=Hq, Hkv=Hkv, D=128, seed=900 + S + Hq)
    pl = torch.tensor([max(C - 13 * b - (b & 1), 0) for b in range(len(N))], dtype=torch.int32)
    sl = torch.tensor(N, dtype=torch.int32)
    checked = (0, layers - 1)
    host = {l: W.make_layer_kv(w, l, prefix_len=pl) for l in checked}
    dev = {l: {k: v.cuda() for k, v in host[l].items()} for l in checked}
    names = ("q", "k_suf", "v_suf", "k_cache", "v_cache")
    ops = [dev[l if l in dev else 0] for l in range(layers)]                # the layers between repeat the first one's operands
    outs = [torch.full(ops[0]["q"].shape, 123.0, dtype=torch.bfloat16, device="cuda") for _ in range(layers)]
    lsp.attn_step_layers(lsp.AttnLayerTable(*[[o[k] for o in ops] for k in names], outs), pl.cuda(), sl.cuda())
    for l in checked:
        ref = oracle.attention(**host[l], prefix_len=pl, suffix_len=sl)
        got, act = outs[l].float().cpu(), ~torch.isnan(ref)
        assert (got[act] - ref[act]).abs().max().item() <= 2e-2
        assert torch.all(got[~act] == 123.0)
    assert all(torch.equal(outs[l], outs[0]) for l in range(1, layers - 1))


# cached rows, active rows: both ends ragged and fitting one block, just so, or one row too many; one end, or none; less than a block in all
ENDS = [(50, 100), (60, 68), (63, 97), (63, 98), (64, 97), (63, 96), (64, 96), (1, 33), (0, 40), (31, 33), (5, 34), (200, 65)]


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [33, 100, 300])
def test_ragged_ends_of_cache_and_suffix(lsp, oracle, rows):
    """Sequences with every pair of ends in one launch of tiles of 128 rows, one of whole blocks among them.  The bound is the bf16 one
    of test_gpu_attention.py."""
    B, C = len(ENDS), 200
    w = W.scaled(W.C2, B=B, S=rows, P=C, C=C, Hq=12, Hkv=12, D=128, seed=77 + rows)
    pl = torch.tensor([p for p, _ in ENDS], dtype=torch.int32)
    sl = torch.tensor([min(n + rows - 100, rows) if rows > 100 else min(n, rows) for _, n in ENDS], dtype=torch.int32)
    kv = W.make_layer_kv(w, 0, prefix_len=pl)
    dev = {k: v.cuda() for k, v in kv.items()}
    names = ("q", "k_suf", "v_suf", "k_cache", "v_cache")
    outs = [torch.full(dev["q"].shape, 123.0, dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    lsp.attn_step_layers(lsp.AttnLayerTable(*[[dev[k]] * 3 for k in names], outs), pl.cuda(), sl.cuda())
    ref = oracle.attention(**kv, prefix_len=pl, suffix_len=sl)
    act = ~torch.isnan(ref)
    for o in outs:
        got = o.float().cpu()
        assert (got[act] - ref[act]).abs().max().item() <= 2e-2
        assert torch.all(got[~act] == 123.0)


# S, active rows: blocks that are tiles of their own unpacked (up to 32 rows), waves of taller tiles (whose list ends with a
# single block at 65 and 96 rows of seven heads), both (129 .. 160 rows)
@pytest.mark.gpu
@pytest.mark.parametrize("S,N", [(20, (20, 7, 1)), (32, (32, 31, 9)), (100, (14, 30, 32)), (96, (96, 65, 80)), (128, (33, 64, 97)), (200, (140, 129, 160))])
def test_packed_blocks_are_computed_as_unpacked_ones(lsp, S, N):
    """The same launch with every head's K/V written out, which shares none and packs nothing.  Waves of taller tiles are the same to
    the bit.  Blocks of their own differ in the order of 32-bit sums alone: some 2^-17 of a row at most, so that an output comes
    out as the neighbouring bf16 (2^-9 to 2^-8 away) for 2^-8 of them at most; row sums of rounded probabilities change 2^-6 and
    more of them."""
    layers, Hkv, rep, C = 32, 4, 7, 300
    g = torch.Generator(device="cuda").manual_seed(S)
    q = torch.randn((len(N), S, Hkv * rep, 128), generator=g, device="cuda").to(torch.bfloat16)
    kv = [torch.randn((len(N), n, Hkv, 128), generator=g, device="cuda").to(torch.bfloat16) for n in (S, S, C, C)]
    pl, sl = torch.tensor([C - 13 * b for b in range(len(N))], dtype=torch.int32).cuda(), torch.tensor(N, dtype=torch.int32).cuda()

    def run(operands):
        outs = [torch.zeros_like(q) for _ in range(layers)]
        lsp.attn_step_layers(lsp.AttnLayerTable(*[[t] * layers for t in (q, *operands)], outs), pl, sl)
        assert all(torch.equal(outs[0], o) for o in outs)
        return outs[0]

    packed, plain = run(kv), run([t.repeat_interleave(rep, 2) for t in kv])
    for b, n in enumerate(N):
        own = n - n % 128 if 0 < n % 128 <= 32 else n      # rows from here on are a tile of their own
        assert torch.equal(packed[b, :own], plain[b, :own])
        if own < n:
            assert (packed[b, own:n] != plain[b, own:n]).float().mean().item() <= 2 ** -8


@pytest.mark.gpu
@pytest.mark.parametrize("rows,Hq", [(40, 96), (128, 32), (129, 32)])
def test_last_rows_of_buffers_of_one_tile_and_longer_ones(lsp, oracle, rows, Hq):
    """Up to 32 rows, which the key split merges in pieces of all rows in buffers of up to 128 and as whole rows beyond: numbers of rows
    around what a wave has of either, ragged keys of one block and many.  The bound is the bf16 one of test_gpu_attention.py."""
    N, C = (1, 7, 8, 9, 31, 32, 0, 20, 33), 150
    w = W.scaled(W.C2, B=len(N), S=rows, P=C, C=C, Hq=Hq, Hkv=Hq, D=128, seed=500 + rows)
    pl, sl = torch.tensor([0, 30, 150, 64, 1, 96, 9, 149, 0], dtype=torch.int32), torch.tensor(N, dtype=torch.int32)
    kv = W.make_layer_kv(w, 0, prefix_len=pl)
    dev = {k: v.cuda() for k, v in kv.items()}
    outs = [torch.full(dev["q"].shape, 123.0, dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    lsp.attn_step_layers(lsp.AttnLayerTable(*[[dev[k]] * 3 for k in ("q", "k_suf", "v_suf", "k_cache", "v_cache")], outs), pl.cuda(), sl.cuda())
    ref = oracle.attention(**kv, prefix_len=pl, suffix_len=sl)
    act = ~torch.isnan(ref)
    for o in outs:
        got = o.float().cpu()
        assert (got[act] - ref[act]).abs().max().item() <= 2e-2
        assert torch.all(got[~act] == 123.0)
