"""fp32 attention whose keys are divided between workgroups (csrc/lsp_attn_f32.hip, parts_of): against the CPU oracle at the
edges of the rule and of the parts, with and without a workspace, and replayed.  The bound is 1e-5: outputs of magnitude 1, of
which a sum of up to 2000 weighted values in 128-key parts rounds less than 2e-6 away."""
import ctypes

import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
TOL = 1e-5
OPERANDS = ("q", "k_suf", "v_suf", "k_cache", "v_cache")


@pytest.fixture(scope="module")
def lsp():
    import paper_2603_05454_amd as m
    assert torch.cuda.is_available()
    return m


def _call(lsp, kv, pl, sl, out, workspace, nbytes):
    """Through the C entry, with that workspace."""
    d = lsp.AttnDesc(dtype=lsp._dtype(kv["q"]), B=kv["q"].shape[0], S=kv["q"].shape[1], Hq=kv["q"].shape[2], Hkv=kv["k_suf"].shape[2],
                     D=kv["q"].shape[3], C=kv["k_cache"].shape[1])
    d.q_stride, d.kv_suf_stride, d.cache_stride, d.o_stride = (lsp._strides3(t) for t in (kv["q"], kv["k_suf"], kv["k_cache"], out))
    rc = lsp.lib().lsp_attn_step(ctypes.byref(d), *[lsp._ptr(kv[n]) for n in OPERANDS], lsp._ptr(pl), lsp._ptr(sl), lsp._ptr(out),
                                 ctypes.c_void_p(workspace), ctypes.c_size_t(nbytes), lsp._stream())
    assert rc == 0, lsp.lib().lsp_last_error()


# keys in all of each sequence, rows, heads, head_dim: 303 | 304 and 227 | 228 (fewest keys that are divided: a part of 128
# has 176 fewer, 100 at head_dim 128), parts of one or more rounds with a remainder, 16 parts and more rounds than parts; an empty suffix, one row, tiles with a remainder; few parts where
# there are many tiles
CASES = [([303, 304, 305, 306], [16, 7, 16, 1], 4, 4, 64), ([227, 228, 229, 384], [5, 0, 17, 17], 4, 2, 128),
         ([2048], [16], 4, 4, 64), ([2049, 1], [3, 1], 7, 1, 64), ([1921], [40], 3, 3, 128), ([1280], [256], 4, 4, 64),
         ([1281, 640], [100, 70], 6, 2, 128)]


@pytest.mark.parametrize("T,N,Hq,Hkv,D", CASES)
def test_keys_divided_between_workgroups(lsp, oracle, T, N, Hq, Hkv, D):
    pl, sl = torch.tensor([t - n for t, n in zip(T, N)], dtype=torch.int32), torch.tensor(N, dtype=torch.int32)
    w = W.scaled(W.C2, dtype="f32", B=len(T), S=max(N) + 3, P=max(1, int(pl.max())), C=int(pl.max()) + 9, Hq=Hq, Hkv=Hkv, D=D, seed=900 + T[0])
    kv = W.make_layer_kv(w, 0, prefix_len=pl)
    ref = oracle.attention(**kv, prefix_len=pl, suffix_len=sl)
    act = ~torch.isnan(ref)
    g = {k: v.cuda() for k, v in kv.items()}
    need = lsp.attn_workspace_bytes(lsp._dtype(g["q"]), w.B, w.S, Hq, Hkv, D, w.C)
    assert need > 0
    ws = torch.randint(0, 256, (need + 16,), dtype=torch.uint8).cuda()     # holds anything
    held = ws.clone()
    for pointer, nbytes in ((None, 0), (ws.data_ptr(), need - 1), (ws.data_ptr() + 8, need), (ws.data_ptr(), need), (ws.data_ptr(), need)):
        out = torch.full(g["q"].shape, 123.0, device="cuda")
        _call(lsp, g, pl.cuda(), sl.cuda(), out, pointer, nbytes)
        got = out.cpu()
        assert (got[act] - ref[act]).abs().max().item() <= TOL and torch.all(got[~act] == 123.0)
        assert torch.equal(ws, held) or (pointer == ws.data_ptr() and nbytes == need)       # one that will not do is left alone
    out = lsp.attn_step(*[g[n] for n in OPERANDS], pl.cuda(), sl.cuda(), out=torch.full(g["q"].shape, 123.0, device="cuda"))
    assert torch.equal(out.cpu(), got) and not torch.equal(ws, held)       # the Python call divides as well
    rows = torch.arange(w.C, dtype=torch.int32, device="cuda").repeat(w.B, 1)
    out = lsp.attn_step(*[g[n] for n in OPERANDS], pl.cuda(), sl.cuda(), out=torch.full(g["q"].shape, 123.0, device="cuda"), cache_row_index=rows)
    assert torch.equal(out.cpu(), got)


@pytest.mark.parametrize("lo,hi", [(0, 128), (256, 384), (0, 640), (128, 700)])
def test_parts_of_scores_of_minus_infinity(lsp, oracle, lo, hi):
    """Parts all of whose scores are -infinity add nothing, the first one or the last, several or the only others."""
    w = W.scaled(W.C2, dtype="f32", B=1, S=20, P=700, C=700, Hq=2, Hkv=2, D=64, seed=47)
    kv, (pl, sl) = W.make_layer_kv(w, 0), W.make_lengths(w)
    kv["q"][..., 5] = 1.0
    kv["k_cache"][:, lo:hi, :, 5] = -float("inf")
    got = lsp.attn_step(*[kv[n].cuda() for n in OPERANDS], pl.cuda(), sl.cuda()).cpu()
    ref = oracle.attention(**kv, prefix_len=pl, suffix_len=sl)
    assert torch.isfinite(ref).all() and (got - ref).abs().max().item() <= TOL


def test_divided_keys_under_graph_replay(lsp):
    """Every replay carries the same tag, on other operands and lengths, so that the parts of a tile change from one to the next."""
    w = W.scaled(W.C2, dtype="f32", B=2, S=40, P=1200, C=1200, Hq=4, Hkv=4, D=64, seed=53)
    g = {k: v.cuda() for k, v in W.make_layer_kv(w, 0).items()}
    args = [g[n] for n in OPERANDS]
    pl, sl = torch.tensor([1200, 300], dtype=torch.int32).cuda(), torch.tensor([40, 9], dtype=torch.int32).cuda()
    out = torch.zeros_like(g["q"])
    lsp.attn_step(*args, pl, sl, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lsp.attn_step(*args, pl, sl, out=out)
    for k in range(6):
        g["q"].copy_(g["q"].roll(1, dims=1))
        pl.copy_(torch.tensor([1200 - 230 * k, 300 + 170 * k], dtype=torch.int32))
        sl.copy_(torch.tensor([40 - 7 * k, 9 + 6 * k], dtype=torch.int32))
        ref = lsp.attn_step(*args, pl, sl, out=torch.zeros_like(out))
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)


def test_workspace_of_sizes_that_are_not_divided(lsp):
    """0 for few keys, for more tiles than half as many as there are compute units, and for any sizes whatever."""
    most = 2 ** 31 - 1
    for sizes in ((1, 16, 4, 4, 64, 287), (1, 16, 4, 4, 128, 211), (129, 16, 1, 1, 64, 2000), (most, 16, 1, 1, 64, 2000), (most,) * 4 + (64, most)):
        assert lsp.attn_workspace_bytes(0, *sizes) == 0
    for sizes in ((1, 16, 4, 4, 64, 288), (1, 16, 4, 4, 128, 212), (128, 16, 1, 1, 64, 2000), (1, 16, 4, 4, 64, most)):
        assert 0 < lsp.attn_workspace_bytes(0, *sizes) < 1 << 22


@pytest.mark.parametrize("native", [True, False])
def test_a_workspace_that_is_handed_over(lsp, native, monkeypatch):
    """One that will do is used and nothing is allocated; one that is too small, misaligned, strided or on the host is left alone, and
    the result is that of the call's own workspace."""
    lsp.lib()
    if not native:
        monkeypatch.setattr(lsp, "_nat", None)
    w = W.scaled(W.C2, dtype="f32", B=1, S=16, P=900, C=900, Hq=4, Hkv=4, D=64, seed=61)
    g = {k: v.cuda() for k, v in W.make_layer_kv(w, 0).items()}
    args, (pl, sl) = [g[n] for n in OPERANDS], [t.cuda() for t in W.make_lengths(w)]
    need = lsp.attn_workspace_bytes(lsp._dtype(g["q"]), w.B, w.S, w.Hq, w.Hkv, w.D, w.C)
    want, layered = lsp.attn_step(*args, pl, sl), torch.zeros_like(g["q"])
    table = lsp.AttnLayerTable(*[[t] for t in args], [layered])
    before = torch.randint(0, 256, (4 * need + 16,), dtype=torch.uint8).cuda()
    held = before.clone()
    rows = torch.arange(w.C, dtype=torch.int32, device="cuda").repeat(w.B, 1)
    good, bad = [held[:need], held[need - need % 16:2 * need]], [held[:need - 1], held[8:8 + need], held[::4][:need], held[:need].cpu()]
    for ws, used in [(t, True) for t in good] + [(t, False) for t in bad]:
        for more in ({}, {"cache_row_index": rows}):
            out = torch.zeros_like(want)
            held.copy_(before)
            allocated = torch.cuda.memory_stats()["allocation.all.allocated"]
            lsp.attn_step(*args, pl, sl, out=out, workspace=ws, **more)
            assert (torch.cuda.memory_stats()["allocation.all.allocated"] == allocated) == used
            assert torch.equal(out, want) and torch.equal(held, before) != used
        held.copy_(before)
        layered.zero_()
        lsp.attn_step_layers(table, pl, sl, workspace=ws)
        assert torch.equal(layered, want) and torch.equal(held, before) != used
