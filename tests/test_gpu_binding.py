"""The native marshalling module (csrc/binding.cpp) against the general path in Python: same results, and
arguments that are not in their ordinary form are left to the general path, which refuses or handles them."""
import ctypes
import subprocess
import threading
import time

import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lsp():
    import paper_2603_05454_amd as m
    m.lib()
    return m


def _state(tokens=True):
    w = W.scaled(W.C2, B=2, S=70, P=40, C=120, Hq=4, Hkv=2, V=1000, layers=3, n_delim=40, seed=77)
    kv = [{k: v.cuda() for k, v in W.make_layer_kv(w, i).items()} for i in range(w.layers)]
    pl, sl = W.make_lengths(w)
    z, _ = W.make_logits(w)
    return w, kv, pl.cuda(), sl.cuda(), z.cuda(), W.make_delimiters(w)[1].cuda(), W.make_tokens(w, w.C).cuda() if tokens else None


def _conf_out(B, S):
    return (torch.zeros((B, S), dtype=torch.int32, device="cuda"), torch.zeros((B, S), device="cuda"), torch.zeros((B, S), device="cuda"))


def _commit_out(B, S):
    out = {k: torch.zeros(B, dtype=torch.int32, device="cuda") for k in ("raw_boundary", "snapped_boundary", "commit_len", "status_flags")}
    out["stable_mask"] = torch.zeros((B, S), dtype=torch.uint8, device="cuda")
    out["tau_used"] = torch.zeros(B, device="cuda")
    return out


def _step(lsp, with_tokens, with_layers, counts):
    w, kv, pl, sl, z, bm, tok = _state(with_tokens)
    res = [lsp.attn_step(kv[0]["q"], *[kv[0][k] for k in ("k_suf", "v_suf", "k_cache", "v_cache")], pl, sl, scale=0.1,
                         out=torch.zeros_like(kv[0]["q"])).clone()]
    cols = {k: [l[k] for l in kv] for k in kv[0]}
    table = lsp.AttnLayerTable(cols["q"], cols["k_suf"], cols["v_suf"], cols["k_cache"], cols["v_cache"], [torch.zeros_like(q) for q in cols["q"]])
    res += [t.clone() for t in lsp.attn_step_layers(table, pl, sl)]
    ws = torch.empty(max(16, lsp.confidence_workspace_bytes(w.B, w.S, w.V)), dtype=torch.uint8, device="cuda")
    conf = lsp.confidence(z, sl, out=_conf_out(w.B, w.S), workspace=ws)
    res += [t.clone() for t in conf]
    h, wt, _ = W.make_lm_head(w, 64)
    lm_ws = torch.empty(lsp.lm_head_confidence_workspace_bytes(w.B, w.S, w.V), dtype=torch.uint8, device="cuda")
    res += [t.clone() for t in lsp.lm_head_confidence(h.cuda(), wt.cuda(), sl, out=_conf_out(w.B, w.S), workspace=lm_ws)]
    last = torch.full((w.B, w.S), -1, dtype=torch.int32, device="cuda")
    counters = torch.zeros(4, dtype=torch.int64, device="cuda")
    sc = torch.zeros((w.B, 2), dtype=torch.int32, device="cuda") if counts else None
    for _ in range(2):
        lsp.flip_update(conf[0], pl, sl, pl.clone(), last, counters, window=(0, 5) if counts else None, step_counts=sc)
    layers = lsp.LayerTable(cols["k_suf"], cols["v_suf"], cols["k_cache"], cols["v_cache"]) if with_layers else None
    out = lsp.commit(conf[2], conf[0], bm, w.V, w.tau, w.window, w.min_commit, True, pl, sl, tokens=tok, layers=layers,
                     C=None if with_layers else w.C, out=_commit_out(w.B, w.S), adaptive=True, alpha=0.25, beta=0.5, max_commit=31)
    res += [out[k] for k in sorted(out)] + [pl, sl, last, counters] + [t for t in (tok, sc) if t is not None] + cols["k_cache"] + cols["v_cache"]
    return res


@pytest.mark.parametrize("with_tokens,with_layers,counts", [(True, True, True), (False, False, False)])
def test_native_and_general_path_agree(lsp, monkeypatch, with_tokens, with_layers, counts):
    taken = []

    class Spy:      # every one of these calls is in its ordinary form
        def __getattr__(self, name):
            def call(*a):
                rc = getattr(native, name)(*a)
                taken.append((name, rc))
                return rc
            return call

    native = lsp._nat
    monkeypatch.setattr(lsp, "_nat", Spy())
    a = _step(lsp, with_tokens, with_layers, counts)
    assert {n for n, _ in taken} == {"attn_step", "attn_step_layers", "confidence", "lm_head_confidence", "flip_update", "commit"}
    assert all(rc == 0 for _, rc in taken)
    monkeypatch.setattr(lsp, "_nat", None)
    b = _step(lsp, with_tokens, with_layers, counts)
    assert len(a) == len(b) and all(torch.equal(x, y) for x, y in zip(a, b))


def test_replaced_attributes_of_a_table_are_the_ones_used(lsp):
    """A table's descriptor and pointer arrays belong to the table: a caller that exchanges them (to point one table at another
    set of buffers) gets what the new ones say, on the native path as on the general one."""
    w, kv, pl, sl, _, bm, tok = _state()
    cols = {k: [l[k] for l in kv] for k in kv[0]}
    names = ("q", "k_suf", "v_suf", "k_cache", "v_cache")
    other = {k: [torch.randn_like(t) for t in cols[k]] for k in names}
    table = lsp.AttnLayerTable(*[cols[k] for k in names], [torch.zeros_like(q) for q in cols["q"]])
    want = lsp.AttnLayerTable(*[other[k] for k in names], [torch.zeros_like(q) for q in cols["q"]])
    lsp.attn_step_layers(want, pl, sl)
    table.arrays = [type(a)(*a) for a in want.arrays[:5]] + [table.arrays[5]]
    table.desc = lsp.AttnDesc.from_buffer_copy(table.desc)
    rc = lsp._nat.attn_step_layers(table.desc, table.n, table.arrays, pl, sl, 0.0, None)
    assert rc == 0 and all(torch.equal(a, b) for a, b in zip(table.out, want.out))
    assert lsp._nat.attn_step_layers(table.desc, table.n + 1, table.arrays, pl, sl, 0.0, None) is None     # arrays too short
    kvt = lsp.LayerTable(*[cols[k] for k in names[1:]])
    before = [t.clone() for t in cols["k_cache"]]
    kvt.arrays = [type(a)(*a) for a in lsp.LayerTable(*[other[k] for k in names[1:]]).arrays]
    margin, ids, p0 = torch.ones((w.B, w.S), device="cuda"), torch.zeros((w.B, w.S), dtype=torch.int32, device="cuda"), pl.clone()
    got = lsp.commit(margin, ids, bm, w.V, 0.5, 0, 1, 0, pl, sl, tokens=tok, layers=kvt, out=_commit_out(w.B, w.S))
    assert (got["commit_len"] > 0).all() and all(torch.equal(a, b) for a, b in zip(before, cols["k_cache"]))
    for b, (p, n) in enumerate(zip(p0.tolist(), got["commit_len"].tolist())):
        assert all(torch.equal(c[b, p:p + n], s[b, :n]) for c, s in zip(other["k_cache"], other["k_suf"]))


def test_other_threads_run_during_a_call(lsp, tmp_path):
    """The entry point is replaced by a host function that waits up to two seconds for a flag, which another Python thread sets."""
    src = tmp_path / "wait.c"
    src.write_text("#include <unistd.h>\nvolatile int flag;\nint wait_for_flag(void) {\n"
                   "  for (int i = 0; i < 2000 && !flag; ++i) usleep(1000);\n  return flag ? 0 : 7;\n}\n")
    subprocess.run(["gcc", "-shared", "-fPIC", str(src), "-o", str(tmp_path / "wait.so")], check=True)
    fake = ctypes.CDLL(str(tmp_path / "wait.so"))
    addr = [ctypes.cast(getattr(lsp.lib(), n), ctypes.c_void_p).value for n in lsp.NATIVE_ENTRIES]
    i32 = [torch.zeros(n, dtype=torch.int32, device="cuda") for n in ((2, 3), 2, 2, 2, (2, 3))]

    def release():
        time.sleep(0.05)
        ctypes.c_int.in_dll(fake, "flag").value = 1

    lsp._nat.bind(*[ctypes.cast(fake.wait_for_flag, ctypes.c_void_p).value if n == "lsp_flip_update" else a for n, a in zip(lsp.NATIVE_ENTRIES, addr)])
    try:
        t = threading.Thread(target=release)
        t.start()
        rc = lsp._nat.flip_update(*i32, torch.zeros(4, dtype=torch.int64, device="cuda"), 1, 0, None)
        t.join()
    finally:
        lsp._nat.bind(*addr)
    assert rc == 0


def test_unusual_arguments_reach_the_general_path(lsp):
    w, kv, pl, sl, z, bm, tok = _state()
    out = _conf_out(w.B, w.S)
    k = kv[0]
    with pytest.raises(lsp.LspError, match="suffix_len must be torch.int32"):
        lsp.confidence(z, sl.long(), out=out)
    with pytest.raises(lsp.LspError, match="device tensors only"):
        lsp.attn_step(k["q"].cpu(), k["k_suf"], k["v_suf"], k["k_cache"], k["v_cache"], pl, sl)
    with pytest.raises(lsp.LspError, match="v_cache must be"):
        lsp.attn_step(k["q"], k["k_suf"], k["v_suf"], k["k_cache"], k["v_cache"].float(), pl, sl)
    with pytest.raises(lsp.LspError, match="bitmap holds"):
        lsp.commit(out[2], out[0], bm[:1].contiguous(), w.V, 0.9, 4, 1, 1, pl, sl, C=w.C, out=_commit_out(w.B, w.S))
    with pytest.raises(lsp.LspError, match="NaN"):         # an error of the library itself
        lsp.commit(out[2], out[0], bm, w.V, float("nan"), 4, 1, 1, pl, sl, C=w.C, out=_commit_out(w.B, w.S))


def test_a_missing_workspace_is_allocated_by_the_general_path(lsp):
    g = torch.Generator(device="cuda").manual_seed(5)
    z = torch.randn((1, 5, 40000), generator=g, device="cuda")         # few long rows are split over workgroups
    out = _conf_out(1, 5)
    assert lsp.confidence_workspace_bytes(*z.shape) > 0 and lsp._nat.confidence(z, None, out, None) is None
    assert torch.equal(lsp.confidence(z, None, out=out)[0].long(), z.argmax(-1))
    h, wt = (torch.randint(-3, 4, s, generator=g, device="cuda").to(torch.bfloat16) for s in ((1, 5, 64), (600, 64)))
    small = torch.empty(lsp.lm_head_confidence_workspace_bytes(1, 5, 600) - 16, dtype=torch.uint8, device="cuda")
    assert lsp._nat.lm_head_confidence(h, wt, None, out, small) is None
    top = (h.float() @ wt.float().T).topk(2, -1).values                # integers: exact
    assert torch.equal(lsp.lm_head_confidence(h, wt, None, out=out, workspace=small)[2], top[..., 0] - top[..., 1])
