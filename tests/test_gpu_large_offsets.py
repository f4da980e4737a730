"""GPU parity on tensors of more than 2**31 elements (more than 2**32 bytes): the shapes a
288 GB device holds once the batch or the cache grows past the workload sizes.  Element
and byte offsets of the later sequences no longer fit 32 bits, so any index arithmetic
done in int would read or write the wrong rows: sampled outputs are compared with the
oracle, and the structure planted by the input generator is checked on every row."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lsp():
    import paper_2603_05454_amd as m
    assert torch.cuda.is_available()
    return m


def test_confidence_on_logits_beyond_2_31_elements(lsp, oracle):
    """20 x 1024 x 126464 bf16 logits (2.59e9 elements, 5.2 GB).  Eq. 1 on rows at both ends,
    on the rows either side of the 2**31-element and 2**32-byte marks, and on a seeded sample."""
    w = W.scaled(W.C4, B=20)
    z, info = W.make_logits(w, device="cuda")
    assert z.numel() > 2**31
    ids, p, m = lsp.confidence(z)
    torch.cuda.synchronize()
    R = w.B * w.S
    marks = [2**31 // w.V, 2**32 // (2 * w.V), 2**32 // w.V]
    g = torch.Generator().manual_seed(11)
    rows = torch.cat([torch.tensor([0, R - 1] + [r + d for r in marks for d in (-1, 0, 1) if r + d < R]),
                      torch.randint(R // 2, R, (100,), generator=g)])
    zs = z.view(-1, w.V)[rows.cuda()].cpu().unsqueeze(0)
    ids_r, p_r, m_r = oracle.confidence(zs)
    assert torch.equal(ids.view(-1)[rows.cuda()].cpu(), ids_r[0])
    assert torch.equal(m.view(-1)[rows.cuda()].cpu(), m_r[0])
    assert (p.view(-1)[rows.cuda()].cpu() - p_r[0]).abs().max().item() <= 2e-2
    # every sequence, also those stored beyond the marks: the planted token wins where the boost is large
    assert torch.equal(ids[:, :32].long(), info["planted_id"][:, :32])
    assert torch.all(m >= 0) and torch.all(p <= 1.0 + 1e-6) and torch.all(p >= 1.0 / w.V)


def test_commit_appends_into_caches_beyond_2_31_elements(lsp, oracle):
    """One layer whose K and V cache hold 8 x 73728 x 32 x 128 bf16 (2.4e9 elements, 4.8 GB each), every
    sequence's prefix close to the end of its slab: boundaries, tokens, lengths and the WHOLE caches
    bit-exact against the oracle (a stray row anywhere in the 9.6 GB would show)."""
    B, S, C, Hkv, D, Vv = 8, 1024, 73728, 32, 128, 4096
    assert B * C * Hkv * D > 2**31
    w = W.scaled(W.C4, B=B, S=S, C=C, P=C - S, Hkv=Hkv, D=D, seed=77)
    src = W.make_layer_kv(W.scaled(w, C=1, P=1), 0)          # suffix K/V from the generator; the caches start at zero
    g = torch.Generator().manual_seed(3)
    margin = 1.0 + torch.rand((B, S), generator=g)
    firsts = [0, 1, 63, 500, 777, 1000, 1023, 1024]
    for b, f in enumerate(firsts):
        if f < S:
            margin[b, f] = 0.25
    ids = torch.randint(0, Vv, (B, S), generator=g, dtype=torch.int32)
    bm = torch.zeros(Vv // 32, dtype=torch.int32)             # no delimiters: the boundary is the first unstable row
    pl = torch.tensor([C - S - 3 * b for b in range(B)], dtype=torch.int32)
    sl = torch.full((B,), S, dtype=torch.int32)
    tokens = torch.full((B, C), -1, dtype=torch.int32)

    pl_r, sl_r, tok_r = pl.clone(), sl.clone(), tokens.clone()
    kc_r = torch.zeros((B, C, Hkv, D), dtype=torch.bfloat16)
    vc_r = torch.zeros((B, C, Hkv, D), dtype=torch.bfloat16)
    ref = oracle.commit(margin, ids, bm, Vv, 0.9, 0, 1, 0, pl_r, sl_r, tokens=tok_r,
                        k_suf=[src["k_suf"]], v_suf=[src["v_suf"]], k_cache=[kc_r], v_cache=[vc_r])
    assert ref["commit_len"].tolist() == [max(f, 1) for f in firsts]

    pl_g, sl_g, tok_g = pl.cuda(), sl.cuda(), tokens.cuda()
    kc_g = torch.zeros((B, C, Hkv, D), dtype=torch.bfloat16, device="cuda")
    vc_g = torch.zeros((B, C, Hkv, D), dtype=torch.bfloat16, device="cuda")
    table = lsp.LayerTable([src["k_suf"].cuda()], [src["v_suf"].cuda()], [kc_g], [vc_g])
    got = lsp.commit(margin.cuda(), ids.cuda(), bm.cuda(), Vv, 0.9, 0, 1, 0, pl_g, sl_g, tokens=tok_g, layers=table, C=C)
    torch.cuda.synchronize()
    for k in ("raw_boundary", "snapped_boundary", "commit_len", "status_flags", "stable_mask"):
        assert torch.equal(got[k].cpu(), ref[k]), k
    assert torch.equal(pl_g.cpu(), pl_r) and torch.equal(sl_g.cpu(), sl_r) and torch.equal(tok_g.cpu(), tok_r)
    for got_c, ref_c, name in ((kc_g, kc_r, "k_cache"), (vc_g, vc_r, "v_cache")):
        host = got_c.cpu()
        for b in range(B):                                    # sequence by sequence: a failure names its slab
            assert torch.equal(host[b].view(torch.int16), ref_c[b].view(torch.int16)), (name, b)
        del host


@pytest.mark.parametrize("S", [48, 300])
def test_attention_over_caches_beyond_2_31_elements(lsp, oracle, S):
    """17 sequences of 131072 cache rows x 8 KV heads x 128 (2.28e9 elements, 4.6 GB per cache tensor):
    the last sequences' keys start beyond the 2**31-element mark.  S = 48 takes the short-suffix launch,
    S = 300 the long-suffix one.  Oracle on sampled (sequence, row, head) of the first and last sequences,
    each given to it as a batch of one."""
    B, C, Hkv, Hq, D = 17, 131072, 8, 16, 128
    assert B * C * Hkv * D > 2**31
    w = W.scaled(W.C2, B=B, S=S, P=C, C=C, Hq=Hq, Hkv=Hkv, D=D, seed=515)
    pl = torch.tensor([130000 - 4099 * b for b in range(B)], dtype=torch.int32)
    sl = torch.tensor([S - (b % 3) for b in range(B)], dtype=torch.int32)
    kv = W.make_layer_kv(w, 0, device="cuda", prefix_len=pl)
    out = torch.full((B, S, Hq, D), 123.0, dtype=torch.bfloat16, device="cuda")
    lsp.attn_step(kv["q"], kv["k_suf"], kv["v_suf"], kv["k_cache"], kv["v_cache"], pl.cuda(), sl.cuda(), out=out)
    torch.cuda.synchronize()
    worst = 0.0
    for b in (0, B - 2, B - 1):
        n = int(sl[b])
        one = {k: v[b:b + 1].cpu() for k, v in kv.items()}
        rows = torch.tensor([[0, i, h] for i in (0, n // 2, n - 1) for h in (0, 7, Hq - 1)], dtype=torch.int32)
        ref = oracle.attention(**one, prefix_len=pl[b:b + 1], suffix_len=sl[b:b + 1], rows=rows)
        sel = out[b, rows[:, 1].long().cuda(), rows[:, 2].long().cuda()].float().cpu()
        worst = max(worst, (sel - ref).abs().max().item())
        assert torch.all(out[b, n:].float() == 123.0) and not torch.isnan(out[b, :n].float()).any()
    assert worst <= 2e-2, worst


def test_f32_attention_in_more_workgroups_than_one_grid_dimension_holds(lsp, oracle):
    """65535 sequences x 32 heads x 5 query tiles: 10.5 million workgroups of 512 threads, where a grid dimension ends at
    2**32 threads.  All sequences share one set of operands (batch stride 0) and all but two have no active row."""
    B, S, H, D, P = 65535, 65, 32, 64, 20
    w = W.scaled(W.C2, dtype="f32", B=1, S=S, P=P, C=P, Hq=H, Hkv=H, D=D, seed=91)
    kv = W.make_layer_kv(w, 0)
    for b, n in ((0, 17), (B - 1, S)):
        sl = torch.zeros(B, dtype=torch.int32, device="cuda")
        sl[b] = n
        out = torch.full((1, S, H, D), 123.0, device="cuda")
        g = {k: v.cuda().expand(B, -1, -1, -1) for k, v in kv.items()}
        lsp.attn_step(g["q"], g["k_suf"], g["v_suf"], g["k_cache"], g["v_cache"], torch.full_like(sl, P), sl, out=out.expand(B, -1, -1, -1))
        torch.cuda.synchronize()
        ref = oracle.attention(**kv, prefix_len=torch.tensor([P], dtype=torch.int32), suffix_len=torch.tensor([n], dtype=torch.int32))
        assert (out[:, :n].cpu() - ref[:, :n]).abs().max().item() <= 1e-5 and torch.all(out[:, n:] == 123.0)


def test_lm_head_on_more_rows_than_one_grid_dimension_holds_waves(lsp, oracle):
    """1100 x 61440 rows (67.6 million, one wave each in the second kernel, where a grid dimension ends at 2**26 waves): rows at
    both ends, either side of the mark and around the last full grid are bit-exact on small integers, and none is left out."""
    B, S, K, V = 1100, 61440, 8, 5
    g = torch.Generator(device="cuda").manual_seed(8)
    h = torch.randint(-3, 4, (B, S, K), generator=g, device="cuda", dtype=torch.int8).to(torch.bfloat16)
    w = torch.randint(-3, 4, (V, K), generator=g, device="cuda").to(torch.bfloat16)
    out = (torch.full((B, S), -7, dtype=torch.int32, device="cuda"), torch.full((B, S), -7.0, device="cuda"), torch.full((B, S), -7.0, device="cuda"))
    ids, p, m = (x.view(-1) for x in lsp.lm_head_confidence(h, w, out=out))
    torch.cuda.synchronize()
    R = B * S
    rows = torch.tensor([0, 1, 2**22 - 1, 2**22, 2**26 - 1, 2**26, 2**26 + 1, 2**26 + 300000, R - 2, R - 1], device="cuda")
    ids_r, p_r, m_r = oracle.lm_head_confidence(h.view(-1, K)[rows].cpu().unsqueeze(0), w.cpu())
    assert torch.equal(ids[rows].cpu(), ids_r[0]) and torch.equal(m[rows].cpu(), m_r[0])
    assert (p[rows].cpu() - p_r[0]).abs().max().item() <= 1e-6
    # p = 1 / (fp32 sum of V exponentials, the largest of which is 1 up to rounding): within 1e-6 of [1 / V, 1]
    assert ((ids >= 0) & (ids < V)).all() and (m >= 0).all() and ((p >= 1 / V - 1e-6) & (p <= 1 + 1e-6)).all()
