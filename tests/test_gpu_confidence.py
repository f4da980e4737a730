"""GPU parity: lsp_confidence against the CPU oracle (Eq. 1, Algorithm 1 line 5).
ids and margins bit-exact; top-1 probability within 1e-5 (fp32) / 2e-2 (bf16)."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
TOL = {torch.float32: 1e-5, torch.bfloat16: 2e-2}


@pytest.fixture(scope="module")
def lsp():
    import paper_2603_05454_amd as m
    assert torch.cuda.is_available()
    return m


def _check(lsp, oracle, z, sl=None, z_gpu=None):
    zg = z.cuda() if z_gpu is None else z_gpu
    B, S, V = z.shape
    out = (torch.full((B, S), -7, dtype=torch.int32, device="cuda"),
           torch.full((B, S), -7.0, device="cuda"), torch.full((B, S), -7.0, device="cuda"))
    slg = None if sl is None else sl.cuda()
    ids, p, m = lsp.confidence(zg, slg, out=out)
    torch.cuda.synchronize()
    ids_r, p_r, m_r = oracle.confidence(z, sl)
    act = ids_r >= 0
    assert torch.equal(ids.cpu()[act], ids_r[act])
    assert torch.equal(m.cpu()[act], m_r[act])
    assert (p.cpu()[act] - p_r[act]).abs().max().item() <= TOL[z.dtype]
    # inactive rows are not written
    assert torch.all(ids.cpu()[~act] == -7) and torch.all(m.cpu()[~act] == -7.0)
    return ids_r, p_r, m_r


def test_c1_tiny_fp32(lsp, oracle):
    z, _ = W.make_logits(W.C1)
    _check(lsp, oracle, z)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V", [2, 7, 63, 1000, 4099, 40007])
def test_ragged_vocab_sizes(lsp, oracle, dtype, V):
    """V not a multiple of the vector width: rows start at every alignment, so
    the scalar head/tail paths and several tiles per row are exercised."""
    g = torch.Generator().manual_seed(V)
    z = (2 * torch.randn((2, 9, V), generator=g)).to(dtype)
    _check(lsp, oracle, z)


def test_ties_and_lowest_index(lsp, oracle):
    g = torch.Generator().manual_seed(5)
    z = torch.randn((1, 128, 20000), generator=g).to(torch.bfloat16)
    # plant exact duplicates of the maximum at many distances (same lane, other lanes, other waves)
    for i in range(64):
        a, b = (37 * i) % 20000, (37 * i + 1 + 311 * i) % 20000
        z[0, i, a] = 9.0
        z[0, i, b] = 9.0
    ids_r, _, m_r = _check(lsp, oracle, z)
    assert torch.all(m_r[0, :64] == 0)


def test_minus_inf_entries(lsp, oracle):
    z = torch.randn((1, 4, 5000), generator=torch.Generator().manual_seed(1))
    z[0, 0, 100:4000] = -float("inf")
    z[0, 1, :] = -float("inf")
    z[0, 1, 4321] = 2.0
    z[0, 1, 17] = 1.0
    z[0, 2, :4990] = -float("inf")
    _check(lsp, oracle, z)
    _check(lsp, oracle, z.to(torch.bfloat16))


def test_suffix_len_rows_skipped(lsp, oracle):
    z = torch.randn((3, 10, 3000), generator=torch.Generator().manual_seed(2)).to(torch.bfloat16)
    _check(lsp, oracle, z, torch.tensor([10, 0, 4], dtype=torch.int32))


def test_strided_rows(lsp, oracle):
    """Rows taken out of a wider buffer (row stride > V, odd offsets)."""
    big = torch.randn((2, 6, 5003), generator=torch.Generator().manual_seed(3)).to(torch.bfloat16)
    view_cpu = big[:, :, 1:4098]
    ids, p, m = lsp.confidence(big.cuda()[:, :, 1:4098])
    torch.cuda.synchronize()
    ids_r, p_r, m_r = oracle.confidence(view_cpu.contiguous())
    assert torch.equal(ids.cpu(), ids_r) and torch.equal(m.cpu(), m_r)
    assert (p.cpu() - p_r).abs().max().item() <= 2e-2


@pytest.mark.parametrize("rows", [1, 3, 40])
def test_few_rows_split_over_workgroups(lsp, oracle, rows):
    """With few rows each row is cut into segments reduced by separate
    workgroups; one of them merges the row."""
    V = 126464
    assert lsp.confidence_workspace_bytes(1, rows, V) > 0
    g = torch.Generator().manual_seed(rows)
    z = torch.randn((1, rows, V), generator=g).to(torch.bfloat16)
    z[0, 0, 70000] = 9.0
    z[0, 0, 3] = 9.0           # tie across segments: the earlier one must win
    ids_r, _, _ = _check(lsp, oracle, z)
    assert ids_r[0, 0] == 3


def test_c2_full_size(lsp, oracle):
    z, info = W.make_logits(W.C2)
    ids_r, p_r, m_r = _check(lsp, oracle, z)
    assert torch.equal(ids_r[0, :64].long(), info["planted_id"][0, :64])


def test_c3_full_size_gqa_vocab(lsp, oracle):
    w = W.C3
    z, info = W.make_logits(w, device="cuda")
    ids, p, m = lsp.confidence(z)
    torch.cuda.synchronize()
    # oracle on a seeded sample of rows (all of sequence 0's first 64 + 64 random rows)
    g = torch.Generator().manual_seed(7)
    rows = torch.cat([torch.arange(64), torch.randint(0, w.B * w.S, (64,), generator=g)])
    zs = z.view(-1, w.V)[rows.cuda()].cpu().unsqueeze(0)
    ids_r, p_r, m_r = oracle.confidence(zs)
    assert torch.equal(ids.view(-1)[rows.cuda()].cpu(), ids_r[0])
    assert torch.equal(m.view(-1)[rows.cuda()].cpu(), m_r[0])
    assert (p.view(-1)[rows.cuda()].cpu() - p_r[0]).abs().max().item() <= 2e-2
    # properties that hold on every row: bounds and the planted structure
    assert torch.all(p <= 1.0 + 1e-6) and torch.all(p >= 1.0 / w.V) and torch.all(m >= 0)
    for b in range(w.B):
        lb = int(info["stable_len"][b])
        assert torch.all(m[b, :lb] > w.tau)
        if lb < w.S:
            assert m[b, lb].item() == 0.0


def test_c4_shape_sampled(lsp, oracle):
    """Config-4 logits (8 x 1024 x 126464 bf16, 2.07 GB): whole tensor on the
    GPU, oracle on sampled rows."""
    w = W.C4
    z, info = W.make_logits(w, device="cuda")
    ids, p, m = lsp.confidence(z)
    torch.cuda.synchronize()
    g = torch.Generator().manual_seed(9)
    rows = torch.cat([torch.tensor([0, 1, w.S - 1, w.B * w.S - 1]), torch.randint(0, w.B * w.S, (124,), generator=g)])
    zs = z.view(-1, w.V)[rows.cuda()].cpu().unsqueeze(0)
    ids_r, p_r, m_r = oracle.confidence(zs)
    assert torch.equal(ids.view(-1)[rows.cuda()].cpu(), ids_r[0])
    assert torch.equal(m.view(-1)[rows.cuda()].cpu(), m_r[0])
    assert (p.view(-1)[rows.cuda()].cpu() - p_r[0]).abs().max().item() <= 2e-2
    assert torch.equal(ids[:, :32].long(), info["planted_id"][:, :32])


def test_deterministic(lsp):
    z = torch.randn((1, 300, 50000), generator=torch.Generator().manual_seed(4)).to(torch.bfloat16).cuda()
    a = lsp.confidence(z)
    b = lsp.confidence(z)
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x, y)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_wide_dynamic_range_and_moving_maximum(lsp, oracle, dtype):
    """Rows that force the lagging soft-max reference to move: a slow ramp (every
    lane's maximum keeps rising), a late spike far above everything before it, an
    early spike followed by a long flat tail, large negative offsets, and a row
    whose sum is dominated by many near-maximal entries."""
    V = 50021
    z = torch.zeros((1, 6, V))
    idx = torch.arange(V, dtype=torch.float32)
    z[0, 0] = idx * (300.0 / V) - 150.0                    # ramp over 300 units
    z[0, 1] = torch.randn(V, generator=torch.Generator().manual_seed(1))
    z[0, 1, V - 5] = 500.0                                 # late spike
    z[0, 2] = torch.randn(V, generator=torch.Generator().manual_seed(2))
    z[0, 2, 2] = 250.0                                     # early spike
    z[0, 3] = torch.randn(V, generator=torch.Generator().manual_seed(3)) - 3000.0
    z[0, 4] = 40.0 - (idx % 7) * 0.125                     # thousands of entries at and near the maximum
    z[0, 5] = -(idx * (200.0 / V))                         # falling ramp: the first entry is the maximum
    z = z.to(dtype)
    ids_r, p_r, m_r = _check(lsp, oracle, z)
    assert ids_r[0, 1] == V - 5 and ids_r[0, 2] == 2 and ids_r[0, 5] == 0 and ids_r[0, 4] == 0
    assert m_r[0, 4] == 0.0


def test_unaligned_start_and_odd_lengths(lsp, oracle):
    """Every alignment of the first element against a 16-byte boundary, vocab sizes
    around the vector and group sizes, in both element types."""
    g = torch.Generator().manual_seed(9)
    for dtype, per16 in ((torch.bfloat16, 8), (torch.float32, 4)):
        for off in range(per16):
            for V in (per16 * 64 * 4 - 1, per16 * 64 * 4 + 1, 1031):
                big = torch.randn((1, 3, V + off + 3), generator=g).to(dtype)
                view = big[:, :, off:off + V]
                ids, p, m = lsp.confidence(big.cuda()[:, :, off:off + V])
                torch.cuda.synchronize()
                ids_r, p_r, m_r = oracle.confidence(view.contiguous())
                assert torch.equal(ids.cpu(), ids_r) and torch.equal(m.cpu(), m_r), (dtype, off, V)
                assert (p.cpu() - p_r).abs().max().item() <= TOL[dtype]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,S,V,n", [
    (1, 300, 20000, [5]),               # 4 segments a row
    (1, 256, 126464, [256]),            # as many rows as workgroups: whole
    (1, 256, 126464, [129]), (1, 256, 126464, [128]),   # first count that is not halved, last one that is
    (3, 150, 70001, [0, 1, 149]),       # rows of every alignment, an empty sequence, whole
    (3, 150, 70001, [0, 1, 99]),        # the same, halved
    (70, 2, 20011, None),               # lengths of more sequences than a wave has lanes
    (300, 1, 17000, None),              # more sequences than the kernel counts: whole rows
    (2, 37, 126464, [33, 32]),          # fp32 rows in four segments, bf16 in two
    (1, 150, 20011, [100]),             # bf16 rows not halved
    (4, 200, 100003, [61, 0, 7, 200]),  # lengths through the scalar cache
    (8, 100, 60011, [100, 99, 0, 1, 100, 0, 0, 13]),
])
def test_active_rows_cut_into_segments(lsp, dtype, B, S, V, n):
    """Rows are cut by the number of ACTIVE ones.  The workspace holds anything; ids and margins are those of whole
    rows bit for bit, and a probability differs by the order of one fp32 sum: rel 2e-6 is 16 roundings of a sum of
    at most 16 segments, each of which is itself within a few."""
    g = torch.Generator().manual_seed(B * S + V)
    z = (2 * torch.randn((B, S, V), generator=g)).to(dtype).cuda()
    n = torch.tensor(n) if n is not None else torch.randint(0, S + 1, (B,), generator=g)
    sl = n.to(torch.int32).cuda()
    active = [(b, i) for b in range(B) for i in range(int(n[b]))]
    tie, low, high = active[0], active[-1], active[len(active) // 2]
    assert len({tie, low, high}) == 3
    z[tie][V - 1] = z[tie][7] = 15.0        # a tie between the first and the last segment
    z[low][:V // 2] = -float("inf")         # first segments without a finite entry
    z[high][V // 2:] = -float("inf")        # last ones
    out = [(torch.full((B, S), -7, dtype=torch.int32, device="cuda"), torch.full((B, S), -7.0, device="cuda"),
            torch.full((B, S), -7.0, device="cuda")) for _ in range(3)]
    # against fp64 sums of all active rows, and against whole rows (no workspace, where that is allowed)
    ws = torch.randint(0, 256, (lsp.confidence_workspace_bytes(B, S, V),), dtype=torch.uint8, generator=g).cuda()
    lsp.confidence(z, sl, out=out[0], workspace=ws)
    lsp.confidence(z, sl, out=out[1], workspace=ws)                 # left clean by the first
    act = torch.arange(S, device="cuda")[None] < sl[:, None]
    for a, b in zip(out[0], out[1]):
        assert torch.equal(a, b) and torch.all(a[~act] == -7)
    zz = z.float()
    top2 = zz.topk(2, dim=-1).values
    first = (zz == top2[..., :1]).to(torch.int8).argmax(-1).to(torch.int32)     # argmax of a mask: the first of equals
    prob = 1 / (zz.double() - top2[..., :1].double()).exp().sum(-1)
    assert out[0][0][tie] == 7 and out[0][2][tie] == 0 and out[0][0][low] >= V // 2 and out[0][0][high] < V // 2
    assert torch.equal(out[0][0][act], first[act])
    assert torch.equal(out[0][2][act], (top2[..., 0] - top2[..., 1])[act])
    assert ((out[0][1].double() - prob)[act] / prob[act]).abs().max() <= 2e-6
    if B * S >= 128:
        lsp.confidence(z, sl, out=out[2])       # whole rows
        assert torch.equal(out[0][0], out[2][0]) and torch.equal(out[0][2], out[2][2])


def test_segments_under_graph_replay(lsp):
    """Every replay carries the same tag: what one leaves in the workspace must not pass for the next one's."""
    B, S, V = 1, 200, 65536
    z = torch.randn((B, S, V), device="cuda", dtype=torch.bfloat16, generator=torch.Generator(device="cuda").manual_seed(3))
    sl = torch.tensor([30], dtype=torch.int32, device="cuda")
    out = (torch.zeros((B, S), dtype=torch.int32, device="cuda"), torch.zeros((B, S), device="cuda"), torch.zeros((B, S), device="cuda"))
    ws = torch.zeros(lsp.confidence_workspace_bytes(B, S, V), dtype=torch.uint8, device="cuda")
    lsp.confidence(z, sl, out=out, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lsp.confidence(z, sl, out=out, workspace=ws)
    for k in range(6):
        z.copy_(z.roll(1000 * k + 1, dims=-1))
        sl.fill_(30 - 5 * k)
        ref = lsp.confidence(z, sl, out=tuple(torch.zeros_like(t) for t in out), workspace=torch.zeros_like(ws))
        for t in out:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(out, ref):
            assert torch.equal(a, b)


@pytest.mark.parametrize("native", [True, False])
@pytest.mark.parametrize("rows", [60, 200])
def test_strided_workspace_is_not_written(lsp, rows, native, monkeypatch):
    """A workspace that is one column of something else: the call does without it, and what lies between stays."""
    lsp.lib()
    if not native:
        monkeypatch.setattr(lsp, "_nat", None)
    V = 40000
    z = torch.randn((1, rows, V), generator=torch.Generator().manual_seed(rows)).to(torch.bfloat16).cuda()
    sl = torch.tensor([20], dtype=torch.int32, device="cuda")
    held = torch.full((lsp.confidence_workspace_bytes(1, rows, V), 4), 77, dtype=torch.uint8, device="cuda")
    ids, prob, margin = lsp.confidence(z, sl, workspace=held[:, 0])
    assert torch.all(held == 77)
    zz = z[0, :20].float()
    top2 = zz.topk(2, dim=-1).values
    assert torch.equal(zz.gather(1, ids[0, :20, None].long()), top2[:, :1]) and torch.equal(margin[0, :20], top2[:, 0] - top2[:, 1])


@pytest.mark.parametrize("native", [True, False])
@pytest.mark.parametrize("given", ["none", "small", "unaligned", "host", "right"])
def test_workspace_that_is_needed(lsp, given, native, monkeypatch):
    """Few long rows: a call without a workspace that will do brings its own, and no call is made in vain where it can be seen
    beforehand."""
    lsp.lib()
    if not native:
        monkeypatch.setattr(lsp, "_nat", None)
    library, tried = lsp.lib(), []

    class Counted:      # the library, as the general path calls it
        def __getattr__(self, name):
            return getattr(library, name)

        def lsp_confidence(self, *a):
            tried.append(library.lsp_confidence(*a))
            return tried[-1]

    z = torch.randn((1, 6, 40000), generator=torch.Generator().manual_seed(1)).cuda()
    need = lsp.confidence_workspace_bytes(1, 6, 40000)
    ws = dict(none=None, small=torch.empty(16, dtype=torch.uint8, device="cuda"), unaligned=torch.empty(need + 4, dtype=torch.uint8, device="cuda")[4:],
              host=torch.empty(need, dtype=torch.uint8), right=torch.empty(need, dtype=torch.uint8, device="cuda"))[given]
    monkeypatch.setattr(lsp, "_lib", Counted())
    ids, prob, margin = lsp.confidence(z, workspace=ws)
    top2 = z.topk(2, dim=-1)
    assert torch.equal(ids.long(), top2.indices[..., 0]) and torch.equal(margin, top2.values[..., 0] - top2.values[..., 1])
    assert tried == ([-3, 0] if given == "unaligned" else [] if native and given == "right" else [0])
