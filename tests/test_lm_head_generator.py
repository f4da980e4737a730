"""Host checks of the output head's generated K loops (csrc/gen_lm_head.py -> csrc/lsp_lm_head_loop_*.inc)."""
import importlib.util
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_05454_amd", "csrc")


def _gen():
    spec = importlib.util.spec_from_file_location("gen_lm_head", os.path.join(CSRC, "gen_lm_head.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


@pytest.mark.parametrize("height", [256, 128, 64])
def test_committed_loop_is_what_the_generator_emits(height):
    g = _gen()
    with open(os.path.join(CSRC, f"lsp_lm_head_loop_{height}.inc")) as f:
        assert f.read() == g.text(g.MODES[height])


@pytest.mark.parametrize("height", [256, 128, 64])
def test_fragments_and_stages_of_every_step(height):
    """Each matrix instruction's fragments were requested before the last wait that covers them; a stage is
    refilled only behind the barrier that follows its last reads; every accumulator block is updated once per
    k-slice; the loads of a step cover its stage exactly once."""
    g = _gen()
    M = g.MODES[height]
    lines = g.generate(M)
    body = lines[lines.index(".Lloop_%=:") + 1:lines.index("s_branch .Lloop_%=")]
    pending, updates, filled, reads = {}, {}, [], []
    for ln in body + body:      # twice: the step boundary as well
        m = re.match(r"ds_read_b128 v\[(\d+):", ln)
        if m:
            pending[int(m.group(1))] = True
            stage = (int(re.search(r", v(\d+) ", ln).group(1)) - M.addr) // (2 * M.NK)
            reads.append(stage)
        elif "lgkmcnt(0)" in ln:
            pending.clear()
        elif ln == "s_barrier":
            reads.clear()
        elif ln.startswith("s_add_u32 m0"):
            dst = int(ln.split(",")[-1])
            filled.append(dst)
            assert dst // M.STAGE not in reads      # nothing of that stage has been read since the barrier
        elif ln.startswith("v_mfma"):
            c, a, b = (int(x) for x in re.findall(r"v\[(\d+):", ln)[:3])
            assert a not in pending and b not in pending
            updates[c] = updates.get(c, 0) + 1
    assert set(updates) == {M.c(i, j) for i in range(M.MV) for j in range(M.MR)}
    assert set(updates.values()) == {2 * M.NSTG * M.NK}
    per_stage = sorted(set(filled))
    assert len(filled) == 2 * len(per_stage) and len(per_stage) == M.NSTG * (M.LW + M.LH)
    assert all(d % M.STAGE % 8192 == 0 for d in per_stage)


class _Wave:
    """The loop's scalar part and its loads, run for one wave and two of its lanes (chunks 0 and 7 of a row): what every
    load fetches, what every matrix instruction therefore multiplies, in which order a tile sums."""
    ZEROS = 1 << 50

    def __init__(self, M, lines):
        self.M, self.lines = M, lines
        self.label = {x[:-1]: n for n, x in enumerate(lines) if x.endswith(":")}
        self.flight, self.lds = [], {}

    def request(self, dst, addr):
        self.flight.append((dst, tuple(addr)))

    def run(self, env, ptr, nxt):
        """`ptr`: register -> [address per lane]; `nxt`: the next tile's hidden pointers."""
        M, s, m0, scc, frag, acc, pc = self.M, {}, 0, False, {}, {}, 0
        on = [True, True]

        def val(x):
            return env[x[2:-1]] if x.startswith("%[") else s[x] if x.startswith("s") else int(x) & 0xffffffff

        while pc < len(self.lines):
            op, _, rest = self.lines[pc].partition(" ")
            a = [x.strip() for x in rest.split(",")]
            pc += 1
            if op.endswith(":") or op in ("s_barrier", "s_nop") or "m0" in a[1:]:
                continue
            if op in ("s_mov_b32", "s_movk_i32"):
                if a[0] != "m0":
                    s[a[0]] = val(a[1])
            elif op == "s_add_u32":
                if a[0] == "m0":
                    m0 = int(a[2])
                else:
                    s[a[0]] = val(a[1]) + val(a[2])
            elif op == "s_cmp_eq_u32":
                scc = val(a[0]) == val(a[1])
            elif op == "s_cmp_lt_u32":
                scc = val(a[0]) < val(a[1])
            elif op == "s_branch" or (op == "s_cbranch_scc1" and scc) or (op == "s_cbranch_scc0" and not scc):
                pc = self.label[a[0]]
            elif op == "s_cselect_b64":
                on = env["zmask"] if scc else [True, True]
            elif op == "s_mov_b64":
                on = [True, True]
            elif op == "s_waitcnt":
                m = re.search(r"vmcnt\((\d+)\)", rest)
                while m and len(self.flight) > int(m.group(1)):
                    dst, addr = self.flight.pop(0)
                    self.lds[dst] = addr
            elif op == "global_load_lds_dwordx4":
                self.request(m0, ptr[int(re.match(r"v\[(\d+)", a[0]).group(1))])
            elif op == "v_lshl_add_u64":
                r, by = int(re.match(r"v\[(\d+)", a[0]).group(1)), 2 * M.KB if a[3].startswith("s[") else env[a[3][2:-1]]
                ptr[r] = [x + by if o else x for x, o in zip(ptr[r], on)]
            elif op == "v_mov_b32":
                r = int(a[0][1:])
                if r in ptr:      # the low half stands for the pointer
                    new = [self.ZEROS] * 2 if a[1] == "%[zlo]" else nxt[(int(a[1][1:]) - M.next) // 2]
                    ptr[r] = [y if o else x for x, y, o in zip(ptr[r], new, on)]
            elif op == "ds_read_b128":
                r, base, off = int(re.match(r"v\[(\d+)", a[0]).group(1)), int(re.match(r"v(\d+)", a[1]).group(1)), int(re.search(r"offset:(\d+)", a[1]).group(1))
                if base == M.next and M.TR == 256:
                    ptr[r], ptr[r + 2] = nxt[off // 4096], nxt[off // 4096 + 1]
                else:
                    stage, kk, hidden = (base - M.addr) // (2 * M.NK), (base - M.addr) // 2 % M.NK, (base - M.addr) % 2
                    at = stage * M.STAGE + (M.TILE_W if hidden else 0)
                    pieces = [self.lds[at + 8192 * i] for i in range(M.LH if hidden else M.LW)]
                    assert all(d != at + 8192 * i for d, _ in self.flight for i in range(len(pieces)))     # nothing of it is still on its way
                    frag[r] = (pieces, kk)
            elif op.startswith("v_mfma"):
                c, x, y = (int(re.match(r"v\[(\d+)", t).group(1)) for t in a[:3])
                acc.setdefault(c, []).append((frag[x], frag[y]))
            else:
                assert op in ("s_cbranch_scc0", "s_cbranch_scc1"), op
        return acc


@pytest.mark.parametrize("height", [256, 128, 64])
@pytest.mark.parametrize("K", [8, 64, 72, 128, 136, 192, 200, 256, 320, 328, 64 * 37])
def test_every_tile_sums_its_own_steps_in_order(height, K):
    """Four tiles of a workgroup, handed over by the loop where the kernel allows it (whole K steps, more of them than
    stages) except into the last one, which stands for a ragged vocabulary tile: every matrix instruction gets both operands of
    one k-slice of this tile, from k = 0 upwards, zeros beyond K; the stage of step 0 is whatever the tile before left."""
    g = _gen()
    M = g.MODES[height]
    W = _Wave(M, g.generate(M))
    NS, KB, chunks = M.NSTG, M.KB, (0, 7)
    real = (K + KB - 1) // KB
    KS, tail, stage, requested = max(real, NS), K % KB // 8, 0, False

    def row(tile, i, hidden):      # addresses at k = 0 of load i of a tile's operand, per lane
        return [(tile + 1) * (1 << 40) + hidden * (1 << 39) + i * (1 << 30) + 16 * c for c in chunks]

    for t in range(4):
        w, h = [row(t, i, 0) for i in range(M.LW)], [row(t, i, 1) for i in range(M.LH)]
        if not requested:
            stage = 0
            for p in range(NS):
                for i, (at, base) in enumerate([(0, x) for x in w] + [(M.TILE_W, x) for x in h]):
                    k = i if at == 0 else i - M.LW
                    W.request(p * M.STAGE + at + 8192 * k, [x + p * 2 * KB if p * KB + 8 * c < K else W.ZEROS for x, c in zip(base, chunks)])
        cross = t < 2 and tail == 0 and real > NS
        ptr = {M.wptr + 2 * i: [x + NS * 2 * KB for x in w[i]] for i in range(M.LW)}
        ptr.update({M.hptr + 2 * i: [x + NS * 2 * KB for x in h[i]] for i in range(M.LH)})
        env = dict(ks=KS, event=min(KS, max(K // KB, NS)), phase=stage, more=int(cross), wstep=(1 << 40) - KS * 2 * KB, zmask=[c >= tail for c in chunks])
        acc = W.run(env, ptr, [row(t + 1, i, 1) for i in range(M.LH)])
        requested, stage = cross, (stage + KS) % NS
        assert set(acc) == {M.c(i, j) for i in range(M.MV) for j in range(M.MR)}
        want = [(k, kk) for k in range(KS) for kk in range(M.NK)]

        def fetched(base, k):
            return tuple(x + k * 2 * KB if k * KB + 8 * c < K else None for x, c in zip(base, chunks))

        def seen(addr):
            return tuple(None if W.ZEROS <= x < W.ZEROS + 1024 - 16 else x for x in addr)

        for steps in acc.values():
            assert len(steps) == len(want)
            for (k, kk), ((wp, wk), (hp, hk)) in zip(want, steps):
                assert wk == hk == kk
                assert [seen(x) for x in wp] == [fetched(x, k) for x in w] and [seen(x) for x in hp] == [fetched(x, k) for x in h]
