"""Host-side checks of the generated block loop of four-wave workgroups (csrc/gen_attn_pipe.py ->
csrc/lsp_attn_half_loop.inc, lsp_attn_half_idle_loop.inc): what the generator emits is committed, every LDS
result is waited for, and the scalar skeleton of both loops, run on concrete key streams, requests every
block once, in order, into a stage that nobody reads any more, and has waited for what is read after each barrier."""
import os
import re

import pytest

from test_attn_pipe_generator import CSRC, _split, _vregs, _walk, gen  # noqa: F401

M = 0xFFFFFFFF
KC, VC, KS, VS, CSTEP, SSTEP, LDSK = 0x1FFFF0000, 0x2FFFF0000, 0x3FFFF0000, 0x4FFFF0000, 0x8000, 0x2000, 0x800


def _loops(gen):
    return {"half_loop": gen.generate_half(), "half_idle_loop": gen.generate_half_idle()}


@pytest.mark.parametrize("name", ["half_loop", "half_idle_loop"])
def test_committed_include_and_fields(gen, name):
    lines = _loops(gen)[name]
    with open(os.path.join(CSRC, f"lsp_attn_{name}.inc")) as f:
        assert re.findall(r'^    "(.*)\\n"$', f.read(), flags=re.M) == lines
    labels = {l[:-1] for l in lines if l.endswith(":")}
    for l in lines:
        mnem, rest = _split(l)
        assert not mnem.startswith(("s_store", "s_buffer_store", "s_atomic", "s_buffer_atomic", "s_dcache", "s_scratch_store", "v_pk_")), l
        assert all(int(n) <= 15 for n in re.findall(r"lgkmcnt\((\d+)\)", l)) and all(int(n) <= 63 for n in re.findall(r"vmcnt\((\d+)\)", l)), l
        assert all(int(n) <= 65535 for n in re.findall(r"offset:(\d+)", l)) and all(r < 244 for r in _vregs(l)), l
        if mnem.startswith(("s_cbranch", "s_branch")):
            assert rest in labels, l
        if name == "half_idle_loop":
            assert not mnem.startswith(("v_mfma", "ds_", "v_exp", "v_fma", "v_max", "v_cvt", "v_dot", "s_setprio")), l


def test_every_lds_result_is_waited_for(gen):
    lines = gen.generate_half()
    labels = {l[:-1]: k for k, l in enumerate(lines) if l.endswith(":")}
    conds, _, _ = _walk(lines, 0, [], labels, lambda t: t == ".Lloop_%=", max_steps=len(lines) * 3)
    for idx, target, pend in conds:
        if not target.startswith(".Lexit"):
            sub, _, end = _walk(lines, labels[target], pend, labels, lambda t: False, max_steps=400)
            assert not sub and lines[end].startswith("s_branch")
    assert lines[labels[".Lexit_%="] + 1] == "s_waitcnt vmcnt(0) lgkmcnt(0)"
    # K fragments of the block after next are the only reads in flight at a barrier, and K(j)'s stage is given away an
    # iteration later than they are waited for
    assert sum(l == "s_barrier" for l in lines) == 2 + gen.UNROLL_H


def _run(lines, nc, ns, nsh):
    """Events of a run on nc cache and ns suffix blocks: ("K" or "V", stage, half, address, offset register),
    ("read", "K" or "V", stage), ("wait", n) for loads, ("returned", n) for reads, ("barrier",), ("iteration",)."""
    labels = {l[:-1]: k for k, l in enumerate(lines) if l.endswith(":")}
    sym = {"%[kc]": KC, "%[vc]": VC, "%[ks]": KS, "%[vs]": VS, "%[cstep]": CSTEP, "%[sstep]": SSTEP, "%[nc]": nc, "%[nsuf]": ns, "%[ldsk]": LDSK}
    reg, scc, off = {"m0": 0}, 0, {164: "c0", 165: "c1", 166: "c0", 167: "c1"}
    off.update({240 + k: ("s" if ns > 0 else "c") + str(k % 2) for k in range(4)})       # (what the kernel passes in)

    def val(x):
        m = re.fullmatch(r"s\[(\d+):(\d+)\]", x)
        if m:
            return reg["s" + m[1]] | reg["s" + m[2]] << 32
        return sym[x] if x in sym else reg[x] if x in reg else int(x, 0) & M

    def put(x, v):
        m = re.fullmatch(r"s\[(\d+):(\d+)\]", x)
        if m:
            reg["s" + m[1]], reg["s" + m[2]] = v & M, v >> 32
        else:
            reg[x] = v & M

    ev, i = [], 0
    for _ in range(200000):
        if i >= len(lines):
            return ev
        l = lines[i]
        i += 1
        if l.endswith(":"):
            if l.startswith(".Lafter"):
                ev.append(("iteration",))
            continue
        mnem, rest = _split(l)
        o = [x.strip() for x in rest.split(",")]
        if mnem.startswith("s_mov"):
            put(o[0], val(o[1]))
        elif mnem in ("s_add_u32", "s_addc_u32"):
            t = val(o[1]) + val(o[2]) + (scc if "addc" in mnem else 0)
            put(o[0], t)
            scc = int(t > M)
        elif mnem in ("s_sub_u32", "s_subb_u32"):
            t = val(o[1]) - val(o[2]) - (scc if "subb" in mnem else 0)
            put(o[0], t)
            scc = int(t < 0)
        elif mnem == "s_cmp_eq_u32":
            scc = int(val(o[0]) == val(o[1]))
        elif mnem.startswith("s_cselect"):
            put(o[0], val(o[1]) if scc else val(o[2]))
        elif mnem in ("s_cbranch_scc0", "s_cbranch_scc1"):
            i = labels[rest] if scc == int(mnem[-1]) else i
        elif mnem == "s_branch":
            i = labels[rest]
        elif mnem == "v_mov_b32" and o[0] in ("v164", "v165", "v166", "v167"):
            off[int(o[0][1:])] = off[int(o[1][1:])]
        elif mnem.startswith("global_load_lds"):
            at, v = reg["m0"] - LDSK, int(o[0][1:])
            which = "V" if at >= nsh * 8192 else "K"
            assert (which == "V") == (v >= 166)
            ev.append((which, at % (nsh * 8192) // 8192, at % 8192 // 1024, val(o[1]), off[v]))
        elif mnem == "ds_read_b128":
            ev.append(("read", "K", int(re.search(r"offset:(\d+)", l)[1]) // 8192))
        elif mnem == "ds_read_b64_tr_b16":
            ev.append(("read", "V", int(re.search(r"offset:(\d+)", l)[1]) // 8192))
        elif mnem == "s_waitcnt":
            if "vmcnt" in l:
                ev.append(("wait", int(re.search(r"vmcnt\((\d+)\)", l)[1])))
            if "lgkmcnt" in l:
                ev.append(("returned", int(re.search(r"lgkmcnt\((\d+)\)", l)[1])))
        elif mnem == "s_barrier":
            ev.append(("barrier",))
    raise AssertionError("the loop does not end")


def test_ring_protocol_on_concrete_streams(gen):
    full, idle, N = gen.generate_half(), gen.generate_half_idle(), gen.NSH
    for nb in range(1, 36):
        for nc in sorted({0, 1, nb // 2, nb - 1, nb}):
            ev = _run(full, nc, nb - nc, N)
            skeleton = [e for e in ev if e[0] not in ("read", "returned", "iteration")]
            assert skeleton == [e for e in _run(idle, nc, nb - nc, N) if e[0] != "iteration"]
            assert sum(e[0] == "iteration" for e in ev) == nb
            # every block in order, each half from this wave's row offsets; beyond the end the last block again
            for which, c, s in (("K", KC, KS), ("V", VC, VS)):
                loads = [e for e in ev if e[0] == which]
                assert len(loads) == 2 * (nb + (N if which == "K" else N - 1))
                for i, (_, stage, half, addr, off) in enumerate(loads):
                    b = min(i // 2, nb - 1)
                    want = (c + b * CSTEP, f"c{i % 2}") if b < nc else (s + (b - nc) * SSTEP, f"s{i % 2}")
                    assert (stage, half) == (i // 2 % N, i % 2) and (addr, off) == want, (nb, nc, which, i)
            # every fragment read finds its block: requested, waited for before the last barrier, and not overwritten
            # by a request made in the same or an earlier interval between barriers
            order, held, landed, j, nk, nv = [], {}, 0, -1, 0, 0
            visible = 0             # loads landed at the last barrier
            reads, done = [], 0     # stages read since the last barrier, or read and not yet waited for when it was passed
            for e in ev:
                if e[0] in ("K", "V"):
                    order.append(e[0])
                    blk = sum(x == e[0] for x in order[:-1]) // 2
                    assert e[:2] not in reads, (nb, nc, e)
                    held[e[0], e[1]] = (blk, len(order))
                elif e[0] == "wait":
                    landed = max(landed, len(order) - e[1])
                elif e[0] == "returned":
                    done = max(done, len(reads) - e[1])
                elif e[0] == "barrier":
                    visible, reads, done = landed, reads[done:], 0
                elif e[0] == "iteration":
                    j += 1
                elif e[0] == "read":
                    blk = {"V": j, "K": 0 if j < 0 and e[2] == 0 else 1 if j < 0 else j + 2}[e[1]]
                    if blk < nb:    # (fragments beyond the last block are read and not used)
                        have, last = held[e[1], e[2]]
                        assert have == blk and last <= visible, (nb, nc, j, e, have, last, visible)
                    reads.append((e[1], e[2]))


def test_either_loop_is_the_loop_twice(gen):
    """lsp_attn_half_either_loop.inc: committed as generated; either way through it is the loop checked above, the second with
    two additions of unrounded probabilities in the place of each dot product of a rounded pair."""
    half, either = gen.generate_half(), gen.generate_half(True)
    with open(os.path.join(CSRC, "lsp_attn_half_either_loop.inc")) as f:
        assert re.findall(r'^    "(.*)\\n"$', f.read(), flags=re.M) == either

    def parts(lines):       # prologue, loops by label, exit, out-of-line blocks by label
        begin = next(k for k, l in enumerate(lines) if l.startswith(".Lloop"))
        leave, cold = lines.index(".Lexit_%=:"), lines.index("s_branch .Lend_%=") + 1
        loops, outer = {}, {}
        for into, part in ((loops, lines[begin:leave]), (outer, lines[cold:-1])):
            for l in part:
                if l.startswith((".Lloop", ".Lresc", ".Lev")) and l.endswith(":"):
                    into[l] = []
                elif not into:
                    raise AssertionError(l)
                list(into.values())[-1].append(l)
        return lines[:begin], loops, lines[leave:cold], outer

    (pro, loops, leave, outer), (pro2, loops2, leave2, outer2) = parts(half), parts(either)
    assert pro2[-2:] == ["s_cmp_lg_u32 %[wide], 0", "s_cbranch_scc1 .Lloopw_%="] and pro2[:-2] == pro and leave == leave2
    assert list(loops2) == [".Lloop_%=:", ".Lloopw_%=:"] and loops2[".Lloop_%=:"] == loops[".Lloop_%=:"]

    def narrow(l):
        return re.sub(r"\.L(loop|resc_|after_|isk_i|isv_i|evk_i|evv_i)w", r".L\1", l)

    first = {f"v_cvt_pk_bf16_f32 v{p}, v{gen.T[2 * i]}, v{gen.T[2 * i + 1]}": i for i, p in enumerate(gen.PF)}
    want, i = [], None
    for l in loops[".Lloop_%=:"]:
        if l.startswith("v_dot2c_f32_bf16"):
            want += [f"v_add_f32 v{gen.LSUM}, v{gen.LSUM}, v{gen.T[e]}" for e in (2 * i, 2 * i + 1)]
            continue
        i = first.get(l, i)
        want.append(l)
    assert [narrow(l) for l in loops2[".Lloopw_%=:"]] == want and sum("v_dot2c" in l for l in half) == 8 * gen.UNROLL_H
    assert {k: v for k, v in outer2.items() if narrow(k) == k} == outer
    assert {narrow(k): [narrow(l) for l in v] for k, v in outer2.items() if narrow(k) != k} == {k: v for k, v in outer.items() if "_p" not in k}
