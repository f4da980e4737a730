#!/usr/bin/env python3
"""Generator of lsp_lm_head_loop_{256,128,64}.inc: the hand-scheduled K loops of the
output-head kernel (lsp_lm_head.hip), one inline-asm statement per tile height.

A workgroup of eight waves (two per SIMD) computes a TV (vocabulary) x TR (rows)
tile with v_mfma_f32_16x16x32_bf16.  Both operand tiles of a K step of KB = 64
elements sit in one of NSTG stages of LDS, rows of 128 bytes whose 16-byte chunk c
is kept at position c ^ ((row >> 1) & 7); the loads that fill them go from global
memory to LDS directly, one wave-wide load = 1 KB = 8 rows.

Why generated assembly: with compiler scheduling every K step ended in a wait for
ALL loads in flight and the fragments of a step were read in a burst.  Here
  * the fragments of k-slice kk+1 are read between the matrix instructions of slice
    kk (two register sets), also across the step boundary;
  * the workgroup meets ONCE per step, in the middle of the step's second-last
    slice, when its last fragment reads have returned: from there on the stage of
    this step is free and is refilled with step + NSTG, one load per matrix
    instruction, while the matrix pipe works on what is in registers;
  * loads never drain: when a tile's last steps have been requested the stream goes
    on with the first steps of the workgroup's next tile (per-lane pointers are
    swapped out of line), so the tile's epilogue runs under them.

The statement takes the stage that step 0 sits in (`phase`) and enters the unrolled
loop there.  Loads in flight at entry: steps 0 .. NSTG-1 of this tile, in order.

Every tile is summed from k = 0 upwards, whatever its height, place and workgroup: a logit
has the same bits wherever its row stands in the batch and however many rows are
active, and equal weight rows give equal logits.  (Starting K at a different step in
different workgroups spreads a power-of-two row pitch over the memory channels, but
gives that up; the kernel gives its XCDs runs of tiles and its workgroups different start TIMES.)
"""
import os

NW = 8


class Mode:
    """TV x TR unit, K steps of KB elements in NSTG stages, WV x WR waves; `bar`: matrix instruction of the
    step's second-last slice before which the workgroup meets."""

    def __init__(self, TV, TR, KB, WV, WR, NSTG, bar):
        self.TV, self.TR, self.KB, self.WV, self.WR, self.NSTG, self.bar = TV, TR, KB, WV, WR, NSTG, bar
        self.ROWB, self.NK = KB * 2, KB // 32
        self.MV, self.MR = TV // WV // 16, TR // WR // 16
        self.TILE_W, self.TILE_H = TV * self.ROWB, TR * self.ROWB
        self.STAGE = self.TILE_W + self.TILE_H
        self.LW, self.LH = self.TILE_W // 1024 // NW, self.TILE_H // 1024 // NW
        # registers
        self.setr = 4 * (self.MV + self.MR)
        r = 2 * self.setr           # two fragment sets
        self.wptr = r; r += 2 * self.LW
        self.hptr = r; r += 2 * self.LH
        self.addr = r; r += 2 * self.NK * NSTG
        self.nacc = self.MV * self.MR * 4
        self.acc = 256 - self.nacc
        self.next = r; r += 1 if TR == 256 else 2 * self.LH     # LDS address of the next pointers, or the pointers
        self.top = r
        assert r <= self.acc

    def a(self, s, i):
        return s * self.setr + 4 * i

    def b(self, s, j):
        return s * self.setr + 4 * self.MV + 4 * j

    def c(self, i, j):
        return self.acc + 4 * (j * self.MV + i)

    def addr_a(self, stage, kk):
        return self.addr + (stage * self.NK + kk) * 2

    def addr_b(self, stage, kk):
        return self.addr_a(stage, kk) + 1


MODES = {256: Mode(256, 256, 64, 2, 4, 2, 18), 128: Mode(256, 128, 64, 4, 2, 3, 11), 64: Mode(256, 64, 64, 4, 2, 3, 6)}

HINT = "<weight hint>"     # in the emitted text: a string macro of the including code

SG = dict(m0save=64, inc=66, li=68, js=69, ev=70)


def v(r, n=1):
    return f"v{r}" if n == 1 else f"v[{r}:{r + n - 1}]"


def generate(M):
    out = []
    e = out.append
    inc = f"s[{SG['inc']}:{SG['inc'] + 1}]"
    li, js, ev = f"s{SG['li']}", f"s{SG['js']}", f"s{SG['ev']}"
    L = M.LW + M.LH
    NS, NK = M.NSTG, M.NK
    tags = []

    def reads(st, kk, s):
        r = [f"ds_read_b128 {v(M.b(s, j), 4)}, {v(M.addr_b(st, kk))} offset:{16 * M.ROWB * j}" for j in range(M.MR)]
        return r + [f"ds_read_b128 {v(M.a(s, i), 4)}, {v(M.addr_a(st, kk))} offset:{16 * M.ROWB * i}" for i in range(M.MV)]

    def loads(tag, st):
        """Requests of one step into stage st; the first entry is the check for the end of K."""
        r = [(f"s_cmp_eq_u32 {li}, {ev}", f"s_cbranch_scc1 .Lcold_{tag}_%=", f".Lback_{tag}_%=:", f"s_add_u32 {li}, {li}, 1")]
        tags.append(tag)
        for k in range(L):
            w = k < M.LW
            i = k if w else k - M.LW
            p = (M.wptr if w else M.hptr) + 2 * i
            dst = st * M.STAGE + (0 if w else M.TILE_W) + 1024 * NW * i
            r.append((f"s_add_u32 m0, %[ldsw], {dst}", f"global_load_lds_dwordx4 {v(p, 2)}, off{HINT if w else ''}",
                      f"v_lshl_add_u64 {v(p, 2)}, {v(p, 2)}, 0, {inc}"))
        return r

    def step(u):
        """Step held in stage u."""
        st = u
        pending = []
        for kk in range(NK):
            s = kk & 1
            order = [(i, j) for j in range(M.MR) for i in range(M.MV)]
            rd = reads(st, kk + 1, s ^ 1) if kk + 1 < NK else reads((st + 1) % NS, 0, 0)
            n = len(order)
            if kk < NK - 1:
                e("s_waitcnt lgkmcnt(0)")       # this slice's fragments, requested during the previous one
            for q, (i, j) in enumerate(order):
                if kk == NK - 2 and q == M.bar:
                    # this wave holds its last fragments of this stage, and the next step has landed as far as it was its to load
                    for x in rd:
                        e(x)
                    rd = []
                    e(f"s_waitcnt vmcnt({(NS - 2) * L}) lgkmcnt(0)")
                    e("s_barrier")
                    pending = loads(f"{u}", st)
                ld = pending.pop(0) if pending else None
                if ld and len(ld) == 4:
                    for x in ld:
                        e(x)
                    ld = pending.pop(0)
                if ld:
                    e(ld[0])
                e(f"v_mfma_f32_16x16x32_bf16 {v(M.c(i, j), 4)}, {v(M.a(s, i), 4)}, {v(M.b(s, j), 4)}, {v(M.c(i, j), 4)}")
                if ld:
                    e(ld[1])
                    e(ld[2])
                k = 1 if len(rd) <= n - q or not rd else 2
                for _ in range(k):
                    if rd:
                        e(rd.pop(0))
            assert not rd
            # (slice kk+1 starts when its reads have returned; for the last slice the barrier has seen to it)
        for ld in pending:
            for x in ld:
                e(x)
        e(f"s_add_u32 {js}, {js}, 1")
        e(f"s_cmp_lt_u32 {js}, %[ks]")
        e("s_cbranch_scc0 .Lexit_%=")

    e(f"s_mov_b32 s{SG['m0save']}, m0")
    e(f"s_movk_i32 s{SG['inc']}, {M.ROWB}")
    e(f"s_mov_b32 s{SG['inc'] + 1}, 0")
    e(f"s_movk_i32 {li}, {NS}")
    e(f"s_mov_b32 {js}, 0")
    e(f"s_mov_b32 {ev}, %[event]")
    e(f"s_waitcnt vmcnt({(NS - 1) * L}) lgkmcnt(0)")
    e("s_barrier")
    for u in range(1, NS):
        e(f"s_cmp_eq_u32 %[phase], {u}")
        e(f"s_cbranch_scc1 .Lenter_{u}_%=")
    for u in range(NS):
        e(f".Lenter_{u}_%=:")
        for x in reads(u, 0, 0):
            e(x)
        e(f"s_branch .Lstep_{u}_%=")
    e(".Lloop_%=:")
    for u in range(NS):
        e(f".Lstep_{u}_%=:")
        step(u)
    e("s_branch .Lloop_%=")
    for u in tags:
        e(f".Lcold_{u}_%=:")
        e(f"s_cmp_eq_u32 {li}, %[ks]")
        e(f"s_cbranch_scc1 .Lswap_{u}_%=")
        # the end of K: the ragged step (lanes whose chunk lies beyond K fetch zeros), then steps wholly beyond it
        e(f"s_cmp_eq_u32 {li}, %[event]")
        e("s_cselect_b64 exec, %[zmask], -1")
        e(f"s_add_u32 {ev}, {li}, 1")
        e(f".Lzero_{u}_%=:")
        for p in range(M.wptr, M.hptr + 2 * M.LH, 2):
            e(f"v_mov_b32 v{p}, %[zlo]")
            e(f"v_mov_b32 v{p + 1}, %[zhi]")
        e("s_mov_b64 exec, -1")
        e(f"s_branch .Lback_{u}_%=")
        e(f".Lswap_{u}_%=:")
        e(f"s_mov_b32 {ev}, -1")
        e("s_cmp_eq_u32 %[more], 0")                 # nothing to go on with: every lane fetches zeros into stages nobody reads
        e(f"s_cbranch_scc1 .Lzero_{u}_%=")
        for i in range(M.LW):
            p = M.wptr + 2 * i
            e(f"v_lshl_add_u64 {v(p, 2)}, {v(p, 2)}, 0, %[wstep]")
        if M.TR == 256:
            for i in range(0, M.LH, 2):
                e(f"ds_read_b128 {v(M.hptr + 2 * i, 4)}, {v(M.next)} offset:{8192 * (i // 2)}")
            e("s_waitcnt lgkmcnt(0)")
        else:
            for k in range(2 * M.LH):
                e(f"v_mov_b32 v{M.hptr + k}, v{M.next + k}")
        e(f"s_branch .Lback_{u}_%=")
    e(".Lexit_%=:")
    e("s_waitcnt lgkmcnt(0)")
    e(f"s_mov_b32 m0, s{SG['m0save']}")
    e("s_nop 15")
    e("s_nop 15")
    return out


def text(M):
    lines = generate(M)
    body = "\n".join(f'    "{x}\\n"' for x in lines).replace(HINT, '" LSP_WEIGHT_HINT "')
    nv = M.nacc // 16
    acc = ", ".join(f'"+{{{v(M.acc + 16 * k, 16)}}}"(acc[{k}])' for k in range(nv))
    clob = [f"v{r}" for r in range(2 * M.setr)] + [f"s{r}" for r in range(64, 71)] + ["scc", "memory"]
    t = f"""// GENERATED by gen_lm_head.py - do not edit; the pipeline and the register map are described there.
// Expects in scope: f32x16 acc[{nv}]; u32x{2 * M.LW} wptr; u32x{2 * M.LH} hptr; u32x{2 * M.NK} addr[{M.NSTG}]; next;
// uint32_t ldsw, ks, event, phase, go_on, zlo, zhi; uint64_t zmask, wstep;
// LSP_WEIGHT_HINT: cache hint of the weight loads ("" or " nt").
asm volatile(
{body}
    : {acc},
      "+{{{v(M.wptr, 2 * M.LW)}}}"(wptr), "+{{{v(M.hptr, 2 * M.LH)}}}"(hptr)
    : {", ".join(f'"{{{v(M.addr + 2 * M.NK * k, 2 * M.NK)}}}"(addr[{k}])' for k in range(M.NSTG))}, "{{{v(M.next, 1 if M.TR == 256 else 2 * M.LH)}}}"(next),
      [ldsw] "s"(ldsw), [ks] "s"(ks), [event] "s"(event), [phase] "s"(phase), [zlo] "s"(zlo), [zhi] "s"(zhi),
      [more] "s"(go_on), [zmask] "s"(zmask), [wstep] "s"(wstep)
    : {", ".join(f'"{c}"' for c in clob)});
"""
    return t


def main():
    here = os.path.dirname(os.path.abspath(__file__))
    for tr, M in MODES.items():
        with open(os.path.join(here, f"lsp_lm_head_loop_{tr}.inc"), "w") as f:
            f.write(text(M))


if __name__ == "__main__":
    main()
