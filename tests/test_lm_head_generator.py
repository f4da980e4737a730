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
