"""Output head: heights of row tiles by rounds (lsp_lm_head.hip, cut_rows), every height with several tiles per workgroup."""
import pytest
import torch

from test_gpu_lm_head import _compare, _run, lsp  # noqa: F401

pytestmark = pytest.mark.gpu


def _plan(rows, vt):
    """Rows per tile, row tiles, tiles of the busiest workgroup, for more than 128 active rows."""
    tiles = lambda h: -(-vt // 8) * -(-rows // h)
    rounds = {h: -(-tiles(h) // 32) for h in (256, 128, 64)}
    h = min((256, 128, 64), key=lambda h: {256: 17, 128: 10, 64: 7}[h] * rounds[h])     # (of equals the first)
    return h, -(-rows // h), rounds[h]


@pytest.mark.parametrize("rows,vt,plan", [(250, 494, (256, 1, 2)), (700, 157, (256, 3, 2)), (300, 103, (256, 2, 1)), (208, 594, (128, 2, 5)),
                                          (580, 103, (128, 5, 3)), (140, 157, (64, 3, 2)), (129, 261, (64, 3, 4))])
@pytest.mark.parametrize("K", [64, 136, 320])
def test_heights_by_rounds(lsp, oracle, rows, vt, plan, K):  # noqa: F811
    """Small integers: bit-exact on rows from all over the list; the last vocabulary tile is ragged, K has one step, a ragged end, or
    more steps than are in flight."""
    assert _plan(rows, vt) == plan
    g = torch.Generator(device="cuda").manual_seed(rows + K)
    h = torch.randint(-3, 4, (1, rows, K), generator=g, device="cuda").to(torch.bfloat16)
    w = torch.randint(-3, 4, (vt * 256 - 3, K), generator=g, device="cuda").to(torch.bfloat16)
    got = _run(lsp, h, w)
    pick = torch.unique(torch.linspace(0, rows - 1, 24).round().long())
    _compare(tuple(x[:, pick] for x in got), oracle.lm_head_confidence(h[:, pick].cpu(), w.cpu()), None, exact=True)
