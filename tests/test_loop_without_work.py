"""A decode loop whose sequences are all complete calls nothing of the library: lengths of any type and place."""
import pytest
import torch

from paper_2603_05454_amd.loop import decode_loop


@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
@pytest.mark.parametrize("strided", [False, True])
def test_nothing_left(dtype, strided):
    lens = torch.tensor([[5, 0], [9, 0], [2, 0]], dtype=dtype)
    prefix, suffix = (lens[:, 0], lens[:, 1]) if strided else lens.t().contiguous()
    res = decode_loop(None, None, 100, 0.9, 16, 1, 1, prefix, suffix, torch.zeros((3, 12), dtype=torch.int32), gen_len=4)
    assert (res["steps"], res["flips"], res["flip_denominator"], res["committed"]) == (0, 0, 0, 0)
