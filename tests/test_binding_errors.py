"""The native marshalling module (csrc/binding.cpp) keeps torch's C++ exceptions to itself: the call is left to the
general path, which raises in Python, where an exception through the C entry would end the process."""
import pytest
import torch

import paper_2603_05454_amd as lsp


@pytest.mark.skipif(torch.cuda.is_available(), reason="the exception is the one a missing device gives")
def test_an_exception_from_torch_is_raised_in_python():
    from torch._subclasses.fake_tensor import FakeTensorMode
    lsp.lib()
    with FakeTensorMode():
        z = torch.empty(2, 4, 64, device="cuda")
        out = (torch.empty(2, 4, dtype=torch.int32, device="cuda"), torch.empty(2, 4, device="cuda"), torch.empty(2, 4, device="cuda"))
        assert lsp._nat.confidence(z, None, out, None) is None
        with pytest.raises((RuntimeError, lsp.LspError)):
            lsp.confidence(z, None, out=out)


@pytest.mark.gpu
def test_a_sparse_tensor_is_refused_in_python():
    lsp.lib()
    z = torch.zeros(2, 4, 64, device="cuda").to_sparse()
    with pytest.raises((RuntimeError, lsp.LspError)):
        lsp.confidence(z, None)
