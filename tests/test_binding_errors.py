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


def test_a_wrong_number_of_arguments_is_an_error():
    lsp.lib()
    for name in ("bind", "attn_step", "attn_step_layers", "confidence", "lm_head_confidence", "commit", "flip_update"):
        with pytest.raises(TypeError, match=name):
            getattr(lsp._nat, name)(1, 2)


def test_the_library_loads_without_the_module(monkeypatch):
    """liblsp.so alone is enough: the general path makes every call."""
    import sys
    monkeypatch.setattr(lsp, "_lib", None)
    monkeypatch.setattr(lsp, "_nat", None)
    monkeypatch.delattr(lsp, "_binding", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2603_05454_amd._binding", None)
    with pytest.warns(RuntimeWarning, match="native binding module"):
        assert "gfx950" in lsp.version()
    assert lsp._nat is None
    with pytest.raises(lsp.LspError, match="device tensors only"):
        lsp.confidence(torch.zeros(1, 2, 8))


class _Raises(torch.Tensor):
    """A device tensor of a subclass whose own Python code raises when its layout is asked for."""

    @staticmethod
    def __new__(cls, *shape, dtype=torch.float32):
        return torch.Tensor._make_wrapper_subclass(cls, shape, dtype=dtype, device="cuda", dispatch_sizes_strides_policy="strides")

    @classmethod
    def __torch_dispatch__(cls, func, types, args=(), kwargs=None):
        raise KeyError("asked for its layout")


def test_an_exception_from_python_code_under_torch_is_the_one_raised():
    lsp.lib()
    z = _Raises(2, 4, 64)
    out = (torch.empty(2, 4, dtype=torch.int32), torch.empty(2, 4), torch.empty(2, 4))
    assert lsp._nat.confidence(z, None, out, None) is None
    with pytest.raises(KeyError, match="asked for its layout"):
        lsp.confidence(z, None, out=out)


@pytest.mark.gpu
def test_numbers_and_outputs_of_rarer_forms_go_to_the_general_path():
    """A scale that float() makes a number of is taken, an output dict with a stray host tensor refused, as without the module."""
    lsp.lib()
    q = torch.randn(1, 20, 2, 64, device="cuda")
    pl, sl = (torch.tensor([x], dtype=torch.int32, device="cuda") for x in (9, 20))
    a, b = (lsp.attn_step(q, q, q, q, q, pl, sl, scale=s, out=torch.zeros_like(q)) for s in (0.5, "0.5"))
    assert torch.equal(a, b)
    table = lsp.AttnLayerTable([q], [q], [q], [q], [q], [torch.zeros_like(q)])
    assert torch.equal(lsp.attn_step_layers(table, pl, sl, scale="0.5")[0], a)
    out = {k: torch.zeros(1, dtype=torch.int32, device="cuda") for k in ("raw_boundary", "snapped_boundary", "commit_len", "status_flags")}
    out.update(stable_mask=torch.zeros((1, 20), dtype=torch.uint8, device="cuda"), tau_used=torch.zeros(1, device="cuda"), notes=torch.zeros(1))
    m, ids = torch.ones((1, 20), device="cuda"), torch.zeros((1, 20), dtype=torch.int32, device="cuda")
    with pytest.raises(lsp.LspError, match="device tensors only"):
        lsp.commit(m, ids, torch.zeros(2, dtype=torch.int32, device="cuda"), 64, 0.5, 4, 1, 1, pl, sl, C=64, out=out)


@pytest.mark.gpu
def test_a_sparse_tensor_is_refused_in_python():
    lsp.lib()
    z = torch.zeros(2, 4, 64, device="cuda").to_sparse()
    with pytest.raises((RuntimeError, lsp.LspError)):
        lsp.confidence(z, None)


WORKSPACE = r"""
#include <stdio.h>
#include <string.h>
#include <stdexcept>
#include "binding_workspace.h"
struct Failing : c10::Allocator {
  int how = 0;
  c10::DataPtr allocate(size_t n) override {
    if (how == 1) TORCH_CHECK_WITH(OutOfMemoryError, false, "none left");
    if (how == 2) TORCH_CHECK(false, "device error");
    if (how == 3) throw std::runtime_error("other");
    static char memory[64];
    return {memory, c10::Device(c10::DeviceType::CUDA, 0)};
  }
  void copy_data(void *to, const void *from, size_t n) const override { memcpy(to, from, n); }
};
int main() {
  static Failing f;
  c10::SetAllocator(c10::DeviceType::CUDA, &f, 127);
  for (f.how = 0; f.how < 4; ++f.how) {
    try {
      const Workspace w(48, nullptr);
      printf("%d %d\n", w.at != nullptr, int(w.bytes));
    } catch (...) {
      printf("raised\n");
    }
  }
}
"""


def test_only_a_lack_of_memory_does_without_a_workspace(tmp_path):
    """Any other failure of the allocator reaches the caller of the attention."""
    import os
    import subprocess
    from paper_2603_05454_amd import build
    (tmp_path / "w.cpp").write_text(WORKSPACE)
    cmd = build.binding_command()
    cmd = [x for x in cmd[:cmd.index("-o")] if x not in ("-shared", os.path.join(build.CSRC, "binding.cpp"))]
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    subprocess.run(cmd + ["-I", build.CSRC, str(tmp_path / "w.cpp"), "-o", str(tmp_path / "w"), "-L", libs, "-lc10", "-ltorch_cpu", f"-Wl,-rpath,{libs}"], check=True)
    out = subprocess.run([str(tmp_path / "w")], capture_output=True, text=True, check=True).stdout
    assert out.split("\n") == ["1 48", "0 0", "raised", "raised", ""]
