"""Host-side check of what the small kernels of a step are launched with: compiled for gfx950 here, read from the compiler's
own metadata.  A kernel that asks the hardware for the size of its workgroup takes 256 bytes of implicit arguments, which
the host writes and the kernel fetches at every launch."""
import os
import re
import subprocess

import pytest

from paper_2603_05454_amd.build import CSRC, FLAGS


def _kernels(source, tmp_path):
    out = tmp_path / "device.s"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *FLAGS, "--cuda-device-only", "-S", os.path.join(CSRC, source), "-o", str(out)],
                   check=True, stderr=subprocess.DEVNULL)
    meta = out.read_text().split("amdhsa.kernels:")[1].split("amdhsa.target:")[0]
    found = {}
    for k in re.split(r"\n  - ", meta)[1:]:
        found[re.search(r"\.name:\s+(\S+)", k)[1]] = (int(re.search(r"\.kernarg_segment_size:\s+(\d+)", k)[1]), "hidden_" in k)
    return found


@pytest.mark.parametrize("source,kernels", [("lsp_commit.hip", {"boundary_kernelIJE": 144, "boundary_kernelIJNS_8FlipArgs": 192}),
                                            ("lsp_common.hip", {"flip_kernel": 80, "poll_kernel": 32})])
def test_no_implicit_arguments(source, kernels, tmp_path):
    """A plain commit carries nothing of the flip count that lsp_commit_step adds to it."""
    found = _kernels(source, tmp_path)
    for part, most in kernels.items():
        (size, hidden), = [v for n, v in found.items() if part in n]
        assert size <= most and not hidden, (part, size, hidden)
