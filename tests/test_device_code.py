"""What the compiler reports about the kernels, here without a GPU."""
from __future__ import annotations

import os
import re
import subprocess

import pytest

from paper_1310_4645_amd import build


@pytest.mark.parametrize("source", ["prs_uni_list.hip", "prs_uni_sched.hip", "prs_uni_times.hip"])
def test_kernels_that_address_lds_from_zero_have_none_of_their_own(source):
    """These kernels reach the LDS that the launch asks for by its address, which is 0 only if the compiler puts nothing there itself:
    a private array indexed by a variable is moved to LDS, below what the launch asks for."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    out = subprocess.run([hipcc, *build.FLAGS, "-Rpass-analysis=kernel-resource-usage", "--cuda-device-only", "-c", os.path.join(build.CSRC, source),
                          "-o", os.devnull], capture_output=True, text=True, check=True).stderr
    sizes = re.findall(r"LDS Size \[bytes/block\]: (\d+)", out)
    assert sizes and set(sizes) == {"0"}, sizes
