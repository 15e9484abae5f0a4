"""The kernel names that the bench line prints are kernels of the built library."""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

import bench
from paper_2609_00224_amd.build import LIB


@pytest.mark.parametrize("B", range(1, 17))
def test_names_are_in_the_library(B):
    if not os.path.exists(LIB) or shutil.which("nm") is None:
        pytest.skip("no built library or no nm")
    out = subprocess.run(["nm", "-C", "--defined-only", LIB], check=True, capture_output=True, text=True).stdout
    have = set(re.findall(r"\w+_kernel<[^>]*>", out))
    names = [bench.kernel_name(B, grouped, rp, e4m3=e4m3)
             for grouped in (False, True) for rp in (512, 1024) for e4m3 in (False, True)]
    names += [bench.kernel_name(B, grouped, g128=True) for grouped in ((False, True) if B == 1 else (False,))]
    for name in names:
        for one in name.split(" / "):
            assert one in have, one
