"""One matrix on its own on both sides of the lines between its kernels: bit for
bit against the fp64 oracle on sampled rows of dyadic inputs."""
from __future__ import annotations

import numpy as np
import pytest

from tests.gpu_cases import dyadic_case, e4m3_dyadic_case, gpu_gemm, gpu_pack, gpu_pack_e4m3, oracle_rows

pytestmark = pytest.mark.gpu


def _check(c, pm, B):
    N = c["N"]
    rows = np.unique(np.concatenate([np.arange(0, N, 1013), np.arange(N - 130, N), np.arange(500, 530)]))
    ref, _ = oracle_rows(c, rows=rows, need_wmax=False)
    y = gpu_gemm(pm, c["x"][:B])
    assert np.array_equal(y[:, rows].astype(np.float64), ref[:B]), (N, c["K"], B)


@pytest.mark.parametrize("fmt", ["fp16", "e4m3"])
@pytest.mark.parametrize("N", [52224, 52228])
def test_batch_5_to_8_either_side_of_two_units(N, fmt):
    # five slices; 256 workgroups take two units each at 102 panels, three at 103
    print(f"[case] {N}x1600 {fmt}, batch 5 and 8", flush=True)
    c = (dyadic_case if fmt == "fp16" else e4m3_dyadic_case)(81, N, 1600, 8, 70)
    pm = gpu_pack(c) if fmt == "fp16" else gpu_pack_e4m3(c)
    for B in (5, 8):
        _check(c, pm, B)
