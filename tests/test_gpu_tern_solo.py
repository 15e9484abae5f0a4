"""The task kernel (one matrix at batch 1) at the edges of its dispatch and
tiles: one and several parts, residual tasks of 32 to 96 columns, whole and cut
64-row tiles, more tiles than workgroups; bit for bit against the fp64 oracle
on dyadic inputs, twice on one workspace whose counters end at zero."""
from __future__ import annotations

import numpy as np
import pytest

from tests.gpu_cases import dyadic_case, gpu_gemm, gpu_pack, oracle_rows

pytestmark = pytest.mark.gpu

# (N, K, salient): 16 slices and none, one column more (two parts), 13 slices
# with 3, 4 and 9 tasks of 32 salient columns (96 a task keeps one part), all
# columns salient, rows around a tile and its pieces, 64 / 65 / 128 / 129 / 257 tiles
# (four of them are the table kernel's by now: 5121 and 14336 columns, 288 and 289
# salient columns of 4096); several parts with tasks of 32, 64 and 96 salient
# columns and one part with 96, which are the task kernel's
SHAPES = [(64, 5120, 0), (68, 5121, 0), (132, 4096, 96), (60, 4096, 97), (256, 4096, 288), (4, 4096, 289), (8, 1, 1),
          (192, 700, 700), (4096, 1601, 33), (4100, 4800, 31), (8192, 640, 5), (8196, 640, 64), (16388, 321, 20),
          (320, 14336, 700), (4096, 2999, 600), (516, 1603, 1603), (68, 3200, 3200), (1028, 6000, 2500), (28672, 4096, 205)]


@pytest.mark.parametrize("N,K,nS", SHAPES)
def test_solo_dyadic_exact(N, K, nS):
    import torch

    import paper_2609_00224_amd as q

    print(f"[case] batch 1 by tasks, {N}x{K}, {nS} salient", flush=True)
    c = dyadic_case(8000 + N + K + nS, N, K, 1, nS)
    pm = gpu_pack(c)
    ws = q.new_workspace(pm.desc, 1)
    ref, _ = oracle_rows(c, need_wmax=False)
    for _ in range(2):
        assert np.array_equal(gpu_gemm(pm, c["x"], ws=ws).astype(np.float64), ref)
    torch.cuda.synchronize()
    assert int(ws[:65536].view(torch.int32).abs().sum().item()) == 0


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_activation_not_finite(bad):
    """Every output is NaN (the digits of its block have the NaN scale)."""
    c = dyadic_case(73, 256, 700, 1, 9)
    c["x"][0, 350] = bad
    assert np.all(np.isnan(gpu_gemm(gpu_pack(c), c["x"])))
