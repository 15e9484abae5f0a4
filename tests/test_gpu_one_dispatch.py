"""One matrix on its own on both sides of the lines between its kernels: bit for
bit against the fp64 oracle on sampled rows of dyadic inputs."""
from __future__ import annotations

import numpy as np
import pytest
import torch

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


# by tasks: four parts of whole tiles (in fp16), of half and of quarter ones (residual tasks
# only in the last ones), two of whole tiles, two of quarter tiles, six, as many tiles
# as workgroups; by tables: three parts, more tiles than workgroups of one and two
# slices, five tasks more than one part holds, a long matrix of few rows, residual
# tasks of 96 columns in a small one
BATCH1 = [(4100, 14340, 1500), (2048, 4096, 4096), (1024, 4096, 4096), (9000, 9000, 0), (132, 1600, 1600), (4, 28672, 0),
          (16384, 320, 9), (4100, 14340, 287), (16388, 320, 9), (49156, 640, 19), (5124, 5120, 154), (68, 8200, 300),
          (260, 4096, 205)]


@pytest.mark.parametrize("fmt", ["fp16", "e4m3"])
@pytest.mark.parametrize("N,K,nS", BATCH1)
def test_batch_1_either_side_of_the_task_kernel(N, K, nS, fmt):
    import paper_2609_00224_amd as q

    print(f"[case] {N}x{K} {fmt}, {nS} salient, batch 1", flush=True)
    c = (dyadic_case if fmt == "fp16" else e4m3_dyadic_case)(83, N, K, 1, nS)
    pm = gpu_pack(c) if fmt == "fp16" else gpu_pack_e4m3(c)
    ws = q.new_workspace(pm.desc, 1)
    rows = np.unique(np.concatenate([np.arange(0, N, 61), np.arange(max(0, N - 130), N), np.arange(0, min(N, 70))]))
    ref, _ = oracle_rows(c, rows=rows, need_wmax=False)
    for _ in range(2):
        assert np.array_equal(gpu_gemm(pm, c["x"], ws=ws)[:, rows].astype(np.float64), ref)
    assert int(ws[:65536].view(torch.int32).abs().sum().item()) == 0
