"""One zero-filled workspace serves any sequence of matrices: a matrix of more
than 64, or of more than 16384, panels of 512 rows keeps its arrival counters
where a smaller matrix's partial rows do not come (its panels past those were
left unsummed when they did)."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from tests.gpu_cases import (dyadic_case, g128_dyadic_case, gpu_gemm, gpu_pack, gpu_pack_g128, oracle_rows,
                             oracle_rows_g128, to_dev)

pytestmark = pytest.mark.gpu


def test_small_matrix_before_one_of_65_panels():
    import torch

    import paper_2609_00224_amd as q

    # seven slices of 65 panels: 455 units over as many workgroups, every panel split
    big = g128_dyadic_case(61, 65 * 512, 1700, 1, 3)
    small = dyadic_case(62, 512, 14336, 2, 40)
    pb, ps = gpu_pack_g128(big), gpu_pack(small)
    need = max(q.qtea_workspace_bytes(pb.desc, 1), q.qtea_workspace_bytes(ps.desc, 2))
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    print("[case] 512x14336 batch 2, then 33280x1700 in the grouped format, one workspace", flush=True)
    for _ in range(2):
        assert np.array_equal(gpu_gemm(ps, small["x"], ws=ws).astype(np.float64), oracle_rows(small, need_wmax=False)[0])
        y = gpu_gemm(pb, big["x"], ws=ws).astype(np.float64)
        rows = np.concatenate([np.arange(0, 65 * 512, 97), np.arange(64 * 512, 65 * 512)])
        assert np.array_equal(y[:, rows], oracle_rows_g128(big, rows=rows, need_wmax=False)[0])


def test_small_matrix_before_one_of_16600_panels():
    import torch

    import paper_2609_00224_amd as q

    # two slices of 16600 panels over 511 workgroups: the last one's first unit is the
    # second of panel 16567; the matrix repeats 5120 rows
    N0, K, times = 5120, 300, 1660
    base = g128_dyadic_case(63, N0, K, 1, 3)
    small = dyadic_case(64, 512, 14336, 2, 40)
    ps = gpu_pack(small)
    rep = lambda a, axis: to_dev(a).repeat(*((times, 1) if axis == 0 else (1, times)))
    bitmap = to_dev(synth.column_bitmap(base["S"], K))
    pb = q.pack_matrix_g128(rep(base["trits"], 0), rep(base["alpha_g"], 0), rep(base["beta_g"], 0), to_dev(base["v"]), bitmap,
                            int(base["S"].size), rep(base["R8"], 1), rep(base["idx"], 1))
    need = max(q.qtea_workspace_bytes(pb.desc, 1), q.qtea_workspace_bytes(ps.desc, 2))
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    ref = torch.from_numpy(oracle_rows_g128(base, need_wmax=False)[0]).to("cuda")
    x, y = to_dev(base["x"]), torch.empty((1, N0 * times), dtype=torch.float32, device="cuda")
    print(f"[case] 512x14336 batch 2, then {N0 * times}x{K} in the grouped format, one workspace", flush=True)
    for _ in range(2):
        assert np.array_equal(gpu_gemm(ps, small["x"], ws=ws).astype(np.float64), oracle_rows(small, need_wmax=False)[0])
        y.fill_(float("nan"))
        q.qtea_gemm_lowbatch(pb.desc, pb.packed, x, 1, y, ws)
        assert torch.equal(y.view(times, N0).double(), ref.expand(times, N0))
    assert int(ws[:65536].view(torch.int32).abs().sum().item()) == 0
