"""One zero-filled workspace serves any sequence of matrices: a matrix of more
than 64 panels of 512 rows keeps its arrival counters where a smaller matrix's
partial rows do not come (its panels past the 64th were left unsummed when
they did)."""
from __future__ import annotations

import numpy as np
import pytest

from tests.gpu_cases import dyadic_case, g128_dyadic_case, gpu_gemm, gpu_pack, gpu_pack_g128, oracle_rows, oracle_rows_g128

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
