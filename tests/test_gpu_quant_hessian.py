"""The Hessian's bits: the matrix cores add the rows' products one after another,
each rounded, so H equals the fp64 sum in ascending row order (a product of two
fp32 values is exact in fp64), at the edges of the 64-column tiles and of the
32-row stages, symmetric, every element written."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 63, 64, 65, 200])
@pytest.mark.parametrize("n", [1, 3, 32, 33, 130])
def test_hessian_bits(n, K):
    import torch

    import paper_2609_00224_amd as q

    print(f"[case] hessian n={n} K={K}", flush=True)
    rng = np.random.default_rng(1000 * n + K)
    X = (rng.standard_normal((n, K)) * np.exp(3 * rng.standard_normal((n, K)))).astype(np.float32)
    acc = np.zeros((K, K))
    for row in X.astype(np.float64):
        acc += np.outer(row, row)
    H = torch.full((K, K), float("nan"), dtype=torch.float64, device="cuda")
    q.qtea_quant_hessian(torch.from_numpy(X).cuda(), H)
    assert np.array_equal(H.cpu().numpy(), (2.0 / n) * acc)
