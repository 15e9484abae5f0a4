"""The FP4 matrix-core kernels (batch 1..8 of one matrix, 2..4 of a plan) on
activations with outliers: a row whose codes are 0 in the outliers' columns has
the error of its other columns' sums, whatever the outliers."""
from __future__ import annotations

import numpy as np
import pytest

from tests.gpu_cases import gpu_gemm, gpu_pack, oracle_rows, synth_case
from tests.test_gpu_tern_mfma import _grouped

pytestmark = pytest.mark.gpu

# A row's sum over 5 slices and 6 to 10 digits: at most some 20 roundings or
# truncations of 2^-23 of a partial sum, of independent sizes, so about sqrt(20)
# 2^-24 = 2.7e-7 (fp32 sums of the exact products measure 0.7e-7 to 1.2e-7).  The
# rounding of the smaller columns to 2^-28 of an outlier of 4000 gave 1e-6.
BAR = 3e-7

# columns of the outliers (one alone; in every pack of a block; a run that
# leaves half a block; next to the last column), their size, the others' size
OUTLIERS = [([7], 4000.0, 1.0), ([320, 640, 1282], 60000.0, 1.0), ([41, 46], 16000.0, 1.0),
            (list(range(100, 113)), 16000.0, 1.0), ([1442], 600.0, 0.01)]


@pytest.mark.parametrize("B", [1, 2, 4, 5, 8])
@pytest.mark.parametrize("cols,size,others", OUTLIERS)
def test_rows_without_the_outliers(B, cols, size, others):
    N, K = 256, 1443
    c = synth_case(77, N, K, B, nS=0)
    c["N"], c["K"] = N, K
    c["x"] = (c["x"].astype(np.float64) * others).astype(np.float16)
    # every batch row its own outliers: the last one has none
    for b in range(B if B == 1 else B - 1):
        c["x"][b, cols] = size * (1.0 if b % 2 else -1.0)
    c["trits"][: N // 2, cols] = 0
    print(f"[case] {len(cols)} outliers of {size} among {others}, batch {B}", flush=True)
    ref, _ = oracle_rows(c, need_wmax=False)
    ys = [gpu_gemm(gpu_pack(c), c["x"])]
    if 2 <= B <= 4:
        ys.append(_grouped([c, c], B)[1])
    for y in ys:
        for half in (slice(0, N // 2), slice(N // 2, N)):
            d = np.linalg.norm(y[:, half].astype(np.float64) - ref[:, half], axis=1)
            assert np.all(d <= BAR * np.linalg.norm(ref[:, half], axis=1))
