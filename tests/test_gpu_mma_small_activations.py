"""The fp16 matrix-core kernel (batch 9..16 of one matrix, 5..16 of a plan) on
activations of 0.01 and 0.001: its two fp16 halves hold them as they hold
activations of 1."""
from __future__ import annotations

import numpy as np
import pytest

from tests.gpu_cases import gpu_gemm, gpu_pack, oracle_rows, synth_case
from tests.test_gpu_tern_mfma import _grouped

pytestmark = pytest.mark.gpu

# fp32 sums of 1443 exact products measure 0.7e-7 to 1.2e-7; the halves hold an
# activation of 2^-14 or more exactly, the few below it (|x| < 0.06 of 0.001) to
# 2^-36, 1.5e-8 of 0.001.  With the second half in units of 1: 1.7e-6 and 1.7e-5.
BAR = 3e-7


@pytest.mark.parametrize("scale", [0.01, 0.001])
@pytest.mark.parametrize("B", [5, 8, 9, 16])
def test_small_activations(B, scale):
    N, K = 256, 1443
    c = synth_case(79, N, K, B, nS=20)
    c["N"], c["K"] = N, K
    c["x"] = (c["x"].astype(np.float64) * scale).astype(np.float16)
    c["R"] = np.zeros_like(c["R"])
    print(f"[case] activations of {scale}, batch {B}", flush=True)
    ref, _ = oracle_rows(c, need_wmax=False)
    for y in [gpu_gemm(gpu_pack(c), c["x"]), _grouped([c, c], B)[1]]:
        d = np.linalg.norm(y.astype(np.float64) - ref, axis=1)
        assert np.all(d <= BAR * np.linalg.norm(ref, axis=1))
