"""Every bit of every activation reaches the output, through every kernel: one
nonzero code per row, at every column of two slices and a part of a third, on
products v x of 22 significant bits down to 2^-6 of their block's largest power
of two.  Such a product is exact in each kernel's form of the activations (six
base-32 digits of 2^28, two fp16 halves, fp32 tables), its digits' partial
sums are multiples of its last bit below 2^24 of them, and the row has no other
term: the outputs are the products, bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

from tests.gpu_cases import gpu_gemm, gpu_pack
from tests.test_gpu_tern_mfma import _grouped

pytestmark = pytest.mark.gpu


def _case(seed, K, B):
    rng = np.random.default_rng(seed)
    N = -(-K // 4) * 4
    T = np.zeros((N, K), np.int8)
    T[np.arange(N), np.arange(N) % K] = rng.choice([-1, 1], size=N)
    sig = lambda shape: (1024 + rng.integers(0, 1024, size=shape)) / 1024.0
    x = sig((B, K)) * 2.0 ** -rng.integers(0, 6, size=(B, K)) * rng.choice([-1.0, 1.0], size=(B, K))
    return {"N": N, "K": K, "trits": T, "alpha": np.ones(N, np.float16), "v": sig(K).astype(np.float16),
            "S": np.zeros(0, np.int32), "R": np.zeros((0, N // 4), np.float16), "idx": np.zeros((0, N // 4), np.uint8),
            "x": x.astype(np.float16)}


@pytest.mark.parametrize("B", [1, 2, 4, 5, 8, 9, 16])
def test_one_code_per_row(B):
    c = _case(91 + B, 803, B)
    a = c["x"].astype(np.float64) * c["v"].astype(np.float64)
    j = np.arange(c["N"]) % c["K"]
    want = a[:, j] * c["trits"][np.arange(c["N"]), j]
    print(f"[case] one code per row, batch {B}", flush=True)
    assert np.array_equal(gpu_gemm(gpu_pack(c), c["x"]).astype(np.float64), want)
    assert np.array_equal(_grouped([c, c], B)[1].astype(np.float64), want)
