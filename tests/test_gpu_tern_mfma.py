"""The FP4 matrix-core kernel (batch 2..8 of one matrix, 2..4 of a grouped
plan) at the edges of its tiles, panels, slices and 32-column residual chunks:
bit for bit against the fp64 oracle on dyadic inputs; within its digit
split's bound on activations of very different magnitudes; and an activation
that is not finite."""
from __future__ import annotations

import numpy as np
import pytest

from tests.gpu_cases import dyadic_case, gpu_gemm, gpu_pack, oracle_rows, synth_case, to_dev

pytestmark = pytest.mark.gpu

# rows around 64 and 512, columns around a pack, a 16-pack group (80) and a
# slice (320), salient columns around the chunk of 32, up to every column
SHAPES = [(4, 1, 0), (4, 5, 5), (60, 79, 31), (64, 80, 32), (68, 81, 33), (512, 319, 64), (516, 320, 65),
          (1028, 321, 321), (124, 961, 700), (2052, 1601, 97)]


def _grouped(cases, B):
    import torch

    import paper_2609_00224_amd as q

    ys = [torch.full((B, c["N"]), float("nan"), dtype=torch.float32, device="cuda") for c in cases]
    gp = q.plan_grouped([gpu_pack(c) for c in cases], [to_dev(c["x"]) for c in cases], ys, batch=B)
    gp.run()
    torch.cuda.synchronize()
    return [y.cpu().numpy() for y in ys]


@pytest.mark.parametrize("B", [2, 3, 4, 5, 7, 8])
def test_edges_dyadic_exact(B):
    cases = [dyadic_case(7000 + 31 * B + i, N, K, B, nS) for i, (N, K, nS) in enumerate(SHAPES)]
    print(f"[case] FP4 kernel, batch {B}, {SHAPES}", flush=True)
    refs = [oracle_rows(c, need_wmax=False)[0] for c in cases]
    for c, ref in zip(cases, refs):
        y = gpu_gemm(gpu_pack(c), c["x"])
        assert np.array_equal(y.astype(np.float64), ref), (c["N"], c["K"], B)
    if B <= 4:
        for c, ref, y in zip(cases, refs, _grouped(cases, B)):
            assert np.array_equal(y.astype(np.float64), ref), ("grouped", c["N"], c["K"], B)


@pytest.mark.parametrize("B", [1, 3, 8])
def test_wide_range_of_magnitudes(B):
    """Activations over eight powers of ten: an a_j below 2^-6 of the largest
    power of two of its block of 20 columns is rounded by at most 2^-28 of that
    power, so a row's error is at most the sum of that over the row's nonzero codes
    (plus 32-bit roundings of the digit sums and of y, 2^-22 of sum |a|)."""
    c = synth_case(71, 192, 1003, B, nS=0)
    rng = np.random.default_rng(5)
    c["x"] = (c["x"].astype(np.float64) * 10.0 ** rng.uniform(-4, 4, size=c["x"].shape)).clip(-6e4, 6e4).astype(np.float16)
    c["N"], c["K"] = 192, 1003
    y = gpu_gemm(gpu_pack(c), c["x"]).astype(np.float64)
    ref, _ = oracle_rows(c, need_wmax=False)
    a = np.abs(c["x"].astype(np.float64) * c["v"].astype(np.float64))
    most = np.pad(a, ((0, 0), (0, -a.shape[1] % 20))).reshape(B, -1, 20).max(2)
    unit = np.repeat(2.0 ** np.floor(np.log2(most)), 20, axis=1)[:, : a.shape[1]]
    nonzero = np.abs(c["trits"]).astype(np.float64)
    bound = c["alpha"].astype(np.float64) * ((2.0 ** -28 * unit + 2.0 ** -22 * a) @ nonzero.T)
    assert np.all(np.abs(y - ref) <= bound)


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_activation_not_finite(bad):
    """Every output of that batch row is NaN (the digits of its block have the
    NaN scale); the other rows keep their values."""
    c = dyadic_case(72, 256, 700, 4, 9)
    ref, _ = oracle_rows(c, need_wmax=False)
    c["x"][2, 350] = bad
    for y in (gpu_gemm(gpu_pack(c), c["x"]), _grouped([c], 4)[0]):
        assert np.all(np.isnan(y[2]))
        assert np.array_equal(np.delete(y, 2, 0).astype(np.float64), np.delete(ref, 2, 0))
