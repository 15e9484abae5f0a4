"""An activation that is not finite: every output of its batch row NaN on the
matrix cores; in the table kernel the infinity, or NaN, where the code in its
column is not 0 and NaN or the other columns' sum where it is, in the grouped
format not finite anywhere, through the bias.  The other batch rows keep their
values."""
from __future__ import annotations

import numpy as np
import pytest

from tests.gpu_cases import (dyadic_case, e4m3_dyadic_case, g128_dyadic_case, gpu_gemm, gpu_pack, gpu_pack_e4m3, gpu_pack_g128,
                             oracle_rows, oracle_rows_g128)

pytestmark = pytest.mark.gpu
BAD = [np.inf, -np.inf, np.nan]


def _case(fmt, N, K, B, nS, col):
    c = {"fp16": dyadic_case, "e4m3": e4m3_dyadic_case, "g128": g128_dyadic_case}[fmt](87, N, K, B, nS)
    assert col not in c["S"]
    pm = {"fp16": gpu_pack, "e4m3": gpu_pack_e4m3, "g128": gpu_pack_g128}[fmt](c)
    ref = (oracle_rows_g128 if fmt == "g128" else oracle_rows)(c, need_wmax=False)[0]
    return c, pm, ref


@pytest.mark.parametrize("bad", BAD)
@pytest.mark.parametrize("fmt", ["fp16", "e4m3"])
@pytest.mark.parametrize("B", [1, 3, 7, 9, 16])
def test_matrix_cores(B, fmt, bad):
    c, pm, ref = _case(fmt, 256, 700, B, 9, 350)
    c["x"][B // 2, 350] = bad
    y = gpu_gemm(pm, c["x"])
    assert np.all(np.isnan(y[B // 2]))
    assert np.array_equal(np.delete(y, B // 2, 0).astype(np.float64), np.delete(ref, B // 2, 0))


@pytest.mark.parametrize("bad", BAD)
@pytest.mark.parametrize("fmt", ["fp16", "e4m3"])
@pytest.mark.parametrize("col", [120, 121, 122, 123, 124])  # every place in a pack
def test_table_kernel(col, fmt, bad):
    c, pm, _ = _case(fmt, 16388, 320, 1, 9, col)
    c["x"][0, col] = 0.0
    without = oracle_rows(c, need_wmax=False)[0][0]
    c["x"][0, col] = bad
    t = c["trits"][:, col]
    y = gpu_gemm(pm, c["x"])[0].astype(np.float64)
    assert np.array_equal(y[t != 0], t[t != 0] * bad, equal_nan=True)
    assert np.all(np.isnan(y[t == 0]) | (y[t == 0] == without[t == 0]))


@pytest.mark.parametrize("bad", BAD)
@pytest.mark.parametrize("B", [1, 4])
def test_grouped_format(B, bad):
    c, pm, ref = _case("g128", 260, 700, B, 9, 350)
    c["x"][B // 2, 350] = bad
    y = gpu_gemm(pm, c["x"])
    assert not np.any(np.isfinite(y[B // 2]))
    assert np.array_equal(np.delete(y, B // 2, 0).astype(np.float64), np.delete(ref, B // 2, 0))
