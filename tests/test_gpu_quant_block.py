"""The quantizer's column phase on both sides of its dispatch (one launch per
128-column block up to 8192 rows, a launch per column stage above) and at the
edges of the block kernel: one workgroup and the most it takes, a last chunk
of columns that is not full, no and several refinement rounds.  Integer and
fp16 results equal the fp64 oracle's bit for bit; the Hessian's mirrored tiles
are exactly symmetric."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from oracle import quantizer as qz

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K,nS,iters", [(8192, 140, 3, 2), (8196, 140, 3, 2), (64, 17, 2, 2), (68, 144, 5, 1),
                                          (132, 129, 4, 0), (256, 300, 9, 4)])
def test_column_phase_matches_oracle(N, K, nS, iters):
    import torch

    import paper_2609_00224_amd as q

    print(f"[case] quantize {N}x{K}, {nS} salient, {iters} rounds", flush=True)
    W, X = synth.quant_inputs(900 + N + K, N, K, 3 * K)
    H = qz.hessian(X)
    ref = qz.quantize(W, H, nS, iters=iters)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")
    out = q.quantize_matrix(dev(W), dev(H), nS, iters=iters)
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in out.items() if v is not None}
    assert np.array_equal(got["S"], ref["S"])
    assert np.array_equal(got["v"].astype(np.float64), ref["v"])
    assert np.array_equal(got["alpha"].astype(np.float64), ref["alpha"])
    assert np.array_equal(got["beta"].astype(np.float64), ref["beta"])
    assert np.array_equal(got["T"], ref["T"])
    assert np.array_equal(got["R8"], ref["rval"]) and np.array_equal(got["idx"], ref["ridx"])


@pytest.mark.parametrize("N,K,nS,iters", [(8192, 140, 3, 2), (132, 300, 4, 3)])
def test_columns_again_when_an_exchange_runs_out(N, K, nS, iters):
    """The debug build's waits between workgroups run out at once: its call
    marks that in the workspace, quantizes the columns again by the launches
    per column and gives the release build's bits."""
    import torch

    import paper_2609_00224_amd as q

    print(f"[case] quantize again {N}x{K}, {nS} salient, {iters} rounds", flush=True)
    W, X = synth.quant_inputs(300 + K, N, K, 3 * K)
    W, H = torch.from_numpy(W).to("cuda"), torch.from_numpy(qz.hessian(X)).to("cuda")
    want = q.quantize_matrix(W, H, nS, iters=iters)
    # the word after the factorization's status, 12 bytes behind the regions of
    # W, H_d, U, a block's errors, scores, flags, ranks and block means
    up = lambda n: -(-n // 256) * 256
    mark = sum(map(up, (8 * K * N, 8 * K * K, 8 * K * K, 8 * 128 * N, 8 * K, 4 * K, 4 * K, 8 * -(-K // 128)))) + 12

    def call():
        out = {k: None if v is None else torch.zeros_like(v) for k, v in want.items()}
        ws = torch.zeros(q.qtea_quant_workspace_bytes(N, K), dtype=torch.uint8, device="cuda")
        p = q.QteaQuantParams(nS, 1.0, 0.01, iters, 0)
        q.qtea_quantize(W, H, p, *(out[k] for k in ("T", "alpha", "beta", "v", "S", "bitmap", "R8", "idx")), None, ws)
        return out, int(ws[mark:mark + 4].view(torch.int32).item())

    assert call()[1] == 0
    saved = q._lib
    q._lib = q.open_library(q.DEBUG_LIB_PATH)
    try:
        got, ran_out = call()
    finally:
        q._lib = saved
    assert ran_out == 1
    for k, v in want.items():
        assert v is None or torch.equal(v, got[k]), k


@pytest.mark.parametrize("K", [1, 127, 128, 129, 300])
def test_hessian_tiles_symmetric(K):
    """Every product is exact in 64 bits and both orders of a pair are summed
    alike: the mirror is the same bits; against numpy to n + 2 roundings of
    the sum of magnitudes."""
    import torch

    import paper_2609_00224_amd as q

    n = 37
    X = np.random.default_rng(K).standard_normal((n, K)).astype(np.float32)
    H = torch.full((K, K), float("nan"), dtype=torch.float64, device="cuda")
    q.qtea_quant_hessian(torch.from_numpy(X).to("cuda"), H)
    got = H.cpu().numpy()
    X64 = X.astype(np.float64)
    assert np.array_equal(got, got.T)
    bound = (n + 2) * 2.0 ** -53 * (2.0 / n) * (np.abs(X64).T @ np.abs(X64))
    assert np.all(np.abs(got - qz.hessian(X)) <= 2 * bound)
