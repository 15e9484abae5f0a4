"""The work that a user of this library has it do, as cases to time.

Four kinds of call, each through the Python binding's entry points:

  gemv    one matrix on its own (qtea_gemm_lowbatch), what a decoder calls
          for one linear layer: any of the three packed formats, batch 1..16;
  token   the products of a decoder's layers one after another on one stream,
          a call per matrix (the latency of one decoded token);
  group   the same products as one planned launch (GroupedPlan.run), the
          throughput form for independent products;
  quant   the offline quantizer of one linear layer: the Hessian of its
          calibration rows, then the quantization.

Shapes are the linears of the Llama-3-8B-, Qwen3-14B- and Llama-3-70B-shaped
workloads of synth/workloads.py, and generic ragged ones.  Weights, scales,
residuals and activations follow that package's recipe (ternary codes with
P(0) = p0, alpha ~ U(0.01, 0.03), v ~ U(0.8, 1.2), x ~ N(0, 1), residual
~ N(0, 0.01) in 2 to 5 % of the columns), drawn on the GPU.
"""
from __future__ import annotations

import math

import torch

import paper_2609_00224_amd as q

# (role, N, K) of one decoder layer's fused linears (synth/workloads.py)
LAYERS = {
    "8b": (("qkv", 6144, 4096), ("o", 4096, 4096), ("gate_up", 28672, 4096), ("down", 4096, 14336)),
    "14b": (("qkv", 7168, 5120), ("o", 5120, 5120), ("gate_up", 34816, 5120), ("down", 5120, 17408)),
    "70b": (("qkv", 10240, 8192), ("o", 8192, 8192), ("gate_up", 57344, 8192), ("down", 8192, 28672)),
}
FORMATS = ("fp16", "e4m3", "g128")


def listed():
    return [
        # the attention output projection of an 8B decoder at batch 1: the
        # smallest product a token has
        {"name": "gemv_o_b1", "kind": "gemv", "N": 4096, "K": 4096, "fmt": "fp16", "sal": 0.02, "batch": 1},
        # the MLP's down projection, the longest rows, in the paper's E4M3
        # residual storage
        {"name": "gemv_down_e4m3_b1", "kind": "gemv", "N": 4096, "K": 14336, "fmt": "e4m3", "sal": 0.05, "batch": 1},
        # the MLP's up and gate projection for four concurrent sequences
        {"name": "gemv_gate_up_b4", "kind": "gemv", "N": 28672, "K": 4096, "fmt": "fp16", "sal": 0.02, "batch": 4},
        # a 14B QKV projection at the largest batch
        {"name": "gemv_qkv_b16", "kind": "gemv", "N": 7168, "K": 5120, "fmt": "fp16", "sal": 0.03, "batch": 16},
        # sizes that divide nothing: rows, columns and batch all ragged
        {"name": "gemv_ragged_b5", "kind": "gemv", "N": 3076, "K": 2999, "fmt": "e4m3", "sal": 0.03, "batch": 5},
        # the paper's grouped format (128-column scale and bias) for two sequences
        {"name": "gemv_g128_b2", "kind": "gemv", "N": 6144, "K": 4096, "fmt": "g128", "sal": 0.05, "batch": 2},
        # one decoded token of an 8B decoder, a call per linear
        {"name": "token_8b_b1", "kind": "token", "model": "8b", "layers": 32, "fmt": "fp16", "sal": 0.02, "batch": 1},
        # the same weights as independent products in one launch: the
        # repository's headline
        {"name": "group_8b_b1", "kind": "group", "model": "8b", "layers": 32, "fmt": "fp16", "sal": 0.02, "batch": 1},
        # the same at batch 4 in the E4M3 storage
        {"name": "group_8b_e4m3_b4", "kind": "group", "model": "8b", "layers": 32, "fmt": "e4m3", "sal": 0.05, "batch": 4},
        # 14B-shaped layers at the largest batch
        {"name": "group_14b_b16", "kind": "group", "model": "14b", "layers": 12, "fmt": "fp16", "sal": 0.03, "batch": 16},
        # the paper's grouped format, an 8B stack at batch 1
        {"name": "group_8b_g128_b1", "kind": "group", "model": "8b", "layers": 32, "fmt": "g128", "sal": 0.05, "batch": 1},
        # quantizing one 4096 x 4096 linear from 8192 calibration rows at the
        # paper's setting (5 % salient, two refinement rounds)
        {"name": "quant_o", "kind": "quant", "N": 4096, "K": 4096, "rows": 8192, "sal": 0.05, "iters": 2},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("gemv", "gemv", "gemv", "gemv", "token", "group", "group", "quant"))
    fmt = rng.choice(FORMATS)
    sal = rng.choice((0.0, 0.02, 0.03, 0.05))
    batch = rng.choice((1, 1, 2, 3, 4, 5, 8, 11, 16))
    if kind == "gemv":
        return {"kind": kind, "N": 4 * _log_int(rng, 16, 8704), "K": _log_int(rng, 64, 17408), "fmt": fmt,
                "sal": sal, "batch": batch}
    if kind == "quant":
        # (more calibration rows than columns, as in use: the factor of a
        # rank-deficient Hessian amplifies the last bits into other codes)
        K = _log_int(rng, 100, 3000)
        return {"kind": kind, "N": 4 * _log_int(rng, 16, 1024), "K": K, "rows": int(K * rng.uniform(1.5, 3.0)),
                "sal": sal, "iters": rng.choice((0, 1, 2, 2, 3))}
    model = rng.choice(("8b", "8b", "14b", "70b"))
    most = {"8b": 16, "14b": 8, "70b": 3}[model]
    return {"kind": kind, "model": model, "layers": rng.randint(1, most), "fmt": fmt, "sal": sal, "batch": batch}


def _shapes(case):
    if case["kind"] == "gemv":
        return [(case["N"], case["K"])]
    return [(N, K) for _ in range(case["layers"]) for _, N, K in LAYERS[case["model"]]]


def _matrix(gen, N, K, case):
    """Dense inputs of one compressed matrix and its activations (GPU)."""
    dev = "cuda"
    fmt, B = case["fmt"], case["batch"]
    nS = int(math.floor(case["sal"] * K + 0.5))
    # P(-1) = P(+1) = 3/10, P(0) = 2/5
    u = torch.randint(0, 10, (N, K), generator=gen, device=dev, dtype=torch.int8)
    m = {"T": (u > 6).to(torch.int8) - (u < 3).to(torch.int8)}
    del u

    def uniform(shape, lo, hi):
        return (lo + (hi - lo) * torch.rand(shape, generator=gen, device=dev)).to(torch.float16)

    G = -(-K // 128)
    m["alpha"] = uniform((N, G) if fmt == "g128" else (N,), 0.01, 0.03)
    m["beta"] = uniform((N, G), -0.005, 0.005) if fmt == "g128" else None
    m["v"] = uniform((K,), 0.8, 1.2)
    m["S"] = torch.randperm(K, generator=gen, device=dev)[:nS].sort().values.to(torch.int32)
    r = 0.01 * torch.randn((nS, N // 4), generator=gen, device=dev)
    m["R"] = r.to(torch.float16) if fmt == "fp16" else r.to(torch.float8_e4m3fn)
    m["idx"] = torch.randint(0, 4, (nS, N // 4), generator=gen, device=dev, dtype=torch.uint8)
    m["x"] = torch.randn((B, K), generator=gen, device=dev).to(torch.float16)
    return m


def _pack(m, N, K, fmt):
    if fmt == "fp16":
        return q.pack_matrix(m["T"], m["alpha"], m["v"], m["S"], m["R"], m["idx"])
    S = m["S"].to(torch.int64)
    # one bit per column, 32 to a word: distinct bits, so a sum sets them
    words = torch.zeros(-(-K // 32), dtype=torch.int64, device=S.device)
    words.index_add_(0, S // 32, torch.ones_like(S) << (S % 32))
    bitmap = torch.where(words >= 1 << 31, words - (1 << 32), words).to(torch.int32)
    R8 = m["R"].view(torch.uint8)
    if fmt == "e4m3":
        return q.pack_matrix_e4m3(m["T"], m["alpha"], m["v"], bitmap, S.numel(), R8, m["idx"])
    return q.pack_matrix_g128(m["T"], m["alpha"], m["beta"], m["v"], bitmap, S.numel(), R8, m["idx"])


def _quant_inputs(case, seed):
    """Weights and calibration rows as synth.quant_inputs draws them, with a
    pairwise instead of a dense correlation of the channels."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    N, K = case["N"], case["K"]
    W = 0.02 * torch.randn((N, K), generator=gen, device="cuda", dtype=torch.float64)
    cols = torch.randperm(K, generator=gen, device="cuda")
    W[:, cols[:max(1, K // 100)]] *= 4.0
    Z = torch.randn((case["rows"], K), generator=gen, device="cuda")
    X = Z + 0.3 * Z.roll(1, 1) + 0.1 * Z.roll(7, 1)
    X[:, torch.randperm(K, generator=gen, device="cuda")[:max(1, K // 50)]] *= 5.0
    return W, X.contiguous()


def prepare(case, seed):
    if case["kind"] == "quant":
        W, X = _quant_inputs(case, seed)
        K = case["K"]
        return {"kind": "quant", "W": W, "X": X, "H": torch.empty((K, K), dtype=torch.float64, device="cuda"),
                "n_salient": int(math.floor(case["sal"] * K + 0.5)), "iters": case["iters"]}
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B = case["batch"]
    mats, xs, ys = [], [], []
    for N, K in _shapes(case):
        m = _matrix(gen, N, K, case)
        mats.append(_pack(m, N, K, case["fmt"]))
        xs.append(m["x"])
    # the outputs of all products in one buffer, product after product
    Y = torch.zeros(sum(B * m.N for m in mats), dtype=torch.float32, device="cuda")
    ys = [y.view(B, m.N) for y, m in zip(Y.split([B * m.N for m in mats]), mats)]
    state = {"kind": case["kind"], "batch": B, "mats": mats, "xs": xs, "ys": ys, "Y": Y}
    if case["kind"] == "group":
        state["plan"] = q.plan_grouped(mats, xs, ys, batch=B)
    else:
        # one workspace serves a stream-ordered sequence of calls
        need = max(q.qtea_workspace_bytes(m.desc, B) for m in mats)
        state["ws"] = torch.zeros(max(need, 4), dtype=torch.uint8, device="cuda")
    return state


def run(state):
    if state["kind"] == "quant":
        q.qtea_quant_hessian(state["X"], state["H"])
        out = q.quantize_matrix(state["W"], state["H"], state["n_salient"], iters=state["iters"])
        return [state["H"]] + [out[k] for k in ("T", "alpha", "beta", "v", "S", "bitmap", "R8", "idx")]
    if state["kind"] == "group":
        state["plan"].run()
    else:
        B, ws = state["batch"], state["ws"]
        for m, x, y in zip(state["mats"], state["xs"], state["ys"]):
            q.qtea_gemm_lowbatch(m.desc, m.packed, x, B, y, ws)
    return state["Y"]


def work(case):
    """Bytes read and written once, and the operations of the plain product."""
    if case["kind"] == "quant":
        N, K, n = case["N"], case["K"], case["rows"]
        nS = int(math.floor(case["sal"] * K + 0.5))
        G = -(-K // 128)
        nbytes = 4 * n * K + 8 * K * K + 8 * N * K + N * K + 4 * N * G + 2 * K + K // 8 + 4 * nS + 2 * nS * (N // 4)
        # symmetric Hessian, Cholesky factor and triangular inverse (K^3 / 3
        # each), error propagation to the later columns (N K^2)
        return {"bytes": nbytes, "flops": n * K * K + 2 * K ** 3 / 3 + N * K * K}
    B, nbytes, flops = case["batch"], 0, 0
    for N, K in _shapes(case):
        nS = int(math.floor(case["sal"] * K + 0.5))
        if case["fmt"] == "g128":
            w = q.algorithmic_bytes_g128(N, K, nS)
        else:
            w = q.algorithmic_bytes(N, K, nS, 2 if case["fmt"] == "fp16" else 1)
        nbytes += w + 2 * B * K + 4 * B * N
        flops += 2 * B * N * K + 2 * B * nS * (N // 4)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] == "quant":
        # codes and scales are decided in 64 bits: another order of the sums
        # moves a decision only where a value ties to its last bits
        return {"rel": 1e-5, "differ": 1e-5}
    # 32-bit sums of up to 28672 products
    return {"rel": 2e-6}


def _dense(m, N, K, fmt):
    """W_eff [N][K] in 64 bits (without the bias of the grouped format)."""
    W = m["T"].to(torch.float64) * m["v"].to(torch.float64)
    a = m["alpha"].to(torch.float64)
    W *= a.repeat_interleave(128, 1)[:, :K] if fmt == "g128" else a[:, None]
    nS = m["S"].numel()
    if nS:
        rows = (torch.arange(N // 4, device=W.device) * 4)[None, :] + m["idx"].to(torch.int64)
        cols = m["S"].to(torch.int64)[:, None].expand(nS, N // 4)
        R = m["R"].to(torch.float32).to(torch.float64)
        W.index_put_((rows.reshape(-1), cols.reshape(-1)), R.reshape(-1), accumulate=True)
    return W


def _exact_quant(case, seed):
    """The quantizer's method (paper, Eq. 1-9) column by column in 64 bits."""
    W, X = _quant_inputs(case, seed)
    N, K, iters = case["N"], case["K"], case["iters"]
    f64, dev = torch.float64, W.device
    nS = int(math.floor(case["sal"] * K + 0.5))
    H = (X.to(f64).T @ X.to(f64)) * (2.0 / X.shape[0])
    d0 = H.diagonal().clone()
    order = torch.sort((W * W).max(0).values * d0 * d0, descending=True, stable=True).indices
    S = order[:nS].sort().values
    rank = torch.full((K,), -1, dtype=torch.int64)
    rank[S.cpu()] = torch.arange(nS)
    Hd = H + 0.01 * d0.mean() * torch.eye(K, dtype=f64, device=dev)
    # H_d = V V^T with V upper (a Cholesky factor from the last column), so
    # that U = V^-1 is the upper factor of the inverse, H_d^-1 = U^T U
    V = torch.linalg.cholesky(Hd.flip(0, 1).contiguous()).flip(0, 1).contiguous()
    U = torch.linalg.solve_triangular(V, torch.eye(K, dtype=f64, device=dev), upper=True).contiguous()
    du = U.diagonal()
    G = -(-K // 128)

    def half(t):  # nearest fp16 value (a plain conversion would round twice, through 32 bits)
        ulp = torch.ldexp(torch.ones_like(t), torch.frexp(t).exponent.clamp(min=-13) - 11)
        return torch.round(t / ulp) * ulp

    tern = lambda x, thr: (x > thr).to(f64) - (x < -thr).to(f64)
    T = torch.zeros((N, K), dtype=torch.int8, device=dev)
    alpha = torch.zeros((N, G), dtype=torch.float16, device=dev)
    beta = torch.zeros((N, G), dtype=torch.float16, device=dev)
    v16 = torch.ones(K, dtype=torch.float16, device=dev)
    R8 = torch.zeros((nS, N // 4), dtype=torch.uint8, device=dev)
    idx = torch.zeros((nS, N // 4), dtype=torch.uint8, device=dev)
    E4 = torch.arange(127, dtype=torch.uint8).view(torch.float8_e4m3fn).to(f64).to(dev)
    ranks = rank.tolist()
    Wt = W.T.contiguous()
    for g in range(G):
        b0, b1 = g * 128, min(K, (g + 1) * 128)
        n = b1 - b0
        w = Wt[b0:b1]
        sw = w.sum(0)
        be = sw / n
        al = (w - be).abs().sum(0) / n
        for _ in range(2):
            t = tern(w - be, al / 2)
            s1, s2, stw = t.sum(0), (t * t).sum(0), (t * w).sum(0)
            det = s2 * n - s1 * s1
            a = torch.where(det > 0, (n * stw - s1 * sw) / det, torch.zeros_like(det))
            ok = (det > 0) & (a > 0) & (al > 0)
            be = torch.where(ok, (s2 * sw - s1 * stw) / det, be)
            al = torch.where(ok, a, al)
        al, be = half(al), half(be)
        al = torch.where(al == 0, torch.ones_like(al), al)
        alpha[:, g], beta[:, g] = al.to(torch.float16), be.to(torch.float16)
        dmean = du[b0:b1].mean()
        gamma = torch.exp(-(du[b0:b1] / dmean) * (torch.arange(n, device=dev, dtype=f64) / n))
        err = torch.zeros((n, N), dtype=f64, device=dev)
        for i in range(n):
            j = b0 + i
            w = Wt[j]
            x = w - be
            xa = x.abs() / al
            t, vj = tern(x, al / 2), torch.ones((), dtype=f64, device=dev)
            for _ in range(iters):
                c = t.abs().sum()
                vj = torch.where(c > 0, half((xa * t.abs()).sum() / c.clamp(min=1)), vj)
                t = tern(x, vj * al / 2)
            qv = be + (vj * al) * t
            if ranks[j] >= 0:
                r = (w - qv).view(N // 4, 4)
                k = r.abs().argmax(1)
                rk = r.gather(1, k[:, None])[:, 0]
                mid = (E4[1:] + E4[:-1]) / 2
                mag = rk.abs().clamp(max=448.0)
                lo = torch.searchsorted(mid, mag)  # codes whose midpoint lies below
                tie = (lo < 126) & (mid[lo.clamp(max=125)] == mag) & (lo % 2 == 1)
                code = lo + tie.to(lo.dtype)
                R8[ranks[j]] = (code + 128 * (rk < 0)).to(torch.uint8)
                idx[ranks[j]] = k.to(torch.uint8)
                val = torch.where(rk < 0, -E4[code], E4[code])
                qv = qv.view(N // 4, 4).scatter_add(1, k[:, None], val[:, None]).reshape(N)
            T[:, j], v16[j] = t.to(torch.int8), vj.to(torch.float16)
            err[i] = gamma[i] * (w - qv) / du[j]
            if i + 1 < n:
                Wt[j + 1:b1] -= U[j, j + 1:b1, None] * err[i]
        if b1 < K:
            Wt[b1:] -= U[b0:b1, b1:].T.contiguous() @ err
    words = torch.zeros(-(-K // 32), dtype=torch.int64, device=dev)
    words.index_add_(0, S // 32, torch.ones_like(S) << (S % 32))
    bitmap = torch.where(words >= 1 << 31, words - (1 << 32), words).to(torch.int32)
    return [H, T, alpha, beta, v16, S.to(torch.int32), bitmap, R8, idx]


def exact(case, seed):
    if case["kind"] == "quant":
        return _exact_quant(case, seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    out = []
    for N, K in _shapes(case):
        m = _matrix(gen, N, K, case)
        x = m["x"].to(torch.float64)
        y = (_dense(m, N, K, case["fmt"]) @ x.T).T.contiguous()
        if case["fmt"] == "g128":
            G = -(-K // 128)
            xg = torch.nn.functional.pad(x, (0, 128 * G - K)).view(-1, G, 128).sum(2)
            y += (m["beta"].to(torch.float64) @ xg.T).T
        out.append(y.reshape(-1))
    return torch.cat(out)
