"""What this framework is timed on: whole calls of its public entry points.

A case is one call as a user's program makes it: a layer's inference (encode +
lookup-accumulate, with or without the layer output fused, int8 or fp32
tables, one image's rows to a million), or an offline step that produces the
tables (building and quantizing them, fitting them to a layer's outputs).
Inputs are drawn on the GPU in the framework's own distributions
(paper_2207_05808_amd/workloads.py); trees, tables and training rows are made
here in plain torch, so `exact` shares none of the framework's code.
"""
from __future__ import annotations

import math

import torch

import paper_2207_05808_amd as mdn

K, LEVELS, NODES = 16, 4, 15
ROWS = 32768          # rows per block of the plain-torch references
LAMBDA = 1.0          # ridge weight of the table fits


def _layer(name, N, D, C, M, op="matmul", data="normal", table="i8", pad=0):
    return {"name": name, "kind": "layer", "N": N, "D": D, "C": C, "M": M, "op": op, "data": data,
            "table": table, "pad": pad}


def listed():
    return [
        # the last layer of a small classifier on one batch: a single launch whose latency is all there is
        _layer("classifier_tiny", 1024, 64, 4, 10),
        # a 3x3 convolution over 64 channels with bias and ReLU, one 32x32 image: the smallest convolution call
        _layer("conv_image_relu", 1024, 576, 32, 64, op="relu", data="im2col"),
        # the same convolution over a batch of 128 images: the headline layer
        _layer("conv_batch", 131072, 576, 32, 64, data="im2col"),
        # a 100-class softmax classifier on 512 features over a test set of 10000 images
        _layer("classifier_softmax", 10000, 512, 64, 100, op="softmax"),
        # a hidden layer 512 -> 512 with bias and ReLU on a serving batch of an odd number of rows
        _layer("dense_serving_relu", 3001, 512, 64, 512, op="relu"),
        # the same hidden layer over a million rows (token- or pixel-wise layers of a large batch)
        _layer("dense_hidden", 1048576, 512, 64, 512),
        # a wide layer 1024 -> 4096 on a serving batch: its table is larger than the LDS
        _layer("wide_serving", 2048, 1024, 128, 4096, data="zero10"),
        # the same wide layer over a large batch: the largest outputs
        _layer("wide_layer", 262144, 1024, 128, 4096, data="zero10"),
        # one input column per codebook with search-tree thresholds and the unquantized fp32 table
        _layer("f32_layer", 524288, 256, 256, 1024, table="f32", data="search_tree"),
        # offline: the wide layer's table from its prototypes and weights, quantized
        {"name": "build_wide", "kind": "build", "D": 1024, "C": 128, "M": 4096},
        # offline: the hidden layer's table fitted to its outputs on a training set, affine output
        {"name": "fit_ridge_dense", "kind": "ridge", "N": 16384, "D": 512, "C": 64, "M": 512},
        # offline: the convolution's table fitted under a row softmax, ten gradient steps
        {"name": "fit_gd_softmax", "kind": "gd", "N": 16384, "D": 576, "C": 32, "M": 64, "act": "softmax", "iters": 10},
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["classifier", "conv", "dense", "dense", "wide", "f32", "build", "ridge", "gd"])
    if kind == "classifier":
        C = rng.choice([4, 5, 8, 12, 16, 32, 64])
        c = _layer("", _log(rng, 256, 32768), C * rng.randint(4, 16), C, _log(rng, 10, 200),
                   op=rng.choice(["matmul", "softmax"]))
    elif kind == "conv":
        c = _layer("", _log(rng, 900, 131072), 576, rng.choice([16, 32, 64]), rng.choice([24, 32, 48, 64, 96, 128]),
                   op=rng.choice(["matmul", "relu"]), data="im2col")
    elif kind == "dense":
        C = rng.choice([24, 32, 48, 64, 96])
        c = _layer("", _log(rng, 128, 300000), C * rng.randint(4, 12) + rng.choice([0, 0, 1]), C,
                   rng.choice([100, 128, 256, 384, 500, 512, 768, 1000]), op=rng.choice(["matmul", "relu", "softmax"]),
                   pad=rng.choice([0, 0, 4, 5]))
    elif kind == "wide":
        C = rng.choice([64, 96, 112, 128])
        c = _layer("", _log(rng, 128, 100000), C * rng.choice([4, 8]), C, rng.choice([1024, 1536, 2000, 3072, 4096]),
                   op=rng.choice(["matmul", "relu"]), data="zero10")
    elif kind == "f32":
        C = rng.choice([16, 50, 64, 128, 256])
        c = _layer("", _log(rng, 500, 200000), C, C, rng.choice([64, 100, 256, 510, 1024]), table="f32",
                   data="search_tree", op=rng.choice(["matmul", "relu"]))
    elif kind == "build":
        C = rng.choice([4, 16, 32, 60, 64, 100, 128])
        c = {"kind": "build", "D": C * rng.randint(1, 10) + rng.choice([0, 3]), "C": C, "M": _log(rng, 10, 4096)}
    elif kind == "ridge":
        C = rng.choice([4, 10, 16, 32, 48, 64])
        c = {"kind": "ridge", "N": _log(rng, 1000, 16384), "D": C * rng.randint(4, 10), "C": C, "M": _log(rng, 10, 512)}
    else:
        C = rng.choice([4, 8, 16, 20, 32])
        c = {"kind": "gd", "N": _log(rng, 500, 16384), "D": C * rng.randint(4, 18), "C": C, "M": _log(rng, 8, 64),
             "act": rng.choice(["relu", "softmax", "softmax_sqerr"]), "iters": rng.choice([5, 10])}
    c.pop("name", None)
    return c


# ------------------------------------------------------------------ inputs


def _gen(seed, k):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000003 + k)
    return g


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)


def _subspaces(D, C):
    """Column -> codebook: C contiguous blocks, the first D % C of them one column wider."""
    q, r = divmod(D, C)
    return [(c * q + min(c, r), q + (1 if c < r else 0)) for c in range(C)]


def _activations(case, seed):
    """Rows of A [N][D] (row stride D + pad)."""
    g = _gen(seed, 1)
    N, D, pad, data = case["N"], case["D"], case.get("pad", 0), case.get("data", "normal")
    if data == "im2col":   # post-ReLU |N(0,1)| images of 32x32, 3x3 window, zero padding; columns (ky, kx, channel)
        ch = D // 9
        imgs = (N + 1023) // 1024
        x = torch.zeros(imgs, 34, 34, ch, device="cuda")
        x[:, 1:-1, 1:-1] = _randn(g, imgs, 32, 32, ch).abs_()
        A = torch.empty(imgs, 32, 32, 9, ch, device="cuda")
        for k in range(9):
            A[:, :, :, k] = x[:, k // 3:k // 3 + 32, k % 3:k % 3 + 32]
        return A.view(imgs * 1024, D)[:N]
    A = _randn(g, N, D + pad)
    if data == "zero10":
        A[torch.rand(N, D + pad, generator=g, device="cuda") < 0.1] = 0.0
    return A[:, :D]


def _trees(case, seed):
    """Split columns [C][4] inside each codebook's subspace and thresholds [C][15]."""
    g = _gen(seed, 2)
    D, C, data = case["D"], case["C"], case.get("data", "normal")
    sub = torch.tensor(_subspaces(D, C), device="cuda")
    thr = _randn(g, C, NODES)
    if data == "im2col":
        thr.abs_()
    pick = torch.rand(C, LEVELS, generator=g, device="cuda")
    if data == "search_tree":   # one column per codebook, sorted thresholds in heap order
        pick.zero_()
        srt = thr.sort(dim=1).values
        at = [(2 * i + 1) * (1 << (3 - t)) - 1 for t in range(LEVELS) for i in range(1 << t)]
        thr = srt[:, at].contiguous()
    split = sub[:, :1] + (pick * sub[:, 1:]).long()
    return split.to(torch.int32).contiguous(), thr


def _weights(case, seed):
    """Prototypes P [C][16][D] (zero outside each subspace) and weights B [D][M]."""
    g = _gen(seed, 3)
    D, C, M, data = case["D"], case["C"], case["M"], case.get("data", "normal")
    P = torch.zeros(C, K, D, device="cuda")
    for c, (lo, n) in enumerate(_subspaces(D, C)):
        v = _randn(g, K, n)
        P[c, :, lo:lo + n] = v.abs_() if data == "im2col" else v
    return P, _randn(g, D, M) / math.sqrt(D)


def _table(P, B, C):
    """T = P B [C][16][M] in float64."""
    Pd, Bd = P.double(), B.double()
    D = B.shape[0]
    return torch.stack([Pd[c, :, lo:lo + n] @ Bd[lo:lo + n] for c, (lo, n) in enumerate(_subspaces(D, C))])


def _quantize(T):
    """8-bit block floating point: codes, power-of-two scales and offsets per codebook."""
    C = T.shape[0]
    lo, hi = T.amin(dim=(1, 2)), T.amax(dim=(1, 2))
    off = ((lo + hi) / 2).float()
    X = T - off.double()[:, None, None]
    r = X.abs().amax(dim=(1, 2))
    m, e = torch.frexp(r / 127.0)
    e = e.long() - (m == 0.5).long()          # the smallest e with r <= 127 2^e
    e = torch.where(127.0 * torch.ldexp(torch.ones_like(r), e) < r, e + 1, e)
    e = torch.where(r == 0, torch.full_like(e, -126), e.clamp(-126, 127))
    cap = 0
    while 127.0 * C * (1 << (cap + 1)) < (1 << 24):
        cap += 1
    e = torch.maximum(e, e.max() - cap)
    s = torch.ldexp(torch.ones_like(r), e)
    return torch.round(X / s[:, None, None]).to(torch.int8), s.float(), off


def _encode(A, split, thr):
    """The indices [N][C] of every row, in plain torch."""
    out = []
    for r in range(0, A.shape[0], ROWS):
        a = A[r:r + ROWS]
        i = torch.zeros(a.shape[0], split.shape[0], dtype=torch.long, device=a.device)
        for t in range(LEVELS):
            th = thr[:, (1 << t) - 1:(2 << t) - 1].t().contiguous().gather(0, i)
            i = 2 * i + (a[:, split[:, t].long()] > th).long()
        out.append(i.to(torch.uint8))
    return torch.cat(out)


def _layer_inputs(case, seed):
    s = {"A": _activations(case, seed)}
    s["split"], s["thr"] = _trees(case, seed)
    P, B = _weights(case, seed)
    T = _table(P, B, case["C"])
    if case["table"] == "f32":
        s["lut"] = T.float()
    else:
        s["lut"], s["scale"], s["offset"] = _quantize(T)
    if case["op"] != "matmul":
        s["bias"] = _randn(_gen(seed, 4), case["M"])
    return s


def _fit_inputs(case, seed):
    A = _activations(case, seed)
    split, thr = _trees(case, seed)
    P, B = _weights(case, seed)
    s = {"idx": _encode(A, split, thr), "Y": (A.double() @ B.double()).float(), "T0": _table(P, B, case["C"]).float()}
    if case["kind"] == "gd":
        s["bias"] = _randn(_gen(seed, 4), case["M"])
        most = int((s["idx"].long() + K * torch.arange(case["C"], device="cuda")).flatten().bincount().max())
        s["eta"] = 1.0 / (2.0 * case["C"] * most + 2.0 * LAMBDA)
    return s


def prepare(case, seed):
    if case["kind"] == "layer":
        s = _layer_inputs(case, seed)
    elif case["kind"] == "build":
        s = dict(zip(("P", "B"), _weights(case, seed)))
    else:
        s = _fit_inputs(case, seed)
    s["case"] = case
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "build":
        return mdn.build_lut(s["P"], s["B"])
    if case["kind"] == "ridge":
        return mdn.fit_lut_ridge(s["idx"], s["Y"], s["T0"], LAMBDA)
    if case["kind"] == "gd":
        return mdn.fit_lut_gd(s["idx"], s["Y"], s["T0"], case["act"], LAMBDA, s["eta"], case["iters"],
                              col_bias=s["bias"])
    if case["table"] == "f32":
        if case["op"] == "matmul":
            return mdn.matmul_f32(s["A"], s["split"], s["thr"], s["lut"])[0]
        return mdn.matmul_act_f32(s["A"], s["split"], s["thr"], s["lut"], col_bias=s["bias"], act=case["op"])
    if case["op"] == "matmul":
        return mdn.matmul(s["A"], s["split"], s["thr"], s["lut"], s["scale"], s["offset"])[0]
    return mdn.matmul_act(s["A"], s["split"], s["thr"], s["lut"], s["scale"], s["offset"], col_bias=s["bias"],
                          act=case["op"])


def work(case):
    C, M = case["C"], case["M"]
    n = K * C
    if case["kind"] == "layer":
        N, D, e = case["N"], case["D"], 4 if case["table"] == "f32" else 1
        return {"bytes": 4 * N * D + 4 * N * M + n * M * e + C * (4 * LEVELS + 4 * NODES + (8 if e == 1 else 0)),
                "flops": N * C * (LEVELS + M)}
    if case["kind"] == "build":
        D = case["D"]
        return {"bytes": 4 * n * D + 4 * D * M + n * M + 8 * C, "flops": 2 * K * D * M}
    N = case["N"]
    one = N * C + 4 * N * M + 12 * n * M
    if case["kind"] == "ridge":
        return {"bytes": one, "flops": N * C * (C + 1) // 2 + N * C * M + n ** 3 // 3 + 2 * n * n * M}
    return {"bytes": one, "flops": case["iters"] * 2 * N * C * M}


def tolerance(case):
    # Integer sums, the quantizer and the ordered fp32 sums are defined to the bit by the entry points.
    if case["kind"] == "build":
        return "exact"
    if case["kind"] == "layer":
        # softmax: 1.1e-7 to 1.7e-7 against 64 bits
        return {"rel": 8e-7, "max": 4e-6} if case["op"] == "softmax" else "exact"
    # ridge: 3e-13 against another factorisation in 64 bits; gradient steps: 9e-18 (the steps are small)
    return {"rel": 1.5e-12, "max": 1e-10} if case["kind"] == "ridge" else {"rel": 1e-15, "max": 1e-13}


# --------------------------------------------------- references in 64 bits


def _sums(T, idx, bias=None):
    """sum_c T[c][idx[n][c]] (+ bias) in float64."""
    z = torch.zeros(idx.shape[0], T.shape[2], dtype=torch.float64, device=T.device)
    for c in range(T.shape[0]):
        z += T[c][idx[:, c].long()]
    return z if bias is None else z + bias.double()


def _sigma(z, op):
    return z.clamp_min(0.0) if op == "relu" else torch.softmax(z, dim=1) if op.startswith("softmax") else z


def exact(case, seed):
    if case["kind"] == "build":
        P, B = _weights(case, seed)
        return _quantize(_table(P, B, case["C"]))
    if case["kind"] == "layer":
        s = _layer_inputs(case, seed)
        T = s["lut"].double()
        if case["table"] != "f32":
            T = T * s["scale"].double()[:, None, None] + s["offset"].double()[:, None, None]
        A = s["A"]
        out = []
        for r in range(0, A.shape[0], ROWS):
            idx = _encode(A[r:r + ROWS], s["split"], s["thr"])
            out.append(_sigma(_sums(T, idx, s.get("bias")), case["op"]))
        return torch.cat(out)
    s = _fit_inputs(case, seed)
    C, M, n = case["C"], case["M"], K * case["C"]
    idx, Y, T0 = s["idx"], s["Y"].double(), s["T0"].double()
    at = idx.long() + K * torch.arange(C, device="cuda")

    def scatter(X):   # G^T X
        R = torch.zeros(n, X.shape[1], dtype=torch.float64, device="cuda")
        for c in range(C):
            R.index_add_(0, at[:, c], X)
        return R

    if case["kind"] == "ridge":
        G = torch.zeros(case["N"], n, dtype=torch.float64, device="cuda")
        G.scatter_(1, at, 1.0)
        H = (G.t().contiguous() @ G + LAMBDA * torch.eye(n, dtype=torch.float64, device="cuda")).cpu()
        rhs = (scatter(Y) + LAMBDA * T0.view(n, M)).cpu()
        return torch.cholesky_solve(rhs, torch.linalg.cholesky(H)).view(C, K, M)
    act, b = case["act"], s["bias"].double()
    P = _sigma(Y + b, act)
    T = T0.clone()
    for _ in range(case["iters"]):
        z = _sums(T, idx, s["bias"])
        Q = _sigma(z, act)
        if act == "relu":
            X = 2 * (Q - P) * (z > 0)
        elif act == "softmax":
            X = Q - P
        else:
            d = Q - P
            X = 2 * Q * (d - (d * Q).sum(dim=1, keepdim=True))
        T = T - s["eta"] * (scatter(X).view(C, K, M) + 2 * LAMBDA * (T - T0))
    return T
