"""The calls whose speed counts: training steps of every model of the library, through its public entry points.

A case is one step of a worker (sufficient factors of its mini-batch, then the summed rank-1 updates of its own
and its peers' factor blocks applied to W), or, where W is kept as two 16-bit planes, a run of steps that ends with
the parameters written back to the fp32 array, as a program does that trains on the planes and then evaluates or
saves.  Inputs are drawn on the GPU from the seed alone.
"""
from __future__ import annotations

import math

import torch

import paper_1409_5705_amd as sfb

DEV = "cuda:0"
SPLIT_STEPS = 5          # steps between two exports of a matrix kept as planes


def listed():
    return [
        # the smallest model: a step is a handful of launches, nothing but latency
        dict(name="mlr_f32_small", family="mlr_f32", J=64, D=128, B=32, P=1),
        # a thousand classes, the worker's own 256 samples and seven peers' blocks
        dict(name="mlr_f32_peers", family="mlr_f32", J=1000, D=2048, B=256, P=8),
        # the mini-batch of a hundred that the method works best with, sizes as data sets have them (nothing aligned)
        dict(name="mlr_f32_ragged", family="mlr_f32", J=1003, D=2047, B=100, P=8),
        # distance metric learning, half the hinge terms active
        dict(name="dml_f32", family="dml", J=1024, D=4096, B=512),
        # sparse coding: 20 ISTA iterations, 10 power iterations, update, row projection
        dict(name="sc_f32", family="sc", J=4096, D=1024, B=512, ista=20, power=10),
        # sparse coding with a small dictionary and a mini-batch of a hundred: many short contractions
        dict(name="sc_f32_small", family="sc", J=1000, D=300, B=100, ista=20, power=10),
        # stochastic dual coordinate ascent at the size of mlr_f32_peers
        dict(name="sdca_f32_peers", family="sdca", J=1000, D=2048, B=256, P=8),
        # bf16 factors, W a plain fp32 array with nothing attached: the path without any preparation
        dict(name="mlr_bf16_plain", family="mlr_bf16", J=8192, D=4096, B=256, P=1, layout="plain"),
        # bf16 factors of eight workers on the fp32 array with its bf16 working copy
        dict(name="mlr_bf16_peers", family="mlr_bf16", J=65000, D=10000, B=256, P=8, layout="copy"),
        # the large model on the two planes: mini-batch of a hundred, and of 1024
        dict(name="mlr_bf16_large_b100", family="mlr_bf16", J=325000, D=10000, B=100, P=1, layout="planes"),
        dict(name="mlr_bf16_large", family="mlr_bf16", J=325000, D=10000, B=1024, P=1, layout="planes"),
        # the large model on samples stored as CSR rows, half a per cent of non-zeros
        dict(name="mlr_csr_large", family="mlr_csr", J=325000, D=10000, B=1024, nonzero=0.005, layout="planes"),
    ]


def draw(rng):
    def log(lo, hi, step=1):
        return max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step)

    def size(lo, hi):      # as they come (often odd), or a multiple of eight
        return log(lo, hi, 8 if rng.random() < 0.4 else 1)

    family = rng.choice(["mlr_f32", "dml", "sc", "sdca", "mlr_bf16", "mlr_csr"])
    if family == "mlr_f32":
        return dict(family=family, J=size(16, 4000), D=size(50, 8192), B=size(16, 512), P=rng.randint(1, 8))
    if family == "dml":
        return dict(family=family, J=size(32, 1024), D=size(64, 4096), B=size(32, 512))
    if family == "sc":
        return dict(family=family, J=size(128, 4096), D=size(64, 1024), B=size(32, 512), ista=20, power=10)
    if family == "sdca":
        return dict(family=family, J=size(16, 2000), D=size(50, 4096), B=size(16, 512), P=rng.randint(1, 8))
    layout = rng.choice(["plain", "copy", "planes"])
    J, D, B = log(1000, 325000, 8), log(512, 10000, 8), size(16, 1024)
    if family == "mlr_csr":
        return dict(family=family, J=J, D=D, B=B, nonzero=round(math.exp(rng.uniform(math.log(0.002), math.log(0.1))), 4), layout=layout)
    # (no more work in all than the largest listed case: with peers, fewer classes)
    P = rng.choice([1, 1, 2, 4, 8])
    return dict(family=family, J=max(1000, J // P // 8 * 8), D=D, B=B, P=P, layout=layout)


def prepare(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    f, J, D, B = case["family"], case["J"], case["D"], case["B"]
    N = B * case.get("P", 1)
    bf16 = f in ("mlr_bf16", "mlr_csr")
    dtype = torch.bfloat16 if bf16 else torch.float32

    def normal(*shape, sigma=1.0):
        return torch.randn(shape, generator=g, device=DEV).mul_(sigma)

    def labels(n):
        return torch.randint(0, J, (n,), generator=g, device=DEV, dtype=torch.int32)

    s = {"case": case, "ctx": sfb.Context(0)}
    if f == "sc":
        s["W"] = normal(J, D)
        s["W"] /= s["W"].norm(dim=1, keepdim=True)
        s["X"], s["U"], s["V"] = normal(B, D), torch.zeros(B, J, device=DEV), torch.zeros(B, D, device=DEV)
        return s
    if f == "dml":         # half similar (close) pairs; W such that about half of the dissimilar ones are within the margin
        s["W"] = normal(J, D, sigma=(2 * J * D) ** -0.5)
        s["X"], s["Y"] = normal(B, D), normal(B, D)
        h = B // 2
        s["Y"][:h] = s["X"][:h] + 0.1 * s["Y"][:h]
        s["sim"] = torch.ones(B, dtype=torch.int8, device=DEV)
        s["sim"][h:] = -1
        s["U"], s["V"] = torch.zeros(B, J, device=DEV), torch.zeros(B, D, device=DEV)
        s["n_active"] = torch.zeros(1, dtype=torch.int32, device=DEV)
        return s
    s["W"] = normal(J, D, sigma=0.01)
    s["U"] = torch.zeros(N, J, dtype=dtype, device=DEV)
    # N > B: the peers' blocks, below the worker's own: softmax of N(0,1) logits minus one-hot, and N(0,1)
    for i in range(B, N, B):
        block = torch.softmax(normal(B, J), dim=1)
        block[torch.arange(B, device=DEV), labels(B).long()] -= 1.0
        s["U"][i:i + B] = block.to(dtype)
    if f == "sdca":
        s["V"] = normal(N, D)
        y = labels(B)
        s["P"] = torch.softmax(normal(B, J, sigma=2.0), dim=1)      # after some epochs; a quarter still at the start
        start = torch.rand(B, generator=g, device=DEV) < 0.25
        s["P"][start] = 0.0
        s["P"][start, y[start].long()] = 1.0
        s["lam"] = 1e-3
        s["Z"] = s["W"] * s["lam"]
        return s
    steps = SPLIT_STEPS if case.get("layout") == "planes" else 1
    s["batches"] = []
    for _ in range(steps):
        X = normal(B, D)
        if bf16:           # tf-idf-like: nine tenths zeros stored dense, or the stored entries of a CSR matrix
            X *= torch.rand(B, D, generator=g, device=DEV) < case.get("nonzero", 0.1)
        X = X.to(dtype)
        if f == "mlr_csr":
            at = X.nonzero()
            indptr = torch.zeros(B + 1, dtype=torch.int64, device=DEV)
            indptr[1:] = torch.bincount(at[:, 0], minlength=B).cumsum(0)
            X = (indptr, at[:, 1].to(torch.int32), X[at[:, 0], at[:, 1]].contiguous())
        s["batches"].append((X, labels(B)))
    if N > B:
        s["V"] = torch.zeros(N, D, dtype=dtype, device=DEV)
        s["V"][B:] = normal(N - B, D).to(dtype)
    if case.get("layout") == "copy":
        s["ctx"].sfb_shadow_attach(s["W"])
    elif case.get("layout") == "planes":
        s["ctx"].sfb_split_attach(s["W"])
    return s


def run(s):
    case, ctx, W, U = s["case"], s["ctx"], s["W"], s["U"]
    f, B = case["family"], case["B"]
    if f == "sc":
        ctx.sfb_compute_sf(sfb.SFB_SC, W, s["X"], U=U, V=s["V"], lam=0.1, ista_iters=case["ista"], power_iters=case["power"])
        ctx.sfb_apply(W, U, s["V"], -0.01)
        ctx.sfb_prox_rows(W, sfb.SFB_PROX_NORMALIZE)
        return W, U, s["V"]
    if f == "dml":
        ctx.sfb_compute_sf(sfb.SFB_DML, W, s["X"], Y=s["Y"], sim=s["sim"], U=U, V=s["V"], n_active=s["n_active"])
        ctx.sfb_apply(W, U, s["V"], 1e-4)
        return W, U, s["V"], s["n_active"]
    if f == "sdca":
        n_total = 100000
        ctx.sfb_sdca_mlr_sf(W, s["V"][:B], s["P"], s["lam"], n_total, 0.125, U[:B])
        ctx.sfb_apply(s["Z"], U, s["V"], 1.0 / n_total)
        ctx.sfb_dual_to_primal_l2(s["Z"], W, s["lam"])
        return W, s["Z"], U[:B], s["P"]
    for X, y in s["batches"]:
        if f == "mlr_csr":
            ctx.sfb_mlr_sf_csr(W, *X, y, U)
            ctx.sfb_apply_csr(W, U, *X, 0.01)
        elif case["P"] > 1:
            ctx.sfb_compute_sf(sfb.SFB_MLR, W, X, Y=y, U=U[:B], V=s["V"][:B])
            ctx.sfb_apply(W, U, s["V"], 0.01)
        else:
            ctx.sfb_compute_sf(sfb.SFB_MLR, W, X, Y=y, U=U)
            ctx.sfb_apply(W, U, X, 0.01)
    if case.get("layout") == "planes":
        ctx.sfb_split_export(W)
    return W, U[:B]


def work(case):
    """W read and written once a step, samples and peers' factors read once, the worker's factors written once; the
    contractions' products and sums (over the stored entries where the samples are CSR rows: forward only, the update
    of W is dense)."""
    f, J, D, B = case["family"], case["J"], case["D"], case["B"]
    N = B * case.get("P", 1)
    e = 2 if f in ("mlr_bf16", "mlr_csr") else 4
    if f == "sc":
        return {"bytes": 8 * J * D + 4 * (2 * B * D + B * J), "flops": 2.0 * B * J * D * (2 * case["ista"] + 1) + 4.0 * J * D * case["power"]}
    if f == "dml":
        return {"bytes": 8 * J * D + 4 * (3 * B * D + B * J), "flops": 4.0 * B * J * D}
    if f == "sdca":
        return {"bytes": 16 * J * D + 4 * (N * D + N * J + 2 * B * J), "flops": 2.0 * (B + N) * J * D}
    steps = SPLIT_STEPS if case.get("layout") == "planes" else 1
    samples, forward = B * D * e, 2.0 * B * J * D
    if f == "mlr_csr":
        samples, forward = case["nonzero"] * B * D * (e + 4) + 8 * B, forward * case["nonzero"]
    peers = (N - B) * (J + D) * e
    return {"bytes": steps * (8 * J * D + samples + B * J * e + peers), "flops": steps * (forward + 2.0 * N * J * D)}


def tolerance(case):
    """About four times the difference of a pass from the same pass computed in 64 bits (fp32 models: 2-norm 3e-6 at
    most, the sparse-coding residual; single values 2e-5).  bf16: factors differ by single roundings (2-norm 5e-7
    where no label's entry, next to -1, is among them; one such entry is worth ten times that), a value by one bf16
    spacing at most."""
    if case["family"] in ("mlr_bf16", "mlr_csr"):
        return {"rel": 5e-5, "max": 1e-2}
    return {"rel": 1.2e-5, "max": 1e-4}
