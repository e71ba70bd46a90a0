"""Performance cases of the library's products.

Every case goes through the tensor entry points of paper_2608_10803_amd
(`matmul_tensors`, `addmm_tensors`, `grouped_mm_tensors`, `bmm_tensors`) with
the shape's plan looked up by the call itself, as a program with dynamic
shapes runs them, into output buffers it keeps.

A case is one of four kinds:
  mm    C = A B (epi "bias": + bias), operands row-major ("rr") or transposed
        views ("rc": B column-major, as a layer's N x K weights are; "cr": A
        column-major, as the left operand of a weight gradient; "cc": both)
  bwd   the two products of a linear layer's backward pass: dX = dY W^T and
        dW = X^T dY
  moe   one grouped product over the experts of a mixture-of-experts layer
        (rows sorted by expert, counts on the device)
  bmm   a strided batch of equal products
"""
import math

import numpy as np
import torch

import paper_2608_10803_amd as ac

# no drawn case does more than the largest listed ones
MAX_FLOPS = 1.1e12
MAX_BYTES = 1.2e9


def _mm(name, M, N, K, dtype="bf16", out="16", layout="rr", epi="none"):
    return {"name": name, "kind": "mm", "M": M, "N": N, "K": K, "dtype": dtype, "out": out, "layout": layout,
            "epi": epi}


def listed():
    return [
        # the smallest calls: over half of a dynamic-shape stream takes less than a microsecond of work
        _mm("tiny", 57, 96, 130),
        # a small square product with fp32 output
        _mm("cube_512", 512, 512, 512, out="32"),
        # decode: a batch of 16 sequences through an up-projection
        _mm("decode_up", 16, 14336, 4096),
        # decode: four sequences through a down-projection whose weights are stored N x K, with its bias (fp16)
        _mm("decode_linear", 4, 4096, 14336, dtype="f16", layout="rc", epi="bias"),
        # prefill: a layer's weights as stored (N x K)
        _mm("prefill_linear", 2048, 14336, 4096, layout="rc"),
        # a large compute-bound product
        _mm("square_8k", 8192, 8192, 8192),
        # a skewed compute-bound product with an odd inner dimension
        _mm("skewed_odd_k", 12288, 688, 16991),
        # a write-bound product with odd sizes: tall operands, small inner dimension
        _mm("write_bound", 28921, 20011, 59),
        # small output, very long inner dimension, fp32 output
        _mm("long_k", 128, 256, 131072, out="32"),
        # the backward pass of a linear layer (4096 tokens)
        {"name": "linear_backward", "kind": "bwd", "M": 4096, "N": 1536, "K": 4096, "dtype": "bf16"},
        # the up-projection of a mixture-of-experts layer: 8192 routed rows over 64 experts of unequal load
        {"name": "moe_up", "kind": "moe", "rows": 8192, "groups": 64, "N": 1536, "K": 4096, "dtype": "bf16"},
        # a batch of middle-sized products with ragged rows
        {"name": "batched", "kind": "bmm", "batch": 128, "M": 300, "N": 320, "K": 192, "dtype": "bf16", "out": "16"},
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_once(rng):
    kind = rng.choice(["sweep", "sweep", "sweep", "decode", "linear", "linear", "long_k", "bwd", "moe", "bmm"])
    grain = rng.choice([1, 8, 64])  # odd sizes and those of laid-out layers

    def dim(lo, hi):
        return max(lo, _log(rng, lo, hi) // grain * grain)

    dtype = rng.choice(["bf16", "bf16", "f16"])
    out = rng.choice(["16", "16", "32"])
    epi = rng.choice(["none", "none", "bias"])
    if kind == "sweep":  # any dynamic shape
        c = _mm("", _log(rng, 1, 100000), _log(rng, 1, 100000), _log(rng, 1, 100000), dtype, out)
    elif kind == "decode":
        c = _mm("", _log(rng, 1, 64), dim(1024, 16384), dim(1024, 16384), dtype, "16", rng.choice(["rr", "rc"]), epi)
    elif kind == "linear":
        c = _mm("", _log(rng, 64, 8192), dim(512, 16384), dim(512, 16384), dtype, out, rng.choice(["rr", "rc"]), epi)
    elif kind == "long_k":
        c = _mm("", dim(16, 512), dim(16, 512), dim(8192, 262144), dtype, "32")
    elif kind == "bwd":
        c = {"kind": "bwd", "M": _log(rng, 64, 8192), "N": dim(512, 8192), "K": dim(512, 8192), "dtype": dtype}
    elif kind == "moe":
        c = {"kind": "moe", "rows": _log(rng, 64, 8192), "groups": _log(rng, 4, 64), "N": dim(256, 4096),
             "K": dim(256, 4096), "dtype": dtype}
    else:
        c = {"kind": "bmm", "batch": _log(rng, 8, 512), "M": dim(16, 1024), "N": dim(16, 1024), "K": dim(16, 512),
             "dtype": dtype, "out": out}
    c.pop("name", None)
    return c


def draw(rng):
    while True:
        c = _draw_once(rng)
        w = work(c)
        if w["flops"] <= MAX_FLOPS and w["bytes"] <= MAX_BYTES:
            return c


_DT = {"bf16": torch.bfloat16, "f16": torch.float16}


def _values(g, rows, cols, scale, dt):
    return torch.empty(rows, cols, device="cuda", dtype=torch.float32).normal_(0.0, scale, generator=g).to(dt)


def _operand(g, rows, cols, scale, dt, col):
    """rows x cols; col: a transposed view of a cols x rows tensor."""
    return _values(g, cols, rows, scale, dt).t() if col else _values(g, rows, cols, scale, dt)


def _counts(rows, groups, seed):
    """Rows of every expert: a bounded Zipf(1.2) load over the experts, in an
    order of its own for every seed."""
    r = np.random.default_rng(seed)
    p = np.arange(1, groups + 1, dtype=np.float64) ** -1.2
    return r.multinomial(rows, r.permutation(p / p.sum()))


def prepare(case, seed):
    """Activations of unit variance, weights of variance 1 / K, and the
    output buffers."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = _DT[case["dtype"]]
    s = {"kind": case["kind"]}
    if case["kind"] == "mm":
        M, N, K = case["M"], case["N"], case["K"]
        s["A"] = _operand(g, M, K, 1.0, dt, case["layout"][0] == "c")
        s["B"] = _operand(g, K, N, K ** -0.5, dt, case["layout"][1] == "c")
        s["C"] = torch.empty(M, N, device="cuda", dtype=torch.float32 if case["out"] == "32" else dt)
        s["bias"] = _values(g, 1, N, 0.1, torch.float32).view(N) if case["epi"] == "bias" else None
    elif case["kind"] == "bwd":
        M, N, K = case["M"], case["N"], case["K"]
        s["X"] = _values(g, M, K, 1.0, dt)
        s["W"] = _values(g, K, N, K ** -0.5, dt)
        s["dY"] = _values(g, M, N, M ** -0.5, dt)
        s["dX"] = torch.empty(M, K, device="cuda", dtype=dt)
        s["dW"] = torch.empty(K, N, device="cuda", dtype=torch.float32)
    elif case["kind"] == "moe":
        rows, groups, N, K = case["rows"], case["groups"], case["N"], case["K"]
        s["counts"] = torch.from_numpy(_counts(rows, groups, seed).astype(np.int32)).cuda()
        s["A"] = _values(g, rows, K, 1.0, dt)
        s["B"] = _values(g, groups * K, N, K ** -0.5, dt).view(groups, K, N)
        s["C"] = torch.empty(rows, N, device="cuda", dtype=dt)
    else:
        b, M, N, K = case["batch"], case["M"], case["N"], case["K"]
        s["A"] = _values(g, b * M, K, 1.0, dt).view(b, M, K)
        s["B"] = _values(g, b * K, N, K ** -0.5, dt).view(b, K, N)
        s["C"] = torch.empty(b, M, N, device="cuda", dtype=torch.float32 if case["out"] == "32" else dt)
    return s


def run(s):
    if s["kind"] == "mm":
        if s["bias"] is not None:
            return ac.addmm_tensors(s["A"], s["B"], s["C"], bias=s["bias"])
        return ac.matmul_tensors(s["A"], s["B"], s["C"])
    if s["kind"] == "bwd":
        ac.matmul_tensors(s["dY"], s["W"].t(), s["dX"])
        ac.matmul_tensors(s["X"].t(), s["dY"], s["dW"])
        return s["dX"], s["dW"]
    if s["kind"] == "moe":
        return ac.grouped_mm_tensors(s["A"], s["B"], s["counts"], s["C"])
    return ac.bmm_tensors(s["A"], s["B"], s["C"])


def work(case):
    if case["kind"] == "mm":
        M, N, K = case["M"], case["N"], case["K"]
        cb = 4 if case["out"] == "32" else 2
        return {"bytes": 2 * M * K + 2 * K * N + cb * M * N + (4 * N if case["epi"] == "bias" else 0),
                "flops": 2 * M * N * K}
    if case["kind"] == "bwd":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 2 * (M * N + K * N + M * K) + 2 * M * K + 4 * K * N, "flops": 4 * M * N * K}
    if case["kind"] == "moe":
        rows, groups, N, K = case["rows"], case["groups"], case["N"], case["K"]
        return {"bytes": 2 * rows * K + 2 * min(rows, groups) * K * N + 2 * rows * N, "flops": 2 * rows * N * K}
    b, M, N, K = case["batch"], case["M"], case["N"], case["K"]
    cb = 4 if case["out"] == "32" else 2
    return {"bytes": b * (2 * M * K + 2 * K * N + cb * M * N), "flops": 2 * b * M * N * K}


def tolerance(case):
    """One rounding to the output type of sums accumulated in 32 bits: about
    1.7e-3 (bf16) and 2e-4 (fp16) from the exact result in the 2-norm, each
    value within one unit in its last place; 32-bit outputs 1e-6."""
    if case["kind"] == "bwd" or case.get("out", "16") == "16":
        return {"rel": 5e-3, "max": 1.6e-2} if case["dtype"] == "bf16" else {"rel": 8e-4, "max": 4e-3}
    return {"rel": 1e-5, "max": 1e-4}


def exact(case, seed):
    """The products in 64 bits."""
    s = prepare(case, seed)
    if case["kind"] == "mm":
        c = s["A"].double() @ s["B"].double()
        return c if s["bias"] is None else c + s["bias"].double()
    if case["kind"] == "bwd":
        dy = s["dY"].double()
        return dy @ s["W"].double().t(), s["X"].double().t() @ dy
    if case["kind"] == "moe":
        c = torch.zeros(s["C"].shape, dtype=torch.float64, device="cuda")
        at = 0
        for e, n in enumerate(s["counts"].tolist()):
            if n:
                c[at:at + n] = s["A"][at:at + n].double() @ s["B"][e].double()
            at += n
        return c
    return torch.bmm(s["A"].double(), s["B"].double())
