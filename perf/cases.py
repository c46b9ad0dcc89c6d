"""Timed cases of the FastH library: what a program that uses it has it do, over the range it is used in.

Every case goes through the public entry points of `paper_2009_13977_amd.binding` with inputs, outputs and the
workspace resident in GPU memory, as a training or serving loop keeps them. A case is a dict:

  op         "train"    fasth_forward + fasth_backward (one gradient step's work of an orthogonal layer)
             "apply"    fasth_apply on factors prepared once (recurrent use, inference)
             "svd"      svd_layer_apply + svd_layer_apply_backward (W X and all gradients)
             "inverse"  svd_layer_inverse_apply + its backward (W^-1 X and all gradients)
             "sym"      svd_sym_apply + its backward, one of the symmetric forms ("function")
             "rect"     svd_rect_apply + its backward (W of `rows` x `d`)
  d, n, m, k vector length, reflections, mini-batch columns, block size
  transpose  H^T X instead of H X ("train" and "apply")

The arithmetic is fp32 throughout: the library has no other data type.
"""
import math

import torch

from paper_2009_13977_amd import binding as B

_BLOCKS = (16, 20, 24, 25, 28, 32, 32, 32, 48, 50, 64, 64, 96, 100, 128)
_FUNCTIONS = ("identity", "exp", "cayley")


def _case(name, op, d, m, k, n=None, transpose=False, function="", rows=0, n_u=0):
    case = {"op": op, "d": d, "n": d if n is None else n, "m": m, "k": k, "transpose": transpose,
            "function": function, "rows": rows, "n_u": n_u}
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # The paper's timing experiment (m = 32, square V, k = 32) from its smallest size to its largest. The smallest
        # is a latency test: two calls, a handful of launches.
        _case("train_d64_m32", "train", 64, 32, 32),
        _case("train_d256_m32", "train", 256, 32, 32),
        # The headline size.
        _case("train_d1024_m32", "train", 1024, 32, 32),
        _case("train_d3072_m32", "train", 3072, 32, 32),
        # A layer on 28 x 28 images (the paper's example for the block-size search, k = sqrt(d)): no power of two anywhere.
        _case("train_d784_m100_k28", "train", 784, 100, 28),
        # The large benchmark size.
        _case("train_d2048_m64_k64", "train", 2048, 64, 64),
        # Ordinary to large mini-batches of the same layer, up to one orthogonal 1 x 1 convolution over m h w positions.
        _case("train_d1024_m256", "train", 1024, 256, 32),
        _case("train_d1024_m1024", "train", 1024, 1024, 32),
        _case("train_d1024_m4096", "train", 1024, 4096, 32),
        # The SVD-reparameterised layer of the benchmark.
        _case("svd_d1024_m32", "svd", 1024, 32, 32),
        # A rectangular layer (a narrowing one), sizes and mini-batch off every tile.
        _case("rect_500x1000_m200_k50", "rect", 1000, 200, 50, rows=500, n_u=500),
        # A recurrent step: factors prepared once for the sequence, then one product per time step.
        _case("apply_d512_m16", "apply", 512, 16, 32),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _length(rng):
    """A vector length in [64, 3072]: a third are multiples of 64, a third of 4, a third anything."""
    d = _log_uniform(rng, 64, 3072)
    kind = rng.randrange(3)
    return max(64, d // 64 * 64) if kind == 0 else max(64, d // 4 * 4) if kind == 1 else d


def _count(rng, d, k):
    """Reflections: as many as the block size allows up to d, now and then half of them."""
    full = max(1, d // k)
    return k * (max(1, full // 2) if rng.random() < 0.2 else full)


def draw(rng):
    limit = max(work(c)["flops"] for c in listed())
    while True:
        op = rng.choice(("train", "train", "train", "train", "apply", "apply", "svd", "inverse", "sym", "rect"))
        d = _length(rng)
        k = rng.choice([b for b in _BLOCKS if b <= d])
        m = _log_uniform(rng, 1 if op == "apply" else 8, 4096)
        n = _count(rng, d, k)
        rows = n_u = 0
        if op == "rect":
            rows = _length(rng)
            if rows < k:
                continue
            n_u = _count(rng, rows, k)
        case = _case(None, op, d, m, k, n=n, transpose=op in ("train", "apply") and rng.random() < 0.3,
                     function=rng.choice(_FUNCTIONS) if op == "sym" else "", rows=rows, n_u=n_u)
        # apply alone is a third of a step; bound its columns the same way
        if work(case)["flops"] <= limit and d * n * m <= 1024 * 1024 * 4096:
            return case


class _Inputs:
    """Seeded normal and uniform arrays in GPU memory (the paper's experiment draws X, G and V from N(0, 1))."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.gen, device="cuda", dtype=torch.float32)

    def uniform(self, lo, hi, size):
        return torch.rand(size, generator=self.gen, device="cuda", dtype=torch.float32) * (hi - lo) + lo


def prepare(case, seed):
    op, d, n, m, k = case["op"], case["d"], case["n"], case["m"], case["k"]
    r = _Inputs(seed)
    s = {"op": op, "k": k, "transpose": case["transpose"], "function": case["function"]}
    if op in ("train", "apply"):
        s["V"], s["X"] = r.normal(n, d), r.normal(d, m)
        s["A"] = torch.empty_like(s["X"])
        s["ws"] = B.new_workspace(B.fasth_workspace_bytes(d, n, m, k))
        if op == "train":
            s["G"] = r.normal(d, m)
            s["dV"], s["dX"] = torch.empty_like(s["V"]), torch.empty_like(s["X"])
        else:
            B.fasth_prepare(s["V"], m, s["ws"], k)
    elif op in ("svd", "inverse"):
        s["Uv"], s["Vv"], s["sigma"] = r.normal(n, d), r.normal(n, d), r.uniform(0.5, 2.0, d)
        s["X"], s["G"] = r.normal(d, m), r.normal(d, m)
        for out, like in (("Y", "X"), ("dX", "X"), ("dUv", "Uv"), ("dVv", "Vv"), ("dsigma", "sigma")):
            s[out] = torch.empty_like(s[like])
        s["ws"] = B.new_workspace(B.svd_layer_workspace_bytes(d, n, m, k))
    elif op == "sym":
        s["Uv"], s["sigma"] = r.normal(n, d), r.uniform(-0.8, 0.9, d)
        s["X"], s["G"] = r.normal(d, m), r.normal(d, m)
        for out, like in (("Y", "X"), ("dX", "X"), ("dUv", "Uv"), ("dsigma", "sigma")):
            s[out] = torch.empty_like(s[like])
        s["ws"] = B.new_workspace(B.svd_layer_workspace_bytes(d, n, m, k))
    else:
        rows, n_u = case["rows"], case["n_u"]
        s["Uv"], s["Vv"], s["sigma"] = r.normal(n_u, rows), r.normal(n, d), r.uniform(0.5, 2.0, min(rows, d))
        s["X"], s["G"] = r.normal(d, m), r.normal(rows, m)
        for out, like in (("Y", "G"), ("dX", "X"), ("dUv", "Uv"), ("dVv", "Vv"), ("dsigma", "sigma")):
            s[out] = torch.empty_like(s[like])
        s["ws"] = B.new_workspace(B.svd_rect_workspace_bytes(rows, d, n_u, n, m, k))
    return s


def run(s):
    op, k, ws = s["op"], s["k"], s["ws"]
    if op == "train":
        B.fasth_forward(s["V"], s["X"], s["A"], ws, k, s["transpose"])
        B.fasth_backward(s["V"], s["G"], s["dV"], s["dX"], ws, k, s["transpose"])
        return s["A"], s["dV"], s["dX"]
    if op == "apply":
        B.fasth_apply(s["V"], s["X"], s["A"], ws, k, s["transpose"], False)
        return s["A"]
    if op == "sym":
        B.svd_sym_apply(s["Uv"], s["sigma"], s["X"], s["Y"], ws, k, s["function"])
        B.svd_sym_apply_backward(s["Uv"], s["sigma"], s["G"], s["dUv"], s["dsigma"], s["dX"], ws, k, s["function"])
        return s["Y"], s["dUv"], s["dsigma"], s["dX"]
    forward, backward = {
        "svd": (B.svd_layer_apply, B.svd_layer_apply_backward),
        "inverse": (B.svd_layer_inverse_apply, B.svd_layer_inverse_apply_backward),
        "rect": (B.svd_rect_apply, B.svd_rect_apply_backward),
    }[op]
    forward(s["Uv"], s["sigma"], s["Vv"], s["X"], s["Y"], ws, k)
    backward(s["Uv"], s["sigma"], s["Vv"], s["G"], s["dUv"], s["dsigma"], s["dVv"], s["dX"], ws, k)
    return s["Y"], s["dUv"], s["dsigma"], s["dVv"], s["dX"]


def work(case):
    """Floating-point operations of the one-reflection-at-a-time definition (an inner product and an update per
    reflection and column forward, the same on the gradient, two updates per vector gradient), and every input
    read and every output written once."""
    op, d, n, m = case["op"], case["d"], case["n"], case["m"]
    if op == "apply":
        return {"bytes": 4 * (n * d + 2 * d * m), "flops": 4 * d * n * m}
    if op == "train":
        return {"bytes": 4 * (2 * n * d + 4 * d * m), "flops": 12 * d * n * m}
    if op in ("svd", "inverse"):
        return {"bytes": 4 * (4 * n * d + 4 * d * m + 2 * d), "flops": 24 * d * n * m}
    if op == "sym":
        return {"bytes": 4 * (2 * n * d + 4 * d * m + 2 * d), "flops": 24 * d * n * m}
    rows, n_u = case["rows"], case["n_u"]
    return {"bytes": 4 * (2 * n_u * rows + 2 * n * d + 2 * (rows + d) * m + 2 * min(rows, d)),
            "flops": 12 * (d * n + rows * n_u) * m}


def tolerance(case):
    """Against the definition evaluated in fp64 (one reflection at a time), outputs of the listed cases and of drawn
    ones are off by 2e-7 to 1.5e-6 (2-norm) and by at most 1.2e-5 of the root mean square in a single entry: about
    four times that."""
    return {"rel": 6e-6, "max": 5e-5}
