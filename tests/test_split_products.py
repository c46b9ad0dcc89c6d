"""What the three-piece bf16 products (chain_trio_kernel, dv_trio_kernel) keep of fp32: no piece and none of the six products
is missing, sums of one term are as exact as fp32 products, numbers near the ends of the fp32 range, infinities and NaN."""
import numpy as np
import pytest

from helpers import gpu_fasth, to_gpu
from oracle import householder as orc
from paper_2009_13977_amd import synthetic

pytestmark = pytest.mark.gpu


def _rel(got, ref):
    return np.linalg.norm(got - ref) / np.linalg.norm(ref)


# A sixth of the products left out of one contraction (emulated in fp64, n / d and normal numbers as here): 2-norm errors of 1.9e-6
# and more of A and dX, 2.4e-6 and more of a sum such as dV's; a lost piece is two of the six. All six: 1.3e-7 to 2.8e-7
# of A and dX and up to 4.2e-7 of dV measured.
ALL_SIX = 1.2e-6


@pytest.mark.parametrize("d,n,m,transpose", [
    (256, 128, 1100, False), (512, 256, 2100, True), (800, 128, 5300, False),   # one workgroup per tile
    (780, 192, 1100, True), (1000, 160, 3000, False)])                          # teams; from the third on dv_trio_kernel but for the fourth
def test_every_product_counts(d, n, m, transpose):
    print(f"split products d={d} n={n} m={m} transpose={transpose}", flush=True)
    p = synthetic.householder_problem(d, n, m, seed=71000 + d)
    got = gpu_fasth(p["V"], p["X"], p["G"], 32, transpose)
    ref = orc.product_gradients(p["V"], p["X"], p["G"], transpose=transpose)
    for name, g, r in zip(("A", "dV", "dX"), got, ref):
        err = _rel(g, r)
        print(f"  {name} {err:.2e}", flush=True)
        assert err <= ALL_SIX, (name, err)


def test_sums_of_one_term():
    """Rows with a single non-zero: H turns the sign of n entries, each through one product b = v a, one c = T b with T = 2 / v^2 and
    one a - v c. Relative to a, the roundings of b, c, v^2 and its inverse count twice (rms 2.5e-8 each, at most 2^-24), that of the
    difference once, and twice the left-out part of each of the two products (rms 2^-27.5, at most 2^-24):
    rms 1.05e-7, largest 2^-24 (2 * 6 + 1) = 7.7e-7. With the leading piece cut off instead of rounded: rms 1.3e-7 measured.
    Entries that no row reaches stay as they are, also those beyond the largest bf16 number."""
    d, n, m = 800, 128, 1040
    rng = np.random.default_rng(72000)
    V = np.zeros((n, d), np.float32)
    V[np.arange(n), rng.permutation(d)[:n]] = (1 + rng.random(n)) * rng.choice([-1.0, 1.0], n)
    X = rng.standard_normal((d, m)).astype(np.float32)
    turned = V.any(axis=0)
    X[~turned, 5] = np.float32(3.4e38)
    X[~turned, 6] = -np.finfo(np.float32).max
    A, _, _ = gpu_fasth(V, X, X, 32, False)
    err = np.abs(A[turned] + X[turned]) / np.abs(X[turned])
    rms = np.sqrt((err.astype(np.float64) ** 2).mean())
    print(f"  largest {err.max():.2e} rms {rms:.2e}", flush=True)
    assert err.max() <= 7.7e-7 and rms <= 1.15e-7
    assert np.array_equal(A[~turned], X[~turned])


def test_columns_of_any_magnitude():
    """Away from the ends of the range every column is as exact as the others."""
    d, n, m = 800, 128, 1040
    p = synthetic.householder_problem(d, n, m, seed=73000)
    scale = 10.0 ** np.linspace(-25, 25, m)
    X = (p["X"] * scale).astype(np.float32)
    A, _, _ = gpu_fasth(p["V"], X, p["G"], 32, False)
    A0 = orc.product_apply(p["V"], X)
    err = np.linalg.norm((A - A0) / scale, axis=0) / np.linalg.norm(A0 / scale, axis=0)
    print(f"  largest {err.max():.2e}", flush=True)
    assert err.max() <= ALL_SIX


@pytest.mark.parametrize("d,n,m", [(250, 128, 1100), (800, 128, 1040), (800, 128, 5300)])
def test_bad_columns_stay_alone(d, n, m):
    """An infinity or NaN in X, or one in G, spoils its own column and no other."""
    import torch
    from paper_2009_13977_amd import binding as B
    print(f"bad columns d={d} n={n} m={m}", flush=True)
    p = synthetic.householder_problem(d, n, m, seed=74000 + d)
    V, X, G = (to_gpu(p[a]) for a in ("V", "X", "G"))
    ws = B.new_workspace(B.fasth_workspace_bytes(d, n, m, 32))

    def run(x, g):
        A, dV, dX = torch.empty_like(X), torch.empty_like(V), torch.empty_like(X)
        B.fasth_forward(V, x, A, ws, 32)
        B.fasth_backward(V, g, dV, dX, ws, 32)
        torch.cuda.synchronize()
        return A, dX

    A0, dX0 = run(X, G)
    bad = {3: float("inf"), 17: float("nan"), 18: -float("inf"), m - 1: float("nan")}
    good = torch.tensor([c for c in range(m) if c not in bad], device="cuda")
    x, g = X.clone(), G.clone()
    for c, value in bad.items():
        x[c % d, c] = value
        g[(c + 5) % d, c] = value
    A, dX = run(x, g)
    assert torch.equal(A[:, good], A0[:, good]) and torch.equal(dX[:, good], dX0[:, good])
    for c in bad:
        assert not A[:, c].isfinite().any() and not dX[:, c].isfinite().any()
