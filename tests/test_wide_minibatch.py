"""The kernels for wide mini-batches that run fp32 products as three-piece bf16 products (chain_trio_kernel, dv_trio_kernel):
the edges of their tiles, parts and ranges, against the fp64 oracle."""
import numpy as np
import pytest

from helpers import assert_close, gpu_fasth, gpu_svd_layer, gpu_svd_rect, gpu_svd_sym
from oracle import householder as orc
from paper_2009_13977_amd import synthetic

pytestmark = pytest.mark.gpu

SHAPES = [
    (256, 65, 1025, 13), (130, 96, 4097, 32),                        # 256 elements per workgroup, 16 and 32 columns
    (512, 65, 2049, 5), (257, 70, 4100, 10),                         # 512 elements per workgroup
    (513, 65, 1025, 65), (1021, 100, 2048, 50), (1024, 128, 2049, 128),  # two parts, 16 and 32 columns
    (1025, 65, 1030, 5), (2047, 66, 1056, 33),                       # three and four parts
    (1023, 65, 4097, 13), (1500, 70, 2561, 7), (2048, 128, 4096, 64),  # 1024 elements per workgroup, one and two parts
    (1030, 65, 4200, 13),                                            # no team fits: fp32 matrix cores
    (1024, 900, 449, 100), (1000, 1000, 1000, 50), (4094, 200, 500, 8), (4100, 64, 1600, 64), (700, 640, 1024, 128),  # dV alone
]


@pytest.mark.parametrize("transpose", [False, True])
@pytest.mark.parametrize("d,n,m,k", SHAPES)
def test_wide_minibatch(d, n, m, k, transpose):
    from paper_2009_13977_amd import binding as B
    print(f"wide d={d} n={n} m={m} k={k} transpose={transpose}", flush=True)
    p = synthetic.householder_problem(d, n, m, seed=31000 + d + n + m + k)
    A, dV, dX = gpu_fasth(p["V"], p["X"], p["G"], k, transpose)
    assert B.fasth_wait_status() == B.FASTH_OK
    A0, dV0, dX0 = orc.product_gradients(p["V"], p["X"], p["G"], transpose=transpose)
    assert_close(A, A0, "A")
    assert_close(dX, dX0, "dX")
    assert_close(dV, dV0, "dV", rows=True)


@pytest.mark.parametrize("d,n,m,k", [(250, 250, 7000, 10), (700, 700, 1100, 20), (1030, 90, 2050, 9)])
def test_wide_layers(d, n, m, k):
    """Diagonal steps in the load, the gradient of sigma beside the chain, two products per launch, accumulated dV."""
    print(f"wide layers d={d} n={n} m={m} k={k}", flush=True)
    p = synthetic.svd_layer_problem(d, n, m, seed=32000 + d)
    for inverse in (False, True):
        got = gpu_svd_layer(p["Uv"], p["sigma"], p["Vv"], p["X"], p["G"], k, inverse)
        fn = orc.svd_layer_inverse_gradients if inverse else orc.svd_layer_gradients
        for name, g, r in zip(("Y", "dUv", "dsigma", "dVv", "dX"), got, fn(p["Uv"], p["sigma"], p["Vv"], p["X"], p["G"])):
            assert_close(g, r, name, rows=name in ("dUv", "dVv"))
    sigma = np.random.default_rng(d).uniform(-0.8, 0.9, d).astype(np.float32)
    got = gpu_svd_sym(p["Uv"], sigma, p["X"], p["G"], k, "exp")
    for name, g, r in zip(("Y", "dUv", "dsigma", "dX"), got, orc.symmetric_gradients(p["Uv"], sigma, p["X"], p["G"], "exp")):
        assert_close(g, r, name, rows=name == "dUv")
    q = synthetic.rect_layer_problem(d, d // 2 + 1, n, k * 2, m, seed=33000 + d)
    got = gpu_svd_rect(q["Uv"], q["sigma"], q["Vv"], q["X"], q["G"], k)
    for name, g, r in zip(("Y", "dUv", "dsigma", "dVv", "dX"), got, orc.rectangular_gradients(q["Uv"], q["sigma"], q["Vv"], q["X"], q["G"])):
        assert_close(g, r, name, rows=name in ("dUv", "dVv"))


def test_wide_magnitudes():
    """Columns of very different size, among them the largest and smallest normal numbers that the products leave finite: each
    column of A is as exact, against its own norm, as the others (pieces of an operand neither overflow nor vanish)."""
    d, n, m, k = 600, 128, 1040, 32
    p = synthetic.householder_problem(d, n, m, seed=34000)
    scale = 10.0 ** np.linspace(-35, 35, m)
    X = (p["X"] * scale).astype(np.float32)
    A, _, _ = gpu_fasth(p["V"], X, p["G"], k, False)
    A0, _, _ = orc.product_gradients(p["V"], X.astype(np.float64), p["G"])
    err = np.linalg.norm((A - A0) / scale, axis=0) / np.linalg.norm(A0 / scale, axis=0)
    # operand pieces below 2^-126 keep their place, results do not: 1e-35 is 2^10 above the smallest normal number
    assert err.max() <= 1e-4, (err.argmax(), err.max())


@pytest.mark.parametrize("d,n,m,k", [(250, 128, 1100, 32), (600, 130, 1040, 13), (1024, 1024, 2048, 32)])
def test_wide_static_forward(d, n, m, k):
    """The entry point that allocates nothing: with the operands in its array, and (the last shape) without room for them."""
    import torch
    from helpers import to_gpu
    from paper_2009_13977_amd import binding as B
    print(f"wide static d={d} n={n} m={m} k={k}", flush=True)
    p = synthetic.householder_problem(d, n, m, seed=35000 + d)
    V, X = to_gpu(p["V"]), to_gpu(p["X"])
    A = torch.full_like(X, float("nan"))
    for _ in range(2):
        B.fasth_forward_static(V, X, A, k)
        torch.cuda.synchronize()
        assert B.fasth_wait_status() == B.FASTH_OK
        assert_close(A.cpu().numpy(), orc.product_apply(p["V"], p["X"]), "A")
