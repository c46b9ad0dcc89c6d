"""Shapes that the library pads before its kernels see them: vectors whose length is no multiple of 4, numbers of
reflections around the multiples of 32, 64 and 128, block sizes the kernels are not written for. The padded rows
are zero reflections' slots whose coefficients must stay zero; nothing of the padding may reach an output."""
import numpy as np
import pytest

from helpers import REL_TOL, assert_close, gpu_fasth, gpu_svd_layer, gpu_svd_rect, gpu_svd_sym, rel_err, to_gpu
from oracle import householder as orc
from paper_2009_13977_amd import synthetic

pytestmark = pytest.mark.gpu

# per kernel family: one row short of, at and past its block; d one off a multiple of 4; fewer rows than a block
PADDED = [
    (3, 1, 1, 1), (5, 7, 2, 7), (61, 31, 33, 31), (63, 33, 3, 11), (255, 65, 5, 13), (509, 95, 300, 19),  # a workgroup per column
    (641, 63, 3, 21), (1021, 65, 3, 13), (1022, 127, 9, 127), (1023, 129, 2, 3), (2047, 191, 3, 1),          # steps of 64, 128 rows
    (3001, 65, 3, 5), (4093, 33, 2, 11), (1999, 70, 100, 10),                                              # more parts; two per column
    (769, 65, 450, 5), (300, 129, 900, 43), (1537, 33, 650, 3), (1368, 12, 1030, 12),                       # shared tiles of 16 columns
    (1001, 33, 1025, 11), (129, 100, 2000, 100), (2045, 31, 1100, 31),                                     # a workgroup per tile
]


@pytest.mark.parametrize("transpose", [False, True])
@pytest.mark.parametrize("d,n,m,k", PADDED)
def test_padded_shapes(d, n, m, k, transpose):
    from paper_2009_13977_amd import binding as B
    print(f"padded d={d} n={n} m={m} k={k} transpose={transpose}", flush=True)
    p = synthetic.householder_problem(d, n, m, seed=21000 + d + n + m + k)
    A, dV, dX = gpu_fasth(p["V"], p["X"], p["G"], k, transpose)
    assert B.fasth_wait_status() == B.FASTH_OK
    A0, dV0, dX0 = orc.product_gradients(p["V"], p["X"], p["G"], transpose=transpose)
    assert_close(A, A0, "A")
    assert_close(dX, dX0, "dX")
    assert_close(dV, dV0, "dV", rows=True)


@pytest.mark.parametrize("d,n,m,k", [(61, 33, 5, 11), (1021, 65, 4, 13), (770, 65, 450, 5)])
def test_padded_layers(d, n, m, k):
    """The layers share or split the factor launches, and the symmetric form takes both uses of U from one copy."""
    print(f"padded layers d={d} n={n} m={m} k={k}", flush=True)
    p = synthetic.svd_layer_problem(d, n, m, seed=22000 + d)
    for inverse in (False, True):
        got = gpu_svd_layer(p["Uv"], p["sigma"], p["Vv"], p["X"], p["G"], k, inverse)
        fn = orc.svd_layer_inverse_gradients if inverse else orc.svd_layer_gradients
        for name, g, r in zip(("Y", "dUv", "dsigma", "dVv", "dX"), got, fn(p["Uv"], p["sigma"], p["Vv"], p["X"], p["G"])):
            assert_close(g, r, name, rows=name in ("dUv", "dVv"))
    sigma = np.random.default_rng(d).uniform(-0.8, 0.9, d).astype(np.float32)
    got = gpu_svd_sym(p["Uv"], sigma, p["X"], p["G"], k, "cayley")
    for name, g, r in zip(("Y", "dUv", "dsigma", "dX"), got, orc.symmetric_gradients(p["Uv"], sigma, p["X"], p["G"], "cayley")):
        assert_close(g, r, name, rows=name == "dUv")
    q = synthetic.rect_layer_problem(d, d // 2 + 1, n, n, m, seed=23000 + d)
    got = gpu_svd_rect(q["Uv"], q["sigma"], q["Vv"], q["X"], q["G"], k)
    for name, g, r in zip(("Y", "dUv", "dsigma", "dVv", "dX"), got, orc.rectangular_gradients(q["Uv"], q["sigma"], q["Vv"], q["X"], q["G"])):
        assert_close(g, r, name, rows=name in ("dUv", "dVv"))


@pytest.mark.parametrize("d,n,m,k", [(1023, 7000, 3, 7), (2047, 3500, 2, 28), (3001, 2400, 2, 12), (515, 12200, 2, 20)])
def test_static_forward_without_room_for_the_padded_copy(d, n, m, k):
    """More than 24 MiB of V, so the entry point that allocates nothing runs on rows as the caller has them."""
    import torch
    from paper_2009_13977_amd import binding as B
    print(f"static without a copy d={d} n={n} m={m} k={k}", flush=True)
    p = synthetic.householder_problem(d, n, m, seed=24000 + d)
    V, X = to_gpu(p["V"]), to_gpu(p["X"])
    A = torch.full_like(X, float("nan"))
    B.fasth_forward_static(V, X, A, k)
    torch.cuda.synchronize()
    assert rel_err(A.cpu().numpy(), orc.product_apply(p["V"], p["X"])) <= REL_TOL
