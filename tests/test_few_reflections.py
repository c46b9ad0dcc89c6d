"""Where the layout changes with the number of reflections: blocks of 16 rows for few reflections in small blocks, n rounded up to
the steps of the shared-column kernels only where that pays, wide mini-batches of few steps off chain_trio_kernel. Both sides
of the lines, rows to spare and none, against the fp64 oracle."""
import pytest

from helpers import assert_close, gpu_fasth, gpu_svd_layer, gpu_svd_rect
from oracle import householder as orc
from paper_2009_13977_amd import synthetic

pytestmark = pytest.mark.gpu

SHAPES = [  # d, n, m, k
    (250, 160, 130, 16), (256, 161, 130, 7), (512, 128, 256, 16), (511, 112, 600, 8), (509, 113, 600, 1),  # blocks of 16, short columns
    (1024, 1, 32, 1), (1024, 192, 100, 16), (1021, 193, 33, 1), (777, 448, 300, 14), (784, 96, 700, 12), (1024, 48, 1000, 3),
    (2048, 16, 3, 16), (2047, 112, 64, 8), (1536, 224, 200, 16), (3072, 32, 16, 8), (3069, 250, 50, 10), (4096, 16, 8, 2), (4093, 100, 600, 5),
    (700, 8, 8, 8), (1024, 24, 800, 8), (2048, 40, 900, 8), (1400, 200, 300, 8), (61, 60, 1100, 5), (256, 128, 1280, 4),              # blocks of 8
    (3072, 72, 300, 24), (3001, 350, 64, 7), (4096, 24, 1100, 24),                                                                     # of 24
    (512, 128, 1500, 16), (500, 97, 2100, 97), (1024, 45, 1500, 9), (2048, 48, 1030, 16), (100, 48, 2050, 16), (600, 32, 2050, 16), (3000, 16, 1030, 8),  # tiles
    (1024, 160, 32, 32), (1000, 288, 64, 32), (1024, 352, 100, 32), (1024, 449, 16, 1), (2044, 192, 32, 32), (1600, 449, 8, 1),  # rounded up or not
    (500, 160, 1000, 32), (500, 200, 1000, 50), (1024, 224, 449, 32), (900, 97, 600, 97), (2048, 96, 700, 32),
    (1536, 192, 1000, 64), (1000, 224, 800, 32),                                                        # blocks of 64 from 25 MB on
    (256, 112, 1025, 14), (640, 200, 1280, 50), (640, 97, 1300, 97), (1024, 96, 2049, 32), (1536, 192, 4096, 64), (1400, 64, 1100, 32),  # no operands
    (256, 113, 1025, 1), (130, 128, 4097, 32), (512, 113, 2049, 1), (257, 120, 4100, 10),               # operands, one workgroup per tile
    (640, 161, 2049, 7), (1023, 97, 4097, 1), (1500, 195, 3000, 13), (2048, 193, 4096, 1),             # of 512 and 1024 elements, teams of each
]


# the largest shapes in one direction
CASES = [(*s, transpose) for s in SHAPES for transpose in (False, True) if not transpose or s[0] * s[1] * s[2] <= 3e8]


@pytest.mark.parametrize("d,n,m,k,transpose", CASES)
def test_number_of_reflections(d, n, m, k, transpose):
    from paper_2009_13977_amd import binding as B
    print(f"few d={d} n={n} m={m} k={k} transpose={transpose}", flush=True)
    p = synthetic.householder_problem(d, n, m, seed=81000 + d + n + m + k)
    A, dV, dX = gpu_fasth(p["V"], p["X"], p["G"], k, transpose)
    assert B.fasth_wait_status() == B.FASTH_OK
    A0, dV0, dX0 = orc.product_gradients(p["V"], p["X"], p["G"], transpose=transpose)
    assert_close(A, A0, "A")
    assert_close(dX, dX0, "dX")
    assert_close(dV, dV0, "dV", rows=True)


@pytest.mark.parametrize("d,n,m,k", [(250, 40, 300, 8), (1021, 64, 20, 16), (1500, 30, 1100, 10)])
def test_layers_of_few_reflections(d, n, m, k):
    print(f"few layers d={d} n={n} m={m} k={k}", flush=True)
    p = synthetic.svd_layer_problem(d, n, m, seed=82000 + d)
    got = gpu_svd_layer(p["Uv"], p["sigma"], p["Vv"], p["X"], p["G"], k)
    for name, g, r in zip(("Y", "dUv", "dsigma", "dVv", "dX"), got, orc.svd_layer_gradients(p["Uv"], p["sigma"], p["Vv"], p["X"], p["G"])):
        assert_close(g, r, name, rows=name in ("dUv", "dVv"))
    # one side in blocks of 16, the other of 32
    q = synthetic.rect_layer_problem(d, 200, n, 176 // k * k, m, seed=83000 + d)
    got = gpu_svd_rect(q["Uv"], q["sigma"], q["Vv"], q["X"], q["G"], k)
    for name, g, r in zip(("Y", "dUv", "dsigma", "dVv", "dX"), got, orc.rectangular_gradients(q["Uv"], q["sigma"], q["Vv"], q["X"], q["G"])):
        assert_close(g, r, name, rows=name in ("dUv", "dVv"))
