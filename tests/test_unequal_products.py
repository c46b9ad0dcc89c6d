"""Rectangular layers whose two products are grouped differently: vectors of more than 4096 elements keep the caller's block
size, the other side's reflections are regrouped into blocks of 32 or 64. Mini-batches wide enough that dV is split
over workgroups (both sides alike), against the fp64 oracle."""
import pytest

from helpers import assert_close, gpu_svd_rect
from oracle import householder as orc
from paper_2009_13977_amd import synthetic

pytestmark = pytest.mark.gpu

SHAPES = [  # rows, cols, n_u, n_v, m, k
    (5000, 2200, 20, 40, 512, 20), (2200, 5000, 40, 20, 512, 20),  # blocks of 20 and 32 rows, three parts of the mini-batch
    (4100, 512, 20, 20, 256, 20),                                  # two parts
    (5000, 2200, 50, 50, 512, 50), (4100, 700, 96, 96, 300, 48),   # blocks of 50 or 48 and 64 or 32
]


@pytest.mark.parametrize("rows,cols,n_u,n_v,m,k", SHAPES)
def test_sides_grouped_differently(rows, cols, n_u, n_v, m, k):
    print(f"unequal rows={rows} cols={cols} n_u={n_u} n_v={n_v} m={m} k={k}", flush=True)
    p = synthetic.rect_layer_problem(rows, cols, n_u, n_v, m, seed=51000 + rows + k)
    got = gpu_svd_rect(p["Uv"], p["sigma"], p["Vv"], p["X"], p["G"], k)
    ref = orc.rectangular_gradients(p["Uv"], p["sigma"], p["Vv"], p["X"], p["G"])
    for name, g, r in zip(("Y", "dUv", "dsigma", "dVv", "dX"), got, ref):
        assert_close(g, r, name, rows=name in ("dUv", "dVv"))
