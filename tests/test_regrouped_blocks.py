"""The library regroups the reflections into blocks of its own size: every block size of the caller's gives the same numbers,
bit for bit, on both sides of the line between blocks of 32 and of 64 rows."""
import numpy as np
import pytest

from helpers import assert_close, gpu_fasth
from oracle import householder as orc
from paper_2009_13977_amd import synthetic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,m,blocks", [(100, 128, 7, (1, 32, 64, 128)), (512, 128, 300, (16, 64, 128)), (1024, 384, 5, (12, 32, 96, 128)),
                                          (3072, 1280, 406, (16, 32)), (3072, 1280, 407, (32, 64, 128)), (1536, 128, 9, (32, 64)), (1540, 128, 9, (64, 128))])
def test_caller_block_size_changes_nothing(d, n, m, blocks):
    print(f"regrouped d={d} n={n} m={m} blocks={blocks}", flush=True)
    p = synthetic.householder_problem(d, n, m, seed=41000 + d + m)
    want = None
    for k in blocks:
        got = gpu_fasth(p["V"], p["X"], p["G"], k)
        if want is None:
            want = got
            for name, g, r in zip(("A", "dV", "dX"), got, orc.product_gradients(p["V"], p["X"], p["G"])):
                assert_close(g, r, name, rows=name == "dV")
        for g, w in zip(got, want):
            assert np.array_equal(g, w)
