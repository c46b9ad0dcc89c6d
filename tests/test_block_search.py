"""The block-size search runs every different grouping once: candidates that lead to the same blocks are one, and the first of
them is the answer, whatever the timing noise."""
import pytest

from helpers import to_gpu
from paper_2009_13977_amd import binding as B
from paper_2009_13977_amd import synthetic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,m,candidates,groupings", [
    (784, 784, 32, [112, 56, 28, 98], 1), (784, 784, 32, [28, 98, 112, 56], 1),
    (1024, 128, 32, [128, 64, 16, 32, 8], 2),      # blocks of 16 rows for k < 32
    (5000, 48, 4, [16, 24, 48], 3),                # long vectors keep the caller's blocks
])
def test_each_grouping_once(d, n, m, candidates, groupings):
    import torch
    print(f"search d={d} n={n} m={m} {candidates}", flush=True)
    p = synthetic.householder_problem(d, n, m, seed=95000 + d)
    V, X, G = (to_gpu(p[a]) for a in ("V", "X", "G"))
    A, dV, dX = torch.empty_like(X), torch.empty_like(V), torch.empty_like(X)
    ws = B.new_workspace(max(B.fasth_workspace_bytes(d, n, m, k) for k in candidates))
    B.fasth_profile_enable(True)
    try:
        k, ms = B.fasth_tune_block_size(V, X, G, A, dV, dX, ws, candidates=candidates, repetitions=2)
        launches = B.fasth_profile_collect()["chain_kernel"][1]
    finally:
        B.fasth_profile_enable(False)
    assert launches == groupings * 2 * (1 + 2)  # two chains per pass, one untimed and two timed passes
    assert ms > 0
    if groupings == 1:
        assert k == candidates[0]
    else:
        assert k in ((128, 16) if d == 1024 else candidates)
