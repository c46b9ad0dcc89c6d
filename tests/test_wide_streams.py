"""Wide mini-batches (chain_trio_kernel) on two streams at a time: unsaved applies may overlap on one prepared workspace and
write nothing but A."""
import pytest

from helpers import assert_close, to_gpu
from oracle import householder as orc
from paper_2009_13977_amd import synthetic

pytestmark = pytest.mark.gpu

# two parts (16 and 32 columns per tile, the launch as large as the GPU or larger), three, two parts of 1024 elements, no team
SHAPES = [(600, 128, 1040, 32), (1021, 200, 4097, 50), (1500, 130, 1100, 13), (2048, 128, 4096, 64), (512, 128, 2100, 32), (1030, 65, 4200, 13)]


def _two_streams():
    import torch
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    return streams


@pytest.mark.parametrize("transpose", [False, True])
@pytest.mark.parametrize("d,n,m,k", SHAPES)
def test_unsaved_applies_share_a_workspace(d, n, m, k, transpose):
    import torch
    from paper_2009_13977_amd import binding as B
    print(f"shared workspace d={d} n={n} m={m} k={k} transpose={transpose}", flush=True)
    p = synthetic.householder_problem(d, n, m, seed=62000 + d)
    V = to_gpu(p["V"])
    X = [to_gpu(p["X"]), to_gpu(p["G"])]
    A = [torch.full_like(x, float("nan")) for x in X]
    ws = B.new_workspace(B.fasth_workspace_bytes(d, n, m, k))
    B.fasth_prepare(V, m, ws, k)
    torch.cuda.synchronize()
    untouched = ws.clone()
    streams = _two_streams()
    for _ in range(4):
        for x, a, stream in zip(X, A, streams):
            with torch.cuda.stream(stream):
                B.fasth_apply(V, x, a, ws, k, transpose, False)
    torch.cuda.synchronize()
    assert B.fasth_wait_status() == B.FASTH_OK
    assert torch.equal(ws, untouched)  # nothing but A is written
    for a, name in zip(A, ("X", "G")):
        assert_close(a.cpu().numpy(), orc.product_apply(p["V"], p[name], transpose=transpose), name)
