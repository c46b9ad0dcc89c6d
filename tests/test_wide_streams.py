"""Wide mini-batches (chain_trio_kernel, chain_team_tile_kernel beyond 1024 columns) on two streams at a time. Calls on workspaces of their own may overlap although the
workgroups of a team wait for each other, and so may unsaved applies on one prepared workspace, which run
without teams: every result is the one of the same call alone, bit for bit."""
import pytest

from helpers import assert_close, to_gpu
from oracle import householder as orc
from paper_2009_13977_amd import synthetic

pytestmark = pytest.mark.gpu

# two parts (16 and 32 columns per tile, the launch as large as the GPU or larger), three, two parts of 1024 elements, no team, no team;
# tiles of 16 columns shared by three workgroups
SHAPES = [(800, 128, 1040, 32), (1021, 200, 3000, 50), (1500, 130, 1100, 13), (2048, 193, 4096, 1), (512, 128, 2100, 32), (1030, 65, 4200, 13), (640, 200, 1280, 50), (1400, 64, 1100, 32)]


def _two_streams():
    import torch
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    return streams


@pytest.mark.parametrize("d,n,m,k", SHAPES)
def test_gradient_steps_on_two_streams(d, n, m, k):
    import torch
    from paper_2009_13977_amd import binding as B
    print(f"two streams d={d} n={n} m={m} k={k}", flush=True)
    jobs = []
    for s in range(2):
        p = synthetic.householder_problem(d, n, m, seed=61000 + d + s)
        V, X, G = (to_gpu(p[a]) for a in ("V", "X", "G"))
        jobs.append((V, X, G, torch.empty_like(X), torch.empty_like(V), torch.empty_like(X),
                     B.new_workspace(B.fasth_workspace_bytes(d, n, m, k))))

    def step(job):
        V, X, G, A, dV, dX, ws = job
        B.fasth_forward(V, X, A, ws, k)
        B.fasth_backward(V, G, dV, dX, ws, k)

    want = []
    for job in jobs:
        step(job)
        torch.cuda.synchronize()
        want.append([t.clone() for t in job[3:6]])
        for t in job[3:6]:
            t.fill_(float("nan"))
    assert B.fasth_wait_status() == B.FASTH_OK
    streams = _two_streams()
    for _ in range(4):
        for job, stream in zip(jobs, streams):
            with torch.cuda.stream(stream):
                step(job)
    torch.cuda.synchronize()
    assert B.fasth_wait_status() == B.FASTH_OK
    for job, w in zip(jobs, want):
        for got, ref in zip(job[3:6], w):
            assert torch.equal(got, ref)


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


def test_wait_gives_up_and_recovers():
    """The limit is forced to zero from the host, so the first unsuccessful poll of a team gives up and every kernel ends; the
    starting order and the tags are whole again for the next call."""
    import torch
    from paper_2009_13977_amd import binding as B
    d, n, m, k = 1021, 130, 1100, 13
    print(f"wide: wait limit 0, d={d} n={n} m={m} k={k}", flush=True)
    p = synthetic.householder_problem(d, n, m, seed=63000)
    V, X, G = (to_gpu(p[a]) for a in ("V", "X", "G"))
    A, dV, dX = torch.empty_like(X), torch.empty_like(V), torch.empty_like(X)
    ws = B.new_workspace(B.fasth_workspace_bytes(d, n, m, k))
    B.fasth_prepare(V, m, ws, k)
    assert B.fasth_wait_status() == B.FASTH_OK
    B.fasth_set_wait_limit(0)
    try:
        B.fasth_apply(V, X, A, ws, k, False, True)
        assert B.fasth_wait_status() == B.FASTH_ETIMEOUT
    finally:
        B.fasth_set_wait_limit(-1)
    A0, dV0, dX0 = orc.product_gradients(p["V"], p["X"], p["G"])
    for _ in range(2):
        B.fasth_apply(V, X, A, ws, k, False, True)
        B.fasth_backward(V, G, dV, dX, ws, k)
        assert B.fasth_wait_status() == B.FASTH_OK
        assert_close(A.cpu().numpy(), A0, "A")
        assert_close(dX.cpu().numpy(), dX0, "dX")
        assert_close(dV.cpu().numpy(), dV0, "dV", rows=True)


def test_captured_and_replayed():
    """The starting order is drawn from counters in the workspace that every launch puts back: replays with new inputs, with eager
    work on the same workspace in between."""
    import torch
    from paper_2009_13977_amd import binding as B
    d, n, m, k = 1500, 130, 1100, 13
    print(f"wide: graph d={d} n={n} m={m} k={k}", flush=True)
    probs = [synthetic.householder_problem(d, n, m, seed=64000 + r) for r in range(3)]
    V, X, G = (to_gpu(probs[0][a]) for a in ("V", "X", "G"))
    A, dV, dX = torch.empty_like(X), torch.empty_like(V), torch.empty_like(X)
    ws = B.new_workspace(B.fasth_workspace_bytes(d, n, m, k))

    def step():
        B.fasth_forward(V, X, A, ws, k)
        B.fasth_backward(V, G, dV, dX, ws, k)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for r in (1, 2, 1):
        for t, name in zip((V, X, G), ("V", "X", "G")):
            t.copy_(to_gpu(probs[r][name]))
        graph.replay()
        torch.cuda.synchronize()
        assert B.fasth_wait_status() == B.FASTH_OK
        replayed = [t.clone() for t in (A, dV, dX)]
        step()  # eagerly, on the same inputs and workspace
        torch.cuda.synchronize()
        for got, ref in zip(replayed, (A, dV, dX)):
            assert torch.equal(got, ref)
    A0, _, dX0 = orc.product_gradients(probs[1]["V"], probs[1]["X"], probs[1]["G"])
    assert_close(A.cpu().numpy(), A0, "A")
    assert_close(dX.cpu().numpy(), dX0, "dX")
