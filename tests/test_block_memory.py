"""A caller's large blocks bound the workspace: smaller blocks than the caller's are taken only while the saved inputs grow by at most
1 GiB. Sizes on the host, and the kernels on blocks of 128 rows that serve beyond; more reflections than a grid has rows."""
import pytest

from helpers import REL_TOL, rel_err
from paper_2009_13977_amd import binding as B

GIB = 1 << 30


@pytest.mark.parametrize("d,n,m", [(2048, 16384, 4096), (4096, 16384, 16384), (256, 1152, 65535), (512, 16512, 2048), (1024, 4096, 4096),
                                   (128, 2048, 65535), (1500, 32000, 900), (3000, 6400, 3000)])
def test_large_blocks_bound_the_workspace(d, n, m):
    saved = lambda rows: 2 * (-(-n // rows)) * m * d * 4  # the inputs that both chains save
    sizes = {k: B.fasth_workspace_bytes(d, n, m, k) for k in (16, 32, 64, 128) if n % k == 0}
    for k, size in sizes.items():
        # beside the saved inputs: coefficients, V padded and as operands (16 bytes per element and padding), factors and
        # partial Gram matrices (64 floats per row and 128 elements of it, half as much again for pairs), hand-off words, parts of dV
        rest = 8 * m * (n + 128) + 20 * (n + 128) * (d + 32) + 24 * 64 * (n + 128) * 16 + 64 * GIB // 1024 + 4 * 16 * (n + 128) * d
        assert size <= saved(k) + GIB + rest, (k, size / GIB, saved(k) / GIB)
    assert sizes[128] == min(sizes.values())


def test_small_workspaces_are_not_split():
    """Within 1 GiB the library's own blocks serve every block size alike."""
    assert B.fasth_workspace_bytes(1024, 384, 4096, 128) == B.fasth_workspace_bytes(1024, 384, 4096, 32) > 6 * 2 * 4096 * 1024 * 4


@pytest.mark.gpu
@pytest.mark.parametrize("d,n,m", [
    (256, 1152, 65535), (124, 2304, 65535),  # operands, one workgroup per tile; more Z than partial Gram matrices
    (512, 16512, 2048),                       # shared tiles
    (1300, 4608, 3000),                       # teams of 1024 elements
    (3000, 2176, 2700)])                      # a workgroup per column
def test_blocks_of_128_rows(d, n, m):
    """Against blocks of 64 (a caller's k = 64), which other tests hold against the oracle, and in fp64 on some columns."""
    import torch
    print(f"blocks of 128: d={d} n={n} m={m}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + n)
    V, X, G = (torch.randn(*shape, generator=gen, device="cuda") for shape in ((n, d), (d, m), (d, m)))
    out = {}
    for k in (128, 64):
        A, dV, dX = torch.full_like(X, float("nan")), torch.full_like(V, float("nan")), torch.full_like(X, float("nan"))
        ws = B.new_workspace(B.fasth_workspace_bytes(d, n, m, k))
        B.fasth_forward(V, X, A, ws, k)
        B.fasth_backward(V, G, dV, dX, ws, k)
        torch.cuda.synchronize()
        assert B.fasth_wait_status() == B.FASTH_OK
        if k == 128:
            Y = torch.full_like(X, float("nan"))
            B.fasth_apply(V, X, Y, ws, k, False, False)
            torch.cuda.synchronize()
            assert rel_err(Y.cpu().numpy(), A.cpu().numpy()) <= REL_TOL
        out[k] = [t.cpu().numpy() for t in (A, dV, dX)]
        del ws
    for a, b in zip(out[128], out[64]):
        assert rel_err(a, b) <= REL_TOL
    cols = [0, 1, m // 2, m - 1]
    ref = X[:, cols].double()
    W = V.double() / V.double().norm(dim=1, keepdim=True)
    for j in range(n - 1, -1, -1):
        ref -= torch.outer(2 * W[j], W[j] @ ref)
    assert rel_err(out[128][0][:, cols], ref.cpu().numpy()) <= REL_TOL


@pytest.mark.gpu
def test_more_reflections_than_a_grid_has_rows():
    """n / 32 blocks would be more than 65535. Every vector comes twice, so the product is the identity and the gradients of
    the two cancel. The two share the rounding of v^2 and of its inverse, which makes the pair's error along v one-sided: at most
    2^-24 a pair on the average, so n / 2 times that after 2.1 million reflections."""
    import torch
    d, n, m, k = 4, 2101248, 1, 128
    print(f"many reflections d={d} n={n}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    V = torch.randn(n // 2, d, generator=gen, device="cuda").repeat_interleave(2, dim=0).contiguous()
    X, G = torch.randn(d, m, generator=gen, device="cuda"), torch.randn(d, m, generator=gen, device="cuda")
    A, dV, dX = torch.empty_like(X), torch.full_like(V, float("nan")), torch.empty_like(X)
    ws = B.new_workspace(B.fasth_workspace_bytes(d, n, m, k))
    B.fasth_forward(V, X, A, ws, k)
    B.fasth_backward(V, G, dV, dX, ws, k)
    torch.cuda.synchronize()
    bound = n / 2 * 2.0 ** -24
    print(f"  A off by {float((A - X).norm() / X.norm()):.2e}, bound {bound:.2e}", flush=True)
    assert (A - X).norm() <= bound * X.norm() and (dX - G).norm() <= bound * G.norm()
    assert bool(dV.isfinite().all())
    assert (dV[0::2] + dV[1::2]).norm() <= bound * dV.norm()
