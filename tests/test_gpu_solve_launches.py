"""The solve sweeps at the edges of their launches: few blocks (no block, one
or two in front of the neighbour), ragged last blocks, passes of two and four
columns, launches in and around the window that takes one workgroup a CU (449
to 512 blocks on 256 CUs), more than 16 passes, and the server's launch of
many solves.  Tolerances, fixed in advance: a column's bits do not depend on
the columns beside it (every pass sums in the same order); a backward error of
at most 1e-12, the bar of the parity tests."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_11937_amd import tilechol
    return tilechol


def columns_alone(tc, L, B, X, cols):
    import torch
    for c in cols:
        x = torch.empty(len(B), 1, dtype=torch.float64, device="cuda")
        x.copy_(B[:, c:c + 1])
        tc.chol_solve(L, x, 128)
        assert torch.equal(x[:, 0], X[:, c]), c


@pytest.mark.parametrize("nrhs", [1, 2, 3, 4, 5, 66])
@pytest.mark.parametrize("n", [1, 15, 64, 65, 127, 128, 129, 191, 192, 193, 257, 700])
def test_small(tc, n, nrhs):
    import torch
    from paper_2606_11937_amd import inputs
    A = torch.from_numpy(inputs.gg_plus_identity(n, seed=n)).cuda()
    buf = torch.full((n, n + 3), float("nan"), dtype=torch.float64, device="cuda")
    L = buf[:, :n]
    L.copy_(torch.tril(A) + torch.triu(torch.full_like(A, float("nan")), 1))  # garbage above the diagonal
    assert tc.chol_factor(L, 128, "fork_join") == 0
    B = torch.from_numpy(np.random.default_rng(n).standard_normal((n, nrhs))).cuda()
    X = B.clone()
    tc.chol_solve(L, X, 128)
    columns_alone(tc, L, B, X, {0, nrhs - 1, nrhs // 2})
    eta = ((A @ X - B).abs().amax(0) / (A.abs().sum(1).max() * X.abs().amax(0) + B.abs().amax(0))).max().item()
    print(f"n={n} nrhs={nrhs}: eta {eta:.2e}")
    assert eta <= 1e-12


@pytest.mark.parametrize("n,nrhs,blocks", [(7100, 16, 444), (7180, 16, 452), (8192, 16, 512), (8200, 16, 516),
                                           (4040, 29, 512), (4100, 66, 1040)])
def test_launch_sizes(tc, n, nrhs, blocks):
    import torch
    from paper_2606_11937_amd import inputs
    per_launch = min(-(-nrhs // 4), 16)
    assert -(-n // 64) * per_launch == blocks
    A = inputs.se_kernel_device(n, 3)
    L = A.clone()
    assert tc.chol_factor(L, 128, "fork_join") == 0
    B = torch.randn(n, nrhs, generator=torch.Generator(device="cuda").manual_seed(5), dtype=torch.float64,
                    device="cuda")
    X = B.clone()
    tc.chol_solve(L, X, 128)
    columns_alone(tc, L, B, X, {0, nrhs - 1, nrhs // 2})
    R = A @ X - B
    eta = (R.abs().amax(0) / (A.abs().sum(1).max() * X.abs().amax(0) + B.abs().amax(0))).max().item()
    print(f"n={n} nrhs={nrhs}: eta {eta:.2e}")
    assert eta <= 1e-12


def test_one_column_beyond_1024_blocks(tc):
    """Order 65600 (1025 blocks, one column): a factor whose last 64 rows are
    the identity leaves the first 65536 rows the solution of the leading
    factor, bit for bit."""
    import torch
    n, m = 65600, 65536
    L = torch.zeros(n, n, dtype=torch.float64, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(1)
    for j in (1, 2, 63, 64, 130, 200, 1000, 30000):
        torch.diagonal(L, -j).copy_(0.1 * torch.rand(n - j, generator=g, dtype=torch.float64, device="cuda"))
    L[m:].zero_()
    torch.diagonal(L).copy_(1.5 + torch.rand(n, generator=g, dtype=torch.float64, device="cuda"))
    b = torch.randn(n, 1, generator=g, dtype=torch.float64, device="cuda")
    x, y = b.clone(), b[:m].clone()
    tc.chol_solve(L, x, 128)
    tc.chol_solve(L[:m, :m], y, 128)
    assert torch.equal(x[:m], y)
    r = (L @ (L.T @ x) - b).abs().max().item()
    norm = (L.abs().sum(1).max() * L.abs().sum(0).max() * x.abs().max() + b.abs().max()).item()
    print(f"eta {r / norm:.2e}")
    assert r / norm <= 1e-12


def test_many_solves_in_a_tick(tc):
    """The same request alone and 250 times over: every copy has the same bits,
    whichever the tick's number of blocks (10 a request, up to 2500)."""
    import torch
    rng = np.random.default_rng(7)
    p, B = rng.random((300, 2)), rng.standard_normal((300, 8))
    with tc.Server(torch.empty(8 << 30, dtype=torch.uint8, device="cuda"), 512 << 20, "continuous") as srv:
        st, X, eta, _, _ = srv.wait(srv.submit(p, B, 0.2, 1e-2, 1e-12))
        assert st == tc.CHOL_OK
        t0 = srv.ticks()
        ids = [srv.submit(p, B, 0.2, 1e-2, 1e-12) for _ in range(250)]
        for rid in ids:
            st, Y, e, _, _ = srv.wait(rid)
            assert st == tc.CHOL_OK and e == eta and np.array_equal(X, Y)
        print(f"{len(ids)} requests in {srv.ticks() - t0} ticks")
