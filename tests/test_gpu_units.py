"""Edges of the POTRF and TRSM bodies, through chol_factor.

A pivot below 2^-700 or not finite takes the plain form of the 16 x 16
diagonal factorization, every other one the fast form; ragged tiles take the
clamped loads and masked stores; a full diagonal block with an update depth
that is a multiple of 16 takes its update and POTRF in one body (T = 136 has
full blocks of a depth that is not).  Tolerances, fixed in advance:
  scaling   A 4^k has the factor 2^k L.  Nothing underflows at the scales
            used, so the two factors are factorizations of the same matrix by
            the same operations up to one rounding of a pivot's reciprocal;
            they agree within the row-scaled error of a stable factorization,
            n u kappa <= 200 * 2^-53 * 5 < 1.2e-13.
  shapes    e_row <= 1e-10 against the oracle, the bar of the parity tests.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2606_11937_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_11937_amd import tilechol
    return tilechol


def factor(tc, A, T, sched="fork_join"):
    import torch
    L = torch.from_numpy(A.copy()).cuda()
    info = tc.chol_factor(L, T, sched)
    return L.cpu().numpy(), info


@pytest.mark.parametrize("n,T", [(1, 128), (5, 128), (16, 128), (33, 128), (130, 128), (200, 64)])
@pytest.mark.parametrize("half", [-390, -351, 480])
def test_pivot_range(tc, n, T, half):
    """Pivots near 2^-780 and 2^-702 (plain form) and 2^960 (fast form)."""
    A = inputs.gg_plus_identity(n, seed=n)
    L, info = factor(tc, A, T)
    S, info_s = factor(tc, A * 2.0 ** (2 * half), T)
    assert info == info_s == 0
    d = np.abs(np.tril(S) * 2.0 ** -half - np.tril(L)) / np.sqrt(np.diag(A))[:, None]
    print(f"n={n} T={T} 2^{2 * half}: row-scaled difference {d.max():.2e}")
    assert d.max() <= 1.2e-13


@pytest.mark.parametrize("k", [0, 1, 15, 16, 31, 100, 127, 128, 129])
@pytest.mark.parametrize("value", [-1.0, 0.0, float("nan")])
def test_failing_pivot_position(tc, k, value):
    """The first failing pivot is reported wherever it lies in a 16-column
    block, with earlier blocks factored by the fast form."""
    A = np.eye(130) * 4.0
    A[k, k] = value
    for j in range(k + 1, 130):
        A[j, j] = -2.0  # later failures do not count
    for sched in ("fork_join", "async_dag"):
        _, info = factor(tc, A, 128, sched)
        assert info == k + 1


@pytest.mark.parametrize("T,n", [(1, 5), (3, 10), (15, 40), (16, 33), (17, 60), (100, 260), (127, 300), (128, 129),
                                 (128, 143), (128, 192), (128, 193), (129, 300), (136, 420), (144, 420), (256, 700)])
def test_ragged_tiles(tc, T, n):
    A = inputs.gg_plus_identity(n, seed=T)
    ref, info = oracle.potrf(A)
    assert info == 0
    for sched in ("fork_join", "async_dag"):
        L, got = factor(tc, A, T, sched)
        assert got == 0
        e = oracle.row_scaled_error(L, ref, A)
        print(f"T={T} n={n} {sched}: e_row {e:.2e}")
        assert e <= 1e-10
        assert np.array_equal(np.triu(L, 1), np.triu(A, 1))


def test_solve_forms_agree(tc):
    """A launch of more than 1024 block steps takes the sweeps' two-workgroup
    form; a column's result is the same bits as alone (the wide form), and its
    backward error meets the bar of the parity tests."""
    import torch
    n, nrhs = 4200, 64  # 66 blocks x 16 passes
    A = inputs.se_kernel_device(n, 3)
    L = A.clone()
    assert tc.chol_factor(L, 128, "fork_join") == 0
    B = torch.randn(n, nrhs, generator=torch.Generator(device="cuda").manual_seed(5), dtype=torch.float64,
                    device="cuda")
    X = B.clone()
    tc.chol_solve(L, X, 128)
    for c in (0, 3, 37, 63):
        x = B[:, c:c + 1].contiguous()
        tc.chol_solve(L, x, 128)
        assert torch.equal(x[:, 0], X[:, c])
    R = A @ X - B
    eta = (R.abs().amax(0) / (A.abs().sum(1).max() * X.abs().amax(0) + B.abs().amax(0))).max().item()
    print(f"eta {eta:.2e}")
    assert eta <= 1e-12


def test_server_residual_rows(tc):
    """The reported backward error at the edges of the residual's 16-row
    blocks and 16 column parts.  The host's residual has the kernel matrix
    with entries a few ulp apart and sums in another order: the two differ by
    at most 4 (n + 8) 2^-53, relative to the same denominator."""
    import torch
    rng = np.random.default_rng(11)
    reqs = [(rng.random((n, 2)), rng.standard_normal((n, k)))
            for n, k in ((1, 1), (2, 8), (15, 3), (16, 1), (17, 8), (31, 2), (33, 4), (65, 5), (150, 8))]
    with tc.Server(torch.empty(1 << 30, dtype=torch.uint8, device="cuda"), 256 << 20, "continuous") as srv:
        ids = [srv.submit(p, B, 0.2, 1e-2, 1e-12) for p, B in reqs]
        for rid, (p, B) in zip(ids, reqs):
            st, X, eta, _, _ = srv.wait(rid)
            assert st == tc.CHOL_OK
            d = p[:, None, :] - p[None, :, :]
            A = np.exp(-(d * d).sum(-1) / (2 * 0.2 ** 2)) + 1e-2 * np.eye(len(p))
            eh = oracle.backward_error(A, X, B)
            print(f"n={len(p)} nrhs={B.shape[1]}: reported {eta:.2e}, host {eh:.2e}")
            assert abs(eta - eh) <= 4 * (len(p) + 8) * 2.0 ** -53
