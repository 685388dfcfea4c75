"""A solution that is not finite is never reported as converged: the backward
error of an overflowed or NaN solution is NaN."""
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


def served(tc, pts, B, mode="continuous"):
    import torch
    with tc.Server(torch.empty(256 << 20, dtype=torch.uint8, device="cuda"), 16 << 20, mode) as srv:
        st, X, eta, _, _ = srv.wait(srv.submit(pts, B, 0.2, 1e-2, 1e-12))
    print(f"n={len(pts)} nrhs={B.shape[1]} {mode}: status {st} eta {eta}")
    return st, X, eta


@pytest.mark.parametrize("mode", ["continuous", "fifo"])
def test_server_overflowed_solution(tc, mode):
    """Two coincident points, A = [[1.01, 1], [1, 1.01]], and b of 1.7e308:
    x overflows, b - A x is NaN in both rows, and the residual's wave holds
    two rows past the matrix beside them."""
    st, X, eta = served(tc, np.zeros((2, 2)), np.array([[1.7e308], [-1.7e308]]), mode)
    assert not np.isfinite(X).any()
    assert st == tc.CHOL_NOT_CONVERGED and np.isnan(eta)


@pytest.mark.parametrize("n,nrhs", [(1, 1), (3, 2), (65, 1), (65, 8), (200, 3)])
def test_server_nan_right_hand_side(tc, n, nrhs):
    """One or three rows leave rows past the matrix in the residual's only wave."""
    rng = np.random.default_rng(n)
    B = rng.standard_normal((n, nrhs))
    B[n // 2, nrhs - 1] = np.nan
    st, X, eta = served(tc, rng.random((n, 2)), B)
    assert np.isnan(X[:, nrhs - 1]).any()
    assert st == tc.CHOL_NOT_CONVERGED and np.isnan(eta)


@pytest.mark.parametrize("method", ["ir", "pcg"])
@pytest.mark.parametrize("n", [1, 65, 300])
def test_refine_nan_column(tc, method, n):
    """One NaN column: its backward error is NaN and the call not converged;
    the other columns meet the tolerance."""
    import torch
    from paper_2606_11937_amd import inputs
    A = torch.from_numpy(inputs.gg_plus_identity(n, seed=n)).cuda()
    L = A.clone()
    assert tc.chol_factor_mixed(L, 128, "fp32") == 0
    B = torch.from_numpy(np.random.default_rng(n).standard_normal((n, 3))).cuda()
    B[n // 2, 1] = float("nan")
    X = torch.zeros_like(B)
    ok, it, eta = tc.chol_solve_refine(A, L, B, X, 128, method, 1e-12, 5)
    print(f"{method} n={n}: converged {ok} after {it}, eta {eta}")
    assert not ok and np.isnan(eta[1])
    assert eta[0] <= 1e-12 and eta[2] <= 1e-12


def test_refined_batch_nan_right_hand_side(tc):
    """The matrices with a NaN in b report a NaN backward error, the others
    meet the tolerance."""
    import torch
    from paper_2606_11937_amd import inputs
    ns = [1, 3, 64, 65, 200, 300]
    As = [torch.from_numpy(inputs.gg_plus_identity(n, seed=n)).cuda() for n in ns]
    Ls = [torch.empty_like(a) for a in As]
    Bs = [torch.from_numpy(np.random.default_rng(n).standard_normal(n)).cuda() for n in ns]
    for k in (0, 1, 3, 5):
        Bs[k][ns[k] // 2] = float("nan")
    Xs = [torch.empty_like(b) for b in Bs]
    infos, its, etas = tc.chol_factor_solve_batched_mixed(As, Ls, Bs, Xs, precs=["fp64", "fp32"] * 3)
    print(f"infos {infos} corrections {its} etas {etas}")
    assert infos == [0] * len(ns)
    for k, e in enumerate(etas):
        assert np.isnan(e) if k in (0, 1, 3, 5) else e <= 1e-12
