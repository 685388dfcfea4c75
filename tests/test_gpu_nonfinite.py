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
