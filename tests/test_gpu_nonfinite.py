"""A solution that is not finite is never reported as converged: the backward
error of a NaN solution is NaN."""
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


@pytest.mark.parametrize("n,nrhs", [(65, 1), (65, 8), (200, 3)])
def test_server_nan_right_hand_side(tc, n, nrhs):
    rng = np.random.default_rng(n)
    B = rng.standard_normal((n, nrhs))
    B[n // 2, nrhs - 1] = np.nan
    st, X, eta = served(tc, rng.random((n, 2)), B)
    assert np.isnan(X[:, nrhs - 1]).any()
    assert st == tc.CHOL_NOT_CONVERGED and np.isnan(eta)
