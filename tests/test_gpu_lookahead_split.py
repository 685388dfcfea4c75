"""The lookahead schedule where it splits a step's update over two streams
(more units than fit on the chip, tiles of more than one block), at orders
that the tiles do not divide, through the change from split to unsplit steps,
and with a pivot that fails in a split step.  FP64 against fork-join, FP32
against the batched launch: the same bits.  All precisions on a matrix whose
factor has entries 0, 1 and -1: every product and sum is a small integer, so
the factor is exact in any order of summation."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# order, tile side: ragged last tile, ragged last block, tiles of two blocks,
# of two and a half and of four
SIZES = [(4700, 256), (4993, 320), (5120, 256), (5300, 512)]


@pytest.fixture(scope="module")
def tc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_11937_amd import tilechol
    return tilechol


def steps(tc, n, T):
    """How many steps have an update of more, and of at most, a chip full of units."""
    units = [len(tc.chol_dag_forkjoin_update(n, T, J)) for J in range(-(-n // T) - 1)]
    more = sum(u > tc.chol_async_grid() for u in units)
    return more, len(units) - more


def integer_factor(n, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    L = torch.randint(-1, 2, (n, n), generator=g, device="cuda").to(torch.float64).tril_(-1)
    L.diagonal().fill_(1.0)
    return L


@pytest.mark.parametrize("n,T", SIZES)
def test_bits_of_fork_join(tc, n, T):
    import torch
    from paper_2606_11937_amd import inputs
    more, less = steps(tc, n, T)
    print(f"n={n} T={T}: {more} steps split, {less} not")
    assert more >= 2 and less >= 2
    A = inputs.se_kernel_device(n, 3)
    ref, L = A.clone(), A.clone()
    assert tc.chol_factor(ref, T, "fork_join") == 0
    for _ in range(2):
        L.copy_(A)
        assert tc.chol_factor(L, T, "fork_join_lookahead") == 0
        assert torch.equal(L, ref)


@pytest.mark.parametrize("n,T", SIZES[:2])
@pytest.mark.parametrize("k", [0, 100, 255, 300, 700, 4690])
def test_failing_pivot(tc, n, T, k):
    """In the first panel, in the column that the next panel takes, in the bulk
    of a split step, and in the last tile."""
    from paper_2606_11937_amd import inputs
    A = inputs.se_kernel_device(n, 3)
    A[k, k] = -1.0
    for j in (k + 1, k + 500):
        if j < n:
            A[j, j] = -2.0  # later failures do not count
    B = A.clone()
    assert tc.chol_factor(B, T, "fork_join") == k + 1
    assert tc.chol_factor(A, T, "fork_join_lookahead") == k + 1
    A = inputs.se_kernel_device(n, 3)  # the next call starts afresh
    assert tc.chol_factor(A, T, "fork_join_lookahead") == 0


@pytest.mark.parametrize("n,T", SIZES)
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_integer_exact(tc, n, T, prec):
    import torch
    L = integer_factor(n, T)
    A = L @ L.T
    assert A.abs().max().item() < 2 ** 24
    if prec == "fp64":
        assert tc.chol_factor(A, T, "fork_join_lookahead") == 0
    else:
        assert tc.chol_factor_mixed(A, T, prec, scale=False) == 0
    assert torch.equal(torch.tril(A), L)


@pytest.mark.parametrize("n,T", SIZES[:2])
def test_fp32_bits_of_the_batched_launch(tc, n, T):
    import torch
    from paper_2606_11937_amd import inputs
    A = inputs.se_kernel_device(n, 3)
    L = A.clone()
    assert tc.chol_factor_mixed(L, T, "fp32", scale=False) == 0
    M = torch.zeros_like(A)
    b = torch.ones(n, dtype=torch.float64, device="cuda")
    x = torch.empty_like(b)
    infos, _, etas = tc.chol_factor_solve_batched_mixed([A], [M], [b], [x], Ts=[T], precs=["fp32"])
    assert infos == [0] and etas[0] <= 1e-12
    assert torch.equal(torch.tril(L), torch.tril(M))


@pytest.mark.parametrize("prec,shift", [("fp32", 0.0), ("bf16", 0.064)])
def test_failing_pivot_low_precision(tc, prec, shift):
    from paper_2606_11937_amd import inputs
    n, T = SIZES[0]
    for k in (300, 700):
        A = inputs.se_kernel_device(n, 3)
        A[k, k] = 0.5 * A[k, k]  # positive, so the scaling passes, and too small for the rows above
        A[k, k - 1] = A[k - 1, k] = 0.999 * (A[k, k] * A[k - 1, k - 1]).sqrt() * 1.9
        assert tc.chol_factor_mixed(A, T, prec, shift=shift) == k + 1
