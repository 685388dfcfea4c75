"""The pivot's root and reciprocal in the fast form of the diagonal blocks:
the bits of sqrt(d) and of 1 / sqrt(d) as IEEE division by that root, for
pivots over two octaves, for exact squares, one unit in the last place beside
them, and over the form's range of exponents.  Factors of block diagonal
matrices of [[d, a], [a, 4]] with a power of two a <= sqrt(d) hold both: L_00
is the root and L_10 / a, exactly, the reciprocal."""
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


def roots(tc, d):
    """(root, reciprocal) of each of the pivots d, 4096 to a factorization."""
    import torch
    n = 8192
    A = torch.zeros(n, n, dtype=torch.float64, device="cuda")
    out = []
    for i in range(0, len(d), n // 2):
        v = np.ones(n // 2)
        v[:len(d[i:i + n // 2])] = d[i:i + n // 2]
        a = np.exp2(np.floor(np.log2(v) / 2))
        A.zero_()
        A.diagonal()[0::2] = torch.from_numpy(v).cuda()
        A.diagonal()[1::2] = 4.0
        A.diagonal(-1)[0::2] = torch.from_numpy(a).cuda()
        assert tc.chol_factor(A, 128, "fork_join") == 0
        out.append(np.stack([A.diagonal()[0::2].cpu().numpy(), A.diagonal(-1)[0::2].cpu().numpy() / a]))
    return np.concatenate(out, axis=1)[:, :len(d)]


def octaves():
    return np.random.default_rng(1).uniform(1.0, 4.0, 1 << 18)


def squares():
    return np.arange(1, 60001, dtype=np.float64) ** 2


def beside_squares():
    s = np.random.default_rng(2).integers(1, 60001, 16384).astype(np.float64) ** 2
    return np.concatenate([np.nextafter(s, 0.0), np.nextafter(s, np.inf)])


def exponents():
    rng = np.random.default_rng(3)
    return rng.uniform(1.0, 4.0, 1 << 16) * 4.0 ** rng.integers(-349, 500, 1 << 16)


@pytest.mark.parametrize("pivots", [octaves, squares, beside_squares, exponents])
def test_bits_of_root_and_reciprocal(tc, pivots):
    d = pivots()
    s, r = roots(tc, d)
    want = np.sqrt(d)
    print(f"{pivots.__name__}: {len(d)} pivots, {(s != want).sum()} roots and {(r != 1.0 / want).sum()} reciprocals differ")
    assert np.array_equal(s, want)
    assert np.array_equal(r, 1.0 / want)
