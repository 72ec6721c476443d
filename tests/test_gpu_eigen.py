"""The eigenpairs behind the compression (angles one round ahead of the
rotations) at both parities of n, its smallest and largest, on moment-like arrays
with full, deficient and rank-one spectra, against numpy's SVD of the same array;
and operands written next to, over and apart from the moments.

Tolerances: the Gram matrix of the second pass carries singular values to 1e-13 of
the largest; the basis is orthonormal to n times the rounding of some 300 rotations
of a row, 1e-12."""
import numpy as np
import pytest

from paper_2210_13069_amd import inputs as I

pytestmark = pytest.mark.gpu
NPAIR = 401


def _array(n, kind):
    rng = np.random.default_rng(900 + n)
    rank = {"full": n, "half": max(1, n // 2), "one": 1}[kind]
    f = rng.standard_normal((n, rank)) @ (10.0 ** -np.linspace(0, 5, rank)[:, None] *
                                          rng.standard_normal((rank, 3 * NPAIR)))
    return np.ascontiguousarray(f.reshape(n, 3, NPAIR).transpose(1, 0, 2))


@pytest.mark.parametrize("kind", ["full", "half", "one"])
@pytest.mark.parametrize("n", [2, 3, 4, 5, 16, 17, 33, 48, 63, 64])
def test_singular_values(tai, n, kind):
    import torch
    M = _array(n, kind)
    s = np.linalg.svd(M.transpose(1, 0, 2).reshape(n, -1), compute_uv=False)
    P = I.Params(omega=0.4, nq=8, n=n, L=8.0, rank_tol=1e-9)
    rank, sigma, V = tai.compress(torch.as_tensor(M, device="cuda"), P)
    sigma, V = sigma.cpu().numpy(), V.cpu().numpy()
    assert np.all(np.diff(sigma) <= 0)
    assert np.max(np.abs(sigma - s)) <= 1e-13 * s[0]
    assert rank == int(np.sum(s > 1e-9 * s[0]))
    assert np.max(np.abs(V.T @ V - np.eye(n))) <= 1e-12
    # the kept vectors carry everything above the tolerance
    W = M.transpose(1, 0, 2).reshape(n, -1)
    assert np.linalg.norm(W - V[:, :rank] @ (V[:, :rank].T @ W), 2) <= 2e-9 * s[0]


def test_operands_over_the_moments(tai):
    """U may lie over M (the moments are then gone); apart from it, M stays."""
    import torch
    n = 24
    M = torch.as_tensor(_array(n, "full"), device="cuda")
    P = I.Params(omega=0.4, nq=8, n=n, L=8.0, rank_tol=1e-4)
    keep = M.clone()
    R, U, Kc = tai.compress_operands(M, P)
    assert torch.equal(M, keep)
    Rp = tai.padded_rank(R, n)
    flat = M.reshape(-1)
    assert tai.context().compress(M, NPAIR, P, U=flat) == R
    assert torch.equal(flat[:3 * Rp * NPAIR].view(3, Rp, NPAIR), U)


@pytest.mark.parametrize("n", [5, 33, 64])
@pytest.mark.parametrize("exponent", [-333, -260, 260, 333])
def test_scale_of_the_moments(tai, n, exponent):
    """Moments times a power of two, to 1e-100 and 1e100, give the same basis and
    rank and singular values times it, bit for bit: no step leaves the range of a
    double (the smallest product, of two values of the last singular vector, is
    1e-15 of the largest)."""
    import torch
    M = torch.as_tensor(_array(n, "full"), device="cuda")
    P = I.Params(omega=0.4, nq=8, n=n, L=8.0, rank_tol=1e-4)
    rank, sigma, V = tai.compress(M, P)
    got_rank, got_sigma, got_V = tai.compress(M * 2.0 ** exponent, P)
    assert got_rank == rank
    assert torch.equal(got_V, V)
    assert np.array_equal(np.ldexp(got_sigma.cpu().numpy(), -exponent), sigma.cpu().numpy())
