"""Partial sums and split dot products at the edges of their work split: fewer
parts than rows of threads, outputs that end inside a work group, more
orbitals than the split product's partials have room for.

Tolerance 1e-11 of the largest entry: FP64 sums of at most n^3 npair terms of
mixed sign in another order than the oracle's; the repository's FP64 bar is
1e-10."""
import numpy as np
import pytest

from oracle import tairef as T
from paper_2210_13069_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,norb", [(4, 40), (4, 70), (5, 33), (7, 1), (9, 65), (16, 64), (17, 12), (33, 3)])
def test_orbital_dots(tai, n, norb):
    import torch
    b = I.small_random(n, natoms=2, shells=("s", "p"), box=2.0)
    P = I.Params(omega=0.4, nq=5, n=n, L=6.0)
    Q = np.random.default_rng(norb).standard_normal((norb, b.nb))
    t, w = T.time_nodes(P.omega, P.nq)
    K = T.ktables(t, T.cheb_nodes(n, P.L)[0])
    ref = T.coulomb_mo(T.moments(b.center, b.alpha, b.lxyz, P.L, n), K, w, Q)
    M = tai.moments(b, P)
    got = tai.coulomb_mo(M, b.nb, torch.as_tensor(Q, device=M.device), P).cpu().numpy()
    assert np.max(np.abs(got - ref)) <= 1e-11 * np.max(np.abs(ref))


@pytest.mark.parametrize("natoms", [1, 3, 9, 20])
@pytest.mark.parametrize("n", [3, 20, 35])
def test_pair_sum_parts(tai, natoms, n):
    """From one chunk of pairs (4 functions) to a few more than the rows of threads."""
    import torch
    b = I.small_random(natoms, natoms=natoms, shells=("s", "p"), box=3.0)
    P = I.Params(omega=0.5, nq=6, n=n, L=8.0)
    D = I.random_density(np.random.default_rng(n), b)
    t, w = T.time_nodes(P.omega, P.nq)
    K = T.ktables(t, T.cheb_nodes(n, P.L)[0])
    ref = T.J_grid(T.moments(b.center, b.alpha, b.lxyz, P.L, n), K, w, D)
    M = tai.moments(b, P)
    got = tai.apply_J(M, torch.as_tensor(D, device=M.device), P).cpu().numpy()
    assert np.max(np.abs(got - ref)) <= 1e-11 * np.max(np.abs(ref))


def test_exchange_of_many_functions(tai):
    """11600 functions: 32 threads for each of nb^2 entries in the sum over the
    slices, past 2^32.  Every entry is written, and sampled ones are the equation in
    FP64 torch."""
    import torch
    dev, f64, nb, n = torch.device("cuda"), torch.float64, 11600, 2
    rng = torch.Generator(device=dev).manual_seed(6)
    M = torch.randn((3, n, nb * (nb + 1) // 2), dtype=f64, device=dev, generator=rng)
    Q = torch.randn((1, nb), dtype=f64, device=dev, generator=rng) / np.sqrt(nb)
    P = I.Params(omega=0.5, nq=2, n=n, L=6.0)
    ctx = tai.Context(0)
    Kx = torch.full((nb, nb), float("nan"), dtype=f64, device=dev)
    ctx.exchange(M, nb, tai.make_params(P, tai.FP64), Q, 1, Kx)
    torch.cuda.synchronize()
    ctx.close()
    t, w = T.time_nodes(P.omega, P.nq)
    K = torch.as_tensor(T.ktables(t, T.cheb_nodes(n, P.L)[0]), device=dev)
    W = sum(w[k] * torch.kron(torch.kron(K[k], K[k]), K[k]) for k in range(P.nq))

    def grid(mu):
        lam = torch.arange(nb, device=dev)
        a, b = lam.clamp(max=mu), lam.clamp(min=mu)
        m = M[:, :, a * nb - a * (a - 1) // 2 + (b - a)]
        return (m[0][:, None, None] * m[1][:, None] * m[2]).reshape(n ** 3, nb) @ Q[0]

    assert bool(torch.isfinite(Kx).all()) and torch.equal(Kx, Kx.T)
    scale = float(Kx.abs().max())
    rows = (0, 1, 5800, nb - 2, nb - 1)
    X = {mu: grid(mu) for mu in rows}
    for mu in rows:
        for nu in rows:
            ref = 4.0 / np.sqrt(np.pi) * float(X[mu] @ (W @ X[nu]))
            assert abs(float(Kx[mu, nu]) - ref) <= 1e-11 * scale


@pytest.mark.parametrize("prec", ["FP32", "BF16X6"])
def test_fp32_copy_beyond_one_grid(tai, prec):
    """7730 functions at n = 48: the moments' FP32 copy is past 2^32 values.  J against
    the FP64 form, relative 2-norm to the repository's 1e-6."""
    import torch
    dev, f64, nb, n = torch.device("cuda"), torch.float64, 7730, 48
    assert 3 * n * (nb * (nb + 1) // 2) > 2 ** 32
    rng = torch.Generator(device=dev).manual_seed(7)
    M = torch.randn((3, n, nb * (nb + 1) // 2), dtype=f64, device=dev, generator=rng)
    D = torch.randn((nb, nb), dtype=f64, device=dev, generator=rng)
    P = I.Params(omega=0.5, nq=2, n=n, L=6.0)
    J = [torch.full((nb, nb), float("nan"), dtype=f64, device=dev) for _ in range(2)]
    ctx = tai.Context(0)
    for out, pr in zip(J, (tai.FP64, getattr(tai, prec))):
        ctx.apply_J(M, nb, tai.make_params(P, pr), D, out)
        torch.cuda.synchronize()
    ctx.close()
    assert float((J[1] - J[0]).norm() / J[0].norm()) <= 1e-6
