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
