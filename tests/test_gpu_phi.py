"""The mode products by parity at every number of 4-row steps and both
parities of n, in the paths that use them: J (one tensor, node runs), J over
boxes (sources and cross tables), orbital dots and the exchange (tensors kept in
parity form), with both node kinds and with truncated tables.

Tolerance 1e-11 of the largest entry: sums of the oracle's terms in another
order, each mode's sums and differences adding one rounding."""
import numpy as np
import pytest

from oracle import tairef as T
from paper_2210_13069_amd import inputs as I

pytestmark = pytest.mark.gpu
NS = [2, 3, 4, 7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32, 33, 39, 40, 41, 47, 48, 49]


def _case(n, kind=0, nq=5):
    b = I.small_random(300 + n, natoms=3, shells=("s", "p"), box=3.0)
    P = I.Params(omega=0.6, nq=nq, n=n, L=7.0, nodes=kind)
    t, w = T.time_nodes(P.omega, nq)
    K = T.ktables(t, T.cheb_nodes(n, P.L, kind)[0])
    return b, P, K, w, T.moments(b.center, b.alpha, b.lxyz, P.L, n, kind=kind)


def _close(got, ref, tol=1e-11):
    assert np.max(np.abs(got - ref)) <= tol * np.max(np.abs(ref))


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("n", NS)
def test_phi_single_tensor(tai, n, kind):
    import torch
    b, P, K, w, Mr = _case(n, kind, nq=7)
    D = I.random_density(np.random.default_rng(n), b)
    M = tai.moments(b, P)
    _close(tai.apply_J(M, torch.as_tensor(D, device=M.device), P).cpu().numpy(), T.J_grid(Mr, K, w, D))


@pytest.mark.parametrize("n", NS)
def test_phi_many_tensors(tai, n):
    import torch
    b, P, K, w, Mr = _case(n)
    Q = np.random.default_rng(n).standard_normal((3, b.nb))
    M = tai.moments(b, P)
    Qg = torch.as_tensor(Q, device=M.device)
    _close(tai.exchange(M, b.nb, Qg, P).cpu().numpy(), T.exchange_grid(Mr, K, w, Q))
    _close(tai.coulomb_mo(M, b.nb, Qg, P).cpu().numpy(), T.coulomb_mo(Mr, K, w, Q))


@pytest.mark.parametrize("n", [3, 8, 15, 24, 29, 32, 37, 48])
def test_phi_boxes(tai, n):
    import torch
    b, P, _, w, _ = _case(n)
    D = I.random_density(np.random.default_rng(n), b)
    pairs, counts, boxes = tai.partition_pairs(b, 1e-20, 3)
    M = tai.moments_partitioned(b, P, pairs, counts, boxes)
    part, bx = T.adaptive_partitions(T.pair_supports(b.center, b.alpha, 1e-20), 3)
    pm = T.partition_moments(b.center, b.alpha, b.lxyz, part, bx, n)
    t, _ = T.time_nodes(P.omega, P.nq)
    ref = T.J_partitioned(pm, bx, t, w, n, D)
    got = tai.apply_J_partitioned(M, torch.as_tensor(D, device=M.device), pairs, counts, boxes, P).cpu().numpy()
    _close(got, ref)


@pytest.mark.parametrize("n", [9, 24, 31, 40])
def test_phi_truncated_tables(tai, n):
    import dataclasses
    import torch
    b, P, _, w, Mr = _case(n)
    P = dataclasses.replace(P, degree_tol=1e-6)
    t, _ = T.time_nodes(P.omega, P.nq)
    _, _, Kt = T.truncated_tables(t, T.cheb_nodes(n, P.L)[0], P.L, P.degree_tol)
    D = I.random_density(np.random.default_rng(n), b)
    M = tai.moments(b, P)
    _close(tai.apply_J(M, torch.as_tensor(D, device=M.device), P).cpu().numpy(), T.J_grid(Mr, Kt, w, D))


@pytest.mark.parametrize("n", [8, 9, 13, 14])
@pytest.mark.parametrize("norb", [16, 17])
def test_both_sides_of_256_tensors(tai, n, norb):
    """256 and 272 tensors: octants, and for 9 <= n <= 13 the slab products beyond 256."""
    import torch
    b = I.small_random(400 + n, natoms=4, shells=("s", "p"), box=3.0)
    assert b.nb == 16
    P = I.Params(omega=0.6, nq=5, n=n, L=7.0)
    t, w = T.time_nodes(P.omega, P.nq)
    K = T.ktables(t, T.cheb_nodes(n, P.L)[0])
    Mr = T.moments(b.center, b.alpha, b.lxyz, P.L, n)
    Q = np.random.default_rng(n).standard_normal((norb, b.nb))
    M = tai.moments(b, P)
    Qg = torch.as_tensor(Q, device=M.device)
    _close(tai.exchange(M, b.nb, Qg, P).cpu().numpy(), T.exchange_grid(Mr, K, w, Q))
    _close(tai.coulomb_mo(M, b.nb, Qg, P).cpu().numpy(), T.coulomb_mo(Mr, K, w, Q))


@pytest.mark.parametrize("prec,n,nb", [(0, 4, 4100), (1, 4, 4100), (1, 31, 140)])
def test_exchange_beyond_one_grid(tai, prec, n, nb):
    """1024 orbitals: 4.2 million tensors (n = 4: 1024 threads each in one launch),
    and X and Phi of 64 GiB at an odd n (32^3 threads per 31^3 values), both past
    2^32 threads.  Sampled entries against the equation in FP64 torch; FP32 to the
    repository's 1e-6."""
    import torch
    dev, f64 = torch.device("cuda"), torch.float64
    rng = torch.Generator(device=dev).manual_seed(5)
    npair = nb * (nb + 1) // 2
    M = torch.randn((3, n, npair), dtype=f64, device=dev, generator=rng)
    Q = torch.randn((1024, nb), dtype=f64, device=dev, generator=rng) / np.sqrt(nb)
    P = I.Params(omega=0.5, nq=2, n=n, L=6.0)
    ctx = tai.Context(0)
    Kx = torch.full((nb, nb), float("nan"), dtype=f64, device=dev)
    ctx.exchange(M, nb, tai.make_params(P, prec), Q, 1024, Kx)
    torch.cuda.synchronize()
    ctx.close()
    t, w = T.time_nodes(P.omega, P.nq)
    K = torch.as_tensor(T.ktables(t, T.cheb_nodes(n, P.L)[0]), device=dev)

    def grids(mu):
        lam = torch.arange(nb, device=dev)
        a, b = lam.clamp(max=mu), lam.clamp(min=mu)
        m = M[:, :, a * nb - a * (a - 1) // 2 + (b - a)]
        return (Q[:, None] * m[0]).reshape(1024 * n, nb) @ (m[1][:, None] * m[2]).reshape(n * n, nb).T.contiguous()

    def phi(X):
        out = torch.zeros_like(X)
        for k in range(P.nq):
            y = (X.view(-1, n) @ K[k]).view(-1, n, n).transpose(1, 2).reshape(-1, n) @ K[k]
            y = y.view(-1, n, n, n).permute(0, 2, 3, 1).reshape(-1, n) @ K[k]   # (a2, a1, a0)
            out += w[k] * y.view(-1, n, n, n).permute(0, 3, 2, 1).reshape(X.shape)
        return out

    assert bool(torch.isfinite(Kx).all()) and torch.equal(Kx, Kx.T)
    scale = float(Kx.abs().max())
    for mu in (0, nb // 2, nb - 1):
        Phi = phi(grids(mu))
        for nu in (0, 1, nb // 2, nb - 1):
            ref = 4.0 / np.sqrt(np.pi) * float((grids(nu) * Phi).sum())
            assert abs(float(Kx[mu, nu]) - ref) <= (1e-11 if prec == 0 else 1e-6) * scale
