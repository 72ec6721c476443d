"""J_p at the edges of its tiles and splits: inner lengths with and without two
a0 values per slab (n <= 16 NT - 8), odd n, from one pair to several work
groups, a0 values split and not, in every arithmetic; and adaptive boxes whose
counts leave part-filled and empty work groups.

Tolerances: FP64 1e-11 (sums in another order than the oracle's), FP32 and
BF16X6 1e-6, BF16X3 3e-5, the repository's bars, normwise."""
import numpy as np
import pytest

from oracle import tairef as T
from paper_2210_13069_amd import inputs as I

pytestmark = pytest.mark.gpu
TOL = {0: 1e-11, 1: 1e-6, 2: 3e-5, 3: 1e-6}


def _case(n, natoms, shells=("s", "p")):
    b = I.small_random(100 + n, natoms=natoms, shells=shells, box=3.0)
    P = I.Params(omega=0.5, nq=6, n=n, L=8.0)
    D = I.random_density(np.random.default_rng(n), b)
    t, w = T.time_nodes(P.omega, P.nq)
    K = T.ktables(t, T.cheb_nodes(n, P.L)[0])
    return b, P, D, K, w


@pytest.mark.parametrize("prec", [0, 1, 2, 3])
@pytest.mark.parametrize("n,natoms", [(2, 1), (7, 4), (8, 7), (9, 7), (16, 12), (17, 5), (23, 7), (24, 12), (25, 7),
                                      (32, 6), (33, 5), (39, 6), (40, 12), (41, 6), (48, 5), (49, 6), (56, 6), (64, 5)])
def test_projection_sizes(tai, n, natoms, prec):
    import torch
    b, P, D, K, w = _case(n, natoms)
    ref = T.J_grid(T.moments(b.center, b.alpha, b.lxyz, P.L, n), K, w, D)
    M = tai.moments(b, P)
    got = tai.apply_J(M, torch.as_tensor(D, device=M.device), P, prec=prec).cpu().numpy()
    assert np.max(np.abs(got - ref)) <= TOL[prec] * np.max(np.abs(ref))


@pytest.mark.parametrize("prec", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [12, 24, 32, 37, 48])
def test_projection_boxes(tai, n, prec):
    """Three boxes, the middle one empty, the others 150 and 150 pairs."""
    import torch
    b, P, D, K, w = _case(n, 6)
    pairs, counts, boxes = tai.partition_pairs(b, 1e-20, 2)
    counts3, boxes3 = [counts[0], 0, counts[1]], [boxes[0], boxes[0], boxes[1]]
    M = tai.moments_partitioned(b, P, pairs, counts3, boxes3)
    part, bx = T.adaptive_partitions(T.pair_supports(b.center, b.alpha, 1e-20), 2)
    pm = T.partition_moments(b.center, b.alpha, b.lxyz, part, bx, n)
    t, _ = T.time_nodes(P.omega, P.nq)
    ref = T.J_partitioned(pm, bx, t, w, n, D)
    got = tai.apply_J_partitioned(M, torch.as_tensor(D, device=M.device), pairs, counts3, boxes3, P,
                                  prec=prec).cpu().numpy()
    assert np.max(np.abs(got - ref)) <= TOL[prec] * np.max(np.abs(ref))
