"""The operands of B (packing, projection by the tables' mirror symmetry,
coefficient moments and per-node degrees) at both parities of n, the edges of
their tiles, and node counts that the runs of nodes do not divide: B of a small
molecule in every arithmetic against the oracle.

Tolerances are the repository's bars, normwise: FP64 1e-10, FP32, BF16X6 and
F16X3 1e-6, BF16X3 3e-5."""
import dataclasses

import numpy as np
import pytest

from oracle import tairef as T
from paper_2210_13069_amd import inputs as I

pytestmark = pytest.mark.gpu
TOL = {0: 1e-10, 1: 1e-6, 2: 3e-5, 3: 1e-6, 4: 1e-6}
SIZES = [(2, 3), (3, 16), (7, 5), (8, 1), (15, 7), (16, 16), (17, 13), (24, 24), (25, 9), (31, 2), (32, 24), (33, 11),
         (40, 32), (41, 17), (47, 12), (48, 16), (49, 6), (63, 5), (64, 8)]


def _case(n, nq, kind):
    b = I.small_random(500 + n, natoms=3, shells=("s", "p", "d"), box=2.5, alpha_lo=0.2, alpha_hi=20.0)
    P = I.Params(omega=0.5, nq=nq, n=n, L=7.0, nodes=kind)
    t, w = T.time_nodes(P.omega, nq)
    xi, _ = T.cheb_nodes(n, P.L, kind)
    return b, P, t, w, xi, T.moments(b.center, b.alpha, b.lxyz, P.L, n, kind=kind)


@pytest.mark.parametrize("prec", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("n,nq", SIZES)
def test_operands(tai, n, nq, prec):
    b, P, t, w, xi, Mr = _case(n, nq, (n + nq) % 2)
    ref = T.B_full(Mr, T.ktables(t, xi), w)
    got = tai.assemble_B(tai.moments(b, P), P, prec=prec).cpu().numpy()
    assert np.max(np.abs(got - ref)) <= TOL[prec] * np.max(np.abs(ref))


@pytest.mark.parametrize("prec", [0, 1, 4])
@pytest.mark.parametrize("n,nq", [s for s in SIZES if s[0] > 3])
def test_operands_with_degrees(tai, n, nq, prec):
    """Coefficient form (FP64, FP32) and truncated tables (F16X3)."""
    b, P, t, w, xi, Mr = _case(n, nq, 0)
    P = dataclasses.replace(P, degree_tol=1e-7)
    N, _, Kt = T.truncated_tables(t, xi, P.L, P.degree_tol)
    nk, _ = tai.degrees(P)
    assert np.array_equal(nk.cpu().numpy(), N)
    ref = T.B_full(Mr, Kt, w)
    got = tai.assemble_B(tai.moments(b, P), P, prec=prec).cpu().numpy()
    assert np.max(np.abs(got - ref)) <= TOL[prec] * np.max(np.abs(ref))


@pytest.mark.parametrize("prec", [0, 1, 4])
def test_operands_mixed_batch(tai, prec):
    """A batch that mixes the node form, per-node degrees and compression
    gives each molecule what a call of its own gives."""
    import torch
    mols, bufs, keep, single = [], [], [], []
    for i, extra in enumerate([{}, {"degree_tol": 1e-7}, {"rank_tol": 1e-7}, {}]):
        b = I.small_random(600 + i, natoms=2 + i, shells=("s", "p"), box=3.0)
        P = I.Params(omega=0.4, nq=11, n=27, L=8.0, **extra)
        ba = tai.BasisArrays(b)
        M = torch.empty((3, P.n, b.npair), dtype=torch.float64, device="cuda")
        B = torch.empty((b.npair, b.npair), dtype=torch.float64 if prec == 0 else torch.float32, device="cuda")
        keep.append(ba)
        bufs.append((M, B))
        mols.append(tai.tai_mol(ba.struct, tai.make_params(P, prec), M.data_ptr(), B.data_ptr(), b.npair))
        single.append(tai.assemble_B(tai.moments(b, P), P, prec=prec))
    tai.context().assemble_B_batched(mols)
    for (_, B), S in zip(bufs, single):
        if prec in (0, 1):
            assert torch.equal(B, S)
        else:
            assert float((B - S).abs().max()) <= TOL[prec] * float(S.abs().max())
