"""The persistent ring kernels of B in FP64 and FP32 (TAI_RING_ASSEMBLY: for any
number of pairs) at every inner length, whole and padded, with and without per-node
degrees, node counts below, at and beyond the FP32 sums' groups of 8, pairs that end
inside a row panel and a column block; over boxes (rectangular blocks); and in
batches, recorded and replayed; and all persistent kernels with few nodes, whose work
items are longest.  Against the oracle, the tile kernels and FP64 torch.

Tolerances are the repository's bars, normwise: FP64 1e-10, FP32 1e-6; ring against
tiles 1e-13 and 1e-6 (the same terms in another order)."""
import numpy as np
import pytest

from oracle import tairef as T
from paper_2210_13069_amd import inputs as I

pytestmark = pytest.mark.gpu
TOL = {0: 1e-10, 1: 1e-6}
# (functions, n, nq): 1, 45, 136, 300, 465, 561 pairs; panels hold 128 to 512 rows
SIZES = [(1, 5, 1), (9, 8, 3), (16, 13, 8), (24, 16, 9), (33, 21, 5), (30, 24, 17), (33, 32, 7), (24, 29, 2), (30, 37, 9),
         (33, 40, 8), (24, 41, 5), (33, 48, 9), (16, 53, 8), (24, 56, 4), (30, 59, 3), (33, 64, 9)]


def _shells(nb):
    rng = np.random.default_rng(800 + nb)
    return I.Basis(center=rng.uniform(-2.5, 2.5, (nb, 3)), alpha=np.exp(rng.uniform(np.log(0.2), np.log(20.0), nb)),
                   lxyz=rng.integers(0, 2, (nb, 3)).astype(np.int32))


@pytest.fixture
def ring(monkeypatch):
    def use(on):
        if on:
            monkeypatch.setenv("TAI_RING_ASSEMBLY", "1")
        else:
            monkeypatch.delenv("TAI_RING_ASSEMBLY", raising=False)
    return use


def _away(got, ref, scale=None):
    return np.max(np.abs(got - ref)) / np.max(np.abs(ref if scale is None else scale))


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nb,n,nq", SIZES)
def test_inner_lengths_and_degrees(tai, ring, nb, n, nq, prec):
    b = _shells(nb)
    for tol in (0.0, 1e-7):
        P = I.Params(omega=0.5, nq=nq, n=n, L=7.0, degree_tol=tol)
        t, w = T.time_nodes(P.omega, nq)
        xi, _ = T.cheb_nodes(n, P.L)
        K = T.truncated_tables(t, xi, P.L, tol)[2] if tol else T.ktables(t, xi)
        ref = T.B_full(T.moments(b.center, b.alpha, b.lxyz, P.L, n), K, w)
        M = tai.moments(b, P)
        tiles = tai.assemble_B(M, P, prec=prec).cpu().numpy().astype(np.float64)
        ring(True)
        got = tai.assemble_B(M, P, prec=prec).cpu().numpy().astype(np.float64)
        ring(False)
        assert _away(got, ref) <= TOL[prec]
        assert _away(got, tiles) <= (1e-13 if prec == 0 else 1e-6)
        assert np.array_equal(got, got.T)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,nparts", [(12, 3), (24, 2), (40, 3), (48, 4)])
def test_boxes(tai, ring, n, nparts, prec):
    """Diagonal and rectangular blocks, rows of B at an odd stride; one box is the
    plain B, bit for bit."""
    import torch
    b = _shells(30)
    P = I.Params(omega=0.4, nq=9, n=n, L=0.0)
    ring(True)
    pairs, counts, boxes = tai.partition_pairs(b, 1e-16, nparts)
    M = tai.moments_partitioned(b, P, pairs, counts, boxes)
    got = tai.assemble_B_partitioned(M, counts, boxes, P, prec=prec, ldb=b.npair + 3)[:, :b.npair].cpu().numpy()
    part, bx = T.adaptive_partitions(T.pair_supports(b.center, b.alpha, 1e-16), nparts)
    pm = T.partition_moments(b.center, b.alpha, b.lxyz, part, bx, n)
    t, w = T.time_nodes(P.omega, P.nq)
    order = pairs.cpu().numpy().astype(np.int64)
    rng = np.random.default_rng(n)
    i, j = rng.integers(0, b.npair, 400), rng.integers(0, b.npair, 400)
    ref = T.B_partitioned_entries(pm, bx, t, w, n, order[i], order[j])
    assert _away(got[i, j].astype(np.float64), ref, T.B_partitioned_entries(pm, bx, t, w, n, order, order)) <= TOL[prec]
    assert np.array_equal(got, got.T)
    pairs, counts, boxes = tai.partition_pairs(b, 1e-16, 1)
    one = tai.assemble_B_partitioned(tai.moments_partitioned(b, P, pairs, counts, boxes), counts, boxes, P, prec=prec)
    Pl = I.Params(omega=0.4, nq=9, n=n, L=boxes[0])
    assert torch.equal(one, tai.assemble_B(tai.moments(b, Pl), Pl, prec=prec))


@pytest.mark.parametrize("prec", [0, 1])
def test_batch_recorded_and_switched(tai, ring, prec):
    """A batch of plain molecules and ones with degrees or compression on a side
    stream, the ring asked for in some of the replays: each replay gives the bits of
    the single calls under the same switch."""
    import torch
    mols, bufs, keep, cases = [], [], [], []
    for nb, extra in ((33, {}), (9, {"degree_tol": 1e-7}), (24, {"rank_tol": 1e-7}), (3, {})):
        b = _shells(nb)
        P = I.Params(omega=0.4, nq=9, n=27, L=8.0, **extra)
        ba = tai.BasisArrays(b)
        M = torch.empty((3, P.n, b.npair), dtype=torch.float64, device="cuda")
        B = torch.zeros((b.npair, b.npair), dtype=torch.float64 if prec == 0 else torch.float32, device="cuda")
        keep.append(ba)
        cases.append((b, P))
        bufs.append(B)
        mols.append(tai.tai_mol(ba.struct, tai.make_params(P, prec), M.data_ptr(), B.data_ptr(), b.npair))
        keep.append(M)
    s = torch.cuda.Stream()
    for on in (False, True, True, False, True):
        ring(on)
        single = [tai.assemble_B(tai.moments(b, P), P, prec=prec) for b, P in cases]
        for B in bufs:
            B.zero_()
        torch.cuda.synchronize()
        tai.context().assemble_B_batched(mols, stream=s)
        torch.cuda.synchronize()
        for B, S in zip(bufs, single):
            assert torch.equal(B, S)


@pytest.mark.parametrize("prec", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("nq", [1, 2, 3])
def test_few_nodes(tai, ring, nq, prec):
    """3003 and 5050 pairs: the longest runs of column blocks per work item."""
    import torch
    ring(True)
    for nb, n in ((77, 16), (100, 24)):
        b = _shells(nb)
        P = I.Params(omega=0.5, nq=nq, n=n, L=7.0)
        M = tai.moments(b, P)
        t, w = T.time_nodes(P.omega, nq)
        K = torch.as_tensor(T.ktables(t, T.cheb_nodes(n, P.L)[0]), device=M.device)
        ref = torch.zeros((b.npair, b.npair), dtype=torch.float64, device=M.device)
        for k in range(nq):
            ref += w[k] * (M[0].T @ (K[k] @ M[0])) * (M[1].T @ (K[k] @ M[1])) * (M[2].T @ (K[k] @ M[2]))
        ref *= 2.0 / np.sqrt(np.pi)
        got = tai.assemble_B(M, P, prec=prec)
        assert float((got - ref).abs().max()) <= {0: 1e-10, 2: 3e-5}.get(prec, 1e-6) * float(ref.abs().max())
        assert torch.equal(got, got.T) or prec > 1
