"""The moment kernel's two quadrature rules and padded inner lengths, against
the oracle's composite rule (8 panels of 48 points).

Tolerance: each moment is a sum of at most 96 terms, each carrying at most
about n + 30 roundings (the recurrence, the powers and the weight), mapped to
the nodes by rows of gam whose absolute sums stay below 4: (96 + 64 + 30) * 4
* 1.1e-16 < 1e-13 of the largest moment, here with a factor of ten for the
oracle's own rounding."""
import numpy as np
import pytest

from oracle import tairef as T
from paper_2210_13069_amd import inputs as I

pytestmark = pytest.mark.gpu


def _basis(seed, nb):
    """Exponents from diffuse (the box cuts the pair) to tight (it lies inside),
    centres up to the box's edge, powers 0 .. 4."""
    rng = np.random.default_rng(seed)
    return I.Basis(rng.uniform(-7.5, 7.5, (nb, 3)), np.exp(rng.uniform(np.log(0.05), np.log(60.0), nb)),
                   rng.integers(0, 5, (nb, 3)).astype(np.int32))


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("n", [2, 3, 5, 16, 17, 24, 25, 32, 33, 40, 41, 47, 48, 49, 63, 64])
def test_moments_both_rules(n, kind):
    from paper_2210_13069_amd import tai
    b = _basis(n, 23)                      # 276 pairs: blocks of 256 items that mix the rules
    P = I.Params(0.5, 8, n, 8.0, nodes=kind)
    M = tai.moments(b, P).cpu().numpy()
    R = T.moments(b.center, b.alpha, b.lxyz, P.L, n, kind=kind)
    a, A = b.alpha, b.center
    mu, nu = T.pair_list(b.nb)
    p = a[mu] + a[nu]
    ctr = (a[mu, None] * A[mu] + a[nu, None] * A[nu]) / p[:, None]
    inside = np.abs(ctr) + 8.0 / np.sqrt(p)[:, None] <= P.L
    assert 0.1 < inside.mean() < 0.9       # both rules are in use
    assert np.max(np.abs(M - R)) <= 1e-12 * np.max(np.abs(R))


def test_moments_list_and_parts_same_bits():
    """A pair's moments do not depend on the pairs beside it."""
    import torch
    from paper_2210_13069_amd import tai
    b = _basis(3, 41)
    P = I.Params(0.5, 8, 37, 8.0)
    M = tai.moments(b, P)
    rng = np.random.default_rng(0)
    sel = rng.permutation(b.npair)[:517].astype(np.int32)
    pairs = torch.as_tensor(sel, device="cuda")
    assert torch.equal(tai.moments_pairs(b, P, pairs), M[:, :, pairs.long()])
    bad = pairs.clone()
    bad[::7] = b.npair + 5                 # entries outside the list: zero moments
    Mb = tai.moments_pairs(b, P, bad)
    assert torch.count_nonzero(Mb[:, :, ::7]) == 0
    assert torch.equal(Mb[:, :, 1::7], M[:, :, pairs.long()][:, :, 1::7])
    counts = [300, 0, 217]
    blocks = tai.moments_partitioned(b, P, pairs, counts, [8.0, 8.0, 8.0])
    n = P.n
    assert torch.equal(blocks[:3 * n * 300].view(3, n, 300), M[:, :, pairs[:300].long()])
    assert torch.equal(blocks[3 * n * 300:].view(3, n, 217), M[:, :, pairs[300:].long()])
