"""Sparse products of the AMG setup at the edges of their work split: rows of A
with one entry fewer and one more than the 64 that a wave takes at a time, rows
of R = P^T over several of those, pair lists refilled within a row, and rows of
the Galerkin product that fit in the LDS accumulators or do not.

Compared with the oracle's hierarchy of the same matrix.  Tolerance: a smoothed
P, an A P and a Galerkin product each sum at most ~2000 terms per entry, so two
correct orders differ by at most 3 * 2000 eps = 1.4e-12 of the sum of
magnitudes; 1e-11 of the operator's largest entry allows for their cancellation,
as in the other hierarchy tests."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import amg, fem
from tests.gpu_util import dev, oracle_bsr_to_device, say, torch_cuda

pytestmark = pytest.mark.gpu


def _spring_network(n, pairs, seed):
    """Springs of unit stiffness plus a grounded part: SPD 3x3 block operator."""
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, 3))
    i, j = pairs
    d = X[i] - X[j]
    d /= np.linalg.norm(d, axis=1)[:, None]
    k = np.einsum("ea,eb->eab", d, d) + 0.1 * np.eye(3)
    blocks = np.concatenate([-k, -np.swapaxes(k, 1, 2)])
    r, c = np.concatenate([i, j]), np.concatenate([j, i])
    diag = np.zeros((n, 3, 3))
    np.add.at(diag, i, k)
    np.add.at(diag, j, k)
    diag += 0.05 * np.eye(3)
    r, c = np.concatenate([r, np.arange(n)]), np.concatenate([c, np.arange(n)])
    data = np.concatenate([blocks, diag])
    o = np.lexsort((c, r))
    ptr = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))])
    return sp.bsr_matrix((data[o], c[o], ptr), shape=(3 * n, 3 * n)), X


def _band(n, h):
    i = np.repeat(np.arange(n), h)
    return i, (i + np.tile(np.arange(1, h + 1), n)) % n     # rows of 2 h + 1 entries


def _random(n, deg, seed):
    rng = np.random.default_rng(seed)
    e = np.concatenate([np.stack([np.arange(n), (np.arange(n) + 1) % n], 1),
                        rng.integers(0, n, (n * deg // 2, 2))])
    e = np.unique(np.sort(e[e[:, 0] != e[:, 1]], axis=1), axis=0)
    return e[:, 0], e[:, 1]


CASES = {"rows3": lambda: (400, _band(400, 1)), "rows63": lambda: (900, _band(900, 31)),
         "rows65": lambda: (900, _band(900, 32)), "rows129": lambda: (1500, _band(1500, 64)),
         "dense_coarse": lambda: (4000, _random(4000, 6, 3))}


@pytest.mark.parametrize("case", list(CASES))
def test_products_match_oracle(case):
    import paper_1804_10060_amd as te
    torch = torch_cuda()
    n, pairs = CASES[case]()
    A, X = _spring_network(n, pairs, seed=7)
    mask = np.zeros((n, 3), dtype=np.uint8)
    levels = amg.setup(A, fem.rigid_body_modes(X, mask), amg.AMGOptions(coarse_max=90, theta0=1e-3))
    assert len(levels) >= 2
    if case == "dense_coarse":   # rows beyond the 113 blocks of the LDS accumulators
        assert np.diff(levels[1].A.indptr).max() > 128
    say("products", case, [lv.A.shape[0] for lv in levels])
    hs = [te.AMG(oracle_bsr_to_device(A), dev(X, torch.float64), dev(mask), coarse_max=90, theta0=1e-3) for _ in range(2)]
    for l, lv in enumerate(levels):
        if l + 1 < len(levels):
            assert np.array_equal(hs[0].aggregates(l), lv.agg)
        rp, col, val = hs[0].level_matrix(l)
        D = sp.bsr_matrix((val, col, rp), shape=lv.A.shape).tocsr() - lv.A.tocsr()
        err = abs(D).max() if D.nnz else 0.0
        assert err <= 1e-11 * np.abs(lv.A.data).max(), (l, err)
        assert np.array_equal(val, hs[1].level_matrix(l)[2])   # and run to run the same bits


@pytest.mark.parametrize("n", [1, 21, 22, 64, 65, 130, 900])
def test_dense_coarsest_inverse(n):
    """A one-level hierarchy applies the explicit inverse: 3, 63, 66, 192, 195, 390
    and 2700 unknowns (blocks of 64 pivots, full and padded).  The residual of a
    Cholesky-like inverse is at most a few n kappa u |b|; kappa <= 1e4 here."""
    import paper_1804_10060_amd as te
    torch = torch_cuda()
    A, X = _spring_network(n, _random(n, 6, 1) if n > 4 else (np.zeros(0, int), np.zeros(0, int)), seed=2)
    mask = np.zeros((n, 3), dtype=np.uint8)
    say("dense inverse", 3 * n)
    h = te.AMG(oracle_bsr_to_device(A), dev(X, torch.float64), dev(mask), coarse_max=3000)
    assert h.info()["n_levels"] == 1
    b = np.random.default_rng(0).standard_normal(3 * n)
    x = h.apply(0, te.TE_OP_VCYCLE, dev(b, torch.float64)).cpu().numpy()
    assert np.linalg.norm(A @ x - b) <= 3 * n * 1e4 * 2.0 ** -53 * np.linalg.norm(b)


def test_dense_coarsest_inverse_rejects_indefinite():
    import paper_1804_10060_amd as te
    torch = torch_cuda()
    A, X = _spring_network(100, _random(100, 6, 1), seed=2)
    A = A.tocsr()
    A[220, 220] = -5.0   # a pivot in the last, padded block
    with pytest.raises(te.TeError):
        te.AMG(oracle_bsr_to_device(A.tobsr((3, 3))), dev(X, torch.float64), dev(np.zeros((100, 3), np.uint8)))
