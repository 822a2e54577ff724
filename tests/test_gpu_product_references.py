"""Products of every level against references formed entry by entry, and the
columns of a multi-column solve against the solves of these columns alone.

The prolongator is read out by unit vectors (one term of its rows is not zero, so
the summation order does not matter), the restriction is its transpose.

Tolerances.  A product of rows of t terms: (t + 3) u (|A||x|)_i, entry by entry,
with u = 2^-53, or 2^-24 with x and the result rounded to float32.  One iteration
from zero is a multiple of the V-cycle of the right-hand side: some 32 products
of rows of at most 600 terms in either order, 32 * 600 * 2^-53 = 2e-12, with a
factor of 5 for the norms between them 1e-11; in float32 with rounding that adds
up like a random walk 32 * sqrt(600) * 2^-24 = 5e-5, bar 1e-4.  Four iterations
multiply that by the sensitivity of the recurrence's scalars: 1e-9."""
import numpy as np
import pytest
import scipy.sparse as sp

import meshgen as mg
from tests.gpu_util import dev, gpu_assemble, say, torch_cuda

pytestmark = pytest.mark.gpu


def _bound(M, x, u):
    return (np.diff(M.indptr) + 3) * u * (abs(M) @ np.abs(x))


@pytest.mark.parametrize("prob", [mg.cube_problem(3, 1), mg.cube_problem(4, 2), mg.disc_problem(7, 30, 2, 1, seed=0)],
                         ids=lambda p: p.name)
def test_level_products_entry_by_entry(prob):
    import paper_1804_10060_amd as te
    torch = torch_cuda()
    A, _, d = gpu_assemble(prob)
    h = te.AMG(A, d["coords"], d["mask"], coarse_max=100, build_fp32=1)
    info = h.info()
    say("products", prob.name, info["n_dof"])
    rng = np.random.default_rng(0)

    def run(l, op, x, prec, n_out):
        return h.apply(l, op, dev(x, torch.float64), y=torch.zeros(n_out, dtype=torch.float64, device="cuda"),
                       precision=prec).cpu().numpy()

    for prec, u in ((te.TE_PREC_FP64, 2.0 ** -53), (te.TE_PREC_MIXED, 2.0 ** -24)):
        for l in range(info["n_levels"]):
            n = info["n_dof"][l]
            rp, col, val = h.level_matrix(l)
            G = sp.bsr_matrix((val if prec == te.TE_PREC_FP64 else val.astype(np.float32).astype(np.float64), col, rp),
                              shape=(n, n)).tocsr()
            x = rng.normal(size=n)
            assert np.all(np.abs(run(l, te.TE_OP_A, x, prec, n) - G @ x) <= _bound(G, x, u)), ("A", l, prec)
            if l + 1 == info["n_levels"]:
                continue
            nc = info["n_dof"][l + 1]
            P = sp.csr_matrix(np.stack([run(l, te.TE_OP_P, e, prec, n) for e in np.eye(nc)], axis=1))
            x, y = rng.normal(size=nc), rng.normal(size=n)
            assert P.nnz > 0
            assert np.all(np.abs(run(l, te.TE_OP_P, x, prec, n) - P @ x) <= _bound(P, x, u)), ("P", l, prec)
            R = P.T.tocsr()
            assert np.all(np.abs(run(l, te.TE_OP_R, y, prec, nc) - R @ y) <= _bound(R, y, u)), ("R", l, prec)


@pytest.mark.parametrize("m", [2, 3, 4, 5, 8, 9, 16, 24, 33, 48, 64])
@pytest.mark.parametrize("precision,degree", [("fp64", 1), ("fp64", 2), ("mixed", 2)])
def test_columns_equal_their_own_solves(m, precision, degree):
    import paper_1804_10060_amd as te
    torch = torch_cuda()
    prob = mg.disc_problem(5, 17, 2, degree, seed=0)
    A, _, d = gpu_assemble(prob)
    n = prob.mesh.n_nodes
    h = te.AMG(A, d["coords"], d["mask"], coarse_max=150, max_nrhs=m, build_fp32=1)
    assert h.info()["n_levels"] >= 2
    B = np.random.default_rng(m).standard_normal((n, 3, m))
    B[prob.mask != 0] = 0.0
    say("columns", m, precision, degree, h.info()["n_dof"])
    for maxit, tol in ((1, 1e-11), (4, 1e-9)) if precision == "fp64" else ((1, 1e-4),):
        opts = dict(precision=precision, maxit=maxit, rtol=1e-15, allow_notconv=True)
        U = h.solve(dev(B, torch.float64), **opts)[0].cpu().numpy().reshape(3 * n, m)
        for j in range(m):
            u1 = h.solve(dev(np.ascontiguousarray(B[:, :, j].reshape(-1)), torch.float64), **opts)[0].cpu().numpy()
            assert np.linalg.norm(U[:, j] - u1) <= tol * np.linalg.norm(u1), (maxit, j)
