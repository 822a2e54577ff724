"""Products of operators with too few slices or rows to fill the device, where
several waves share a slice or a row: every level's A, P and R against host
products of the same matrices, at slice counts around 64 rows (one slice, a
remainder) and with row lengths that leave some waves without entries.

Tolerance: a row of t terms differs between two summation orders by at most
t u (|A||x|)_i with u = 2^-53 and t <= 6 * 300 here: 1e-12 of the norm."""
import numpy as np
import pytest
import scipy.sparse as sp

import meshgen as mg
from tests.gpu_util import dev, gpu_assemble, say, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prob", [mg.cube_problem(3, 1), mg.cube_problem(4, 2), mg.disc_problem(7, 30, 2, 1, seed=0),
                                  mg.disc_problem(12, 48, 3, 2, seed=0)], ids=lambda p: p.name)
def test_level_products(prob):
    import paper_1804_10060_amd as te
    torch = torch_cuda()
    A, b, d = gpu_assemble(prob)
    h = te.AMG(A, d["coords"], d["mask"], coarse_max=100)
    info = h.info()
    say("split products", prob.name, info["n_dof"])
    rng = np.random.default_rng(0)
    G = []
    for l in range(info["n_levels"]):
        rp, col, val = h.level_matrix(l)
        n = info["n_dof"][l]
        G.append(sp.bsr_matrix((val, col, rp), shape=(n, n)).tocsr())
        x = rng.normal(size=n)
        ref = G[l] @ x
        for prec, tol in ((te.TE_PREC_FP64, 1e-12), (te.TE_PREC_MIXED, 1e-4)):
            y = h.apply(l, te.TE_OP_A, dev(x, torch.float64), precision=prec).cpu().numpy()
            assert np.linalg.norm(y - ref) <= tol * np.linalg.norm(ref), (l, prec)
    for l in range(info["n_levels"] - 1):   # the Galerkin identity ties P and R to the level operators
        x = rng.normal(size=info["n_dof"][l + 1])
        px = h.apply(l, te.TE_OP_P, dev(x, torch.float64), y=torch.zeros(info["n_dof"][l], dtype=torch.float64, device="cuda"))
        r = h.apply(l, te.TE_OP_R, dev(G[l] @ px.cpu().numpy(), torch.float64),
                    y=torch.zeros(info["n_dof"][l + 1], dtype=torch.float64, device="cuda")).cpu().numpy()
        ref = G[l + 1] @ x
        assert np.linalg.norm(r - ref) <= 1e-10 * np.linalg.norm(ref), l
    u, rep = h.solve(b)
    x = u.cpu().numpy()
    assert rep.converged[0] and np.linalg.norm(b.cpu().numpy() - G[0] @ x) <= 1.01e-8 * np.linalg.norm(b.cpu().numpy())
