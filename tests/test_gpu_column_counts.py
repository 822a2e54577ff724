"""Several right-hand sides at the column counts where the products change their
lanes per row (4, 8, 16, 16 lanes of two columns, then a lane per column), on meshes whose rows do
not fill the last wave.

Every column against the solve of that column alone: the sums of a row run over
the same entries in the same order, so only the dot products differ, in their
last bits; iteration counts within one and both true residuals at the
tolerance, the bar of the multi-column tests."""
import numpy as np
import pytest
import scipy.sparse as sp

import meshgen as mg
from tests.gpu_util import dev, gpu_assemble, matrix_to_host, say, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [2, 4, 5, 7, 8, 9, 16, 17, 32, 33])
@pytest.mark.parametrize("degree", [1, 2])
def test_columns_match_single_solves(m, degree):
    import paper_1804_10060_amd as te
    torch = torch_cuda()
    prob = mg.disc_problem(5, 17, 2, degree, seed=0)
    A, _, d = gpu_assemble(prob)
    n = prob.mesh.n_nodes
    h = te.AMG(A, d["coords"], d["mask"], coarse_max=150, max_nrhs=m)
    B = np.random.default_rng(m).standard_normal((n, 3, m))
    B[prob.mask != 0] = 0.0
    say("columns", m, degree, h.info()["n_dof"])
    U, rep = h.solve(dev(B, torch.float64))
    U = U.cpu().numpy().reshape(3 * n, m)
    rp, col, val = matrix_to_host(A)
    K = sp.bsr_matrix((val, col, rp), shape=(3 * n, 3 * n)).tocsr()
    bn = np.linalg.norm(B.reshape(3 * n, m), axis=0)
    assert all(rep.converged)
    assert np.all(np.linalg.norm(B.reshape(3 * n, m) - K @ U, axis=0) <= 1.0000001e-8 * bn)
    for j in (0, m - 1):
        u1, rep1 = h.solve(dev(np.ascontiguousarray(B[:, :, j].reshape(-1)), torch.float64))
        assert abs(rep1.iters[0] - rep.iters[j]) <= 1
