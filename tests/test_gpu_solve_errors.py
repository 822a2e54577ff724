"""A solve that breaks down inside the CG loop returns with its stream idle, also
where the next V-cycle is launched before the host has looked at the iteration:
the handle can be used at once on another stream, and its next solve there is bit
for bit that of a fresh handle.

The breakdown is forced from the data: the CG products run with the negated
matrix, so that (p, Ap) < 0 in the first iteration of a small operator (whose
V-cycles are launched ahead)."""
import numpy as np
import pytest

import meshgen as mg
from tests.gpu_util import dev, gpu_assemble, say, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,nrhs", [("fp64", 1), ("fp64", 3), ("mixed", 1)])
def test_breakdown_leaves_the_stream_idle(precision, nrhs):
    import paper_1804_10060_amd as te
    torch = torch_cuda()
    prob = mg.disc_problem(12, 48, 3, 2, seed=0)
    A, _, d = gpu_assemble(prob)
    n = prob.mesh.n_nodes
    B = np.random.default_rng(nrhs).standard_normal((n, 3, nrhs))
    B[prob.mask != 0] = 0.0
    b = dev(B.reshape(-1) if nrhs == 1 else B, torch.float64)
    opts = dict(coarse_max=150, max_nrhs=nrhs, build_fp32=1)
    h, fresh = te.AMG(A, d["coords"], d["mask"], **opts), te.AMG(A, d["coords"], d["mask"], **opts)
    neg = te.Matrix(A.row_ptr, A.col_idx, -A.val)
    torch.cuda.synchronize()
    say("breakdown", precision, nrhs, h.info()["n_dof"])
    first, second = torch.cuda.Stream(), torch.cuda.Stream()
    ref, rref = fresh.solve(b, precision=precision)
    torch.cuda.synchronize()
    for _ in range(3):
        h.set_operator(neg)
        with torch.cuda.stream(first):
            with pytest.raises(te.TeError) as e:
                h.solve(b, precision=precision)
            assert first.query()
        assert e.value.code == te._lib.TE_EINDEF and "(p,Ap)" in str(e.value)
        h.set_operator(None)
        with torch.cuda.stream(second):
            u, rep = h.solve(b, precision=precision)
        assert rep.iters == rref.iters and torch.equal(u, ref)
