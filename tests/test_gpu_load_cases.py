"""Load vectors of several cases at once: case counts around the eight that a
pass takes, with and without body forces, every column against the oracle.

Tolerance: a node's load is a sum of at most a few hundred products, each
rounded a few times: 1e-13 of the load's norm (the bar of the single-case
assembly tests)."""
import numpy as np
import pytest

import meshgen as mg
from tests.gpu_util import dev, say, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("degree", [1, 2])
@pytest.mark.parametrize("nrhs", [1, 2, 7, 8, 9, 17])
@pytest.mark.parametrize("force", [False, True])
def test_load_cases_match_oracle(degree, nrhs, force):
    import dataclasses
    import paper_1804_10060_amd as te
    from oracle import fem
    torch = torch_cuda()
    prob = mg.disc_problem(3, 11, 2, degree, seed=1)
    m = prob.mesh
    rng = np.random.default_rng(nrhs)
    T = 300 + rng.uniform(-50, 250, (nrhs, m.n_nodes))
    f = rng.normal(size=(nrhs, m.n_nodes, 3)) * 1e9 if force else None
    say("load cases", degree, nrhs, force, m.n_nodes)
    b = te.assemble_load(dev(m.coords, torch.float64), dev(m.cells.astype(np.int32)), degree, prob.E, prob.nu,
                         prob.alpha, prob.T_ref, dev(T, torch.float64), f=None if f is None else dev(f, torch.float64),
                         mask=dev(prob.mask)).cpu().numpy()
    for j in range(nrhs):
        pj = dataclasses.replace(prob, T=T[j], f=None if f is None else f[j])
        ref = fem.assemble_problem(pj)[1].reshape(-1, 3)
        assert np.linalg.norm(b[:, :, j] - ref) <= 1e-13 * np.linalg.norm(ref), j
