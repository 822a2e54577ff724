"""Block CG at the column counts where its kernels change their tiling (16
columns each) and at row counts that leave remainders of their 16-row steps.

Random right-hand sides against the oracle's block CG of the same matrix: the
same bars as the load-case tests (iteration counts within one, true residual,
1e-8 of the oracle's solution), which a wrong or missing term in any of the Gram
products or updates would miss, since each step's directions come from them."""
import numpy as np
import pytest

import meshgen as mg
from tests.test_gpu_block_cg import _check, _gpu_block, _oracle_block, _oracle_system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 4, 15, 16, 17, 31, 32, 33, 48, 49, 63, 64])
def test_block_widths(m):
    prob = mg.cube_problem(4, 1) if m % 2 else mg.disc_problem(5, 17, 2, 1, seed=0)
    A, _ = _oracle_system(prob, [1])
    B = np.random.default_rng(m).standard_normal((A.shape[0], m))
    B[prob.mask.reshape(-1) != 0] = 0.0
    h, U, rep = _gpu_block(prob, B, 150)
    _check(A, B, U, rep, _oracle_block(prob, A, B, 150))
