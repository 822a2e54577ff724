"""The hybrid Gauss-Seidel sweep where the number of row blocks is not a
multiple of the eight blocks a wave takes: the spare groups of the last wave
hold no rows and must read no row pointers."""
import numpy as np
import pytest
import scipy.sparse as sp

from tests.gpu_util import dev, say, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [129, 1024, 1025, 5520])
@pytest.mark.parametrize("block", [16, 128])
def test_sweep_with_spare_block_groups(n, block):
    from oracle import camg
    from paper_1804_10060_amd import _lib, heat
    torch = torch_cuda()
    rng = np.random.default_rng(n + block)
    off = [1, 7, 60]
    A = sp.diags([-rng.uniform(0.5, 1.0, n - k) for k in off], off, shape=(n, n))
    A = (A + A.T + sp.diags(np.full(n, 7.0))).tocsr()
    A.sort_indices()
    say("sweep blocks", n, block)
    M = heat.CsrMatrix(dev(A.indptr.astype(np.int64)), dev(A.indices.astype(np.int32)), dev(A.data, torch.float64))
    h = heat.CAMG(M, coarse_max=60, block=block)
    lev = camg.setup(A, camg.CAMGOptions(coarse_max=60, block=block))
    assert h.info()["n_levels"] == len(lev) >= 2
    for l in range(len(lev) - 1):
        m = lev[l].A.shape[0]
        g, x0 = rng.standard_normal(m), rng.standard_normal(m)
        for op, fwd in ((_lib.TE_CAMG_SWEEP_FWD, True), (_lib.TE_CAMG_SWEEP_BWD, False)):
            y = h.apply(l, op, dev(g, torch.float64), dev(x0, torch.float64)).cpu().numpy()
            ref = camg.hybrid_gs(lev[l], g, x0, block, forward=fwd)
            # up to 6 terms a row and a chain of at most `block` rows, contracting: far below 1e-12
            assert np.linalg.norm(y - ref) <= 1e-12 * np.linalg.norm(ref), (l, op)
