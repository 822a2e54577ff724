"""A row pointer of another mesh is refused by both assembly calls before they
write the load vector."""
import ctypes as C

import numpy as np
import pytest

import meshgen as mg
from tests.gpu_util import dev, gpu_assemble, say, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("degree", [1, 2])
@pytest.mark.parametrize("tables", [False, True])
def test_load_vector_is_kept(degree, tables):
    import paper_1804_10060_amd as te
    from paper_1804_10060_amd import _lib
    torch = torch_cuda()
    prob = mg.cube_problem(3, degree)
    A, b, d = gpu_assemble(prob)
    say("refused row pointer", degree, tables)
    n, nc = prob.mesh.n_nodes, len(prob.mesh.cells)
    rp = A.row_ptr.clone()
    rp[1] -= 1                 # the first row one short, the second one long
    m = _lib.TeMesh(n, nc, degree, d["coords"].data_ptr(), d["cells"].data_ptr())
    M = _lib.TeBsr(n, A.nnzb, rp.data_ptr(), A.col_idx.data_ptr(), A.val.data_ptr())
    before = b.clone()
    with pytest.raises(te.TeError, match="row_ptr"):
        if tables:
            tab = [np.array([[200.0, 400.0]]), np.array([[1.0, 1.0]]), np.array([[0.3, 0.3]]), np.array([[1e-3, 1e-3]])]
            mt = _lib.TeMaterialTables(1, 2, *[t.ctypes.data for t in tab], 300.0)
            cm = dev(np.zeros(nc, np.int32))
            _lib.check(_lib.load().fe_assemble_thermoelastic_materials(
                C.byref(m), C.byref(mt), cm.data_ptr(), d["T"].data_ptr(), None, None, None, None, C.byref(M),
                b.data_ptr(), None))
        else:
            mat = _lib.TeMaterial(1.0, 0.3, 1e-3, 300.0)
            _lib.check(_lib.load().fe_assemble_thermoelastic(C.byref(m), C.byref(mat), d["T"].data_ptr(), None, None,
                                                           None, C.byref(M), b.data_ptr(), None))
    torch.cuda.synchronize()
    assert torch.equal(b, before)
