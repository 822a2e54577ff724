"""The network's matrix-core layers at the edges of their vertex tiles: fewer
vertices than a tile, a remainder of the 16-vertex tiles, and a mesh large
enough for the 32-vertex tiles with a remainder of them.

Tolerance: float32 sums of at most 320 terms through four layers against the
float64 oracle with the same float32 parameters, 1e-4 normwise per tensor (the
bar of the network's other tests)."""
import numpy as np
import pytest

import meshgen as mg
from oracle import mpnn as om
from tests.gpu_util import dev, gpu_assemble, say, torch_cuda
from tests.test_gpu_mpnn import _flatten, _unflatten

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(1,), (4, 13, 2), (40, 90, 6)])
def test_forward_and_gradients_at_tile_edges(grid):
    import paper_1804_10060_amd as te
    torch = torch_cuda()
    prob = mg.cube_problem(1, 1) if len(grid) == 1 else mg.disc_problem(*grid, 1, seed=0)
    m = prob.mesh
    say("mpnn tiles", grid, "vertices", m.n_nodes)
    rng = np.random.default_rng(5)
    A, _, d = gpu_assemble(prob)
    net = te.MPNN(A, d["coords"])
    X = net.features(dev(300 + rng.uniform(-50, 250, m.n_nodes), torch.float64), prob.T_ref, d["mask"])
    Xo = X.cpu().numpy().astype(np.float64)
    ptr, nbr = om.vertex_graph(m.cells, m.n_nodes)
    w = om.direction_weights(m.coords, ptr, nbr)
    po = _unflatten(_flatten(om.init_params(2)).astype(np.float32))
    for k in po:   # non-zero biases so both ReLU branches occur
        if k.startswith("b"):
            po[k] = (0.1 * rng.normal(size=po[k].shape)).astype(np.float32).astype(np.float64)
    P = dev(_flatten(po).astype(np.float32))
    target = (rng.normal(size=(m.n_nodes, 3)) * (1 - prob.mask)).astype(np.float32)
    gy = rng.normal(size=(m.n_nodes, 3)).astype(np.float32)
    yo, cache = om.forward(po, Xo, ptr, nbr, prob.mask, w)
    y = net.forward(P, X, d["mask"]).cpu().numpy()
    assert np.linalg.norm(y - yo) <= 1e-4 * np.linalg.norm(yo)
    g, loss = net.backward(P, dev(target))
    assert abs(loss - om.loss(yo, target.astype(np.float64))) <= 1e-5 * loss
    for got, ref in ((g, om.backward(po, Xo, ptr, nbr, w, cache, yo, target.astype(np.float64))),
                     (net.backward_from(P, dev(gy)), om.backward_from(po, Xo, ptr, nbr, w, cache, gy.astype(np.float64)))):
        gg = _unflatten(got.cpu().numpy())
        for k in om.PARAM_ORDER:
            e = np.linalg.norm(gg[k] - ref[k]) / max(np.linalg.norm(ref[k]), 1e-30)
            assert e <= 1e-4, f"{k}: {e:.2e}"
