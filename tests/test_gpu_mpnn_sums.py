"""Sums over the vertices in the network's gradients, on data whose rounding does
not cancel: every vertex contributes the same value 1 + d with d below the last
bit of a long float32 sum, so that a sum of t terms in one chain is off by about
t u (u = 2^-24).

A ring of vertices, all weights zero but a copy of the features into the channels
and of the channels into the outputs, layer biases one: h_l = h_0 + l, every gate
is open, and dL/dy reaches every layer unchanged, so each gradient is n times one
product.

Tolerance: bias gradients are added in double and rounded once (2 u).  Weight
gradients are chains of at most 32 vertices, 32 of which are added before the
rest is added in double; with the products and the sums of four waves: 72 u."""
import numpy as np
import pytest

from tests.gpu_util import dev, say, torch_cuda

pytestmark = pytest.mark.gpu

U = 2.0 ** -24
SIZES = [4111, 334368, 1500001]


def _gradients(n):
    """(gradient by name, h0 per feature channel, sum of dL/dy per channel)"""
    import paper_1804_10060_amd as te
    from oracle import mpnn as om
    from tests.test_gpu_mpnn import _flatten, _unflatten
    torch = torch_cuda()
    i = np.arange(n, dtype=np.int64)
    col = np.stack([(i - 1) % n, (i + 1) % n], 1).astype(np.int32).reshape(-1)
    x = np.zeros((n, 3))
    x[:, 0] = i / n
    A = te.Matrix(dev(2 * np.arange(n + 1, dtype=np.int64)), dev(col), torch.empty(0, dtype=torch.float64, device="cuda"))
    net = te.MPNN(A, dev(x))
    p = {k: np.zeros_like(v) for k, v in om.init_params(0).items()}
    c = np.arange(64)
    p["W_in"][c % 10, c] = 1.0
    p["W_out"][c, c % 3] = 1.0
    for l in range(om.L):
        p[f"b{l}"][:] = 1.0
    P = dev(_flatten(p).astype(np.float32))
    f = (1.0 + np.arange(10) / 16.0).astype(np.float32)
    X = dev(np.tile(f, (n, 1)))
    v = (1.0 + 2.0 ** np.array([-13.5, -14.5, -15.5])).astype(np.float32)
    net.forward(P, X, torch.zeros((n, 3), dtype=torch.uint8, device="cuda"))
    g = _unflatten(net.backward_from(P, dev(np.tile(v, (n, 1)))).cpu().numpy())
    return g, f.astype(np.float64)[c % 10], n * v.astype(np.float64)[c % 3], n * v.astype(np.float64)


def _off(got, ref):
    return float(np.max(np.abs(got - ref) / np.abs(ref)) / U)


@pytest.mark.parametrize("n", SIZES)
def test_bias_gradients_are_rounded_once(n):
    from oracle import mpnn as om
    g, h0, s, sy = _gradients(n)
    errs = {"b_out": _off(g["b_out"], sy), "b_in": _off(g["b_in"], s)}
    errs.update({f"b{l}": _off(g[f"b{l}"], s) for l in range(om.L)})
    say("bias gradients", n, errs)
    assert max(errs.values()) <= 2.0


@pytest.mark.parametrize("n", SIZES)
def test_weight_gradients_do_not_grow_with_the_mesh(n):
    from oracle import mpnn as om
    g, h0, s, sy = _gradients(n)
    errs = {"W_in": _off(g["W_in"], (1.0 + np.arange(10) / 16.0)[:, None] * s), "W_out": _off(g["W_out"], (h0 + om.L)[:, None] * sy)}
    for l in range(om.L):
        errs[f"W_s{l}"] = _off(g[f"W_s{l}"], (h0 + l)[:, None] * s)
        errs[f"W_n{l}"] = _off(g[f"W_n{l}"], (h0 + l)[:, None] * s)
    say("weight gradients", n, errs)
    assert max(errs.values()) <= 72.0
