"""The autotuner chooses only what reaches a launch.  Where an operator of a small
mesh shares a slice (rows of six blocks and more) or a row (of forty and more)
between several waves, the waves per workgroup, slices per wave and block order of
the single-column product do not, so they keep their untuned values; at 24 columns
the tiles 0, 32 and 64 are one launch, one tile wide, so of these the untuned 0 is
kept, and none is spread over the XCDs; and rows shared by several waves keep the
untuned waves per workgroup."""
import json

import numpy as np
import pytest

import meshgen as mg
from tests.gpu_util import dev, gpu_assemble, say, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrhs", [1, 5, 24])
def test_only_distinct_launches_are_chosen(tmp_path, nrhs):
    import paper_1804_10060_amd as te
    torch = torch_cuda()
    prob = mg.disc_problem(10, 40, 3, 2, seed=2)
    A, _, d = gpu_assemble(prob)
    h = te.AMG(A, d["coords"], d["mask"], coarse_max=400, max_nrhs=nrhs, build_fp32=1)
    path = str(tmp_path / "tune.json")
    say(h.autotune(path, use_cache=False))
    with open(path) as fh:
        saved = json.load(fh)
    single = {k: v for k, v in saved.items() if "-nrhs" not in k}
    assert len(single) >= 6 and (nrhs == 1 or len(single) == len(saved) - len(single))
    shared = 0
    for k, (wpb, spw, remap, nt, mwpb, mtile, msplit, xb) in single.items():
        bpr = int(k.rsplit("bpr", 1)[1])
        bpr = 2 * bpr - 1 if k.startswith("rsym") else bpr   # the mirrored blocks count too
        if bpr > (6 if k.startswith("sell") else 40):
            shared += 1
            assert (wpb, spw, remap) == (1 if k.startswith("sell") or "-6x3-" in k else 2, 1, 1), k
    assert shared >= 6
    for k, (wpb, spw, remap, nt, mwpb, mtile, msplit, xb) in saved.items():
        if "-nrhs" not in k:
            continue
        if k.startswith("sell") and nrhs == 24:
            assert mtile in (0, 16) and (mtile == 16 or msplit == 0), k
        else:
            assert (mtile, msplit) == (0, 0) and (mwpb == 4 or k.startswith("sell")), k
    rng = np.random.default_rng(0)
    B = rng.standard_normal((prob.mesh.n_nodes, 3, nrhs))
    B[prob.mask != 0] = 0.0
    b = dev(B.reshape(-1) if nrhs == 1 else B, torch.float64)
    assert all(h.solve(b)[1].converged)
