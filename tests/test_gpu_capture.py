"""Chains whose launches take more than 64 KB of LDS (the 2-D and 3-D multi-step
kernels and the LDS bands) and the others recorded into a HIP graph: every
replay, on new input values and with other work between, equals the eager
call bit for bit."""

import numpy as np
import pytest
import torch

from workloads import biharmonic2d, convdiff2d, convdiff3d_box, randsparse, rhs
from gpu_util import say, dev

pytestmark = pytest.mark.gpu

GRID, LBAND = "grid", "lband"
CASES = {
    "2d": (lambda: convdiff2d(300, 3.0), GRID, (2, 4, 16, 9), 1.0),
    "13_points": (lambda: biharmonic2d(150), GRID, (2, 4, 16, 9), -8.0),
    "3d": (lambda: convdiff3d_box(70, 45, 40, 4.0, 2.0, 1.0), GRID, (1, 2, 16, 3), 1.0),
    "bands": (lambda: randsparse(40_000, 6, seed=6), LBAND, None, 2.0),
}


@pytest.fixture(scope="module")
def pp():
    import paper_1911_07065_amd.api as api

    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    return api


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("name", list(CASES))
def test_replays_equal_eager_calls(pp, name, prec):
    make, what, shape, scale = CASES[name]
    csr = make()
    dt = torch.float64 if prec == "fp64" else torch.float32
    poly = pp.poly_from_roots(scale * np.array([7.5, 3 + 1j, 3 - 1j, 5.0, 2.5, 6 + 0.5j, 6 - 0.5j, 1.0, 4.5, 3.5, 2.0, 6.5]))
    M = pp.Matrix.from_csr(csr)
    M.set_variant(prec, 34 if what == LBAND else 0, 1)
    if shape:
        M.set_grid(prec, *shape)
    v = dev(rhs(csr.n, 1), dt)
    outs = {k: torch.empty_like(v) for k in ("p", "phi")}
    for k, o in outs.items():
        pp.apply(poly, M, v, k, out=o)  # the workspace is there before the recording
    say("capture", name, prec)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for k, o in outs.items():
            pp.apply(poly, M, v, k, out=o)
    for seed in (2, 3, 4):
        v.copy_(dev(rhs(csr.n, seed), dt))
        want = {k: pp.apply(poly, M, v, k) for k in outs}
        for o in outs.values():
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for k, o in outs.items():
            assert torch.equal(o, want[k]), (name, prec, k, seed)
