"""GPU parity of the batch's many-steps-per-launch kernel.

Systems of different sizes (smaller than a region, exactly one wave wide,
leaving partial tiles) and different programs (real roots, conjugate pairs,
added copies) are solved with every built shape and several segment lengths.
Bound for x: the symmetric part of a 2-D convection-diffusion matrix is the
Laplacian, so ||A^-1|| <= 1 / (4 - 4 cos(pi / (N + 1))) and x is within
||A^-1|| ||r|| of the direct solution, r computed on the host. Graph replays
equal eager launches bit for bit.
"""

import numpy as np
import pytest
import scipy.sparse.linalg as sla
import torch

from workloads import convdiff2d, rhs, start_vector
from gpu_util import say, dev, host

pytestmark = pytest.mark.gpu

SIDES = [(9, 2.0), (64, 40.0), (70, 5.0), (33, 0.0), (131, 25.0)]
SHAPES = [(2, 4), (2, 16), (3, 8), (4, 8), (4, 16), (6, 8), (6, 16)]


@pytest.fixture(scope="module")
def pp():
    import paper_1911_07065_amd.api as api

    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    return api


@pytest.fixture(scope="module")
def systems():
    csrs = [convdiff2d(N, a) for N, a in SIDES]
    bs = [rhs(c.n, 40 + i, count=4) for i, c in enumerate(csrs)]
    xs = [np.stack([sla.spsolve(c.to_scipy().tocsc(), b) for b in bb]) for c, bb in zip(csrs, bs)]
    return csrs, bs, xs


def _batch(pp, csrs):
    B = pp.Batch(csrs)
    v0 = dev(np.concatenate([start_vector(c.n, 60 + i) for i, c in enumerate(csrs)]))
    return B, B.setup(v0, 14)


@pytest.mark.parametrize("R", [1, 2, 4])
@pytest.mark.parametrize("inner", ["fp64", "fp32"])
def test_batch_grid_solves(pp, systems, R, inner):
    csrs, bs, xs = systems
    B, polys = _batch(pp, csrs)
    bd = B.interleave(np.concatenate([b[:R] for b in bs], axis=1))
    tol, ran = 1e-10, 0
    B.set_chain_config(R, inner, "box")
    for ry, waves in SHAPES:
        for steps in (2, 5, 13):
            try:
                B.set_grid(R, inner, ry, waves, steps)
            except Exception as e:
                assert "built shape" in str(e) or "no tile" in str(e)
                continue
            assert B.grid(R, inner)[0] == (ry, waves, steps)
            say("batch grid", R, inner, ry, waves, steps)
            x, infos = B.solve(polys, bd, R, tol=tol, m=30, inner=inner, graphs=steps == 5)
            assert all(i["converged"] for i in infos)
            xh = host(B.deinterleave(x, R))
            for s, c in enumerate(csrs):
                lo, A = int(B.row_off[s]), c.to_scipy()
                for r in range(R):
                    got, b = xh[r, lo: lo + c.n], bs[s][r]
                    res = np.linalg.norm(b - A @ got)
                    assert res <= 1.001 * tol * np.linalg.norm(b)
                    inv = 1.0 / (4.0 - 4.0 * np.cos(np.pi / (SIDES[s][0] + 1)))
                    assert np.linalg.norm(got - xs[s][r]) <= 1.01 * inv * res + 1e-12 * np.linalg.norm(xs[s][r])
            ran += 1
    assert ran >= 6


def test_batch_grid_tuned_graphs_and_refusals(pp, systems):
    csrs, bs, _ = systems
    B, polys = _batch(pp, csrs)
    bd = B.interleave(np.concatenate(bs, axis=1))
    with pytest.raises(Exception, match="box copy"):
        B.set_grid(4, "fp32", 4, 8, 5)  # nothing tuned or set yet
    B.tune(4, "fp32")
    assert B.grid(4, "fp32")[0][2] >= 2  # launches of one step are never faster here
    say("batch grid tuned", B.grid(4, "fp32"))
    xe, ie = B.solve(polys, bd, 4, tol=1e-11, m=8, inner="fp32", graphs=False)
    for graph_steps in (3, 0):
        xg, ig = B.solve(polys, bd, 4, tol=1e-11, m=8, inner="fp32", graphs=True, graph_steps=graph_steps)
        assert torch.equal(xe, xg) and [i["iters"] for i in ie] == [i["iters"] for i in ig]
    for bad in ((4, "fp32", 5, 8, 5), (4, "fp32", 4, 17, 5), (4, "fp32", 4, 8, 33), (4, "fp64", 6, 8, 5), (4, "fp32", 2, 2, 4)):
        with pytest.raises(Exception):
            B.set_grid(*bad)
    B.tune(4, "fp32")
    B.set_chain_config(4, "fp32", "box")
    assert B.grid(4, "fp32")[0][2] == 0
    B.set_format("box")
    with pytest.raises(Exception, match="box copy"):
        B.set_grid(4, "fp32", 4, 8, 5)
    # new values that no longer are a constant stencil
    B, _ = _batch(pp, csrs)
    B.tune(4, "fp32")
    vals = np.concatenate([c.val for c in csrs])
    B.set_values(vals * np.linspace(1.0, 1.1, vals.size))
    assert B.grid(4, "fp32")[0][2] == 0


@pytest.mark.parametrize("m", [63, 64, 65, 130, 260])
def test_batch_long_cycles(pp, m):
    # cycles of more columns than a wave has lanes, and than its lanes hold in
    # registers: the rotations and the back substitution of every pair
    sides = [(48, 0.0), (23, 4.0)]
    csrs = [convdiff2d(N, a) for N, a in sides]
    B = pp.Batch(csrs)
    polys = [pp.poly_from_roots([6.0]) for _ in csrs]
    bs = [rhs(c.n, 7 + i, count=2) for i, c in enumerate(csrs)]
    bd = B.interleave(np.concatenate(bs, axis=1))
    x, infos = B.solve(polys, bd, 2, tol=1e-9, m=m, inner="fp64", max_cycles=60)
    say("batch long cycles", m, [i["iters"] for i in infos])
    assert max(i["iters"] for i in infos) > 64
    xh = host(B.deinterleave(x, 2))
    for s, c in enumerate(csrs):
        lo, A = int(B.row_off[s]), c.to_scipy()
        for r in range(2):
            got, b = xh[r, lo: lo + c.n], bs[s][r]
            res = np.linalg.norm(b - A @ got)
            assert infos[2 * s + r]["converged"] and res <= 1.001e-9 * np.linalg.norm(b)
            ref = sla.spsolve(A.tocsc(), b)
            inv = 1.0 / (4.0 - 4.0 * np.cos(np.pi / (sides[s][0] + 1)))
            assert np.linalg.norm(got - ref) <= 1.01 * inv * res + 1e-12 * np.linalg.norm(ref)
