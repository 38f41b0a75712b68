"""The batch tuner over mixes of sides: it finishes for every precision and
number of right-hand sides, and what it picks solves.

In launches with an accumulator a region may be half as high as without (its
registers leave room for half of the waves), so a shape whose full region
spans a system can leave no tile in the lower one. The mixes are ones whose
most promising shapes do that (uniform sides up to two regions' height, sides
a little past one wave), one large system among small ones, and the smallest.
Bound: the residual, formed on the host in FP64, as the solver states it.
"""

import numpy as np
import pytest
import torch

from workloads import convdiff2d, rhs, start_vector
from gpu_util import say, dev, host

pytestmark = pytest.mark.gpu

MIXES = {
    "16x25": [25] * 16,
    "16x40": [40] * 16,
    "96x49": [49] * 96,
    "128x64": [64] * 128,
    "64_to_80": list(range(64, 82)),
    "64_to_150": [64, 76, 89, 101, 113, 125, 138, 150],
    "one_large": [9, 20, 200, 33],
}
TOL = 1e-9


@pytest.fixture(scope="module")
def pp():
    import paper_1911_07065_amd.api as api

    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    return api


def _batch(pp, sides):
    csrs = [convdiff2d(N, 3.0 + i % 5) for i, N in enumerate(sides)]
    B = pp.Batch(csrs)
    polys = B.setup(dev(np.concatenate([start_vector(c.n, 60 + i) for i, c in enumerate(csrs)])), 12)
    return csrs, B, polys


def _solved(B, csrs, polys, R, inner):
    bs = [rhs(c.n, 40 + i, count=R) for i, c in enumerate(csrs)]
    x, infos = B.solve(polys, B.interleave(np.concatenate(bs, axis=1)), R, tol=TOL, m=30, inner=inner)
    assert all(i["converged"] for i in infos)
    xh = host(B.deinterleave(x, R))
    for s, c in enumerate(csrs):
        lo, A = int(B.row_off[s]), c.to_scipy()
        for r in range(R):
            assert np.linalg.norm(bs[s][r] - A @ xh[r, lo: lo + c.n]) <= 1.001 * TOL * np.linalg.norm(bs[s][r])


@pytest.mark.parametrize("mix", list(MIXES))
def test_batch_tunes_and_solves(pp, mix):
    csrs, B, polys = _batch(pp, MIXES[mix])
    for R in (1, 2, 4):
        for inner in ("fp64", "fp32"):
            say("batch tune", mix, R, inner)
            B.tune(R, inner)
            say("batch grid", mix, R, inner, B.grid(R, inner))
        _solved(B, csrs, polys, R, "fp64")
        _solved(B, csrs, polys, R, "fp32")


@pytest.mark.parametrize("inner", ["fp64", "fp32"])
def test_first_solve_tunes_by_itself(pp, inner):
    csrs, B, polys = _batch(pp, MIXES["16x40"] if inner == "fp64" else MIXES["128x64"])
    say("batch first solve", inner)
    _solved(B, csrs, polys, 4, inner)
    assert B.grid(4, inner)[0][2] >= 2  # launches of one step are never faster here
