"""Infinities and NaN in the input of the multi-step kernels and of the
LDS-band product stay where single steps put them: the entries that are
finite are the same ones as with one launch per step, and agree with it.
A batch's right-hand side that is not finite spoils no other one."""

import numpy as np
import pytest
import torch

from workloads import biharmonic2d, convdiff2d, convdiff3d_box, randsparse, rhs, start_vector
from gpu_util import say, dev, host, relerr

pytestmark = pytest.mark.gpu

# finite entries of two kernels differ by roundings of their sums alone
TOL = {"fp64": 1e-12, "fp32": 1e-4}
DTYPE = {"fp64": torch.float64, "fp32": torch.float32}


@pytest.fixture(scope="module")
def pp():
    import paper_1911_07065_amd.api as api

    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    return api


def _varied(csr, seed=4):
    rows = np.repeat(np.arange(csr.n), np.diff(csr.rowptr))
    return csr.with_values(csr.val * np.random.default_rng(seed).uniform(0.5, 1.0, csr.n)[rows])


def _same(pp, M, S, poly, bad, prec, what):
    for kind in ("p", "phi"):
        got, want = (host(pp.apply(poly, X, dev(bad, DTYPE[prec]), kind)) for X in (M, S))
        ok = np.isfinite(want)
        assert np.array_equal(np.isfinite(got), ok), (what, kind)
        assert 0 < ok.sum() < ok.size, (what, kind)
        assert relerr(got[ok], want[ok]) <= TOL[prec], (what, kind)


GRIDS = {
    "const": (lambda: convdiff3d_box(201, 90, 1, 4.0, 2.0, 0.0), (201, 90), [(1, 3, 8, 5), (2, 4, 8, 7)], 1.0),
    "varied": (lambda: _varied(convdiff3d_box(201, 90, 1, 4.0, 2.0, 0.0)), (201, 90), [(1, 4, 8, 5), (2, 2, 16, 7)], 1.0),
    "13_points": (lambda: biharmonic2d(150), (150, 150), [(1, 4, 8, 3), (2, 3, 16, 5)], -8.0),
}


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("name", list(GRIDS))
def test_grid_steps_keep_nonfinite_values_in_place(pp, name, prec):
    make, (gx, gy), shapes, scale = GRIDS[name]
    csr = make()
    poly = pp.poly_from_roots(scale * np.array([7.5, 3 + 1j, 3 - 1j, 5.0, 2.5, 6 + 0.5j, 6 - 0.5j]))
    M, S = pp.Matrix.from_csr(csr), pp.Matrix.from_csr(csr)
    for X in (M, S):
        X.set_variant(prec, 0, 1)
    bad = rhs(csr.n, 7)
    bad[0] = np.inf  # a corner, the end of a line and an inner point
    bad[gx * (gy // 2) + gx - 1] = -np.inf
    bad[gx * (gy // 3) + gx // 3] = np.nan
    for shape in shapes:
        M.set_grid(prec, *shape)
        say("grid nonfinite", name, prec, shape)
        _same(pp, M, S, poly, bad, prec, (name, shape))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_lds_bands_keep_nonfinite_values_in_place(pp, prec):
    csr = randsparse(40_000, 6, seed=6)
    poly = pp.poly_from_roots([11.0, 14.0])
    M, S = pp.Matrix.from_csr(csr), pp.Matrix.from_csr(csr)
    M.set_variant(prec, 34, 1)
    S.set_variant(prec, 0, 1)
    bad = rhs(csr.n, 7)
    for at, v in ((0, np.inf), (20_000, np.nan), (csr.n - 1, -np.inf)):  # the padding's column, a band's edge, the last
        bad[at] = v
    say("lds bands nonfinite", prec)
    _same(pp, M, S, poly, bad, prec, "lds bands")


@pytest.mark.parametrize("inner", ["fp64", "fp32"])
def test_batch_grid_keeps_nonfinite_systems_apart(pp, inner):
    csrs = [convdiff2d(N, 3.0) for N in (70, 33, 64)]
    B = pp.Batch(csrs)
    polys = B.setup(dev(np.concatenate([start_vector(c.n, 60 + i) for i, c in enumerate(csrs)])), 10)
    B.set_chain_config(2, inner, "box")
    B.set_grid(2, inner, 4, 8, 5)
    bs = [rhs(c.n, 40 + i, count=2) for i, c in enumerate(csrs)]
    bs[1][0, 5], bs[0][1, 0] = np.nan, np.inf
    say("batch nonfinite", inner)
    x, infos = B.solve(polys, B.interleave(np.concatenate(bs, axis=1)), 2, tol=1e-9, m=30, inner=inner)
    xh = host(B.deinterleave(x, 2))
    for s, c in enumerate(csrs):
        lo = int(B.row_off[s])
        for r in range(2):
            if np.all(np.isfinite(bs[s][r])):
                assert infos[2 * s + r]["converged"]
                res = np.linalg.norm(bs[s][r] - c.to_scipy() @ xh[r, lo: lo + c.n])
                assert res <= 1.001e-9 * np.linalg.norm(bs[s][r])
