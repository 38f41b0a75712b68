"""GPU parity of many chain steps per launch on 2-D grids against the oracle.

Regions of 64 vx x waves ry points held in registers deliver the tile that
is still exact after the launch's steps. Checked for 5-point stencils with
constant and with varying coefficients and for the 13-point stencil, on grids
that leave partial tiles in both directions, that end with a region, and that
a single region spans; for every built shape, for step counts that divide
the chain and that do not, and for the most a region can take; with real
roots, conjugate pairs and added copies, p, phi and pi, FP64 and FP32. The
bounds are the other chain kernels': 1e-12 relative in FP64, ten times the
error of the chain emulated in float32 in FP32.
"""

import numpy as np
import pytest
import torch

from oracle import chains, roots as oroots
from oracle.mixed import apply_p_low, apply_phi_low
from workloads import biharmonic2d, convdiff2d, convdiff3d, convdiff3d_box, randsparse, rhs
from gpu_util import say, dev, host, maxerr, assert_close, tail_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pp():
    import paper_1911_07065_amd.api as api

    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    return api


def _varied(csr, seed=4):
    # every row scaled on its own: no two rows share their coefficients
    rows = np.repeat(np.arange(csr.n), np.diff(csr.rowptr))
    return csr.with_values(csr.val * np.random.default_rng(seed).uniform(0.5, 1.0, csr.n)[rows])


CASES = {
    "const_50x50": (lambda: convdiff2d(50, 3.0), 5, True),          # one region spans it
    "const_64x33": (lambda: convdiff3d_box(64, 33, 1, 4.0, 2.0, 0.0), 5, True),  # exactly one wave wide
    "const_201x37": (lambda: convdiff3d_box(201, 37, 1, 4.0, 2.0, 0.0), 5, True),
    "const_65x131": (lambda: convdiff3d_box(65, 131, 1, 1.0, 3.0, 0.0), 5, True),
    "var_90x41": (lambda: _varied(convdiff3d_box(90, 41, 1, 4.0, 2.0, 0.0)), 5, False),
    "var_40x150": (lambda: _varied(convdiff3d_box(40, 150, 1, 4.0, 2.0, 0.0)), 5, False),
    "bihar_40": (lambda: biharmonic2d(40), 13, True),
    "bihar_81": (lambda: biharmonic2d(81), 13, True),
}
ONE = [(1, 2), (1, 3), (1, 4), (2, 2)]
MORE = ONE + [(1, 6), (2, 3), (2, 4)]
SHAPES = {(5, True): MORE, (5, False): ONE, (13, True): MORE}


def _roots(nd):
    th = np.array([7.5, 0.2, 3 + 1j, 3 - 1j, 5 + 0.5j, 5 - 0.5j, 1.0, 0.05, 2.5])
    return th if nd == 5 else -8.0 * th


def _most_steps(nd, dims, vx, ry, waves):
    """The most steps that leave a tile, by the region's sides."""
    halo = 2 if nd == 5 else 4
    sides = [(s - 1) // halo for s, g in ((64 * vx, dims[0]), (ry * waves, dims[1])) if g > s]
    return min([32] + sides)


@pytest.mark.parametrize("name", list(CASES))
def test_grid_steps_match_oracle(pp, name):
    make, nd, const = CASES[name]
    csr = make()
    A = csr.to_scipy()
    gx = int(csr.colind[int(csr.rowptr[1]) - 1]) // (1 if nd == 5 else 2)
    dims = (gx, csr.n // gx)
    v = rhs(csr.n, 5)
    v32 = v.astype(np.float32)
    th = _roots(nd)
    P = oroots.poly_from_roots(th, add_roots=True)
    poly = pp.poly_from_roots(th, add_roots=True)
    M = pp.Matrix.from_csr(csr)
    for prec in ("fp64", "fp32"):
        M.set_variant(prec, 0, 1)
    refs = {"p": chains.apply_p(A, P.units, v), "phi": chains.apply_phi(A, P.units, v), "pi": chains.apply_pi(A, P.units, v)}
    A32 = A.astype(np.float32)
    emu = {"p": apply_p_low(A32, P.units, v32, "fp32"), "phi": apply_phi_low(A32, P.units, v32, "fp32")}
    ran = 0
    for vx, ry in SHAPES[nd, const]:
        for waves in (3, 16):
            most = _most_steps(nd, dims, vx, ry, waves)
            for steps in sorted({2, 5, most}):
                if steps < 2 or steps > most:
                    continue
                say("grid", name, vx, ry, waves, steps)
                for prec in ("fp64", "fp32"):
                    M.set_grid(prec, vx, ry, waves, steps)
                    assert M.grid(prec)[0] == (vx, ry, waves, steps)
                    assert pp.chain_bytes(poly, M, "phi", prec)[1] < poly.d_eff
                for kind in ("p", "phi", "pi"):
                    what = f"{name} {vx}x{ry}x{waves} {steps} {kind}"
                    assert_close(host(pp.apply(poly, M, dev(v), kind)), refs[kind], 1e-12, what, (*dims, 1))
                    g32 = host(pp.apply(poly, M, dev(v32, torch.float32), kind))
                    base = "p" if kind == "p" else "phi"
                    for idx in (None, tail_rows(csr.n)):
                        delta = maxerr(emu[base], refs[base], idx)
                        err = maxerr(v32 - g32 if kind == "pi" else g32, refs[base], idx)
                        assert err <= 10 * delta + 1e-6, (what, err, delta)
                ran += 1
    assert ran >= 10


def test_grid_tuned_repeats_and_follows_new_values(pp):
    # the tuner's own choice; repeated products are identical; values that
    # keep the stencil constant, then values that do not, keep it right
    csr = convdiff2d(150, 6.0)
    A = csr.to_scipy()
    th = _roots(5)
    P = oroots.poly_from_roots(th)
    poly = pp.poly_from_roots(th)
    M = pp.Matrix.from_csr(csr)
    v = rhs(csr.n, 7)
    M.tune("fp64")
    say("grid tuned", M.grid("fp64"))
    assert M.grid("fp64")[0][3] >= 2  # a chain of single launches is never faster here
    first = pp.apply(poly, M, dev(v), "phi")
    assert torch.equal(first, pp.apply(poly, M, dev(v), "phi"))
    assert_close(host(first), chains.apply_phi(A, P.units, v), 1e-12, "tuned", (150, 150, 1))
    val = csr.val * np.where(csr.colind == np.repeat(np.arange(csr.n), np.diff(csr.rowptr)), 1.25, 1.0)
    for vals in (val, _varied(csr).val):
        M.set_values(dev(vals))
        ref = chains.apply_p(csr.with_values(vals).to_scipy(), P.units, v)
        assert_close(host(pp.apply(poly, M, dev(v), "p")), ref, 1e-12, "new values", (150, 150, 1))


def test_grid_refused_where_it_does_not_apply(pp):
    for what, csr in {"3-D": convdiff3d(12, 1, 1, 1), "random": randsparse(3000, 8, seed=3),
                      "13 points, varying": _varied(biharmonic2d(30))}.items():
        say("grid refused", what)
        M = pp.Matrix.from_csr(csr)
        M.set_variant("fp64", 0, 1)
        with pytest.raises(Exception, match="2-D grid"):
            M.set_grid("fp64", 1, 2, 8, 4)
    M = pp.Matrix.from_csr(convdiff2d(200, 1.0))
    with pytest.raises(Exception, match="tune"):
        M.set_grid("fp32", 1, 2, 8, 4)
    for prec in ("fp32", "bf16"):
        M.set_variant(prec, 0, 1)
    for bad in (("bf16", 1, 2, 8, 4), ("fp32", 1, 5, 8, 4), ("fp32", 1, 2, 17, 4), ("fp32", 1, 2, 4, 4), ("fp32", 3, 1, 8, 2)):
        with pytest.raises(Exception, match="2-D grid"):
            M.set_grid(*bad)
    M.set_grid("fp32", 1, 2, 8, 4)
    M.set_variant("fp32", 0, 1)
    assert M.grid("fp32")[0][3] == 0
