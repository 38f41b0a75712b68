"""GPU parity of many chain steps per launch on 3-D boxes against the oracle.

Workgroups march through the planes of a tile with two or three steps in
flight. Checked on boxes whose lines, columns and plane counts leave partial
tiles, fill one exactly, and fit inside a single one; on chunks of one plane
and more; for every built shape, for the largest and for small workgroups;
with real roots, conjugate pairs and added copies, p, phi and pi, FP64 and
FP32. The bounds are the other chain kernels': 1e-12 relative in FP64, ten
times the error of the chain emulated in float32 in FP32.
"""

import numpy as np
import pytest
import torch

from oracle import chains, roots as oroots
from oracle.mixed import apply_p_low, apply_phi_low
from workloads import convdiff3d, convdiff3d_box, rhs
from gpu_util import say, dev, host, maxerr, assert_close, tail_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pp():
    import paper_1911_07065_amd.api as api

    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    return api


BOXES = [(64, 32, 9), (20, 17, 5), (3, 40, 30), (65, 33, 7), (201, 15, 11), (131, 75, 4), (59, 130, 40)]
SHAPES = {"fp64": [(1, 2), (1, 4), (2, 2)], "fp32": [(1, 2), (1, 4), (2, 2), (2, 4)]}
TH = np.array([7.5, 0.2, 3 + 1j, 3 - 1j, 5 + 0.5j, 5 - 0.5j, 1.0, 0.05, 2.5, 4 + 2j, 4 - 2j])


@pytest.mark.parametrize("dims", BOXES)
def test_box_steps_match_oracle(pp, dims):
    csr = convdiff3d_box(*dims, 4.0, 2.0, 1.0)
    A = csr.to_scipy()
    v = rhs(csr.n, 5)
    v32 = v.astype(np.float32)
    P = oroots.poly_from_roots(TH, add_roots=True)
    poly = pp.poly_from_roots(TH, add_roots=True)
    M = pp.Matrix.from_csr(csr)
    refs = {"p": chains.apply_p(A, P.units, v), "phi": chains.apply_phi(A, P.units, v), "pi": chains.apply_pi(A, P.units, v)}
    A32 = A.astype(np.float32)
    emu = {"p": apply_p_low(A32, P.units, v32, "fp32"), "phi": apply_phi_low(A32, P.units, v32, "fp32")}
    for prec, shapes in SHAPES.items():
        M.set_variant(prec, 0, 1)
        for vx, ry in shapes:
            for steps in (2, 3):
                for waves in (4, 8, 16):
                    if waves == 16 and vx * ry > (2 if prec == "fp64" else 4):
                        continue
                    say("box", dims, prec, vx, ry, waves, steps)
                    M.set_grid(prec, vx, ry, waves, steps)
                    assert M.grid(prec)[0] == (vx, ry, waves, steps)
                    assert pp.chain_bytes(poly, M, "phi", prec)[1] < poly.d_eff
                    for kind in ("p", "phi", "pi"):
                        what = f"{dims} {prec} {vx}x{ry}x{waves} {steps} {kind}"
                        if prec == "fp64":
                            assert_close(host(pp.apply(poly, M, dev(v), kind)), refs[kind], 1e-12, what, dims)
                            continue
                        g32 = host(pp.apply(poly, M, dev(v32, torch.float32), kind))
                        base = "p" if kind == "p" else "phi"
                        for idx in (None, tail_rows(csr.n)):
                            delta = maxerr(emu[base], refs[base], idx)
                            err = maxerr(v32 - g32 if kind == "pi" else g32, refs[base], idx)
                            assert err <= 10 * delta + 1e-6, (what, err, delta)


def test_box_tuned_repeats_and_follows_new_values(pp):
    # the tuner's own choice; repeated products are identical, infinities stay
    # where the single steps have them; new values that keep the stencil
    # constant, then values that do not (single steps again)
    dims = (150, 101, 60)
    csr = convdiff3d_box(*dims, 4.0, 2.0, 1.0)
    P = oroots.poly_from_roots(TH)
    poly = pp.poly_from_roots(TH)
    M, S = pp.Matrix.from_csr(csr), pp.Matrix.from_csr(csr)
    S.set_variant("fp64", 0, 1)
    v = rhs(csr.n, 7)
    M.tune("fp64")
    say("box tuned", M.grid("fp64"))
    for kind in ("p", "phi"):
        first = pp.apply(poly, M, dev(v), kind)
        assert torch.equal(first, pp.apply(poly, M, dev(v), kind))
    M.set_grid("fp64", 1, 4, 8, 3)
    bad = v.copy()
    bad[0] = np.inf
    bad[csr.n - 150] = np.nan
    for kind in ("p", "phi"):
        got, want = (host(pp.apply(poly, X, dev(bad), kind)) for X in (M, S))
        assert np.array_equal(np.isfinite(got), np.isfinite(want))
    rows = np.repeat(np.arange(csr.n), np.diff(csr.rowptr))
    scaled = csr.val * np.random.default_rng(4).uniform(0.5, 1.0, csr.n)[rows]
    for vals in (csr.val * np.where(csr.colind == rows, 1.25, 1.0), scaled):
        M.set_values(dev(vals))
        ref = chains.apply_p(csr.with_values(vals).to_scipy(), P.units, v)
        assert_close(host(pp.apply(poly, M, dev(v), "p")), ref, 1e-12, "new values", dims)
    assert M.grid("fp64")[0][3] == 0


def test_box_refused_where_it_does_not_apply(pp):
    M = pp.Matrix.from_csr(convdiff3d(100, 1, 1, 1))
    for prec in ("fp64", "fp32", "bf16"):
        M.set_variant(prec, 0, 1)
    for bad in (("bf16", 1, 2, 8, 2), ("fp64", 2, 4, 8, 2), ("fp64", 1, 3, 8, 2), ("fp64", 1, 4, 9, 2), ("fp32", 2, 4, 16, 3),
                ("fp64", 1, 4, 8, 4), ("fp64", 1, 2, 2, 2)):
        with pytest.raises(Exception, match="grid"):
            M.set_grid(*bad)
    M = pp.Matrix.from_csr(convdiff3d(3, 1, 1, 1))  # 27 rows: no diagonal format
    M.set_variant("fp64", 0, 1)
    with pytest.raises(Exception, match="grid"):
        M.set_grid("fp64", 1, 2, 4, 2)
