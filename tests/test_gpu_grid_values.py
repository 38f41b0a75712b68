"""The 2-D multi-step shape in use follows new values: it stays while its kernel
does, and a shape whose kernel changed never reports the old one's time. And
the byte count of a 3-D program whose launches are of different lengths."""

import numpy as np
import pytest
import torch

from oracle import chains, roots as oroots
from workloads import convdiff2d, convdiff3d_box, rhs
from gpu_util import say, dev, host, assert_close

pytestmark = pytest.mark.gpu

TH = np.array([7.5, 0.2, 3 + 1j, 3 - 1j, 1.0, 0.05, 2.5])


@pytest.fixture(scope="module")
def pp():
    import paper_1911_07065_amd.api as api

    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    return api


def _rows(csr):
    return np.repeat(np.arange(csr.n), np.diff(csr.rowptr))


def _varied(csr, seed=4):
    return csr.val * np.random.default_rng(seed).uniform(0.5, 1.0, csr.n)[_rows(csr)]


def _right(pp, M, csr, vals, dims):
    v = rhs(csr.n, 7)
    P = oroots.poly_from_roots(TH)
    got = host(pp.apply(pp.poly_from_roots(TH), M, dev(v), "phi"))
    assert_close(got, chains.apply_phi(csr.with_values(vals).to_scipy(), P.units, v), 1e-12, "new values", (*dims, 1))


DIA = 25  # a single-step variant that new values leave in place


@pytest.mark.parametrize("case", ["two_coefficients", "constant_built", "constant_not_built"])
def test_forced_shape_and_new_values(pp, case):
    dims = (90, 70)
    csr = convdiff3d_box(*dims, 1, 4.0, 2.0, 0.0)
    if case == "two_coefficients":  # few distinct rows, but no constant stencil
        csr = csr.with_values(csr.val * np.where(_rows(csr) < csr.n // 2, 1.0, 0.5))
    shape = (1, 6, 10, 5) if case == "constant_not_built" else (1, 3, 7, 6)
    M = pp.Matrix.from_csr(csr)
    assert pp.chain_variant_name(DIA).startswith("dia")
    M.set_variant("fp64", DIA, 1)
    M.set_grid("fp64", *shape)
    say("grid new values", case)
    vals = _varied(csr)
    M.set_values(dev(vals))
    got, us = M.grid("fp64")
    if case == "constant_not_built":
        assert got != shape and got[3] >= 2 and us == 0.0
    else:
        assert got == shape
    _right(pp, M, csr, vals, dims)


def test_tuned_shape_reports_no_time_of_another_kernel(pp):
    csr = convdiff2d(150, 6.0)
    M = pp.Matrix.from_csr(csr)
    M.tune("fp64")
    assert M.grid("fp64")[0][3] >= 2 and M.grid("fp64")[1] > 0.0
    say("grid tuned, new values")
    vals = _varied(csr)
    M.set_values(dev(vals))
    assert M.grid("fp64")[1] == 0.0
    _right(pp, M, csr, vals, (150, 150))


@pytest.mark.parametrize("variant", ["sell64", "diapv"])
def test_box_chain_bytes_count_single_steps_as_such(pp, variant):
    # a 3-D program's launches of one step run the single-step variant: they
    # read its matrix data, not the interior row's coefficients alone
    csr = convdiff3d_box(40, 30, 20, 4.0, 2.0, 1.0)
    M = pp.Matrix.from_csr(csr)
    names = [pp.chain_variant_name(k) for k in range(pp.N_CHAIN_VARIANTS)]
    one = pp.poly_from_roots([3.0], keep_order=True)
    mixed = pp.poly_from_roots([3.0, 5 + 1j, 5 - 1j], keep_order=True)
    for prec, size in (("fp64", 8), ("fp32", 4)):
        M.set_variant(prec, names.index(variant), 1)
        single = pp.chain_bytes(one, M, "phi", prec)  # matrix data; input, final vector, output
        matrix = single[0] - 3 * csr.n * size
        M.set_grid(prec, 1, 2, 8, 2)
        say("chain bytes, single steps", variant, prec)
        assert pp.chain_bytes(one, M, "phi", prec) == single
        # the real root alone (input, output), then the pair in one launch
        # (input, final vector, output, seven coefficients)
        assert pp.chain_bytes(mixed, M, "phi", prec) == (matrix + 5 * csr.n * size + 7 * size, 2)
