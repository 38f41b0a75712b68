"""GPU parity of the products whose column bands are held in LDS.

Element-wise against the oracle's chains on scattered matrices at the edges
of a band (16384 columns in FP64, 32768 in FP32, 65536 in BF16 storage), of a
window of 512 rows and of a slice of 64; with empty rows and rows of very
different lengths; on vectors that are not 16-byte aligned; after new
values. Bounds as for the other chain kernels.
"""

import numpy as np
import pytest
import scipy.sparse as sp
import torch

from oracle import chains, roots as oroots
from oracle.mixed import apply_p_low
from workloads import CSR, convdiff2d, randsparse, rhs
from gpu_util import say, dev, host, maxerr, assert_close

pytestmark = pytest.mark.gpu

LBAND = 34
ROOTS = np.array([14.0, 9.5, 12 + 4j, 12 - 4j, 18.0])


@pytest.fixture(scope="module")
def pp():
    import paper_1911_07065_amd.api as api

    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    assert api.chain_variant_name(LBAND) == "ldsband"
    return api


def _ragged(n, seed):
    """Rows of 0 to 60 entries: every 50th row empty, every 97th long, the rest 3 or so."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, 6, n)
    lens[::50], lens[::97] = 0, 60
    rows = np.repeat(np.arange(n), lens)
    A = sp.coo_matrix((rng.standard_normal(rows.size), (rows, rng.integers(0, n, rows.size))), shape=(n, n)).tocsr()
    A = (A + sp.diags(np.where(lens > 0, 14.0, 0.0))).tocsr()
    A.eliminate_zeros()
    A.sort_indices()
    return CSR(n, A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data.astype(np.float64))


CASES = {
    "rand_4096": lambda: randsparse(4096, 16, seed=3),
    "rand_16384": lambda: randsparse(16384, 8, seed=4),
    "rand_16385": lambda: randsparse(16385, 8, seed=5),
    "rand_32769": lambda: randsparse(32769, 16, seed=6),
    "rand_65537": lambda: randsparse(65537, 6, seed=7),
    "ragged_20011": lambda: _ragged(20011, 8),
}


@pytest.mark.parametrize("name", list(CASES))
def test_lds_bands_match_oracle(pp, name):
    csr = CASES[name]()
    A = csr.to_scipy()
    A32 = A.astype(np.float32)
    P = oroots.poly_from_roots(ROOTS)
    poly = pp.poly_from_roots(ROOTS)
    v = rhs(csr.n, 5)
    M = pp.Matrix.from_csr(csr)
    for prec in ("fp64", "fp32", "bf16"):
        M.set_variant(prec, LBAND, 1)
    ref_p, ref_phi = chains.apply_p(A, P.units, v), chains.apply_phi(A, P.units, v)
    d32 = maxerr(apply_p_low(A32, P.units, v.astype(np.float32)), ref_p)
    for remap in (0, 1):
        say("lds bands", name, remap)
        for prec in ("fp64", "fp32", "bf16"):
            M.set_variant(prec, LBAND, remap)
        got = pp.apply(poly, M, dev(v), "p")
        assert torch.equal(got, pp.apply(poly, M, dev(v), "p"))
        assert_close(host(got), ref_p, 1e-12, f"{name} p")
        assert_close(host(pp.apply(poly, M, dev(v), "phi")), ref_phi, 1e-12, f"{name} phi")
        assert maxerr(host(pp.apply(poly, M, dev(v, torch.float32), "p")), ref_p) <= 10 * d32 + 1e-6
        vb = dev(v, torch.bfloat16)
        db = maxerr(apply_p_low(A32, P.units, host(vb), "bf16"), ref_p)
        assert maxerr(host(pp.apply(poly, M, vb, "p")), ref_p) <= 10 * db + 1e-6
        # inputs that start in the middle of a 16-byte word
        for dt, ref, tol in ((torch.float64, ref_p, 1e-12), (torch.float32, ref_p, None), (torch.bfloat16, ref_p, None)):
            buf = torch.zeros(csr.n + 1, dtype=dt, device="cuda")
            buf[1:] = dev(v, dt)
            shifted = pp.apply(poly, M, buf[1:], "p")
            assert torch.equal(shifted, pp.apply(poly, M, dev(v, dt), "p"))
    # new values reach the copy
    M.set_values(dev(0.5 * csr.val))
    assert_close(host(pp.apply(poly, M, dev(v), "phi")), chains.apply_phi(0.5 * A, P.units, v), 1e-12, f"{name} new values")


def test_lds_bands_bytes_and_refusals(pp):
    csr = randsparse(5000, 8, seed=9)
    M = pp.Matrix.from_csr(csr)
    M.set_variant("fp32", LBAND, 1)
    poly = pp.poly_from_roots([12.0, 15.0])
    # two launches a step; at least the entries' 8 bytes (column pairs and values)
    by, launches = pp.chain_bytes(poly, M, "phi", "fp32")
    assert launches == 4 and by >= 2 * csr.nnz * 6
    say("lds bands refused")
    heavy = randsparse(5000, 8, seed=9).to_scipy().tolil()
    heavy[17, :300] = 1.0  # more entries in a band than a lane's count holds
    heavy = heavy.tocsr()
    heavy.sort_indices()
    big = randsparse(8 * 16384 + 1, 2, seed=2)  # nine FP64 bands
    for what, c, prec in (("a row of 300", CSR(5000, heavy.indptr.astype(np.int32), heavy.indices.astype(np.int32), heavy.data), "fp32"),
                          ("nine bands", big, "fp64"), ("a stencil", convdiff2d(80, 1.0), "fp32"),
                          ("few rows", randsparse(2000, 8, seed=1), "fp32")):
        Mb = pp.Matrix.from_csr(c)
        with pytest.raises(Exception, match="column bands in LDS"):
            Mb.set_variant(prec, LBAND, 1)
        Mb.tune(prec)
        assert Mb.variant(prec)[0] != "ldsband", what
