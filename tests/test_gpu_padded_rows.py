"""Pattern rows padded to whole lines (handles without a memory budget) and
rows of exactly K samples (handles with one), in the staged translation kernel
and in the one that is best at the number of right-hand sides, against the
tiled translation kernel."""
import numpy as np
import pytest
import torch

import paper_2210_04892_amd as mf
import synth

pytestmark = pytest.mark.gpu

# The three handles share every stage but the translation, whose sums differ in
# order alone.  Rounding as in any two orders: a far field is a sum of samples
# that cancels by 1e4 to 1e5, and a few percent of the product.
TOL = {torch.complex64: 2e-4, torch.complex128: 1e-11}


# 3 levels on the far interactions, leaf rows of 242 samples; one level alone
@pytest.fixture(scope="module", params=[(32, 2.67), (6, 0.5)], ids=["levels", "single"])
def handles(request):
    v, t = synth.icosphere(*request.param)
    kw = dict(k=2 * np.pi, max_rhs=33)
    h = [mf.Geometry(v, t, trans_kernel=tk, hbm_budget_bytes=hb, **kw).precompute()
         for tk, hb in (("tiled", 0), ("lds", 0), ("lds", 32 << 30), ("auto", 32 << 30), ("auto", 0))]
    yield h
    for g in h:
        g.release()


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("nrhs", [1, 2, 4, 5, 8, 9, 16, 31, 33])
def test_padded_rows_match(handles, nrhs, dtype):
    x = torch.from_numpy(synth.gaussian_coeffs(2 * handles[0].n_rwg, nrhs, 90 + nrhs)).to("cuda").to(dtype)
    ref = handles[0].matvec(x, op="C")
    for g in handles[1:]:
        y = g.matvec(x, op="C")
        assert float(torch.linalg.norm(y - ref) / torch.linalg.norm(ref)) < TOL[dtype]
        assert torch.equal(y, g.matvec(x, op="C"))
