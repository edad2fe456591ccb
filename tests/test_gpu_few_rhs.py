"""Products of a few right-hand sides on the matrix cores (packed tiles of 8,
full tiles of 16, the inner index shared by four waves or not) against the
one-right-hand-side vector kernels, column by column."""
import numpy as np
import pytest
import torch

import paper_2210_04892_amd as mf
import synth

pytestmark = pytest.mark.gpu

K = 2 * np.pi
# Rounding: a near-field row sums a few hundred products of order one (error
# some eps), a far-field one is a sum of samples that cancels by 1e4 to 1e5
# (the translation operators' size at the finest level), of which the far
# field is a few percent of the product.
TOL = {torch.complex64: {mf.PART_NEAR: 4e-6, mf.PART_ALL: 2e-4},
       torch.complex128: {mf.PART_NEAR: 1e-13, mf.PART_ALL: 1e-11}}


@pytest.fixture(scope="module", params=["small", "large"])
def geom(request):
    # 1 080 RWGs (fewer than 2048 work items: the inner index split over four
    # waves everywhere) and 30 720 (split in the near field alone)
    v, t = synth.icosphere(6, 0.5) if request.param == "small" else synth.icosphere(32, 2.67)
    g = mf.Geometry(v, t, k=K, max_rhs=17).precompute()
    yield g
    g.release()


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("op", ["C", "EM"])
@pytest.mark.parametrize("nrhs", [2, 3, 7, 8, 9, 15, 17])
def test_few_rhs_match_single(geom, nrhs, op, dtype):
    x = torch.from_numpy(synth.gaussian_coeffs(2 * geom.n_rwg, nrhs, 70 + nrhs)).to("cuda").to(dtype)
    for part, tol in TOL[dtype].items():
        y = geom.matvec(x, op=op, part=part)
        one = torch.stack([geom.matvec(x[:, r].contiguous(), op=op, part=part) for r in range(nrhs)], 1)
        err = torch.linalg.norm(y - one, dim=0) / torch.linalg.norm(one, dim=0)
        assert float(err.max()) < tol, (part, err)
