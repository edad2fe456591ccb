"""Near field of 2 to 15 right-hand sides: its rounding in complex64 and, on a
body with enough work items that each is one wave's, its columns against the
one-right-hand-side kernel's."""
import numpy as np
import pytest
import torch

import paper_2210_04892_amd as mf
import synth

pytestmark = pytest.mark.gpu


# 1 080 and 30 720 RWGs (the inner index shared by four waves) and 122 880
# (above 12 288 items of a box and 16 rows: not shared)
@pytest.fixture(scope="module", params=[(6, 0.5), (32, 2.67), (64, 5.3)], ids=["small", "split", "unsplit"])
def geom(request):
    v, t = synth.icosphere(*request.param)
    g = mf.Geometry(v, t, k=2 * np.pi, max_rhs=15).precompute()
    yield g
    g.release()


def errors(y, ref):
    return torch.linalg.norm(y - ref, dim=0) / torch.linalg.norm(ref, dim=0)


@pytest.mark.parametrize("op", ["C", "EM"])
@pytest.mark.parametrize("nrhs", [2, 3, 7, 8, 9, 15])
def test_rounding_is_that_of_one_vector(geom, nrhs, op):
    """The one-right-hand-side kernel adds up 64 sums of a few products each in a
    tree.  A single-precision sum over the whole row would be two to five times
    further from the complex128 product; 10 % are left for the draw."""
    x = torch.from_numpy(synth.gaussian_coeffs(2 * geom.n_rwg, nrhs, 40 + nrhs)).to("cuda").to(torch.complex64)
    ref = geom.matvec(x.to(torch.complex128), op=op, part=mf.PART_NEAR)
    few = errors(geom.matvec(x, op=op, part=mf.PART_NEAR), ref)
    one = errors(torch.stack([geom.matvec(x[:, r].contiguous(), op=op, part=mf.PART_NEAR) for r in range(nrhs)], 1), ref)
    assert float(few.max()) < 1.1 * float(one.max())


# a row sums a few hundred products of order one
@pytest.mark.parametrize("dtype,tol", [(torch.complex64, 4e-7), (torch.complex128, 1e-13)])
@pytest.mark.parametrize("nrhs", [2, 7, 8, 9, 15])
def test_columns_match_one_vector(geom, nrhs, dtype, tol):
    x = torch.from_numpy(synth.gaussian_coeffs(2 * geom.n_rwg, nrhs, 60 + nrhs)).to("cuda").to(dtype)
    y = geom.matvec(x, op="EM", part=mf.PART_NEAR)
    one = torch.stack([geom.matvec(x[:, r].contiguous(), op="EM", part=mf.PART_NEAR) for r in range(nrhs)], 1)
    assert float(errors(y, one).max()) < tol
