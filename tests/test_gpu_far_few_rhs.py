"""Far field of 2 to 15 right-hand sides against one at a time: received a wave
per RWG (2, 3) or on the matrix cores (packed up to 8, full up to 15, the
samples shared by four waves or not)."""
import numpy as np
import pytest
import torch

import paper_2210_04892_amd as mf
import synth

pytestmark = pytest.mark.gpu


# 1 470 RWGs (a last workgroup of two rows, 242 leaf samples), 7 680 and 38 880
# (more than 2 048 items of a box and 16 rows: the samples are not shared)
MESHES = {"ellipsoid": lambda: synth.ellipsoid(7, (0.6, 0.45, 0.3)), "sphere": lambda: synth.icosphere(16, 1.2),
          "large": lambda: synth.icosphere(36, 3.0)}


@pytest.fixture(scope="module", params=list(MESHES))
def geom(request):
    v, t = MESHES[request.param]()
    g = mf.Geometry(v, t, k=2 * np.pi, max_rhs=15).precompute()
    yield g
    g.release()


def errors(y, ref):
    return torch.linalg.norm(y - ref, dim=0) / torch.linalg.norm(ref, dim=0)


@pytest.mark.parametrize("op", ["C", "EM"])
@pytest.mark.parametrize("nrhs", [2, 3, 4, 7, 8, 9, 15])
def test_far_field_of_few(geom, nrhs, op):
    """complex128: the far field sums samples that cancel by 1e4 to 1e5.
    complex64: no further from the complex128 far field than one right-hand
    side, whose samples are added up in 64 short sums in single precision (2 %
    for the draw; one long sum in single precision leaves them 12 % further)."""
    x = torch.from_numpy(synth.gaussian_coeffs(2 * geom.n_rwg, nrhs, 10 + nrhs)).to("cuda").to(torch.complex64)

    def far(v):
        return geom.matvec(v, op=op, part=mf.PART_FAR)

    def one_by_one(v):
        return torch.stack([far(v[:, r].contiguous()) for r in range(nrhs)], 1)

    d = x.to(torch.complex128)
    ref = one_by_one(d)
    assert float(errors(far(d), ref).max()) < 1e-10
    assert float(errors(far(x), ref).max()) < 1.02 * float(errors(one_by_one(x), ref).max())
