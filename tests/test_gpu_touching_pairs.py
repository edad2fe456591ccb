"""Near-field integrals in double precision over both forms of the kernel's
cosine and sine (pairs whose k R stays below 2, and above it)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2210_04892_amd as mf
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mesh,leaf,k", [
    (synth.rounded_box((0.6, 0.45, 0.3), 0.06, 0.15), 0.3, 4 * np.pi),   # touching pairs with k R up to 5
    (synth.octahedron(0.1), 0.25, 2 * np.pi),                            # k R below 1, every pair touches
])
@pytest.mark.parametrize("op", ["C", "EM"])
def test_near_field_wavenumbers(mesh, leaf, k, op):
    v, t = mesh
    n2 = 3 * len(t)
    x = synth.gaussian_coeffs(n2, 1, 23)[:, 0]
    g = mf.Geometry(v, t, k=k, leaf=leaf).precompute()
    y = g.matvec(torch.from_numpy(x).cuda(), op=op, part=mf.PART_NEAR).cpu().numpy()
    g.release()
    both = oracle.matvec(v, t, k, x, op=oracle.OP_BOTH, leaf=leaf, classes=True)
    ref = both[0 if op == "C" else 1][0]
    # the oracle's own order search stops at 3e-11 of a pair's largest entry
    assert np.linalg.norm(y - ref) / np.linalg.norm(ref) < 1e-10
