"""The solver's orthogonalisation against a least-squares problem on an
explicit Krylov basis: steps below, at and above a batch of inner products,
one and several columns, with and without restarts."""
import numpy as np
import pytest
import torch

import paper_2210_04892_amd as mf
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[4, 12])
def geom(request):
    # 480 RWGs (less than two row chunks) and 4 320
    v, t = synth.icosphere(request.param, request.param / 12.0)
    g = mf.Geometry(v, t, k=2 * np.pi, max_rhs=3).precompute()
    yield g
    g.release()


def reference(g, b, steps):
    """Residual norm of the best correction from the Krylov space of steps vectors."""
    q = [b / torch.linalg.norm(b)]
    aq = []
    for _ in range(steps):
        a = g.matvec(q[-1].contiguous(), op="C")
        aq.append(a)
        w = a.clone()
        for _ in range(3):
            for u in q:
                w -= torch.vdot(u, w) * u
        q.append(w / torch.linalg.norm(w))
    m = torch.stack(aq, 1).cpu()
    r = b.cpu()
    y = torch.linalg.lstsq(m, r.unsqueeze(1)).solution[:, 0]
    return r - m @ y


@pytest.mark.parametrize("nrhs", [1, 3])
@pytest.mark.parametrize("steps,restart", [(1, 8), (3, 8), (4, 8), (5, 8), (9, 12), (9, 4)])
def test_steps_minimise_the_residual(geom, nrhs, steps, restart):
    b = torch.from_numpy(synth.gaussian_coeffs(2 * geom.n_rwg, nrhs, 33)).to("cuda")
    x, iters, rel = geom.gmres(b, op="C", restart=restart, max_iters=steps, tol=1e-14)
    assert iters == steps
    for r in range(nrhs):
        res, left = b[:, r].clone(), steps
        while left:
            res = reference(geom, res, min(left, restart)).to("cuda")
            left -= min(left, restart)
        want = float(torch.linalg.norm(res) / torch.linalg.norm(b[:, r]))
        # products carry 1e-11 of their norm as rounding, ten steps of a
        # second-kind system amplify it by less than its condition (below 1e3)
        assert abs(rel[r] - want) < 1e-8 * max(want, 1e-3) + 1e-9
