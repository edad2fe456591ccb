"""Every translation kernel but the matrix-core one adds up a target's sources
in ascending order with the same fused operations: products of handles that
differ in it alone, and lockstep batches of them, agree bit for bit."""
import numpy as np
import pytest
import torch

import paper_2210_04892_amd as mf
import synth

pytestmark = pytest.mark.gpu

# the level steps fixed, so that the handles share every other stage; tuned at
# 16 right-hand sides, where the LDS-operator shape is kept.  The last one has
# rows of exactly K samples.
KERNELS = [("tiled", 0), ("auto", 0), ("groups", 0), ("lds", 0), ("lds", 32 << 30)]


# 7 680 RWGs (five levels) and 1 080 (three: translations on one level)
@pytest.fixture(scope="module", params=[(16, 1.2), (6, 0.5)], ids=["levels", "single"])
def handles(request):
    v, t = synth.icosphere(*request.param)
    h = [mf.Geometry(v, t, k=2 * np.pi, max_rhs=16, trans_kernel=tk, hbm_budget_bytes=hb, level_kernel="blocked")
         .precompute() for tk, hb in KERNELS]
    yield h
    for g in h:
        g.release()


def vectors(g, nrhs, dtype, seed):
    return torch.from_numpy(synth.gaussian_coeffs(2 * g.n_rwg, nrhs, seed)).to("cuda").to(dtype)


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("nrhs", [1, 2, 3, 4, 5, 7, 8, 9, 15, 16])
def test_far_fields_equal(handles, nrhs, dtype):
    x = vectors(handles[0], nrhs, dtype, 20 + nrhs)
    ref = handles[0].matvec(x, op="C", part=mf.PART_FAR)
    for (name, budget), g in zip(KERNELS[1:], handles[1:]):
        assert torch.equal(g.matvec(x, op="C", part=mf.PART_FAR), ref), (name, budget)


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("nrhs", [1, 2, 5])
def test_lockstep_batch_equals_single_products(handles, nrhs, dtype):
    xs = [vectors(g, nrhs, dtype, 30 + i) for i, g in enumerate(handles)]
    ys = mf.matvec_batch([(g, x, "EM") for g, x in zip(handles, xs)], fused=True)
    for y, g, x in zip(ys, handles, xs):
        assert torch.equal(y, g.matvec(x, op="EM"))


@pytest.mark.parametrize("dtype,tol", [(torch.complex64, 2e-4), (torch.complex128, 1e-11)])
@pytest.mark.parametrize("first", ["matrix", "auto"])
def test_lockstep_batch_with_a_matrix_core_handle(first, dtype, tol):
    """Only handles built for the matrix cores hold that kernel's table of
    groups: beside others they run a kernel all have.  The far field sums
    samples that cancel by 1e4 to 1e5 and is a few percent of the product."""
    big, small = synth.icosphere(16, 1.2), synth.icosphere(6, 0.5)
    kinds = [first, "auto" if first == "matrix" else "matrix"]
    gs = [mf.Geometry(v, t, k=2 * np.pi, max_rhs=4, trans_kernel=tk).precompute()
          for (v, t), tk in zip((big, small), kinds)]
    xs = [vectors(g, 4, dtype, 50 + i) for i, g in enumerate(gs)]
    for y, g, x in zip(mf.matvec_batch([(g, x, "C") for g, x in zip(gs, xs)], fused=True), gs, xs):
        want = g.matvec(x, op="C")
        assert float(torch.linalg.norm(y - want) / torch.linalg.norm(want)) < tol
    for g in gs:
        g.release()
