"""Products whose near field follows the radiation on the caller's stream (few
near-field values) and those just past that line, whose near field runs on a
side stream, against the sum of their near and far parts."""
import pytest
import torch

import paper_2210_04892_amd as mf
import synth

pytestmark = pytest.mark.gpu


# 1 080 RWGs on three levels, 3 630 on four (16 MB of near blocks in
# complex64, 32 in complex128), 7 680 on five (34 MB)
@pytest.fixture(scope="module", params=[6, 11, 16])
def geometry(request):
    v, t = synth.icosphere(request.param, 0.5 if request.param == 6 else 0.075 * request.param)
    g = mf.Geometry(v, t, k=2 * 3.141592653589793, max_rhs=4).precompute()
    yield g
    g.release()


# The parts run the same kernels: their sum differs by the rounding of the last
# addition and, with one right-hand side, of the radiation's sums, which the
# cancellation of the translation raises to 1e5 times that of the type at most.
@pytest.mark.parametrize("dtype,tol", [(torch.complex64, 2e-5), (torch.complex128, 1e-11)])
@pytest.mark.parametrize("op", ["C", "EM"])
@pytest.mark.parametrize("nrhs", [1, 2, 4])
def test_product_is_sum_of_parts(geometry, nrhs, op, dtype, tol):
    xs = [torch.from_numpy(synth.gaussian_coeffs(2 * geometry.n_rwg, nrhs, 70 + s)).to("cuda").to(dtype)
          for s in range(4)]
    want = [geometry.matvec(x, op=op, part=mf.PART_NEAR) + geometry.matvec(x, op=op, part=mf.PART_FAR) for x in xs]
    got = [geometry.matvec(x, op=op) for x in xs]      # in a row, on one workspace
    for a, b in zip(got, want):
        assert float(torch.linalg.norm(a - b) / torch.linalg.norm(b)) < tol


@pytest.mark.parametrize("code,dtype", [(mf.C64, torch.complex64), (mf.C128, torch.complex128)])
def test_captured_product_matches(geometry, code, dtype):
    n = 2 * geometry.n_rwg
    x, x2 = (torch.from_numpy(synth.gaussian_coeffs(n, 1, s)[:, 0].copy()).to("cuda").to(dtype) for s in (5, 6))
    want = geometry.matvec(x, op="C")
    y = torch.empty_like(x)
    graph = geometry.capture("C", code, 1, x.data_ptr(), n, y.data_ptr(), n)
    for _ in range(3):
        y.fill_(7)
        graph.launch(torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(y, want)
        geometry.matvec(x2, op="C")
        torch.cuda.synchronize()
    graph.close()
