"""The whole-box disaggregation (from the second octree level down, where the
parents' samples are many) against the chunked kernels, which add up the same
terms in the same order (and, where a chunk does not fit its limits, the two
kernels through global memory, whose weights are rounded differently)."""
import pytest
import torch

import paper_2210_04892_amd as mf
import synth

pytestmark = pytest.mark.gpu


# 276 480 and 39 600 RWGs: the largest samples and four steps, then rows and
# columns that do not fill a wave
@pytest.fixture(scope="module", params=["sphere", "ellipsoid"])
def handles(request):
    v, t = synth.icosphere(96, 8.0) if request.param == "sphere" else synth.ellipsoid(40, (3.2, 2.4, 1.6))
    kw = dict(k=2 * 3.141592653589793, max_rhs=3)
    h = [mf.Geometry(v, t, level_kernel=lk, **kw).precompute() for lk in ("blocked", "auto")]
    yield h, request.param
    for g in h:
        g.release()


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("nrhs", [1, 2, 3])
def test_box_disaggregation_matches(handles, nrhs, dtype):
    handles, name = handles
    x = torch.from_numpy(synth.gaussian_coeffs(2 * handles[0].n_rwg, nrhs, 50 + nrhs)).to("cuda").to(dtype)
    a, b = (g.matvec(x, op="C", part=mf.PART_FAR) for g in handles)
    if name == "sphere" and dtype == torch.complex128:   # two kernels from 58 x 116 samples down
        # a sum of samples that cancels by 1e4 to 1e5
        assert float(torch.linalg.norm(a - b) / torch.linalg.norm(b)) < 1e-11
    else:
        assert torch.equal(a, b)


@pytest.mark.parametrize("code,dtype", [(mf.C64, torch.complex64), (mf.C128, torch.complex128)])
def test_captured_box_steps_match(handles, code, dtype):
    """A captured product replays the kernels that use more than the default LDS."""
    g = handles[0][1]
    n = 2 * g.n_rwg
    x, x2 = (torch.from_numpy(synth.gaussian_coeffs(n, 1, s)[:, 0].copy()).to("cuda").to(dtype) for s in (5, 6))
    want = g.matvec(x, op="C")
    y = torch.empty_like(x)
    graph = g.capture("C", code, 1, x.data_ptr(), n, y.data_ptr(), n)
    for _ in range(3):
        y.fill_(7)
        graph.launch(torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(y, want)
        g.matvec(x2, op="C")
        torch.cuda.synchronize()
    graph.close()
