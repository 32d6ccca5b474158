"""GPU: gradients written over the parameters they were taken at are the same."""
import math

import ctypes
import numpy as np
import pytest

from paper_2504_07090_amd import workload as w

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vis():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_07090_amd import vis as v
    return v


CFG = w.scaled(w.C0, lmax=8, n_freq=3, n_time=3, grid_nz=24, grid_nphi=48)


@pytest.mark.parametrize("sep", [True, False])
def test_grad_fwhm_over_fwhm(vis, sep):
    basis = vis.basis_for(CFG, vis.STORAGE_SEPARABLE if sep else 1)
    fld = vis.Field.from_config(basis, CFG, vis.VIS_FP32, vis.VIS_SYNTH_SEPARABLE if sep else vis.VIS_SYNTH_DENSE)
    d = w.draw(CFG, with_noise=False)
    rng = np.random.default_rng(5)
    shape = (CFG.n_time, CFG.n_freq, CFG.n_bl)
    # small cotangents: a dL/dF far below any beam width
    y = torch.tensor(1e-9 * (rng.normal(size=shape) + 1j * rng.normal(size=shape)), dtype=torch.complex64, device="cuda")
    alm = torch.tensor(d.alm, dtype=torch.float32, device="cuda")
    g = torch.tensor(d.gains, dtype=torch.complex64, device="cuda")
    f = torch.tensor([math.radians(20.0)], dtype=torch.float32, device="cuda")
    want = vis.adjoint(fld, alm, g, f, y)
    ga, gg, both = torch.empty_like(alm), torch.empty_like(g), f.clone()
    status = vis._lib.vis_adjoint(fld.handle, vis._ptr(alm), vis._ptr(g), vis._ptr(both), vis._ptr(y), vis._ptr(ga),
                                  vis._ptr(gg), vis._ptr(both), ctypes.c_void_p(vis._stream()))
    assert status == 0
    assert all(torch.equal(a, b) for a, b in zip((ga, gg, both), want))


@pytest.mark.parametrize("sep", [True, False])
@pytest.mark.parametrize("entry", ["adjoint", "chi2"])
def test_all_gradients_over_their_parameters(vis, entry, sep):
    basis = vis.basis_for(CFG, vis.STORAGE_SEPARABLE if sep else 1)
    fld = vis.Field.from_config(basis, CFG, vis.VIS_FP32, vis.VIS_SYNTH_SEPARABLE if sep else vis.VIS_SYNTH_DENSE)
    d = w.draw(CFG, with_noise=False)
    rng = np.random.default_rng(6)
    shape = (CFG.n_time, CFG.n_freq, CFG.n_bl)
    y = torch.tensor(rng.normal(size=shape) + 1j * rng.normal(size=shape), dtype=torch.complex64, device="cuda")
    alm = torch.tensor(d.alm, dtype=torch.float32, device="cuda")
    g = torch.tensor(d.gains, dtype=torch.complex64, device="cuda")
    f = torch.tensor([math.radians(20.0)], dtype=torch.float32, device="cuda")
    p, s = vis._ptr, ctypes.c_void_p(vis._stream())
    a2, g2, f2 = alm.clone(), g.clone(), f.clone()
    if entry == "adjoint":
        want = vis.adjoint(fld, alm, g, f, y)
        status = vis._lib.vis_adjoint(fld.handle, p(a2), p(g2), p(f2), p(y), p(a2), p(g2), p(f2), s)
    else:
        x2, *want = vis.chi2_and_grad(fld, y, 1.0, alm, g, f)
        out = torch.empty((), dtype=torch.float64, device="cuda")
        status = vis._lib.chi2_and_grad(fld.handle, p(y), ctypes.c_float(1.0), p(a2), p(g2), p(f2), p(out), p(a2),
                                        p(g2), p(f2), s)
        assert float(out) == float(x2)
    assert status == 0
    assert all(torch.equal(a, b) for a, b in zip((a2, g2, f2), want))
