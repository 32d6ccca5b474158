"""GPU: a map with an undefined beam or gain leaves nothing behind in the field."""
import math

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


# 518 pixels are up at some time: the last chunk of 64 slots holds 58 without a pixel
CFG = w.scaled(w.C0, lmax=8, n_freq=2, n_time=7, dt_s=3600.0, grid_nz=20, grid_nphi=36)


@pytest.mark.parametrize("sep", [True, False])
@pytest.mark.parametrize("what", ["fwhm", "gains", "huge gains"])
def test_evaluation_after_undefined_map(vis, what, sep):
    basis = vis.basis_for(CFG, vis.STORAGE_SEPARABLE if sep else 1)
    syn = vis.VIS_SYNTH_SEPARABLE if sep else vis.VIS_SYNTH_DENSE
    d = w.draw(CFG, with_noise=False)
    rng = np.random.default_rng(1)
    shape = (CFG.n_time, CFG.n_freq, CFG.n_bl)
    y = torch.tensor(rng.normal(size=shape) + 1j * rng.normal(size=shape), dtype=torch.complex64, device="cuda")
    alm = torch.tensor(d.alm, dtype=torch.float32, device="cuda")
    g = torch.tensor(d.gains, dtype=torch.complex64, device="cuda")
    wide = torch.tensor([math.radians(75.0)], dtype=torch.float32, device="cuda")   # every chunk within the beam

    def evaluate(fld):
        return (vis.forward(fld, alm, g, wide),) + tuple(vis.adjoint(fld, alm, g, wide, y))

    want = evaluate(vis.Field.from_config(basis, CFG, vis.VIS_FP32, syn))
    used = vis.Field.from_config(basis, CFG, vis.VIS_FP32, syn)
    bad_f = torch.full_like(wide, math.nan) if what == "fwhm" else wide
    bad_g = g if what == "fwhm" else g * math.nan if what == "gains" else g * 1e30
    vis.make_map(used, y, bad_g, bad_f)
    got = evaluate(used)
    assert all(bool(torch.isfinite(torch.view_as_real(x) if x.is_complex() else x).all()) for x in want)
    assert all(torch.equal(a, b) for a, b in zip(got, want))
