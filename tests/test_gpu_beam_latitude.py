"""GPU: the beam cut far from the equator, for skies that are faint at the beam centre.

A harmonic of |m| = l falls as cos^l(dec) towards the poles, each of its values
exact relative to itself, so at a high latitude the outskirts of the beam carry
its visibilities.  The references sum every pixel above the horizon in FP64;
bounds as in test_gpu_parity: visibilities 1e-5 per channel, gradients of the
single modes max |error| / rms 2e-3.
"""
import numpy as np
import pytest

from paper_2504_07090_amd import workload as w
from oracle import model
from tests.gpu_common import GRAD_ELEM_FP32, chan_rel_err, max_rel, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vis():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_07090_amd import vis as v
    return v


L = 60
BASE = w.scaled(w.C0, array="hex", array_size=3, lmax=L, n_freq=3, n_time=2, dt_s=3600.0, grid_nz=64, grid_nphi=192)


# the largest terms lie 6 to 35 powers of two down the beam; amplitudes of 1e8, so
# that visibilities and gradients (down to 2e-34 of them) stay clear of FP32's smallest numbers
@pytest.mark.parametrize("sep", [True, False])
@pytest.mark.parametrize("lat,fwhm", [(-45.0, 10.0), (-60.0, 8.0), (75.0, 10.0), (-90.0, 10.0), (-90.0, 14.0)])
def test_sectoral_modes(vis, lat, fwhm, sep):
    cfg = w.scaled(BASE, latitude_deg=lat, fwhm_ref_deg=fwhm)
    say("beam latitude", lat, fwhm, sep)
    basis = vis.basis_for(cfg, vis.STORAGE_SEPARABLE if sep else 1)
    fld = vis.Field.from_config(basis, cfg, vis.VIS_FP32, vis.VIS_SYNTH_SEPARABLE if sep else vis.VIS_SYNTH_DENSE)
    of = model.Field(cfg)
    fw = w.fwhm_ref_rad(cfg)
    g = np.ones((cfg.n_freq, cfg.n_ant))
    dev = dict(device="cuda")
    gt, ft = torch.tensor(g, dtype=torch.complex64, **dev), torch.tensor([fw], dtype=torch.float32, **dev)
    rng = np.random.default_rng(3)
    shape = (cfg.n_time, cfg.n_freq, cfg.n_bl)
    y = 1e8 * (rng.normal(size=shape) + 1j * rng.normal(size=shape))
    for m in (L, L // 2):
        alm = np.zeros((cfg.n_freq, cfg.n_modes))
        idx = [m * m + m - m, m * m + m + m]     # l = |m|, both signs
        alm[:, idx] = 1e8 * rng.normal(size=(cfg.n_freq, 2))
        at = torch.tensor(alm, dtype=torch.float32, **dev)
        alm = at.cpu().numpy().astype(np.float64)
        v = vis.forward(fld, at, gt, ft).cpu().numpy().astype(np.complex128)
        ref = model.forward(of, alm, g, fw)
        e = float(np.max(chan_rel_err(v, ref)))
        ga = vis.adjoint(fld, at, gt, ft, torch.tensor(y, dtype=torch.complex64, **dev))[0].cpu().numpy()
        rga = model.adjoint(of, alm, g, fw, y)[0]
        eg = max_rel(ga[:, idx].astype(np.float64), rga[:, idx])
        say(m, e, eg)
        assert e <= 1e-5 and eg <= GRAD_ELEM_FP32
