"""GPU: separable synthesis beyond one segment of degrees and one round of rings, and tiny grids.

The forward Legendre stage gathers 128 degrees at a time and a block's waves take
128 rings per round; a grid of fewer than 64 visible pixels is one partial chunk.
Against the FP64 oracle; bounds as in test_gpu_parity: visibilities 1e-5 per
channel, adjoint gradients 2e-5.
"""
import math

import numpy as np
import pytest

from paper_2504_07090_amd import workload as w
from oracle import model
from tests.gpu_common import chan_rel_err, rel_norm, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vis():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_07090_amd import vis as v
    return v


# lmax, rings, columns, FWHM (deg): degrees 128 and 129 in number, both more rings than
# one round and a narrow beam of few; one partial chunk
@pytest.mark.parametrize("lmax,nz,nphi,fwhm", [(127, 144, 24, 70.0), (128, 144, 24, 70.0), (150, 144, 24, 70.0),
                                               (150, 36, 48, 20.0), (4, 4, 8, 70.0), (3, 6, 10, 30.0)])
def test_sizes_match_oracle(vis, lmax, nz, nphi, fwhm):
    say("separable sizes", lmax, nz, nphi, fwhm)
    cfg = w.scaled(w.C0, lmax=lmax, grid_nz=nz, grid_nphi=nphi, n_freq=3, n_time=2)
    fld = vis.Field.from_config(vis.basis_for(cfg, vis.STORAGE_SEPARABLE), cfg, vis.VIS_FP32, vis.VIS_SYNTH_SEPARABLE)
    of = model.Field(cfg)
    fw = math.radians(fwhm)
    d = w.draw(cfg, with_noise=False)
    rng = np.random.default_rng(8)
    shape = (cfg.n_time, cfg.n_freq, cfg.n_bl)
    y = rng.normal(size=shape) + 1j * rng.normal(size=shape)
    alm = torch.tensor(d.alm, dtype=torch.float32, device="cuda")
    g = torch.tensor(d.gains, dtype=torch.complex64, device="cuda")
    f = torch.tensor([fw], dtype=torch.float32, device="cuda")
    m = vis.forward(fld, alm, g, f).cpu().numpy()
    ga, gg, gf = vis.adjoint(fld, alm, g, f, torch.tensor(y, dtype=torch.complex64, device="cuda"))
    ref, v, img = model.forward(of, d.alm, d.gains, fw, return_parts=True)
    rga, rgg, rgf = model.adjoint(of, d.alm, d.gains, fw, y, parts=(v, img))
    # dL/dF = Re<y, dm/dF>, against the size of its factors (it may cancel)
    h = 1e-4
    dm = (model.forward(of, d.alm, d.gains, fw * (1 + h)) - model.forward(of, d.alm, d.gains, fw * (1 - h))) / (2 * h * fw)
    errs = (float(np.max(chan_rel_err(m, ref))), rel_norm(ga.cpu().numpy(), rga), rel_norm(gg.cpu().numpy(), rgg),
            abs(float(gf) - rgf) / float(np.linalg.norm(y) * np.linalg.norm(dm)))
    say(errs)
    assert errs[0] <= 1e-5 and max(errs[1:]) <= 2e-5
