"""GPU: a beam width without bound is a beam of 1 above the horizon, and still 0 below it.

Pixels below the horizon and slots without a pixel share chunks with pixels
above it here (518 pixels that rise and set); bounds as in test_gpu_parity:
visibilities 1e-5 per channel, adjoint gradients 2e-5, maps 1e-5.
"""
import math

import numpy as np
import pytest

from paper_2504_07090_amd import workload as w
from oracle import mapmaking, model
from tests.gpu_common import chan_rel_err, rel_norm, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vis():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_07090_amd import vis as v
    return v


CFG = w.scaled(w.C0, lmax=8, n_freq=2, n_time=7, dt_s=3600.0, grid_nz=20, grid_nphi=36)


@pytest.mark.parametrize("sep", [True, False])
@pytest.mark.parametrize("value", [math.inf, 1e25, 1e15])   # sigma^2 infinite, finite beyond 1e30, below it
def test_infinite_beam_matches_oracle(vis, value, sep):
    say("infinite beam", value, sep)
    basis = vis.basis_for(CFG, vis.STORAGE_SEPARABLE if sep else 1)
    fld = vis.Field.from_config(basis, CFG, vis.VIS_FP32, vis.VIS_SYNTH_SEPARABLE if sep else vis.VIS_SYNTH_DENSE)
    d = w.draw(CFG, with_noise=False)
    rng = np.random.default_rng(2)
    shape = (CFG.n_time, CFG.n_freq, CFG.n_bl)
    y = rng.normal(size=shape) + 1j * rng.normal(size=shape)
    alm = torch.tensor(d.alm, dtype=torch.float32, device="cuda")
    g = torch.tensor(d.gains, dtype=torch.complex64, device="cuda")
    f = torch.tensor([value], dtype=torch.float32, device="cuda")
    yt = torch.tensor(y, dtype=torch.complex64, device="cuda")
    of = model.Field(CFG)
    m = vis.forward(fld, alm, g, f).cpu().numpy()
    ga, gg, gf = vis.adjoint(fld, alm, g, f, yt)
    mp, wt = vis.make_map(fld, yt, g, f)
    ref = model.forward(of, d.alm, d.gains, 1e6)          # a beam of 1 - 1e-12 at the horizon
    rga, rgg, _ = model.adjoint(of, d.alm, d.gains, 1e6, y)
    rmap, rwt = mapmaking.dirty_map(of, y, d.gains, 1e6)
    errs = (float(np.max(chan_rel_err(m, ref))), rel_norm(ga.cpu().numpy(), rga), rel_norm(gg.cpu().numpy(), rgg))
    emap = (rel_norm(mp.cpu().numpy(), rmap), rel_norm(wt.cpu().numpy(), rwt))
    say(errs, emap, float(gf))
    assert errs[0] <= 1e-5 and max(errs[1:]) <= 2e-5 and max(emap) <= 1e-5
    assert abs(float(gf)) <= 1e-9      # dB/dF = B theta^2 / (sigma^2 F)
