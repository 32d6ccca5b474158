"""GPU: the two ways the adjoint fringe pass takes its (chunk, channel group) items.

Many items: a wave takes whole items (more times than the 64 list entries its
lanes hold, or few times and most chunks outside the beam); few items: a block's
waves share one item.  Sparse arrays reach every tile extent with few baselines, a
short one among them (long ones alone would see next to nothing).
Sampled channels against the FP64 oracle (the cotangent is zero at the others, so
dL/dF is theirs too); bounds as in test_gpu_parity: visibilities 1e-5 per
channel, adjoint gradients 2e-5, ten times as much for the split precision.
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


BASE = w.scaled(w.C0, lmax=4, freq_lo_hz=120e6, freq_hi_hz=130e6, grid_nz=128, grid_nphi=384)
# extent of the array, channels, times, FWHM (deg)
CASES = {
    "whole, 70 times": [(2, 150, 70, 60.0), (4, 301, 70, 60.0), (8, 150, 70, 60.0), (12, 101, 70, 60.0)],
    "whole, some outside": [(4, 81, 5, 10.0), (6, 41, 5, 10.0), (12, 47, 6, 10.0)],
    "shared": [(4, 9, 70, 60.0), (8, 9, 70, 20.0), (12, 9, 20, 20.0)],
    # ... by blocks, those sure to be outside by waves
    "shared, some outside": [(4, 11, 6, 10.0), (8, 6, 5, 10.0), (12, 9, 5, 10.0)],
}


@pytest.mark.parametrize("precision", ["fp32", "fp16x3"])
@pytest.mark.parametrize("kind,case", [(k, c) for k, v in CASES.items() for c in v])
def test_items_match_oracle(vis, monkeypatch, kind, case, precision):
    extent, n_freq, n_time, fwhm = case
    say("adjoint items", kind, case, precision)
    e = extent
    lattice = np.array([(0, 0), (1, 0), (e, 0), (0, e), (e // 2, e // 2), (e, e - 1)], dtype=np.int64)
    monkeypatch.setattr(w, "antenna_lattice", lambda cfg: lattice)
    # a narrow beam needs a sky with structure: lmax 4 would leave 1e-3 of the sum's terms
    cfg = w.scaled(BASE, n_freq=n_freq, n_time=n_time, lmax=4 if fwhm >= 60.0 else 40)
    prec = vis.VIS_FP32 if precision == "fp32" else vis.VIS_FP16X3
    fld = vis.Field.from_config(vis.basis_for(cfg, vis.STORAGE_SEPARABLE), cfg, prec, vis.VIS_SYNTH_SEPARABLE)
    of = model.Field(cfg)
    fw = math.radians(fwhm)
    d = w.draw(cfg, with_noise=False)
    ch = [0, n_freq - 1]
    rng = np.random.default_rng(7)
    y = np.zeros((n_time, n_freq, cfg.n_bl), dtype=np.complex128)
    shape = (n_time, len(ch), cfg.n_bl)
    y[:, ch] = rng.normal(size=shape) + 1j * rng.normal(size=shape)
    alm = torch.tensor(d.alm, dtype=torch.float32, device="cuda")
    g = torch.tensor(d.gains, dtype=torch.complex64, device="cuda")
    f = torch.tensor([fw], dtype=torch.float32, device="cuda")
    m = vis.forward(fld, alm, g, f).cpu().numpy()[:, ch]
    ga, gg, gf = vis.adjoint(fld, alm, g, f, torch.tensor(y, dtype=torch.complex64, device="cuda"))
    ref, v, img = model.forward(of, d.alm, d.gains, fw, ch, return_parts=True)
    rga, rgg, rgf = model.adjoint(of, d.alm, d.gains, fw, y[:, ch], ch, parts=(v, img))
    errs = (float(np.max(chan_rel_err(m, ref))), rel_norm(ga.cpu().numpy()[ch], rga),
            rel_norm(gg.cpu().numpy()[ch], rgg), abs(float(gf) - rgf) / abs(rgf))
    say(errs)
    bar = 1.0 if precision == "fp32" else 10.0
    assert errs[0] <= 1e-5 * bar and max(errs[1:]) <= 2e-5 * bar
    others = np.setdiff1d(np.arange(n_freq), ch)
    assert not ga[others].any() and not gg[others].any()
