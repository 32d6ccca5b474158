"""GPU: the staged gains pass over several times per block, and with many unique baselines.

A block keeps a channel's tables for a slab of consecutive times and loads the
next time's data ahead; with this many slices every size of it takes slabs of
four times and a shorter last one.  An irregular array of 30 antennas has more
unique baselines than the pass has threads in its smallest size.  Every channel
against the FP64 oracle; bounds as in test_gpu_parity: chi^2 1e-4 and its
gradient 2e-4 at 1.2 times the sky, adjoint gradients 2e-5, ten times as much for
the split precision.
"""
import numpy as np
import pytest

from paper_2504_07090_amd import workload as w
from oracle import model
from tests.gpu_common import rel_norm, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vis():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_07090_amd import vis as v
    return v


BASE = w.scaled(w.C0, lmax=4, grid_nz=12, grid_nphi=24)


def _compare(vis, cfg, precision):
    bar = 1.0 if precision == "fp32" else 10.0
    prec = vis.VIS_FP32 if precision == "fp32" else vis.VIS_FP16X3
    fld = vis.Field.from_config(vis.basis_for(cfg, vis.STORAGE_SEPARABLE), cfg, prec, vis.VIS_SYNTH_SEPARABLE)
    d = w.draw(cfg)
    of = model.Field(cfg)
    fw = w.fwhm_ref_rad(cfg)
    _, sig, data = model.make_data(of, d)
    alm = torch.tensor(d.alm * 1.2, dtype=torch.float32, device="cuda")
    g = torch.tensor(d.gains, dtype=torch.complex64, device="cuda")
    f = torch.tensor([fw], dtype=torch.float32, device="cuda")
    y = torch.tensor(np.ascontiguousarray(data), dtype=torch.complex64, device="cuda")
    _, v, img = model.forward(of, d.alm * 1.2, d.gains, fw, return_parts=True)
    x2, ga, gg, gf = vis.chi2_and_grad(fld, y, sig, alm, g, f)
    r = data - model.forward(of, d.alm * 1.2, d.gains, fw)
    r2 = model.chi2(of, data, sig, data - r)
    rga, rgg, rgf = model.adjoint(of, d.alm * 1.2, d.gains, fw, -2.0 * r / sig ** 2, parts=(v, img))
    errs = (rel_norm(ga.cpu().numpy(), rga), rel_norm(gg.cpu().numpy(), rgg), abs(float(gf) - rgf) / abs(rgf))
    say("chi2", abs(float(x2) - r2) / r2, errs)
    assert abs(float(x2) - r2) <= 1e-4 * bar * r2
    assert max(errs) <= 2e-4 * bar
    ga, gg, gf = vis.adjoint(fld, alm, g, f, y)
    rga, rgg, rgf = model.adjoint(of, d.alm * 1.2, d.gains, fw, data, parts=(v, img))
    errs = (rel_norm(ga.cpu().numpy(), rga), rel_norm(gg.cpu().numpy(), rgg), abs(float(gf) - rgf) / abs(rgf))
    say("adjoint", errs)
    assert max(errs) <= 2e-5 * bar


# 2016 baselines (256 threads), 4095 (512), 7260 (1024)
@pytest.mark.parametrize("array,side,n_freq,n_time", [("rhombus", 8, 33, 97), ("hex", 6, 17, 97), ("rhombus", 11, 17, 50)])
def test_slabs_of_times(vis, array, side, n_freq, n_time):
    say("gains slabs", array, side)
    _compare(vis, w.scaled(BASE, array=array, array_size=side, n_freq=n_freq, n_time=n_time), "fp32")


@pytest.mark.parametrize("precision", ["fp32", "fp16x3"])
def test_irregular_array(vis, monkeypatch, precision):
    say("irregular array", precision)
    rng = np.random.default_rng(4)
    cells = rng.choice(17 * 17, size=30, replace=False)
    lattice = np.stack([cells % 17, cells // 17], axis=1).astype(np.int64)
    diffs = {max((a, b), (-a, -b)) for p in lattice for q in lattice if (p != q).any() for a, b in [tuple(p - q)]}
    assert 256 < len(diffs) <= 512
    monkeypatch.setattr(w, "antenna_lattice", lambda cfg: lattice)
    _compare(vis, w.scaled(BASE, n_freq=9, n_time=7), precision)
