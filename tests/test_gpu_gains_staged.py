"""GPU: the gains pass of arrays too large for all staged terms in LDS.

Its sizes: above 61 dishes up to 64 (2048 baselines), 96 (4608) and 128 (8192),
and beyond, where the lists are walked in memory.  The sums are those of the FP32
path, so the bounds are test_gpu_parity's: adjoint gradients 2e-5, chi^2 1e-4
with its gradient 2e-4 at 1.2 times the sky, maps 1e-5.
"""
import numpy as np
import pytest

from paper_2504_07090_amd import workload as w
from oracle import mapmaking, model
from tests.gpu_common import rel_norm, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vis():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_07090_amd import vis as v
    return v


# (array, side): 64 and 81 dishes on a rhombus, 91 and 127 on a hexagon, 121 on a
# rhombus, 144 beyond the staged sizes
@pytest.mark.parametrize("array,side", [("rhombus", 8), ("rhombus", 9), ("hex", 6), ("hex", 7), ("rhombus", 11),
                                        ("rhombus", 12)])
@pytest.mark.parametrize("precision", ["fp32", "fp16x3"])
def test_gains_pass_matches_oracle(vis, array, side, precision):
    cfg = w.scaled(w.C0, array=array, array_size=side, lmax=6, n_freq=3, n_time=5, grid_nz=16, grid_nphi=32)
    say("staged gains", array, side, precision)
    prec = vis.VIS_FP32 if precision == "fp32" else vis.VIS_FP16X3
    basis = vis.basis_for(cfg, vis.STORAGE_SEPARABLE)
    fld = vis.Field.from_config(basis, cfg, prec, vis.VIS_SYNTH_SEPARABLE)
    d = w.draw(cfg)
    of = model.Field(cfg)
    fw = w.fwhm_ref_rad(cfg)
    _, sig, data = model.make_data(of, d)
    alm = torch.tensor(d.alm * 1.2, dtype=torch.float32, device="cuda")
    g = torch.tensor(d.gains, dtype=torch.complex64, device="cuda")
    f = torch.tensor([fw], dtype=torch.float32, device="cuda")
    y = torch.tensor(np.ascontiguousarray(data), dtype=torch.complex64, device="cuda")
    bar = 1.0 if precision == "fp32" else 10.0
    x2, ga, gg, gf = vis.chi2_and_grad(fld, y, sig, alm, g, f)
    r2, rga, rgg, rgf = model.chi2_and_grad(of, data, sig, d.alm * 1.2, d.gains, fw)
    assert abs(float(x2) - r2) <= 1e-4 * bar * r2
    errs = (rel_norm(ga.cpu().numpy(), rga), rel_norm(gg.cpu().numpy(), rgg), abs(float(gf) - rgf) / abs(rgf))
    say("chi2", errs)
    assert max(errs) <= 2e-4 * bar
    ga, gg, gf = vis.adjoint(fld, alm, g, f, y)
    rga, rgg, rgf = model.adjoint(of, d.alm * 1.2, d.gains, fw, data)
    errs = (rel_norm(ga.cpu().numpy(), rga), rel_norm(gg.cpu().numpy(), rgg), abs(float(gf) - rgf) / abs(rgf))
    say("adjoint", errs)
    assert max(errs) <= 2e-5 * bar
    mp, wt = vis.make_map(fld, y, g, f)
    rmap, rwt = mapmaking.dirty_map(of, data, d.gains, fw)
    errs = (rel_norm(mp.cpu().numpy(), rmap), rel_norm(wt.cpu().numpy(), rwt))
    say("map", errs)
    assert max(errs) <= 1e-5 * bar
