"""GPU: the filtered likelihood at the channel counts where its kernels change.

Up to 240 channels one block holds all rows of its columns, a wave per 16; beyond,
the filtered residual passes through memory.  The bounds are those of
test_gpu_filter: the arithmetic is the same.
"""
import numpy as np
import pytest

from oracle import filter as fl
from oracle import model
from paper_2504_07090_amd import workload as w
from tests.gpu_common import GRAD_ELEM_FP32, max_rel, rel_norm, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# 7 dishes (42 real columns, a ragged block) and 19 (342, six blocks)
@pytest.mark.parametrize("side,nf", [(2, 1), (2, 64), (3, 65), (2, 17), (2, 239), (2, 240), (2, 241)])
def test_filtered_chi2_and_gradient(side, nf):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_07090_amd import vis
    cfg = w.scaled(w.C0, array="hex", array_size=side, n_freq=nf, n_time=2, lmax=4, grid_nz=12,
                   grid_nphi=24, freq_lo_hz=120e6, freq_hi_hz=130e6)
    say("filter rows", side, nf)
    fld = vis.Field.from_config(vis.basis_for(cfg), cfg)
    filt = vis.Filter(w.frequencies(cfg))
    d, of = w.draw(cfg), model.Field(cfg)
    _, sig, data = model.make_data(of, d)
    f = fl.delay_filter(w.frequencies(cfg))
    fw = w.fwhm_ref_rad(cfg)
    ref = fl.chi2_filtered_and_grad(of, data, sig, f, d.alm * 1.2, d.gains, fw)
    args = (torch.tensor(np.ascontiguousarray(data), dtype=torch.complex64, device="cuda"), sig,
            torch.tensor(d.alm * 1.2, dtype=torch.float32, device="cuda"),
            torch.tensor(d.gains, dtype=torch.complex64, device="cuda"),
            torch.tensor([fw], dtype=torch.float32, device="cuda"))
    x2, ga, gg, gf = vis.chi2_filtered_and_grad(fld, filt, *args)
    e = [abs(float(x2) - ref[0]) / ref[0], rel_norm(ga.cpu().numpy(), ref[1]), rel_norm(gg.cpu().numpy(), ref[2]),
         abs(float(gf) - ref[3]) / abs(ref[3])]
    em = [max_rel(ga.cpu().numpy(), ref[1]), max_rel(gg.cpu().numpy(), ref[2])]
    say("errs (chi2, a, g, F)", e, "element-wise (a, g)", em)
    assert max(e) <= 2e-4 and max(em) <= GRAD_ELEM_FP32
    x2b, *_ = vis.chi2_filtered_and_grad(fld, filt, *args, grads=False)
    assert float(x2b) == float(x2)
