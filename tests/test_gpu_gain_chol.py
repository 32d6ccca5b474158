"""GPU: Cholesky factors of the dense gain blocks at the edges of its kernels.

Blocks up to 128 rows take 16 x 16 threads, larger ones 32 x 32; the bound is that
of the smaller block in test_gpu_serve (1e-5 of the largest entry).
"""
import numpy as np
import pytest

from paper_2504_07090_amd import workload as w
from oracle import hmc as ohmc
from oracle import model
from tests.gpu_common import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# 4 dishes (8 rows), 64 (128, the last of its kernel), 81 (162), 91 (182), 127 (254)
@pytest.mark.parametrize("array,side", [("rhombus", 2), ("rhombus", 8), ("rhombus", 9), ("hex", 6), ("hex", 7)])
def test_factor_times_transpose_is_the_block(array, side):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_07090_amd import serve, vis
    cfg = w.scaled(w.C0, array=array, array_size=side, lmax=4, n_freq=2, n_time=1, grid_nz=12, grid_nphi=24)
    say("gain chol", array, side)
    fld = vis.Field.from_config(vis.basis_for(cfg), cfg)
    d = w.draw(cfg, with_noise=False)
    sig, fw = 1e-3, w.fwhm_ref_rad(cfg)
    ref = ohmc.gain_gauss_newton_blocks(model.Field(cfg), d.alm, d.gains, fw, sig)
    ref += np.eye(ref.shape[1])[None] * 2.0 / cfg.gain_scatter ** 2
    args = (torch.tensor(d.alm, dtype=torch.float32, device="cuda"),
            torch.tensor(d.gains, dtype=torch.complex64, device="cuda"),
            torch.tensor([fw], dtype=torch.float32, device="cuda"), sig)
    l = serve.gain_mass_blocks(fld, *args, cfg.gain_scatter).double().cpu().numpy()
    err = np.max(np.abs(l @ np.transpose(l, (0, 2, 1)) - ref)) / np.max(np.abs(ref))
    say("rel err", err)
    assert err <= 1e-5 and np.array_equal(l, np.tril(l))
    # a non-finite input leaves no finite factor
    bad = (args[0], args[1], torch.tensor([float("nan")], device="cuda"), sig)
    assert not bool(torch.isfinite(serve.gain_mass_blocks(fld, *bad, cfg.gain_scatter)[:, -1, -1]).any())
