"""Timed cases of the visibility / chi^2 / gradient / HMC library.

Each case is one call (or, for the server, one request per chain) of the
public Python entry points on a synthetic observation: a hexagonal or rhombic
lattice array of 14.6 m spacing, a drift scan of one-minute samples at
latitude -30.7 deg, a band between 120 and 180 MHz, and a sky of spherical
harmonics on an equal-area grid.  Parameters are those of a chain at its start:
a prior draw of the sky coefficients, 5% gains, a beam width a few percent off;
the data are the visibilities of a few dozen point sources, with gains of their
own and noise of half their rms, so the residual is as large as the data.

`listed()` gives the fixed cases, `draw(rng)` others of the same ranges,
`prepare` and `run` one call, `work` what it cannot do without and `exact` its
results in 64 bits from torch alone (no code of this package).
"""
import math

import numpy as np
import torch

from paper_2504_07090_amd import serve, vis, workload

SPACING_M, LAT_DEG, DT_S, REF_HZ = 14.6, -30.7, 60.0, 150e6
OMEGA = 7.2921159e-5            # sidereal rate, rad per solar second
C_LIGHT = 299792458.0
GAIN_SCATTER, NOISE_FRAC, DATA_RMS, N_SOURCES = 0.05, 0.5, 0.003, 24
TAU_MAX_S, NOISE_RATIO = 250e-9, 1e-8   # delay filter half-width and regulariser
PROBES = 4                              # Hutchinson probes of a mass-matrix set-up

PRECISION = {"fp32": vis.VIS_FP32, "bf16x3": vis.VIS_BF16X3, "fp16x3": vis.VIS_FP16X3}
SYNTHESIS = {"dense": vis.VIS_SYNTH_DENSE, "separable": vis.VIS_SYNTH_SEPARABLE}


def _case(name, op, array, side, n_freq, n_time, lmax, grid=(128, 384), band=(120e6, 130e6),
          fwhm_deg=10.0, precision="fp32", synthesis="separable"):
    c = dict(op=op, array=array, side=side, n_freq=n_freq, n_time=n_time, lmax=lmax,
             grid_nz=grid[0], grid_nphi=grid[1], freq_lo_hz=band[0], freq_hi_hz=band[1],
             fwhm_deg=fwhm_deg, precision=precision, synthesis=synthesis)
    return c if name is None else dict(name=name, **c)


def listed():
    return [
        # the smallest likelihood evaluation in use (16 dishes, a coarse sky): latency and launches
        _case("chi2_grad_16", "chi2_grad", "rhombus", 4, 8, 4, 20, (32, 96), (120e6, 180e6)),
        # one chain of a small array with an odd number of channels and times
        _case("chi2_grad_19", "chi2_grad", "hex", 3, 33, 37, 45),
        # the reference observation: 61 dishes, 64 channels, 60 times, lmax 100, FP32
        _case("chi2_grad_61", "chi2_grad", "hex", 5, 64, 60, 100),
        # the same observation in the split precision with the stored basis
        _case("chi2_grad_61_bf16x3", "chi2_grad", "hex", 5, 64, 60, 100, precision="bf16x3",
              synthesis="dense"),
        # a large array and a long scan, FP16 hi + lo fringe products
        _case("chi2_grad_127_fp16x3", "chi2_grad", "hex", 7, 96, 97, 100, precision="fp16x3"),
        # small dishes: a 35 deg beam, most of the sky in it
        _case("chi2_grad_37_wide", "chi2_grad", "hex", 4, 40, 30, 60, fwhm_deg=35.0),
        # simulation only: visibilities of a given sky, stored basis
        _case("forward_37", "forward", "hex", 4, 50, 25, 70, synthesis="dense"),
        # the backward pass under a likelihood of the user's own, for a sampler of the user's own
        _case("adjoint_91", "adjoint", "hex", 6, 48, 45, 80),
        # the delay-filtered likelihood with the beam width held fixed, preallocated outputs
        _case("filtered_61", "filtered", "hex", 5, 64, 60, 100),
        # maps of every channel from one hour of data
        _case("map_61", "map", "hex", 5, 64, 60, 100),
        # mass-matrix set-up of one chain: Hutchinson diagonal and dense gain blocks
        _case("mass_37", "mass", "hex", 4, 24, 20, 50),
        # the server: four chains of uneven size admitted, one trajectory each, read back, released
        _case("serve_4", "serve", "hex", 5, 48, 40, 80),
    ]


#: chains of a serving case relative to its own sizes: array side, channels, times, lmax
_CHAINS = ((-2, 1.0, 1.5, 0.6), (-1, 1.3, 0.4, 1.0), (0, 0.8, 1.0, 0.8), (2, 0.45, 0.35, 0.7))
_LEAPFROG, _EPS = 4, 0.002


def draw(rng):
    most = max(_macs(c) for c in listed())
    while True:
        op = rng.choice(["chi2_grad"] * 5 + ["forward", "adjoint", "filtered", "map", "mass", "serve"])
        array = rng.choice(["hex", "hex", "hex", "rhombus"])
        side = rng.randint(3, 7)

        def log_int(lo, hi):
            return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

        n_freq, n_time = log_int(8, 128), log_int(4, 120)
        lmax = rng.randint(20, 100)
        grid = (128, 384) if lmax > 40 or rng.random() < 0.5 else (32, 96)
        if grid == (32, 96):
            lmax = min(lmax, 30)
        band = rng.choice([(120e6, 130e6), (120e6, 130e6), (120e6, 180e6)])
        fwhm = rng.uniform(8.0, 14.0) if rng.random() < 0.8 else rng.uniform(14.0, 40.0)
        precision = rng.choice(["fp32", "fp32", "bf16x3", "fp16x3"])
        synthesis = rng.choice(["separable", "separable", "dense"])
        if op == "serve":
            array, side = "hex", rng.choice([3, 4, 5])
            n_freq, n_time, lmax = max(8, n_freq // 2), max(6, n_time // 2), min(lmax, 80)
        if op == "mass":
            n_freq, n_time, side = min(n_freq, 32), min(n_time, 24), min(side, 5)
        if op == "filtered":
            n_freq = max(16, n_freq)
        c = _case(None, op, array, side, n_freq, n_time, lmax, grid, band, round(fwhm, 2), precision,
                  synthesis)
        fits = op != "filtered" or 16.1 * n_time * n_freq * _n_bl(c) < 120e6   # its static scratch
        if _macs(c) <= 0.8 * most and fits:
            return c


# ------------------------------------------------------------------ geometry --
def _lattice(case):
    s = case["side"]
    if case["array"] == "rhombus":
        return [(i, j) for j in range(s) for i in range(s)]
    r = s - 1
    return [(i, j) for j in range(-r, r + 1) for i in range(-r, r + 1) if abs(i + j) <= r]


def _n_bl(case):
    n = len(_lattice(case))
    return n * (n - 1) // 2


def _unique(lat):
    """Baseline pairs (i, j), their unique index and sign, and the unique lattice differences."""
    ii, jj, uu, sg, diffs, index = [], [], [], [], [], {}
    for i in range(len(lat)):
        for j in range(i + 1, len(lat)):
            d = (lat[i][0] - lat[j][0], lat[i][1] - lat[j][1])
            s = 1 if d > (0, 0) else -1
            d = (s * d[0], s * d[1])
            if d not in index:
                index[d] = len(diffs)
                diffs.append(d)
            ii.append(i), jj.append(j), uu.append(index[d]), sg.append(s)
    return ii, jj, uu, sg, diffs


def _freqs(case):
    k = np.arange(case["n_freq"])
    return case["freq_lo_hz"] + (k + 0.5) * (case["freq_hi_hz"] - case["freq_lo_hz"]) / case["n_freq"]


def _lsts(case):
    return np.arange(case["n_time"]) * DT_S * OMEGA


def _enu(dec, ra, lst):
    """Topocentric (E, N, U) of directions (dec, ra) at sidereal time lst, FP64 tensors."""
    lat = math.radians(LAT_DEG)
    h = lst - ra
    e = -torch.cos(dec) * torch.sin(h)
    n = math.cos(lat) * torch.sin(dec) - math.sin(lat) * torch.cos(dec) * torch.cos(h)
    u = math.sin(lat) * torch.sin(dec) + math.cos(lat) * torch.cos(dec) * torch.cos(h)
    return e, n, u


def _config(case):
    return workload.FieldConfig(
        name="case", array=case["array"], array_size=case["side"], n_freq=case["n_freq"],
        freq_lo_hz=case["freq_lo_hz"], freq_hi_hz=case["freq_hi_hz"], n_time=case["n_time"],
        grid_nz=case["grid_nz"], grid_nphi=case["grid_nphi"], lmax=case["lmax"], seed=0,
        fwhm_ref_deg=case["fwhm_deg"])


def _chains(case):
    """The chains of a serving case, as cases of their own."""
    out = []
    for ds, kf, kt, kl in _CHAINS:
        out.append(dict(case, op="chi2_grad", side=max(3, min(7, case["side"] + ds)),
                        n_freq=max(4, int(case["n_freq"] * kf)), n_time=max(3, int(case["n_time"] * kt)),
                        lmax=max(8, int(case["lmax"] * kl))))
    return out


# -------------------------------------------------------------------- inputs --
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _inputs(case, seed):
    """Parameters, data and noise level of one observation, from the seed alone."""
    dev = _device()
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed) * 1000003 + 17)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device=dev, dtype=torch.float64)

    nf, nt, lmax = case["n_freq"], case["n_time"], case["lmax"]
    lat = _lattice(case)
    nu = torch.tensor(_freqs(case), device=dev)
    # sky: a(lm, nu) = a0(lm) (nu / 150 MHz)^-2.5, a0 ~ N(0, (l + 1)^-2.5)
    ell = torch.tensor(np.repeat(np.arange(lmax + 1), 2 * np.arange(lmax + 1) + 1), device=dev)
    var0 = (ell.double() + 1.0) ** -2.5
    scale = (nu / REF_HZ) ** -2.5
    alm = scale[:, None] * (var0.sqrt() * normal((lmax + 1) ** 2))[None]
    var = scale[:, None] ** 2 * var0[None]

    def gains():
        z = normal(nf, len(lat), 2) * math.sqrt(0.5)
        return 1.0 + GAIN_SCATTER * torch.view_as_complex(z)

    g, g_true = gains(), gains()
    fwhm = math.radians(case["fwhm_deg"]) * (1.0 + 0.03 * normal(1))
    # data: point sources that drift through the beam, true gains, noise
    fw0 = math.radians(case["fwhm_deg"])
    lat0 = math.radians(LAT_DEG)
    dec = lat0 + 0.5 * fw0 * normal(N_SOURCES)
    ra = 0.5 * float(_lsts(case)[-1]) + 0.7 * fw0 * normal(N_SOURCES) / math.cos(lat0)
    flux = torch.exp(normal(N_SOURCES))
    e1, e2 = (SPACING_M, 0.0), (0.5 * SPACING_M, 0.5 * math.sqrt(3.0) * SPACING_M)
    pos = torch.tensor([[a * e1[0] + b * e2[0], a * e1[1] + b * e2[1]] for a, b in lat],
                       device=dev, dtype=torch.float64)
    sig = fw0 * (REF_HZ / nu) / (2.0 * math.sqrt(2.0 * math.log(2.0)))
    ii, jj = (torch.tensor(x, device=dev) for x in _unique(lat)[:2])
    data = torch.empty(nt, nf, len(ii), dtype=torch.complex128, device=dev)
    for t, lst in enumerate(_lsts(case)):
        e, n, u = _enu(dec, ra, float(lst))
        th = torch.acos(u.clamp(-1.0, 1.0))
        w = flux * torch.exp(-th ** 2 / (2 * sig[:, None] ** 2)) * (u > 0)            # [nf][src]
        delay = (pos[:, :1] * e + pos[:, 1:] * n) / C_LIGHT                            # [ant][src]
        ph = torch.exp(-2j * math.pi * nu[:, None, None] * delay) * g_true[:, :, None]
        cov = torch.bmm(ph * w[:, None, :], ph.conj().transpose(1, 2).resolve_conj().contiguous())
        data[t] = cov[:, ii, jj]
    data *= DATA_RMS / torch.sqrt(torch.mean(data.abs() ** 2))
    sigma = NOISE_FRAC * DATA_RMS / math.sqrt(2.0)
    data += sigma * torch.view_as_complex(normal(nt, nf, len(ii), 2))
    return dict(alm=alm.float(), var=var.float(), gains=g.to(torch.complex64), fwhm=fwhm.float(),
                data=data.to(torch.complex64), sigma=float(np.float32(sigma)))


def _minv(case, var, sigma):
    """A chain's inverse mass in the server's layout: a rough diagonal of the Hessian plus the priors."""
    nf, nt, nm, na, nb = (case["n_freq"], case["n_time"], (case["lmax"] + 1) ** 2, len(_lattice(case)),
                          _n_bl(case))
    sig = math.radians(case["fwhm_deg"]) * 0.42466090014400953
    h_a = 1.0 / var.double().reshape(-1) + nt * nb * math.pi * sig ** 2 / nm / sigma ** 2
    snr = (DATA_RMS / sigma) ** 2
    h_g = (na - 1) * nt * snr + 2.0 / GAIN_SCATTER ** 2
    h_f = 4.0 * nt * nf * nb * snr / math.radians(case["fwhm_deg"]) ** 2
    pad = -(nf * nm) % 64
    one = torch.ones(1, dtype=torch.float64, device=var.device)
    return torch.cat([1.0 / h_a, one.expand(pad), (one / h_g).expand(2 * nf * na), one / h_f]).float()


# ------------------------------------------------------------- prepare / run --
def _field(case, basis):
    return vis.Field.from_config(basis, _config(case), PRECISION[case["precision"]],
                                 SYNTHESIS[case["synthesis"]])


def _basis(case):
    storage = (vis.STORAGE_SEPARABLE if case["synthesis"] == "separable"
               else vis.STORAGE_FOR[PRECISION[case["precision"]]])
    return vis.Basis(case["grid_nz"], case["grid_nphi"], case["lmax"], storage)


def prepare(case, seed):
    basis = _basis(case)
    if case["op"] == "serve":
        chains = []
        for k, c in enumerate(_chains(case)):
            x, fld = _inputs(c, seed * 16 + k), _field(c, basis)
            q0 = serve.Layout(fld).pack(x["alm"], x["gains"], x["fwhm"])
            chains.append(dict(x, field=fld, q0=q0, minv=_minv(c, x["var"], x["sigma"])))
        room = sum(serve.Server.footprint(c["field"]) for c in chains) + (16 << 20)
        return dict(op="serve", chains=chains, server=serve.Server(room, len(chains), len(chains)))
    fld = _field(case, basis)
    s = dict(_inputs(case, seed), op=case["op"], field=fld)
    if case["op"] == "filtered":
        s["filter"] = vis.Filter(_freqs(case), TAU_MAX_S, NOISE_RATIO)
        s["out"] = (torch.empty((), dtype=torch.float64, device=fld.device),
                    torch.empty_like(s["alm"]), torch.empty_like(s["gains"]), None)
    if case["op"] == "adjoint":
        s["dvis"] = s.pop("data")
    return s


def run(s):
    op = s["op"]
    if op == "serve":
        srv = s["server"]
        ids = [srv.admit(c["field"], c["data"], c["sigma"], c["q0"], c["minv"], c["var"], GAIN_SCATTER,
                         _EPS, _LEAPFROG, seed=7, stream_id=k) for k, c in enumerate(s["chains"])]
        for i in ids:
            srv.submit(i, 1)
        res = {r["chain"]: r for r in srv.wait(len(ids))}
        out = [srv.position(i, len(c["q0"]), c["q0"].device) for i, c in zip(ids, s["chains"])]
        for i in ids:
            srv.release(i)
        return dict(q=out, chi2=np.array([res[i]["chi2"] for i in ids], dtype=np.float32),
                    accepted=np.array([res[i]["accepted"] for i in ids], dtype=np.int64))
    f, alm, g, fw = s["field"], s["alm"], s["gains"], s["fwhm"]
    if op == "chi2_grad":
        x2, ga, gg, gf = vis.chi2_and_grad(f, s["data"], s["sigma"], alm, g, fw)
        return dict(chi2=x2.float(), alm=ga, gains=gg, fwhm=gf)
    if op == "forward":
        return dict(vis=vis.forward(f, alm, g, fw))
    if op == "adjoint":
        ga, gg, gf = vis.adjoint(f, alm, g, fw, s["dvis"])
        return dict(grad=serve.Layout(f).pack(ga, gg, gf))   # one vector, as a sampler takes it
    if op == "filtered":
        x2, ga, gg, _ = vis.chi2_filtered_and_grad_noalloc(f, s["filter"], s["data"], s["sigma"], alm, g,
                                                           fw, out=s["out"])
        return dict(chi2=x2.float(), alm=ga, gains=gg)
    if op == "map":
        m, w = vis.make_map(f, s["data"], g, fw)
        return dict(map=m, weight=w)
    if op == "mass":
        # the second result is 1 / h element by element
        h, _ = serve.mass_diag(f, alm, g, fw, s["sigma"], s["var"], GAIN_SCATTER, n_probes=PROBES, seed=5)
        chol = serve.gain_mass_blocks(f, alm, g, fw, s["sigma"], GAIN_SCATTER)
        return dict(h=h, chol=chol)
    raise ValueError(op)


# ---------------------------------------------------------------------- work --
def _beam_pixels(case):
    """Mean number of pixels whose beam an FP32 sum can tell from nothing (above 2^-40 of its peak)."""
    sig = math.radians(case["fwhm_deg"]) * 0.42466090014400953 * REF_HZ / float(np.mean(_freqs(case)))
    th = min(0.5 * math.pi, sig * math.sqrt(2.0 * 40.0 * math.log(2.0)))
    return 0.5 * (1.0 - math.cos(th)) * case["grid_nz"] * case["grid_nphi"]


def _n_ubl(case):
    s = case["side"]
    return ((2 * s - 1) ** 2 - 1) // 2 if case["array"] == "rhombus" else 3 * (2 * s - 1) * (s - 1)


def _macs(case):
    """Complex x real multiply-adds of one fringe contraction over the pixels above the horizon."""
    if case["op"] == "serve":
        return sum((_LEAPFROG + 1) * _macs(c) for c in _chains(case))
    k = PROBES if case["op"] == "mass" else 1
    return 0.5 * k * _n_ubl(case) * case["grid_nz"] * case["grid_nphi"] * case["n_freq"] * case["n_time"]


def work(case):
    if case["op"] == "serve":
        per = [work(c) for c in _chains(case)]
        return {k: (_LEAPFROG + 1.0) * sum(w[k] for w in per) for k in ("bytes", "flops")}
    nf, nt, nm, na = case["n_freq"], case["n_time"], (case["lmax"] + 1) ** 2, len(_lattice(case))
    nvis = nt * nf * _n_bl(case)
    npix = case["grid_nz"] * case["grid_nphi"]
    fringe = 4.0 * _n_ubl(case) * _beam_pixels(case) * nf * nt
    # the separable sum: Legendre over l and |m| for every ring, then m for every pixel above the horizon
    synth = nf * (2.0 * nm * case["grid_nz"] + 2.0 * (2 * case["lmax"] + 1) * npix / 2)
    filt = 2.0 * nf * nf * 2 * _n_bl(case) * nt
    par = 4.0 * nf * nm + 8.0 * nf * na + 4
    vb = 8.0 * nvis
    flops, nbytes = {
        "chi2_grad": (2 * fringe + 2 * synth + 30.0 * nvis, vb + 2 * par),
        "forward": (fringe + synth + 8.0 * nvis, vb + par),
        "adjoint": (2 * fringe + 2 * synth + 30.0 * nvis, vb + 2 * par),
        "filtered": (2 * fringe + 2 * synth + 2 * filt + 40.0 * nvis, vb + 2 * par),
        "map": (fringe + 16.0 * nvis, vb + 8.0 * nf * na + 8.0 * nf * npix),
        "mass": ((PROBES + 1) * fringe + (PROBES + 1) * synth + 60.0 * PROBES * nvis + nf * (2.0 * na) ** 3 / 3,
                 par + 4.0 * nf * nm + 8.0 * nf * nm + 4.0 * nf * (2 * na) ** 2),
    }[case["op"]]
    return {"bytes": nbytes, "flops": flops}


# --------------------------------------------------------------------- exact --
class _Exact:
    """The model of one observation in FP64: sky, visibilities, and their transpose."""

    def __init__(self, case):
        self.case = case
        self.dev = _device()
        nz, nphi, self.lmax = case["grid_nz"], case["grid_nphi"], case["lmax"]
        self.nz, self.nphi, self.npix, self.d_omega = nz, nphi, nz * nphi, 4 * math.pi / (nz * nphi)
        z = -1.0 + (np.arange(nz) + 0.5) * 2.0 / nz
        ra = (np.arange(nphi) + 0.5) * 2 * math.pi / nphi
        lam = self._legendre(z)                                       # [m][l][ring]
        m = np.arange(self.lmax + 1)
        norm = np.where(m == 0, 1.0, math.sqrt(2.0))[:, None]
        self.lam = torch.tensor(lam, device=self.dev)
        self.cos = torch.tensor(norm * np.cos(m[:, None] * ra), device=self.dev)   # [m][col]
        self.sin = torch.tensor(norm * np.sin(m[:, None] * ra), device=self.dev)
        ell, mm = np.meshgrid(np.arange(self.lmax + 1), m, indexing="ij")
        ok = (mm <= ell).T                                            # [m][l]
        col = (ell * ell + ell).T
        self.ok = torch.tensor(ok, device=self.dev)
        self.cplus = torch.tensor(np.where(ok, col + mm.T, 0), device=self.dev)
        self.cminus = torch.tensor(np.where(ok, col - mm.T, 0), device=self.dev)
        self.dec = torch.tensor(np.arcsin(z), device=self.dev)[:, None].expand(nz, nphi).reshape(-1)
        self.ra = torch.tensor(ra, device=self.dev)[None].expand(nz, nphi).reshape(-1)
        self.nu = torch.tensor(_freqs(case), device=self.dev)
        ii, jj, uu, sg, diffs = _unique(_lattice(case))
        self.ii, self.jj, self.uu = (torch.tensor(x, device=self.dev) for x in (ii, jj, uu))
        self.flip = torch.tensor(sg, device=self.dev) < 0
        self.n1 = torch.tensor([d[0] for d in diffs], device=self.dev)
        self.n2 = torch.tensor([d[1] for d in diffs], device=self.dev)
        self.D = int(max(self.n1.max(), self.n2.abs().max()))

    def _legendre(self, z):
        """Normalised associated Legendre values, no Condon-Shortley phase."""
        lm = self.lmax
        out = np.zeros((lm + 1, lm + 1, len(z)))
        diag = np.full(len(z), 1.0 / math.sqrt(4 * math.pi))
        for m in range(lm + 1):
            if m:
                diag = diag * math.sqrt((2 * m + 1) / (2 * m)) * np.sqrt(1 - z * z)
            out[m, m] = diag
            for l in range(m + 1, lm + 1):
                a = math.sqrt((4.0 * l * l - 1) / (l * l - m * m))
                b = math.sqrt(((l - 1.0) ** 2 - m * m) / (4 * (l - 1.0) ** 2 - 1)) if l - 1 > m else 0.0
                out[m, l] = a * (z * out[m, l - 1] - (b * out[m, l - 2] if l - 1 > m else 0.0))
        return out

    def sky(self, alm):
        """I [nf][pix] of a [nf][modes]."""
        img = 0
        for col, trig in ((self.cplus, self.cos), (self.cminus, self.sin)):
            a = (alm[:, col] * self.ok).permute(1, 0, 2).contiguous()            # [m][nf][l]
            g = torch.bmm(a, self.lam).permute(1, 2, 0).reshape(-1, self.lmax + 1)  # [nf ring][m]
            img = img + g @ trig if trig is self.cos else img + g[:, 1:] @ trig[1:]
        return img.reshape(alm.shape[0], self.npix)

    def sky_t(self, dimg):
        """The transpose: dL/da [nf][modes] of dL/dI [nf][pix]."""
        nf = dimg.shape[0]
        d = dimg.reshape(nf * self.nz, self.nphi)
        out = torch.zeros(nf, (self.lmax + 1) ** 2, dtype=torch.float64, device=self.dev)
        for col, trig in ((self.cminus, self.sin), (self.cplus, self.cos)):
            g = (d @ trig.t().contiguous()).reshape(nf, self.nz, -1).permute(2, 0, 1).contiguous()
            a = torch.bmm(g, self.lam.transpose(1, 2).contiguous())              # [m][nf][l]
            out[:, col[self.ok]] = a.permute(1, 0, 2)[:, self.ok]
        return out

    def _tiles(self, lst, fwhm):
        """Beam, theta^2 and fringe powers of the pixels above the horizon at one time, in S slabs."""
        e, n, u = _enu(self.dec, self.ra, lst)
        up = torch.nonzero(u > 0).reshape(-1)
        S = 16
        pad = -len(up) % S
        idx = torch.cat([up, up[:1].expand(pad)])
        th2 = torch.acos(u[idx].clamp(max=1.0)) ** 2
        sig = fwhm * (REF_HZ / self.nu) / (2.0 * math.sqrt(2.0 * math.log(2.0)))
        beam = torch.exp(-th2[None] / (2 * sig[:, None] ** 2))
        beam[:, len(up):] = 0.0
        p1 = SPACING_M * e[idx] / C_LIGHT
        p2 = SPACING_M * (0.5 * e[idx] + 0.5 * math.sqrt(3.0) * n[idx]) / C_LIGHT

        def powers(p, lo, hi):
            x = self.nu[:, None] * p[None]
            k = torch.arange(lo, hi + 1, device=self.dev, dtype=torch.float64)
            c = x.reshape(len(self.nu), S, 1, -1) * k[None, None, :, None]
            c = -2 * math.pi * (c - torch.round(c))
            return torch.complex(torch.cos(c), torch.sin(c)).reshape(len(self.nu) * S, len(k), -1)

        return idx, th2, sig, beam, powers(p1, 0, self.D), powers(p2, -self.D, self.D), S

    def forward(self, img, fwhm):
        """V [nt][nf][unique] without gains."""
        nf, D = len(self.nu), self.D
        out = []
        for lst in _lsts(self.case):
            idx, _, _, beam, a, b, S = self._tiles(float(lst), fwhm)
            w = (self.d_omega * beam * img[:, idx]).reshape(nf * S, 1, -1)
            v = torch.bmm(a * w, b.transpose(1, 2).contiguous()).reshape(nf, S, D + 1, -1).sum(1)
            out.append(v[:, self.n1, self.n2 + D])
        return torch.stack(out)

    def adjoint(self, img, fwhm, ev, want_f=True):
        """dL/dI [nf][pix] and dL/dF of e = dL/dRe V + i dL/dIm V [nt][nf][unique]."""
        nf, D = len(self.nu), self.D
        dimg = torch.zeros(nf, self.npix, dtype=torch.float64, device=self.dev)
        df = torch.zeros(1, dtype=torch.float64, device=self.dev)
        for t, lst in enumerate(_lsts(self.case)):
            idx, th2, sig, beam, a, b, S = self._tiles(float(lst), fwhm)
            om = torch.zeros(nf, D + 1, 2 * D + 1, dtype=torch.complex128, device=self.dev)
            om[:, self.n1, self.n2 + D] = ev[t].conj().resolve_conj()
            x = torch.bmm(om[:, None].expand(nf, S, D + 1, 2 * D + 1).reshape(nf * S, D + 1, -1).contiguous(), b)
            z = (a * x).real.sum(1).reshape(nf, -1) * self.d_omega * beam
            dimg.index_add_(1, idx, z)
            if want_f:
                df += torch.sum(z * img[:, idx] * th2[None] / (sig[:, None] ** 2 * fwhm))
        return dimg, df

    def model(self, vu, g):
        v = vu[:, :, self.uu]
        v = torch.where(self.flip, v.conj(), v)
        return g[:, self.ii] * g[:, self.jj].conj() * v

    def collapse(self, vu, g, loss):
        """dL/dV (unique) and dL/dg of a real loss of the model visibilities."""
        vu, g = vu.detach().requires_grad_(True), g.detach().requires_grad_(True)
        val = loss(self.model(vu, g))
        val.backward()
        return val.detach(), vu.grad, g.grad

    def gradient(self, x, loss, want_f=True):
        """(loss, dL/da, dL/dg, dL/dF) at the parameters x in FP64."""
        img = self.sky(x["alm"])
        val, ev, gg = self.collapse(self.forward(img, x["fwhm"]), x["gains"], loss)
        dimg, df = self.adjoint(img, x["fwhm"], ev, want_f)
        return val, self.sky_t(dimg), gg, df


def _filter64(case):
    nu = torch.tensor(_freqs(case), device=_device())
    c = torch.sinc(2 * TAU_MAX_S * (nu[:, None] - nu[None]))
    eye = torch.eye(len(nu), dtype=torch.float64, device=nu.device)
    return eye - torch.cholesky_solve(c, torch.linalg.cholesky(c + NOISE_RATIO * eye)).t().contiguous()


def _philox(c0, c1, c2, c3, seed):
    """Philox-4x32-10 (Salmon et al. 2011) of counters c0 (array), c1, c2, c3."""
    lo = np.uint64(0xFFFFFFFF)
    c = [np.asarray(v, dtype=np.uint64) + np.zeros_like(c0, dtype=np.uint64) for v in (c0, c1, c2, c3)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for r in range(10):
        p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & lo, (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & lo]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return np.stack(c, axis=-1)


def _normals(n, traj, stream, purpose, seed):
    u = (_philox(np.arange((n + 3) // 4, dtype=np.uint64), traj, stream, purpose, seed).astype(np.float64) + 0.5) / 2 ** 32
    r = np.sqrt(-2 * np.log(u[:, 0::2]))
    z = np.stack([r * np.cos(2 * math.pi * u[:, 1::2]), r * np.sin(2 * math.pi * u[:, 1::2])], axis=-1)
    return torch.tensor(z.reshape(-1)[:n], device=_device())


def _wide(x):
    return {k: v.to(torch.complex128) if torch.is_tensor(v) and v.is_complex() else v.double() if torch.is_tensor(v) else v
            for k, v in x.items()}


def _chi2(x):
    return lambda m: torch.sum(torch.view_as_real(x["data"] - m) ** 2) / x["sigma"] ** 2


def _trajectory64(case, x, minv, stream):
    """One leapfrog trajectory of a chain and its Metropolis test."""
    ex = _Exact(case)
    nf, nm, na = case["n_freq"], (case["lmax"] + 1) ** 2, len(_lattice(case))
    nalm, pad = nf * nm, -(nf * nm) % 64
    prior = 0.5 * GAIN_SCATTER ** 2
    z = _normals(nalm + pad + 2 * nf * na + 1, 0, stream, 0, 7)
    take = torch.cat([torch.arange(nalm), torch.arange(nalm + pad, len(z))]).to(z.device)
    z, minv, var = z[take], minv.double()[take], x["var"].reshape(-1)

    def potential(q):
        g = torch.view_as_complex(q[nalm:-1].reshape(nf, na, 2).clone())
        p = dict(alm=q[:nalm].reshape(nf, nm), gains=g, fwhm=q[-1:])
        x2, ga, gg, gf = ex.gradient(p, _chi2(x))
        dg = torch.view_as_real(g - 1.0).reshape(-1)
        u = 0.5 * x2 + 0.5 * torch.sum(q[:nalm] ** 2 / var) + 0.5 * torch.sum(dg ** 2) / prior
        grad = torch.cat([0.5 * ga.reshape(-1) + q[:nalm] / var,
                          0.5 * torch.view_as_real(gg).reshape(-1) + dg / prior, 0.5 * gf])
        return x2, u, grad

    q = q0 = torch.cat([x["alm"].reshape(-1), torch.view_as_real(x["gains"]).reshape(-1), x["fwhm"]])
    p = z / torch.sqrt(minv)
    x20, u, grad = potential(q)
    x2, h0, eps = x20, u + 0.5 * torch.sum(z * z), float(np.float32(_EPS))
    for _ in range(_LEAPFROG):
        p = p - 0.5 * eps * grad
        q = q + eps * minv * p
        x2, u, grad = potential(q)
        p = p - 0.5 * eps * grad
    h1 = u + 0.5 * torch.sum(p * p * minv)
    uni = (int(_philox(np.array([0xFFFFFFFF], dtype=np.uint64), 0, stream, 1, 7)[0, 0]) + 0.5) / 2 ** 32
    took = uni < math.exp(min(0.0, float(h0 - h1)))
    q, x2 = (q, x2) if took else (q0, x20)
    return torch.cat([q[:nalm], torch.zeros(pad, dtype=q.dtype, device=q.device), q[nalm:]]), float(x2), int(took)


def exact(case, seed):
    op = case["op"]
    if op == "serve":
        got = []
        for k, c in enumerate(_chains(case)):
            x = _inputs(c, seed * 16 + k)
            minv = _minv(c, x["var"], x["sigma"])
            got.append(_trajectory64(c, _wide(x), minv, k))
        return dict(q=[g[0] for g in got], chi2=np.array([g[1] for g in got]),
                    accepted=np.array([g[2] for g in got], dtype=np.int64))
    ex, x = _Exact(case), _wide(_inputs(case, seed))
    if op == "chi2_grad":
        x2, ga, gg, gf = ex.gradient(x, _chi2(x))
        return dict(chi2=x2, alm=ga, gains=gg, fwhm=gf)
    if op == "forward":
        return dict(vis=ex.model(ex.forward(ex.sky(x["alm"]), x["fwhm"]), x["gains"]))
    if op == "adjoint":
        _, ga, gg, gf = ex.gradient(x, lambda m: torch.sum((x["data"].conj() * m).real))
        pad = torch.zeros(-ga.numel() % 64, dtype=torch.float64, device=ex.dev)
        return dict(grad=torch.cat([ga.reshape(-1), pad, torch.view_as_real(gg).reshape(-1), gf]))
    if op == "filtered":
        f = _filter64(case)
        nrm = x["sigma"] ** 2 * torch.sum(f * f, dim=1)
        fc = f.to(torch.complex128)

        def loss(m):
            r = torch.matmul(fc, (x["data"] - m).permute(1, 0, 2).reshape(len(nrm), -1))
            return torch.sum((r.abs() ** 2).sum(1) / nrm)

        x2, ga, gg, _ = ex.gradient(x, loss, want_f=False)
        return dict(chi2=x2, alm=ga, gains=gg)
    if op == "map":
        g = x["gains"]
        zero = torch.zeros(case["n_time"], case["n_freq"], len(ex.n1), dtype=torch.complex128, device=ex.dev)
        _, ev, _ = ex.collapse(zero, g, lambda m: torch.sum((x["data"].conj() * m).real))
        img = torch.zeros(case["n_freq"], ex.npix, dtype=torch.float64, device=ex.dev)
        num, _ = ex.adjoint(img, x["fwhm"], ev, want_f=False)
        b2 = torch.zeros_like(img)
        for lst in _lsts(case):
            idx, _, _, beam, _, _, _ = ex._tiles(float(lst), x["fwhm"])
            b2.index_add_(1, idx, beam ** 2)
        gg = torch.sum(g[:, ex.ii].abs() ** 2 * g[:, ex.jj].abs() ** 2, dim=1)
        wgt = ex.d_omega ** 2 * b2 * gg[:, None]
        ok = wgt >= 1e-6 * wgt.max(dim=1, keepdim=True).values
        return dict(map=torch.where(ok, num / torch.where(ok, wgt, torch.ones_like(wgt)), torch.zeros_like(num)), weight=wgt)
    if op == "mass":
        nf, na, nvis = case["n_freq"], len(_lattice(case)), x["data"].numel()
        img = ex.sky(x["alm"])
        vu = ex.forward(img, x["fwhm"])
        s2, g = x["sigma"] ** 2, x["gains"]
        ha, hf = 0, 0
        for k in range(PROBES):
            z = torch.view_as_complex(_normals(2 * nvis, k, 0, 5, 5).reshape(*x["data"].shape, 2))
            _, ev, _ = ex.collapse(vu, g, lambda m: torch.sum((z.conj() * m).real))
            dimg, df = ex.adjoint(img, x["fwhm"], ev)
            ha, hf = ha + ex.sky_t(dimg) ** 2 / (PROBES * s2), hf + df ** 2 / (PROBES * s2)
        ha = ha + 1.0 / x["var"]
        pw = (vu.abs() ** 2).sum(0)[:, ex.uu] / s2                               # [nf][bl]
        gd = torch.zeros(nf, na, dtype=torch.float64, device=ex.dev)
        gd.index_add_(1, ex.ii, g[:, ex.jj].abs() ** 2 * pw)
        gd.index_add_(1, ex.jj, g[:, ex.ii].abs() ** 2 * pw)
        pri = 2.0 / GAIN_SCATTER ** 2
        hg = (gd + pri)[..., None].expand(nf, na, 2)
        pad = torch.ones(-ha.numel() % 64, dtype=torch.float64, device=ex.dev)
        h = torch.cat([ha.reshape(-1), pad, hg.reshape(-1), hf])
        w = g[:, ex.ii] * g[:, ex.jj] * pw
        blk = torch.zeros(nf, na, 2, na, 2, dtype=torch.float64, device=ex.dev)
        for a, b in ((ex.ii, ex.jj), (ex.jj, ex.ii)):
            blk[:, a, 0, b, 0] = w.real
            blk[:, a, 1, b, 1] = -w.real
            blk[:, a, 0, b, 1] = w.imag
            blk[:, a, 1, b, 0] = w.imag
        blk = blk.reshape(nf, 2 * na, 2 * na) + torch.diag_embed(hg.reshape(nf, 2 * na))
        return dict(h=h, chol=torch.linalg.cholesky(blk))
    return None
