"""Timing cases: the calls a user of the library makes, over the range of sizes
and options the workloads, the serving trace and the tests cover.

Each case is one pass through a public entry point of
`paper_2111_04141_amd.api` (or `autograd`), with inputs made on the GPU from a
seed: Earth-rotation uv tracks of a synthetic array in measurement-set order
([time][baseline][channel]), visibilities of a few point sources plus unit
noise, model grids that are transforms of point-source images, and the kernel
tables of the benchmark workloads.

Keys of a gridding case: `path` (the entry point), `kind` (kernel), `nu`, `nv`,
`npol`, `beta`, `s_min` .. `s_max` over `planes` (separable kernels: s_min =
s_max), `nrec`, `array` and `n_ant`, `n_chan`, `taps` and `uvw` (data types),
`layers` (W-stacking).
"""
import math

import numpy as np
import torch

from paper_2111_04141_amd import api
from paper_2111_04141_amd import autograd as AG
from paper_2111_04141_amd import workload as W

LAT = DEC = math.radians(-30.0)
BASE_SUPPORT = 7
SIGMA = 0.1
TAP_TYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


def _case(name, path, **kw):
    c = {"name": name, "path": path, "kind": "sep", "npol": 4, "beta": 8, "planes": 1,
         "s_min": 7, "s_max": 7, "array": "disc", "n_ant": 64, "n_chan": 50, "taps": "f32",
         "uvw": "f32", "layers": 0}
    c.update(kw)
    return c


WPROJ32 = {"kind": "wproj", "beta": 4, "planes": 32, "s_min": 8, "s_max": 64, "array": "log"}
WPROJ16 = {"kind": "wproj", "beta": 4, "planes": 16, "s_min": 8, "s_max": 32, "array": "log"}


def listed():
    return [
        # the smallest job of the serving trace: a snapshot, bound by latency
        _case("grid-10k-sep-512", "grid", nu=512, nv=512, nrec=10_000),
        # one observation of a 64-antenna array in one channel (the small workload)
        _case("grid-101k-sep-1024", "grid", nu=1024, nv=1024, nrec=100_800, n_chan=1, uvw="f64"),
        # a middle-sized W-projection job of the serving trace
        _case("grid-1M-wproj-2048", "grid", nu=2048, nv=2048, nrec=1_000_003, n_ant=128,
              n_chan=80, **WPROJ16),
        # one step of a major cycle: residual, chi^2 and its gradient
        _case("chi2-10M-sep-2048", "chi2", nu=2048, nv=2048, nrec=10_080_000),
        # wide-field W-projection imaging at full size (the benchmark workload), one shot
        _case("grid-134M-wproj-8192", "grid", nu=8192, nv=8192, nrec=133_693_440, n_ant=256,
              n_chan=128, **WPROJ32),
        # model prediction over the same records with a kept plan
        _case("degrid-134M-wproj-8192", "plan_degrid", nu=8192, nv=8192, nrec=133_693_440,
              n_ant=256, n_chan=128, **WPROJ32),
        # two polarisations, a half-precision bank, a grid of odd sides, a kept plan
        _case("grid-7M-wproj-f16-odd", "plan_grid", nu=6000, nv=5001, npol=2, nrec=7_000_003,
              n_ant=197, n_chan=37, **dict(WPROJ32, beta=6, planes=24, s_max=48, taps="f16")),
        # one polarisation (Stokes I) predicted through a bfloat16 bank, one shot
        _case("degrid-3M-wproj-bf16-I", "degrid", nu=3072, nv=2500, npol=1, nrec=3_000_017,
              n_ant=100, n_chan=64, **dict(WPROJ16, taps="bf16")),
        # the hybrid pipeline: gridding step, column pruning, image
        _case("hybrid-10M-sep-2048", "hybrid", nu=2048, nv=2048, nrec=10_080_000),
        # the image of finished grids
        {"name": "image-4x2048", "path": "image", "nu": 2048, "nv": 2048, "npol": 4},
        # W-stacking: 16 layers gridded, transformed, screened and summed
        _case("wstack-10M-16x2048", "wstack", kind="wstack", nu=2048, nv=2048,
              nrec=10_080_000, layers=16),
        # the benchmark's W-projection bank, built once per observation
        {"name": "bank-32-planes", "path": "bank", "beta": 4, "planes": 32, "s_min": 8,
         "s_max": 64, "fov": 0.02, "taps": "f32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _even(n):
    return n + (n & 1)


def draw(rng):
    path = rng.choice(["grid", "grid", "plan_grid", "plan_grid", "degrid", "plan_degrid", "chi2",
                       "hybrid", "image", "wstack", "bank"])
    if path == "image":
        return {"path": path, "nu": _even(_log(rng, 256, 4096)), "nv": _even(_log(rng, 256, 4096)),
                "npol": rng.randint(1, 4)}
    if path == "bank":
        return {"path": path, "beta": rng.choice([2, 4, 6, 8]), "planes": rng.randint(4, 40),
                "s_min": 8, "s_max": 2 * rng.randint(6, 32), "fov": rng.uniform(0.005, 0.05),
                "taps": rng.choice(["f32", "f16", "bf16"])}
    c = {"path": path, "npol": rng.choice([1, 2, 4, 4, 4]), "layers": 0,
         "taps": rng.choice(["f32", "f32", "f16", "bf16"]),
         "uvw": rng.choice(["f32", "f32", "f64"]), "n_ant": rng.choice([36, 64, 100, 128, 197, 256]),
         "n_chan": _log(rng, 1, 128)}
    if path in ("hybrid", "wstack") or (path == "chi2") or rng.random() < 0.4:
        s = rng.choice([6, 7, 7, 8, 9, 12, 15])
        c.update(kind="wstack" if path == "wstack" else "sep", beta=rng.choice([4, 8, 8]),
                 planes=1, s_min=s, s_max=s, array="disc")
        if path == "hybrid":
            s = rng.choice([6, 7, 8])
            c.update(s_min=s, s_max=s)
        if path == "wstack":
            c["layers"] = rng.randint(3, 16)
    else:
        c.update(kind="wproj", beta=rng.choice([2, 4, 4, 6]), planes=rng.randint(8, 32), s_min=8,
                 s_max=2 * rng.randint(6, 32), array=rng.choice(["log", "log", "disc"]))
    top = 2048 if path in ("hybrid", "wstack") else 8192
    side = _log(rng, 512, top)
    c.update(nu=_even(side), nv=_even(_log(rng, max(512, 0.7 * side), side)))
    if path not in ("hybrid", "wstack", "chi2") and rng.random() < 0.5:
        c["nv"] -= 1
    # at most the records of 40 times, and no more than the grid's size suggests
    b = c["n_ant"] * (c["n_ant"] - 1) // 2
    most = min(60_000_000 if c["array"] == "log" else 10_000_000, 40 * b * c["n_chan"],
               8 * c["nu"] * c["nv"])
    c["nrec"] = _log(rng, 10_000, max(10_001, most)) | 1
    c["nrec"] = min(c["nrec"], 40 * b * c["n_chan"])
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _device():
    return torch.device("cuda") if torch.cuda.is_available() else torch.device("cpu")


def _generator(seed, dev):
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    return g


def _uvw(c, seed, dev):
    """[nrec, 3] wavelengths in measurement-set order, largest |u|, |v| and |w|."""
    aseed = W.SEED_ANTENNAS + int(seed)
    if c["array"] == "disc":
        ant = W.antennas_uniform_disc(c["n_ant"], 1000.0, aseed)
        freqs = np.linspace(1.43e9 * 0.9, 1.43e9 * 1.1, c["n_chan"])
    else:
        ant = W.antennas_log_radial(c["n_ant"], 20.0, 2500.0, aseed)
        freqs = np.linspace(1.2e9, 1.6e9, c["n_chan"], endpoint=False)
    bl = W.baselines_enu(ant)
    per = bl.shape[0] * c["n_chan"]
    times = -(-c["nrec"] // per)
    m = W.baseline_uvw_m(bl, LAT, DEC, W.hour_angles(times) if times > 1 else np.array([0.3]))
    m = torch.from_numpy(m).to(dev)
    f = torch.from_numpy(freqs / W.C_LIGHT).to(dev)
    dt = torch.float64 if c["uvw"] == "f64" else torch.float32
    out = torch.empty(c["nrec"], 3, dtype=dt, device=dev)
    for t in range(times):
        lo = t * per
        hi = min(lo + per, c["nrec"])
        out[lo:hi] = (m[t][:, None, :] * f[None, :, None]).reshape(-1, 3)[: hi - lo].to(dt)
    top = float(f.max())
    return out, float(m[..., :2].abs().max()) * top, float(m[..., 2].abs().max()) * top


def _vis(c, seed, uvw, scale, dev):
    """Three point sources and unit noise, complex64 [nrec, npol]."""
    n = c["nrec"]
    g = _generator(seed + 1, dev)
    v = torch.view_as_complex(torch.randn(n, c["npol"], 2, generator=g, device=dev))
    r = np.random.Generator(np.random.PCG64(int(seed)))
    pol = torch.tensor([1.0, 0.1, 0.1, 0.8][: c["npol"]], device=dev)
    for _ in range(3):
        l, m = (r.uniform(-0.25, 0.25, 2) * scale).tolist()
        flux = r.uniform(0.5, 2.0)
        for lo in range(0, n, 1 << 25):
            u = uvw[lo:lo + (1 << 25)].double()
            ph = ((u[:, 0] * l + u[:, 1] * m) % 1.0).float() * (-2.0 * math.pi)
            v[lo:lo + (1 << 25)] += torch.polar(torch.full_like(ph, flux), ph)[:, None] * pol
    return v


def _model_grid(c, seed, dev):
    """Transform of a tapered image of 50 point sources, complex64 [npol, nv, nu]."""
    nu, nv = c["nu"], c["nv"]
    r = np.random.Generator(np.random.PCG64(int(seed)))
    img = torch.zeros(nv, nu, device=dev)
    x, y = r.integers(nu // 4, 3 * nu // 4, 50), r.integers(nv // 4, 3 * nv // 4, 50)
    flux = r.uniform(0.5, 2.0, 50)
    taper = np.exp(-((x - nu / 2) / (0.3 * nu)) ** 2 - ((y - nv / 2) / (0.3 * nv)) ** 2)
    img[torch.from_numpy(y).to(dev), torch.from_numpy(x).to(dev)] = torch.from_numpy(
        (flux * taper).astype(np.float32)).to(dev)
    g = torch.fft.fftshift(torch.fft.fft2(torch.fft.ifftshift(img)))
    return torch.stack([g * a for a in (1.0, 0.5, 0.25, 0.8)[: c["npol"]]]).contiguous()


def _usable(h):
    """A corrector cut to the central half of the field, the part that is kept:
    towards the edge it grows without bound and amplifies rounding."""
    n = h.numel()
    h = h.clone()
    h[: n // 4] = 0.0
    h[n - n // 4:] = 0.0
    return h


def _planes(supports, ws, beta, fov, dev):
    """W-projection tables in 64 bits, one complex [beta S + 1, beta S + 1] per
    plane: the transform of the kernel's image-domain taper times the inverse
    W-term, sampled every 1/beta cells."""
    base = torch.from_numpy(W.pswf_taps(BASE_SUPPORT, beta)).to(dev)
    half = base.numel() // 2
    found = []
    for s, w in zip(supports, ws):
        m = 2 * beta * s
        pad = torch.zeros(m, dtype=torch.float64, device=dev)
        pad[m // 2 - half: m // 2 - half + base.numel()] = base
        taper = torch.fft.ifft(torch.fft.ifftshift(pad))
        l = torch.fft.ifftshift((torch.arange(m, device=dev, dtype=torch.float64) - m // 2)
                                * (beta / m)) * fov
        n = torch.sqrt((1.0 - (l[:, None] ** 2 + l[None, :] ** 2)).clamp(min=0.0))
        ph = 2.0 * math.pi * w * (n - 1.0)
        k = torch.fft.fftshift(torch.fft.fft2(taper[:, None] * taper[None, :]
                                              * torch.polar(torch.ones_like(ph), ph)))
        lo = m // 2 - beta * s // 2
        found.append(k[lo: lo + beta * s + 1, lo: lo + beta * s + 1].contiguous())
    return found


def _tables(c, wmax, fov, dev):
    """(taps, plane supports, plane offsets, 1 / plane spacing); taps float64,
    or complex128 planes one after another, before rounding."""
    if c["kind"] != "wproj":
        return torch.from_numpy(W.pswf_taps(c["s_min"], c["beta"])).to(dev), [], [], 0.0
    sup = [int(s) for s in W.wproj_support_schedule(c["planes"], c["s_min"], c["s_max"])]
    dw = wmax / max(1, c["planes"] - 1)
    pl = _planes(sup, [p * dw for p in range(len(sup))], c["beta"], fov, dev)
    flat = torch.cat([p.reshape(-1) for p in pl])
    offs, at = [], 0
    for p in pl:
        offs.append(at)
        at += p.numel()
    return flat / flat.abs().max(), sup, offs, 1.0 / dw


def _round_taps(c, taps):
    """The table as the library takes it, in the case's tap type."""
    dt = TAP_TYPES[c["taps"]]
    if not taps.is_complex():
        return taps.to(dt)
    return taps.to(torch.complex64) if c["taps"] == "f32" else torch.view_as_real(taps).to(dt)


def _inputs(c, seed, dev):
    uvw, umax, wmax = _uvw(c, seed, dev)
    scale = 0.5 * (min(c["nu"], c["nv"]) / 2 - c["s_max"]) / umax
    taps, sup, offs, inv_dw = _tables(c, wmax, scale, dev)
    if c["kind"] == "wstack":
        inv_dw = max(1, c["layers"] - 1) / (2.0 * wmax)
    return uvw, scale, _round_taps(c, taps), sup, offs, inv_dw


def prepare(case, seed):
    c, dev = case, _device()
    if c["path"] == "image":
        g = _generator(seed, dev)
        grid = torch.view_as_complex(torch.randn(c["npol"], c["nv"], c["nu"], 2, generator=g,
                                                 device=dev))
        t = torch.from_numpy(W.pswf_taps(7, 8)).float().to(dev)
        return {"c": c, "grid": grid, "hx": _usable(api.corrector(c["nu"], 8, t, 8)),
                "hy": _usable(api.corrector(c["nv"], 8, t, 8)),
                "imager": api.Imager(c["npol"], c["nu"], c["nv"])}
    if c["path"] == "bank":
        sup, ws = _bank_schedule(c, seed)
        return {"c": c, "sup": sup, "ws": ws,
                "base": torch.from_numpy(W.pswf_taps(BASE_SUPPORT, c["beta"])).to(dev)}
    uvw, scale, taps, sup, offs, inv_dw = _inputs(c, seed, dev)
    spec = api.GridSpec(c["nu"], c["nv"], c["npol"], c["beta"], scale, scale)
    if c["kind"] == "wproj":
        bank = api.KernelBank("wproj", taps, plane_support=sup, plane_offset=offs, inv_dw=inv_dw)
    elif c["kind"] == "wstack":
        bank = api.KernelBank("wstack", taps, support=c["s_min"], layers=c["layers"],
                              inv_dw=inv_dw)
    else:
        bank = api.KernelBank("separable", taps, support=c["s_min"])
    s = {"c": c, "spec": spec, "bank": bank, "uvw": uvw}
    if c["path"] in ("degrid", "plan_degrid", "chi2"):
        s["model"] = _model_grid(c, seed, dev)
    if c["path"] not in ("degrid", "plan_degrid"):
        s["vis"] = _vis(c, seed, uvw, scale, dev)
    if c["path"] in ("plan_grid", "plan_degrid", "chi2", "wstack"):
        s["plan"] = api.Plan(spec, bank, uvw)
    t32 = taps.float() if c["kind"] != "wproj" else None
    if c["path"] == "hybrid":
        a = c["beta"] // 2
        s["plan"] = api.HybridPlan(spec, bank, uvw)
        s["ztaps"] = t32
        s["hx"] = _usable(api.corrector(c["nu"], c["beta"], t32, c["beta"]))
        s["hy"] = _usable(api.corrector(c["nv"], c["beta"], t32, a))
        s["imager"] = api.Imager(c["npol"], c["nu"], 2 * c["nv"])
    if c["path"] == "wstack":
        s["hx"] = _usable(api.corrector(c["nu"], c["beta"], t32, c["beta"]))
        s["hy"] = _usable(api.corrector(c["nv"], c["beta"], t32, c["beta"]))
        s["dw"] = 1.0 / inv_dw
        s["imager"] = api.WStackImager(c["npol"], c["layers"], c["nu"], c["nv"])
    return s


def run(s):
    path = s["c"]["path"]
    if path == "grid":
        return api.grid(s["spec"], s["bank"], s["uvw"], s["vis"])
    if path == "degrid":
        return api.degrid(s["spec"], s["bank"], s["uvw"], s["model"])
    if path == "plan_grid":
        return s["plan"].grid(s["vis"])
    if path == "plan_degrid":
        return s["plan"].degrid(s["model"])
    if path == "chi2":
        m = s["model"].detach().requires_grad_(True)
        loss = AG.chi2(m, s["plan"], s["vis"], SIGMA)
        loss.backward()
        return {"chi2": loss.detach().float(), "grad": m.grad}
    if path == "image":
        return s["imager"].image(s["grid"], s["hx"], s["hy"])
    if path == "bank":
        c = s["c"]
        return api.wkernel_bank(s["sup"], s["ws"], c["beta"], s["base"], c["fov"], c["taps"])[0]
    if path == "hybrid":
        c = s["c"]
        hy = s["plan"].grid(s["vis"])
        pr = api.prune_columns(hy, c["beta"] // 2, s["ztaps"], 2 * c["s_min"])
        return s["imager"].image(pr, s["hx"], s["hy"], y0=c["nv"] // 2, out_ny=c["nv"])
    fov = s["spec"].scale_u
    layers = s["plan"].grid(s["vis"])
    return {"layers": layers,
            "image": s["imager"].image(layers, s["hx"], s["hy"], fov, fov, s["dw"])}


# ---------------------------------------------------------------------------
# work and values in 64 bits
# ---------------------------------------------------------------------------
def _bank_schedule(c, seed):
    sup = [int(s) for s in W.wproj_support_schedule(c["planes"], c["s_min"], c["s_max"])]
    top = 400.0 + 10.0 * (int(seed) % 1000)
    return sup, [top * p / max(1, len(sup) - 1) for p in range(len(sup))]


def _fft_flops(n, m):
    return 5.0 * n * m * math.log2(n * m)


def _mean_updates(c):
    """Mean of S^2 over a sample of the case's records."""
    if c["kind"] != "wproj":
        return float(c["s_min"] ** 2)
    few = dict(c, n_chan=min(c["n_chan"], 4))
    few["nrec"] = min(c["nrec"], 40 * (c["n_ant"] * (c["n_ant"] - 1) // 2) * few["n_chan"])
    uvw, _, wmax = _uvw(few, 0, torch.device("cpu"))
    sup = torch.from_numpy(W.wproj_support_schedule(c["planes"], c["s_min"], c["s_max"])).double()
    p = torch.floor(uvw[:, 2].double().abs() * ((c["planes"] - 1) / wmax) + 0.5).long()
    return float((sup[p.clamp(max=c["planes"] - 1)] ** 2).mean())


def work(case):
    c = case
    if c["path"] == "image":
        cells = c["npol"] * c["nu"] * c["nv"]
        return {"bytes": 16 * cells, "flops": c["npol"] * _fft_flops(c["nu"], c["nv"])}
    if c["path"] == "bank":
        sup, _ = _bank_schedule(c, 0)
        el = sum((c["beta"] * s + 1) ** 2 for s in sup)
        return {"bytes": (8 if c["taps"] == "f32" else 4) * el,
                "flops": sum(_fft_flops(2 * c["beta"] * s, 2 * c["beta"] * s) for s in sup)}
    npol, n = c["npol"], c["nrec"]
    cells = npol * c["nu"] * c["nv"]
    flops = 2.0 * npol * (4 if c["kind"] == "wproj" else 2) * n * _mean_updates(c)
    one_shot = c["path"] in ("grid", "degrid")
    data = 8 * npol * n + (3 * n * (8 if c["uvw"] == "f64" else 4) if one_shot else 0)
    if c["path"] == "chi2":
        return {"bytes": data + 16 * cells, "flops": 2 * flops}
    if c["path"] == "hybrid":
        alpha = c["beta"] // 2
        f = flops / c["s_min"] + 4.0 * 2 * c["s_min"] * c["beta"] * cells
        return {"bytes": data + 8 * cells, "flops": f + npol * _fft_flops(c["nu"], 2 * c["nv"])}
    if c["path"] == "wstack":
        return {"bytes": data + 8 * (c["layers"] + 1) * cells,
                "flops": flops + c["layers"] * npol * (_fft_flops(c["nu"], c["nv"])
                                                       + 8.0 * c["nu"] * c["nv"])}
    return {"bytes": data + 8 * cells, "flops": flops}


def _axis(coord, scale, n, beta, s):
    """First cell, first tap and validity of one axis, as the definition states."""
    q = torch.floor((coord.double() * scale + float(n // 2)) * float(beta) + 0.5).long()
    d = q - beta * s // 2
    ok = (d >= -beta) & (d < beta * (n - s))
    k = torch.div(d + beta, beta, rounding_mode="floor")
    return torch.where(ok, k, 0), torch.where(ok, k * beta - d, 1), ok


def _rows(c, uvw, scale, taps, sup, offs, inv_dw):
    """(records, first cell of one footprint row as an index into the grid's
    cells, the row's taps [n, S] in 64 bits) for every plane and row."""
    beta, nu, nv = c["beta"], c["nu"], c["nv"]
    if c["kind"] == "wproj":
        t = taps if taps.is_complex() else torch.view_as_complex(taps.double())
        t = t.to(torch.complex128)
        w = uvw[:, 2].double()
        plane = torch.floor(w.abs() * inv_dw + 0.5).long().clamp(max=len(sup) - 1)
    else:
        t, sup, plane = taps.double(), [c["s_min"]], None
    layer = 0
    if c["kind"] == "wstack":
        layer = torch.floor(uvw[:, 2].double() * inv_dw + 0.5 * c["layers"]).long()
        layer = layer.clamp(0, c["layers"] - 1)
    step = 4_000_000
    for p, s in enumerate(sup):
        every = torch.arange(uvw.shape[0], device=uvw.device) if plane is None else \
            (plane == p).nonzero()[:, 0]
        for lo in range(0, every.numel(), step):
            r = every[lo:lo + step]
            ku, tu, oku = _axis(uvw[r, 0], scale, nu, beta, s)
            kv, tv, okv = _axis(uvw[r, 1], scale, nv, beta, s)
            ok = oku & okv
            r, ku, tu, kv, tv = r[ok], ku[ok], tu[ok], kv[ok], tv[ok]
            if not r.numel():
                continue
            if c["kind"] == "wstack":
                kv = kv + layer[r] * nv
            along = torch.arange(s, device=r.device)
            for j in range(s):
                first = (kv + j) * nu + ku
                if c["kind"] == "wproj":
                    at = offs[p] + (tv + j * beta) * (beta * s + 1) + tu
                    x = t[at[:, None] + beta * along]
                    x = torch.where((uvw[r, 2] < 0)[:, None], x.conj(), x)
                else:
                    x = t[tu[:, None] + beta * along] * t[tv + j * beta][:, None]
                yield r, first, x


def _grid64(c, rows, vis, cells):
    out = torch.zeros(cells * c["npol"], 2, dtype=torch.float64, device=vis.device)
    for r, first, x in rows:
        at = (first[:, None] + torch.arange(x.shape[1], device=x.device)).reshape(-1)
        for p in range(c["npol"]):
            v = (x * vis[r, p].to(torch.complex128)[:, None]).reshape(-1)
            out.index_add_(0, at + p * cells, torch.view_as_real(v))
    return torch.view_as_complex(out)


def _degrid64(c, rows, grid):
    g = grid.reshape(c["npol"], -1).to(torch.complex128)
    out = torch.zeros(c["nrec"], c["npol"], dtype=torch.complex128, device=grid.device)
    for r, first, x in rows:
        at = first[:, None] + torch.arange(x.shape[1], device=x.device)
        for p in range(c["npol"]):
            out[r, p] += (x.conj() * g[p][at]).sum(1)
    return out


def _centred_image64(grid):
    g = torch.fft.ifft2(torch.fft.ifftshift(grid.to(torch.complex128), dim=(-2, -1)), norm="forward")
    return torch.fft.fftshift(g, dim=(-2, -1))


def _corrector64(n, beta, table, phases, dev):
    l = (torch.arange(n, device=dev, dtype=torch.float64) - n // 2) / n
    e = torch.arange(table.numel(), device=dev, dtype=torch.float64) - (table.numel() - 1) / 2
    s = (table.double()[:, None] * torch.cos(2 * math.pi * (e / beta)[:, None] * l)).sum(0) / phases
    return _usable(1.0 / (s * torch.sinc(l / beta)))


def exact(case, seed):
    c, dev = case, _device()
    if c["path"] == "image":
        g = _generator(seed, dev)
        grid = torch.view_as_complex(torch.randn(c["npol"], c["nv"], c["nu"], 2, generator=g,
                                                 device=dev))
        t = torch.from_numpy(W.pswf_taps(7, 8)).float().to(dev)
        hx, hy = (_corrector64(n, 8, t, 8, dev) for n in (c["nu"], c["nv"]))
        return _centred_image64(grid) * hx * hy[:, None]
    if c["path"] == "bank":
        sup, ws = _bank_schedule(c, seed)
        pl = torch.cat([p.reshape(-1) for p in _planes(sup, ws, c["beta"], c["fov"], dev)])
        pl = pl / pl.abs().max()
        return pl if c["taps"] == "f32" else torch.view_as_real(pl)
    # 64-bit sums over more updates than this take too long
    if c["nrec"] * _mean_updates(c) > 2e9:
        return None
    uvw, scale, taps, sup, offs, inv_dw = _inputs(c, seed, dev)
    cells = c["nu"] * c["nv"] * max(1, c["layers"])
    rows = lambda: _rows(c, uvw, scale, taps, sup, offs, inv_dw)  # noqa: E731
    shape = (c["npol"], c["nv"], c["nu"])
    if c["path"] in ("degrid", "plan_degrid"):
        return _degrid64(c, rows(), _model_grid(c, seed, dev))
    vis = _vis(c, seed, uvw, scale, dev)
    if c["path"] in ("grid", "plan_grid"):
        return _grid64(c, rows(), vis, cells).reshape(shape)
    if c["path"] == "chi2":
        r = vis - _degrid64(c, rows(), _model_grid(c, seed, dev))
        loss = (r.real ** 2 + r.imag ** 2).sum() / (SIGMA * SIGMA)
        g = _grid64(c, rows(), r, cells).reshape(shape)
        return {"chi2": loss, "grad": g * (-2.0 / (SIGMA * SIGMA))}
    t32 = taps.float()
    if c["path"] == "wstack":
        layers = _grid64(c, rows(), vis, cells).reshape(c["npol"], c["layers"], c["nv"], c["nu"])
        l, m = ((torch.arange(n, device=dev, dtype=torch.float64) - n // 2) / n * scale
                for n in (c["nu"], c["nv"]))
        nm1 = torch.sqrt((1.0 - (m[:, None] ** 2 + l[None, :] ** 2)).clamp(min=0.0)) - 1.0
        img = torch.zeros(shape, dtype=torch.complex128, device=dev)
        for j in range(c["layers"]):
            ph = 2 * math.pi * ((j - (c["layers"] - 1) / 2) / inv_dw) * nm1
            img += _centred_image64(layers[:, j]) * torch.polar(torch.ones_like(ph), ph)
        hx, hy = (_corrector64(n, c["beta"], t32, c["beta"], dev) for n in (c["nu"], c["nv"]))
        return {"layers": layers, "image": img * hx * hy[:, None]}
    return _hybrid64(c, uvw, scale, t32.double(), vis, dev)


def _hybrid64(c, uvw, scale, t, vis, dev):
    beta, s, nu, nv, npol = c["beta"], c["s_min"], c["nu"], c["nv"], c["npol"]
    rows = beta * nv
    ku, tu, ok = _axis(uvw[:, 0], scale, nu, beta, s)
    q = torch.floor((uvw[:, 1].double() * scale + float(nv // 2)) * float(beta) + 0.5).long()
    r = (ok & (q >= 0) & (q < rows)).nonzero()[:, 0]
    hy = torch.zeros(npol * rows * nu, 2, dtype=torch.float64, device=dev)
    for i in range(s):
        w = t[tu[r] + i * beta]
        at = q[r] * nu + ku[r] + i
        for p in range(npol):
            hy.index_add_(0, at + p * rows * nu,
                          torch.view_as_real(vis[r, p].to(torch.complex128) * w))
    hy = torch.view_as_complex(hy).reshape(npol, rows, nu)
    alpha, sz = beta // 2, 2 * s
    pruned = torch.zeros(npol, 2 * nv, nu, dtype=torch.complex128, device=dev)
    for d in range(-alpha * sz // 2, alpha * sz // 2):
        pruned += t[d + alpha * sz // 2] * torch.roll(hy, -d, 1)[:, ::alpha]
    hx = _corrector64(nu, beta, t, beta, dev)
    hv = _corrector64(nv, beta, t, alpha, dev)
    img = _centred_image64(pruned)[:, nv // 2: nv // 2 + nv]
    return img * hx * hv[:, None]
