"""The imaging work that a user of this package has it do, as cases that can be timed.

Each case is one call (or one training step) through the package's public entry
points at a size of the kind the package is used at: the station and tile arrays
of its synthetic workloads, from a single small image to cubes of thousands, with
the options that observations need (flags, gains, cable lengths, a rotated phase
centre, a gridding kernel, 16-bit storage) and the calls around the imager (the
gridding alone, the 2D transform, dynamic spectra, the correlator). Inputs are
made on the GPU from a seed: antenna positions, a sky of point sources with
noise, flags and gains, all new with every seed.

``exact`` recomputes a case in 64 bits with plain torch operations.
"""
import math

import torch

import paper_2405_13478_amd as blink
from paper_2405_13478_amd import blink as api

C_LIGHT = 299792458.0
OMEGA_EARTH = 7.2921e-5        # rad/s
DT = 0.1                       # s per timestep
N_SRC = 12                     # point sources of the synthetic sky

STORAGE = {"c64": torch.complex64, "f16": torch.float16, "bf16": torch.bfloat16}


def _image(name, **kw):
    c = dict(kind="image", n_ant=128, core_m=300.0, disc_m=3000.0, n_time=1, n_chan=1, f0=170e6, df=40e3,
             grid_n=1024, out_n=512, allsky=False, uniform=False, storage="c64", flagged=False, kernel=0,
             rotate=False, gains=False)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one small snapshot of a 32-antenna station: the smallest call, all latency
        _image("snapshot_128", n_ant=32, core_m=35.0, disc_m=35.0, f0=160e6, grid_n=128, out_n=128),
        # one image of the 128-tile array: the per-image loop of a quick look
        _image("single_1024"),
        # a batch of timesteps of the 128-tile array with all 768 channels: bulk imaging
        _image("widefield_1024_cube", n_time=4, n_chan=768),
        # an odd-sized job with everything applied at load: 117 antennas, 3 x 37 images,
        # gains, cable lengths, a rotated phase centre, flags that differ per timestep
        _image("calibrated_512_ragged", n_ant=117, n_time=3, n_chan=37, grid_n=512, out_n=400, flagged=True,
               rotate=True, gains=True),
        # a 256-antenna station imaging the whole sky, uniform weighting, 2-10% flagged
        _image("allsky_180_uniform", n_ant=256, core_m=35.0, disc_m=35.0, n_time=200, n_chan=32, f0=150e6,
               df=30e6 / 31, grid_n=180, out_n=180, allsky=True, uniform=True, flagged=True),
        # large images of a 256-tile array from FP16 visibilities, uniform weighting
        _image("precision_2048_f16", n_ant=256, core_m=5000.0, disc_m=5000.0, n_chan=128, f0=200e6, grid_n=2048,
               out_n=2048, uniform=True, storage="f16"),
        # anti-aliased widefield images: a Kaiser-Bessel kernel of 6 cells
        _image("kernel6_1024", n_time=2, n_chan=192, kernel=6),
        # one step of a gain fit: images, and gradients of visibilities and gains
        dict(kind="train", name="gain_fit_1024", n_ant=128, core_m=300.0, disc_m=3000.0, n_time=10, n_chan=32,
             f0=170e6, df=40e3, grid_n=1024, out_n=512, uniform=False, flagged=False),
        # the weighted uv grids and counts themselves (for a user's own weighting or transform)
        dict(kind="grid", name="uvgrid_1024", n_ant=128, core_m=300.0, disc_m=3000.0, n_time=1, n_chan=32, f0=170e6,
             df=40e3, grid_n=1024, uniform=True, flagged=False),
        # the batched 2D transform alone, inverse
        dict(kind="fft", name="fft2d_1024", grid_n=1024, batch=64, sign=1),
        # per-pixel time series of an image cube, the mean of 8 preceding images subtracted
        dict(kind="spectra", name="dynspec_512", n_time=100, n_chan=24, n_pix_side=512, ref="mean", ref_len=8),
        # the correlator: 8-bit voltages of 256 antennas, 32 channels x 16 integrations
        dict(kind="correlate", name="correlate_256", n_ant=256, n_time=16, n_chan=32, n_samp=4096),
    ]


# ------------------------------------------------------------------ drawn cases
def _log(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]."""
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _within(c):
    """Whether a drawn case costs no more than the listed ones of its kind."""
    n_img = c.get("n_time", 1) * c.get("n_chan", 1)
    if c["kind"] == "spectra":
        return n_img * c["n_pix_side"] ** 2 <= 2400 * 512 * 512
    if c["kind"] == "correlate":
        return n_img * c["n_ant"] ** 2 * max(c["n_samp"], c["n_ant"]) <= 512 * 256 * 256 * 4096
    n_bl = c["n_ant"] * (c["n_ant"] - 1) // 2
    cells = n_img * c["grid_n"] ** 2
    entries = n_img * n_bl
    if c["kind"] == "image":
        return (cells <= 1536 * 1024 ** 2 and entries <= 3200 * 32640
                and (not c["kernel"] or (cells <= 384 * 1024 ** 2 and entries * c["kernel"] ** 2 <= 384 * 8128 * 36)))
    if c["kind"] == "train":
        return cells <= 320 * 1024 ** 2 and entries <= 320 * 8128
    return cells <= 32 * 1024 ** 2 and entries <= 128 * 8128       # grid


def draw(rng):
    while True:
        kind = rng.choice(["image"] * 6 + ["train", "train", "grid", "fft", "spectra", "correlate", "correlate"])
        if kind == "fft":
            n = rng.choice([128, 180, 256, 512, 1024, 2048])
            return dict(kind="fft", grid_n=n, batch=_log(rng, 1, max(1, 64 * 1024 * 1024 // (n * n))),
                        sign=rng.choice([1, -1]))
        if kind == "spectra":
            c = dict(kind="spectra", n_time=_log(rng, 9, 700), n_chan=_log(rng, 1, 64),
                     n_pix_side=rng.choice([128, 180, 256, 400, 511, 512]), ref=rng.choice(["none", "mean", "model"]),
                     ref_len=rng.choice([1, 4, 8, 25]))
        elif kind == "correlate":
            c = dict(kind="correlate", n_ant=rng.randint(16, 256), n_time=_log(rng, 1, 64), n_chan=_log(rng, 1, 64),
                     n_samp=16 * _log(rng, 4, 256))
        else:
            station = rng.random() < 0.35
            radius = 35.0 if station else rng.choice([1000.0, 3000.0, 5000.0])
            c = dict(kind=kind, n_ant=rng.randint(24, 256) if station else rng.randint(48, 256),
                     core_m=radius if station else 0.1 * radius, disc_m=radius, n_time=_log(rng, 1, 64),
                     n_chan=_log(rng, 1, 768), f0=rng.uniform(80e6, 220e6), df=rng.choice([10e3, 40e3, 200e3]),
                     grid_n=rng.choice([128, 180, 256]) if station else rng.choice([256, 512, 1024, 1024, 2048]),
                     uniform=rng.random() < 0.5, flagged=rng.random() < 0.5)
            n = c["grid_n"]
            out_n = n if station else rng.choice([n, n // 2, n // 2, 2 * rng.randint(n // 8, n // 2)])
            if kind == "image":
                c = _image(None, **{**c, "kind": "image", "out_n": out_n,
                                    "storage": rng.choice(["c64", "c64", "c64", "f16", "bf16"]),
                                    "kernel": rng.choice([0, 0, 0, 0, 4, 6, 7]), "rotate": rng.random() < 0.25,
                                    "gains": rng.random() < 0.25})
            elif kind == "train":
                c["out_n"] = out_n
        if _within(c):
            return c


# ------------------------------------------------------------------ inputs
def _device():
    return torch.device("cuda:0")


def _gens(seed):
    cpu = torch.Generator().manual_seed(20240521 + seed)
    gpu = torch.Generator(device=_device()).manual_seed(40240521 + seed)
    return cpu, gpu


def _disc(n, radius, g):
    r = radius * torch.sqrt(torch.rand(n, generator=g, dtype=torch.float64))
    th = 2 * math.pi * torch.rand(n, generator=g, dtype=torch.float64)
    return torch.stack([r * torch.cos(th), r * torch.sin(th)], 1)


def _freqs(case):
    return case["f0"] + case["df"] * torch.arange(case["n_chan"], dtype=torch.float64)


def _pixscale(case):
    """2 / N for the whole sky, else the longest possible baseline's beam sampled three times."""
    if case.get("allsky"):
        return 2.0 / case["grid_n"]
    return 1.0 / (3.0 * 2.0 * case["disc_m"] * float(_freqs(case).max()) / C_LIGHT)


def _observation(case, seed):
    """Geometry, sky and visibilities of an imaging case, on the GPU."""
    dev = _device()
    cpu, gpu = _gens(seed)
    A, T, C = case["n_ant"], case["n_time"], case["n_chan"]
    xy = torch.cat([_disc(A // 2, case["core_m"], cpu), _disc(A - A // 2, case["disc_m"], cpu)])
    a1, a2 = torch.triu_indices(A, A, 1)
    d = xy[a2] - xy[a1]
    th = (OMEGA_EARTH * DT * torch.arange(T, dtype=torch.float64))[:, None]
    u = d[None, :, 0] * torch.cos(th) - d[None, :, 1] * torch.sin(th)
    v = d[None, :, 0] * torch.sin(th) + d[None, :, 1] * torch.cos(th)
    w = 1e-3 * u + 2e-3 * v if case.get("rotate") else torch.zeros_like(u)
    uvw = torch.stack([u, v, w], -1).contiguous().to(dev)
    freq = _freqs(case).to(dev)
    B = uvw.shape[1]
    # a sky inside the imaged field
    fov = min(1.0, _pixscale(case) * case["grid_n"]) * 0.45
    lm = _disc(N_SRC, fov, cpu)
    flux = 1 + 9 * torch.rand(N_SRC, generator=cpu, dtype=torch.float64)
    vis = torch.empty((T, C, B), dtype=torch.complex64, device=dev)
    tc = max(1, (1 << 25) // max(1, C * B))
    for t in range(0, T, tc):
        re = 0.1 * torch.randn(vis[t:t + tc].shape, generator=gpu, device=dev)
        im = 0.1 * torch.randn(vis[t:t + tc].shape, generator=gpu, device=dev)
        for k in range(N_SRC):
            path = uvw[t:t + tc, :, 0] * float(lm[k, 0]) + uvw[t:t + tc, :, 1] * float(lm[k, 1])
            turns = path[:, None, :] * (freq / C_LIGHT)[None, :, None]
            ph = (turns - torch.round(turns)).float() * (-2.0 * math.pi)
            re.add_(torch.cos(ph), alpha=float(flux[k]))
            im.add_(torch.sin(ph), alpha=float(flux[k]))
        vis[t:t + tc] = torch.complex(re, im)
    s = dict(vis=vis, uvw=uvw, freq=freq, ant1=a1.to(torch.int32).to(dev), ant2=a2.to(torch.int32).to(dev),
             flags=None, gains=None, cable=None, scale=None, lm=(0.0, 0.0))
    if case.get("flagged"):
        frac = 0.02 + 0.08 * torch.rand((T, 1), generator=cpu)
        s["flags"] = (torch.rand((T, B), generator=cpu) < frac).to(torch.uint8).to(dev)
    if case.get("gains") or case["kind"] == "train":
        n = 0.05 * torch.randn((A, 2), generator=cpu)
        s["gains"] = torch.complex(1 + n[:, 0], n[:, 1]).to(dev)
    if case.get("rotate"):
        s["cable"] = (500.0 * torch.rand(A, generator=cpu, dtype=torch.float64)).to(dev)
        s["lm"] = (0.05, 0.03)
    if case.get("storage", "c64") != "c64":
        ri = torch.view_as_real(vis)
        sig = ri.abs().amax(dim=(0, 2, 3))
        s["scale"] = sig.contiguous()
        s["vis"] = (ri / sig[None, :, None, None]).to(STORAGE[case["storage"]]).contiguous()
    return s


def _image_options(case, s):
    return dict(grid_n=case["grid_n"], pixscale=_pixscale(case), out_n=case["out_n"],
                weighting=blink.UNIFORM if case["uniform"] else blink.NATURAL, norm=blink.NORM_WEIGHTS,
                gains=s["gains"], kernel_support=case["kernel"], phase_lm=s["lm"], cable_m=s["cable"])


def prepare(case, seed):
    dev = _device()
    kind = case["kind"]
    if kind == "fft":
        _, gpu = _gens(seed)
        n = case["grid_n"]
        x = torch.randn((case["batch"], n, n), generator=gpu, device=dev, dtype=torch.complex64)
        return dict(case=case, x=x, out=torch.empty_like(x))
    if kind == "spectra":
        _, gpu = _gens(seed)
        T, C, M = case["n_time"], case["n_chan"], case["n_pix_side"]
        sky = 3.0 * torch.rand((1, C, M, M), generator=gpu, device=dev)
        cube = torch.randn((T, C, M, M), generator=gpu, device=dev)
        cube.add_(sky)
        ref = sky[0].contiguous() if case["ref"] == "model" else None
        return dict(case=case, images=cube, ref=ref, out=torch.empty((M * M, C, T), device=dev))
    if kind == "correlate":
        _, gpu = _gens(seed)
        T, C, A, S = case["n_time"], case["n_chan"], case["n_ant"], case["n_samp"]
        volt = torch.empty((T, C, A, S, 2), dtype=torch.int8, device=dev)
        for t in range(T):       # Gaussian noise of 20 counts, the levels an 8-bit channeliser is set to
            volt[t] = (20.0 * torch.randn((C, A, S, 2), generator=gpu, device=dev)).round_().clamp_(-127, 127)
        vis = torch.empty((T, C, A * (A - 1) // 2), dtype=torch.complex64, device=dev)
        return dict(case=case, volt=volt, vis=vis)
    s = _observation(case, seed)
    s["case"] = case
    T, C, M = case["n_time"], case["n_chan"], case.get("out_n", 0)
    if kind == "image":
        opt = _image_options(case, s)
        tun = api.tuning_for(case["grid_n"], M, s["uvw"].shape[1], opt["weighting"], api._vis_type(s["vis"]))
        p = api.make_problem(s["vis"], s["uvw"], s["freq"], **opt, **tun)
        s["ws"] = blink.workspace(p, blink.CALL_IMAGE, dev)
        s["images"] = torch.empty((T * C, M, M), device=dev)
        s["weight_sum"] = torch.empty((T * C,), device=dev)
    elif kind == "train":
        _, gpu = _gens(seed + 1)
        s["model"] = torch.randn((T * C, M, M), generator=gpu, device=dev)
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "image":
        blink.image_batch(s["vis"], s["uvw"], s["freq"], flags=s["flags"], vis_scale=s["scale"], ant1=s["ant1"],
                          ant2=s["ant2"], images=s["images"], weight_sum=s["weight_sum"], ws=s["ws"],
                          **_image_options(case, s))
        return dict(images=s["images"], weight_sum=s["weight_sum"])
    if kind == "train":
        vis, gains = s["vis"].detach().requires_grad_(), s["gains"].detach().requires_grad_()
        images = blink.blink_image(vis, gains, s["uvw"], s["freq"], s["ant1"], s["ant2"], grid_n=case["grid_n"],
                                   pixscale=_pixscale(case), out_n=case["out_n"],
                                   weighting=blink.UNIFORM if case["uniform"] else blink.NATURAL, flags=s["flags"])
        # the gradient of |images - model|^2 / 2
        g_vis, g_gains = torch.autograd.grad(images, (vis, gains), torch.sub(images.detach(), s["model"]))
        return dict(images=images.detach(), g_vis=g_vis, g_gains=g_gains)
    if kind == "grid":
        g, counts, w, dropped = blink.grid(s["vis"], s["uvw"], s["freq"], grid_n=case["grid_n"],
                                           pixscale=_pixscale(case), flags=s["flags"],
                                           weighting=blink.UNIFORM if case["uniform"] else blink.NATURAL)
        return dict(grid=g, counts=counts, weight_sum=w, dropped=dropped)
    if kind == "fft":
        return blink.fft2d(s["x"], sign=case["sign"], out=s["out"])
    if kind == "spectra":
        mode = {"none": blink.REF_NONE, "mean": blink.REF_MEAN, "model": blink.REF_MODEL}[case["ref"]]
        return blink.dynamic_spectra(s["images"], mode, case["ref_len"], s["ref"], out=s["out"])
    vis, autos = blink.correlate(s["volt"], vis=s["vis"], autos=True)
    return dict(vis=vis, autos=autos)


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind == "fft":
        n2 = case["grid_n"] ** 2 * case["batch"]
        return {"bytes": 16 * n2, "flops": 5 * n2 * math.log2(case["grid_n"] ** 2)}
    if kind == "spectra":
        n = case["n_time"] * case["n_chan"] * case["n_pix_side"] ** 2
        return {"bytes": 8 * n, "flops": (3 if case["ref"] == "mean" else 1) * n}
    n_img = case["n_time"] * case["n_chan"]
    A = case["n_ant"]
    B = A * (A - 1) // 2
    if kind == "correlate":
        return {"bytes": n_img * (2 * A * case["n_samp"] + 8 * B + 4 * A),
                "flops": 8 * n_img * (B + A) * case["n_samp"]}
    N = case["grid_n"]
    taps = max(1, case.get("kernel", 0)) ** 2
    vis_bytes = n_img * B * (8 if case.get("storage", "c64") == "c64" else 4)
    uvw_bytes = case["n_time"] * B * (24 + (1 if case["flagged"] else 0))
    if kind == "grid":
        return {"bytes": vis_bytes + uvw_bytes + 12 * n_img * N * N, "flops": n_img * 8 * B}
    fft = 2.5 * N * N * math.log2(N * N)                 # a real image's transform
    image_bytes = 4 * n_img * case["out_n"] ** 2
    if kind == "image":
        return {"bytes": vis_bytes + uvw_bytes + image_bytes, "flops": n_img * (fft + 8 * B * taps)}
    # images out; gradient images and visibilities in, visibility gradients out
    return {"bytes": 3 * vis_bytes + 2 * uvw_bytes + 4 * image_bytes, "flops": n_img * (2 * fft + 24 * B)}


# ------------------------------------------------------------------ 64 bits
def _cells(case, s, t, c0, c1):
    """Exact cell positions of timestep t at channels c0..c1: x_u, x_v [c][B] and the unflagged baselines."""
    scale = (s["freq"][c0:c1] * (case["grid_n"] * _pixscale(case))) / C_LIGHT
    xu = s["uvw"][t, :, 0][None] * scale[:, None]
    xv = s["uvw"][t, :, 1][None] * scale[:, None]
    ok = torch.ones_like(xu[:1], dtype=torch.bool) if s["flags"] is None else (s["flags"][t] == 0)[None]
    return xu, xv, ok.expand_as(xu)


def _visibilities64(case, s, t, c0, c1, gains=None, vis=None):
    """Calibrated and rotated visibilities [c][B] in complex128."""
    v = s["vis"][t, c0:c1] if vis is None else vis
    if not v.is_complex():
        v = torch.view_as_complex(v.double().contiguous()) * s["scale"][c0:c1, None].double()
    v = v.to(torch.complex128)
    g = s["gains"].to(torch.complex128) if gains is None and s["gains"] is not None else gains
    if g is not None:
        v = (g[s["ant1"].long()] * g[s["ant2"].long()].conj())[None] * v
    l, m = s["lm"]
    if s["cable"] is not None:
        n = math.sqrt(1 - l * l - m * m)
        d = s["uvw"][t, :, 0] * l + s["uvw"][t, :, 1] * m + s["uvw"][t, :, 2] * (n - 1)
        d = d + s["cable"][s["ant1"].long()] - s["cable"][s["ant2"].long()]
        ph = d[None] * (s["freq"][c0:c1] / C_LIGHT)[:, None]
        v = v * torch.polar(torch.ones_like(ph), 2 * math.pi * (ph - torch.round(ph)))
    return v


def _scatter(n_img, N, ku, kv, val):
    """Sums of val at the cells (kv, ku) mod N of each image: [c][N][N]."""
    idx = (torch.arange(n_img, device=val.device)[:, None] * N + kv.long() % N) * N + ku.long() % N
    out = torch.zeros(n_img * N * N, dtype=val.dtype, device=val.device)
    return out.index_add(0, idx.reshape(-1), val.reshape(-1)).reshape(n_img, N, N)


def _grid64(case, s, t, c0, c1, v):
    """(weighted grid [c][N][N], counts or None, weight sums [c], dropped [c])."""
    N, H = case["grid_n"], case["grid_n"] // 2
    xu, xv, ok = _cells(case, s, t, c0, c1)
    n = xu.shape[0]
    W = case.get("kernel", 0)
    if not W:
        ku, kv = torch.round(xu), torch.round(xv)
        keep = ok & (ku.abs() < H) & (kv.abs() < H)
        one = keep.double()
        v = v * one
        g = _scatter(n, N, ku, kv, v) + _scatter(n, N, -ku, -kv, v.conj())
        counts = _scatter(n, N, ku, kv, one) + _scatter(n, N, -ku, -kv, one)
        dropped = (ok & ~keep).sum(1)
        if case["uniform"]:
            return g / counts.clamp(min=1), counts, (counts > 0).sum((1, 2)).double(), dropped
        return g, counts, counts.sum((1, 2)), dropped
    hw = 0.5 * W
    keep = ok
    for x in (xu, xv):
        keep = keep & (torch.ceil(x - hw) > -H) & (torch.floor(x + hw) < H)
    one = keep.double()
    share = one
    if case["uniform"]:
        ku, kv = torch.round(xu), torch.round(xv)
        dens = _scatter(n, N, ku, kv, one) + _scatter(n, N, -ku, -kv, one)
        idx = (torch.arange(n, device=xu.device)[:, None] * N + kv.long() % N) * N + ku.long() % N
        share = one / dens.reshape(-1)[idx].clamp(min=1)
    v = v * share
    beta = _beta(W)
    g = torch.zeros((n, N, N), dtype=v.dtype, device=v.device)
    total = torch.zeros(n, dtype=torch.float64, device=v.device)

    def weights(x):
        i = torch.ceil(x - hw)[..., None] + torch.arange(W + 1, device=x.device)
        q = 1 - (2 * (i - x[..., None]) / W) ** 2
        z = beta * torch.sqrt(q.clamp(min=0))
        return i, torch.where(q >= -1e-15, torch.special.i0e(z) * torch.exp(z - beta), 0.0) / float(
            torch.special.i0e(torch.tensor(beta, dtype=torch.float64)))
    iu, wu = weights(xu)
    iv, wv = weights(xv)
    for a in range(W + 1):
        for b in range(W + 1):
            w = wu[..., a] * wv[..., b]
            g += _scatter(n, N, iu[..., a], iv[..., b], v * w) + _scatter(n, N, -iu[..., a], -iv[..., b], (v * w).conj())
            total += 2 * (w * share).sum(1)
    return g, None, total, None


def _beta(W):
    return math.pi * math.sqrt(0.5625 * W * W - 0.8)


def _image64(case, g, weight):
    """The cut, shifted and normalised images of weighted grids."""
    N, M = case["grid_n"], case["out_n"]
    img = torch.fft.ifft2(g, norm="forward").real
    img = torch.roll(img, (M // 2, M // 2), (1, 2))[:, :M, :M]
    img = torch.where(weight[:, None, None] > 0, img / weight.clamp(min=1e-300)[:, None, None], 0.0)
    if case.get("kernel", 0):
        beta = _beta(case["kernel"])
        x = math.pi * case["kernel"] * (torch.arange(M, device=g.device, dtype=torch.float64) - M // 2) / N
        z2 = beta * beta - x * x
        z = torch.sqrt(z2.abs()).clamp(min=1e-12)
        c = torch.where(z2 >= 0, torch.sinh(z), torch.sin(z)) / z / (math.sinh(beta) / beta)
        img = img / c[None, :, None] / c[None, None, :]
    return img


def _spans(case, most):
    """(timestep, first channel, last channel) in pieces of at most `most` images."""
    for t in range(case["n_time"]):
        for c in range(0, case["n_chan"], most):
            yield t, c, min(case["n_chan"], c + most)


def exact(case, seed):
    kind = case["kind"]
    if kind == "correlate":      # integer sums, exact in the result's type up to 2^24
        s = prepare(case, seed)
        T, C, A = case["n_time"], case["n_chan"], case["n_ant"]
        a1, a2 = torch.triu_indices(A, A, 1)
        vis = torch.empty(s["vis"].shape, dtype=torch.complex128, device=s["vis"].device)
        autos = torch.empty((T, C, A), dtype=torch.float64, device=vis.device)
        for t in range(T):
            for c in range(C):
                x = s["volt"][t, c].double()
                r, q = x[..., 0].contiguous(), x[..., 1].contiguous()
                re = r @ r.t().contiguous() + q @ q.t().contiguous()
                im = q @ r.t().contiguous() - r @ q.t().contiguous()
                vis[t, c] = torch.complex(re, im)[a1, a2]
                autos[t, c] = re.diagonal()
        return dict(vis=vis, autos=autos)
    s = prepare(case, seed)
    if kind == "fft":
        out = torch.empty(s["x"].shape, dtype=torch.complex128, device=s["x"].device)
        for b in range(0, case["batch"], 16):
            x = s["x"][b:b + 16].to(torch.complex128)
            out[b:b + 16] = torch.fft.ifft2(x, norm="forward") if case["sign"] > 0 else torch.fft.fft2(x)
        return out
    if kind == "spectra":
        T, C, M = case["n_time"], case["n_chan"], case["n_pix_side"]
        out = torch.empty((M * M, C, T), dtype=torch.float64, device=s["images"].device)
        for c in range(C):
            x = s["images"][:, c].reshape(T, M * M).double()
            if case["ref"] == "model":
                x = x - s["ref"][c].reshape(1, -1).double()
            elif case["ref"] == "mean":
                y = torch.zeros_like(x)
                for t in range(1, T):
                    y[t] = x[t] - x[max(0, t - case["ref_len"]):t].mean(0)
                x = y
            out[:, c] = x.t()
        return out
    most = max(1, (48 << 20) // case["grid_n"] ** 2)
    if kind == "grid":
        parts = []
        for t, c0, c1 in _spans(case, most):
            parts.append(_grid64(case, s, t, c0, c1, _visibilities64(case, s, t, c0, c1)))
        # the counts and the dropped baselines are whole numbers
        return dict(grid=torch.cat([p[0] for p in parts]), counts=torch.cat([p[1] for p in parts]).to(torch.int32),
                    weight_sum=torch.cat([p[2] for p in parts]),
                    dropped=torch.cat([p[3] for p in parts]).to(torch.int32))
    n_img, C = case["n_time"] * case["n_chan"], case["n_chan"]
    M = case["out_n"]
    dev = s["vis"].device
    images = torch.empty((n_img, M, M), dtype=torch.float64, device=dev)
    if kind == "image":
        wsum = torch.empty(n_img, dtype=torch.float64, device=dev)
        for t, c0, c1 in _spans(case, most):
            g, _, w, _ = _grid64(case, s, t, c0, c1, _visibilities64(case, s, t, c0, c1))
            images[t * C + c0:t * C + c1] = _image64(case, g, w)
            wsum[t * C + c0:t * C + c1] = w
        return dict(images=images, weight_sum=wsum)
    g_vis = torch.empty(s["vis"].shape, dtype=torch.complex128, device=dev)
    g_gains = torch.zeros(s["gains"].shape, dtype=torch.complex128, device=dev)
    for t, c0, c1 in _spans(case, max(1, most // 3)):
        vis = s["vis"][t, c0:c1].to(torch.complex128).requires_grad_()
        gains = s["gains"].to(torch.complex128).requires_grad_()
        g, _, w, _ = _grid64(case, s, t, c0, c1, _visibilities64(case, s, t, c0, c1, gains, vis))
        img = _image64(case, g, w)
        at = slice(t * C + c0, t * C + c1)
        images[at] = img.detach()
        gv, gg = torch.autograd.grad(img, (vis, gains), img.detach() - s["model"][at].double())
        g_vis[t, c0:c1] = gv
        g_gains += gg
    return dict(images=images, g_vis=g_vis, g_gains=g_gains)
