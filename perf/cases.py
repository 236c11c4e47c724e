"""Workloads of the haemoglobin-estimation path, for timing it.

A case is one shape of call that a program makes: frame size, Haar levels,
posterior grid, storage type, frames per call, estimator options and the maps
it asks for.  ``listed()`` names the calls that the benchmark, the serving
pattern, the pulse analysis and the parity tests are built on, from one 64x64
frame to sixteen 1920x1080 frames; ``draw()`` gives others of the same
ranges.  Frames are rendered on the GPU from seeded haemoglobin fields (sums
of Gaussian blobs, rigidly moving from frame to frame) by Beer-Lambert
absorption with sensor noise, as ``paper_1706_07263_amd.synth`` does on the
host.
"""
import math

import numpy as np
import torch

from paper_1706_07263_amd import hb, synth

THB_MIN, THB_MAX = synth.THB_RANGE
SO2_MIN, SO2_MAX = synth.SO2_RANGE
LAMBDA = 1e-3
FLOOR = 1e-4
THB_EPS = 1e-3
MAPS = {"all": (1, 1, 1, 1), "thb": (0, 0, 1, 0), "thb+so2": (0, 0, 1, 1)}   # Hb, HbO2, THb, SO2
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
# Share of the grid's nodes whose weight a posterior mean to 1e-6 uM needs
# (measured on the 1080p video frames at sigma 0.01: a tenth).
NODE_SHARE = 0.1


def _case(name, width, height, levels, grid_thb, grid_so2, dtype, batch, sigma=0.01, lowpass="bayes",
          illumination=False, maps="all", call="estimate"):
    c = dict(width=width, height=height, levels=levels, grid_thb=grid_thb, grid_so2=grid_so2, dtype=dtype,
             batch=batch, sigma=sigma, lowpass=lowpass, illumination=illumination, maps=maps, call=call)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one thumbnail frame on a coarse grid, launch latency
        _case("thumbnail", 64, 64, 1, 32, 32, "f32", 1),
        # a served VGA stream: the lane's captured graph replayed for one frame
        _case("vga stream graph", 640, 480, 2, 256, 256, "f16", 1, call="graph"),
        # one HD frame of a live stream through the allocation-free call
        _case("hd stream frame", 1920, 1080, 2, 256, 256, "f16", 1, call="noalloc"),
        # the video benchmark: sixteen HD frames a call
        _case("hd video batch", 1920, 1080, 2, 256, 256, "f32", 16),
        # a stereo laparoscope pair
        _case("stereo pair", 1280, 1024, 1, 128, 128, "f32", 2),
        # the same pair on the fine grid, half-precision storage
        _case("stereo pair fine grid", 1280, 1024, 1, 512, 512, "bf16", 2),
        # one 4K frame of a served stream
        _case("uhd stream frame", 3840, 2160, 2, 128, 128, "f16", 1),
        # pulse analysis: a clip of small frames of which only THb is used
        _case("pulse clip", 320, 240, 1, 128, 128, "f32", 16, maps="thb"),
        # every coefficient by the linear inverse (no posterior), HD batch
        _case("linear hd batch", 1920, 1080, 2, 256, 256, "f32", 16, lowpass="tikhonov"),
        # three Haar levels, HD
        _case("three levels", 1920, 1080, 3, 256, 256, "f32", 4),
        # posterior on every pixel, with the unknown-illumination term
        _case("full resolution lit", 1280, 1024, 0, 128, 128, "f16", 1, illumination=True),
        # a ragged frame size on a coarse ragged grid (quick preview)
        _case("ragged preview", 1006, 758, 1, 24, 20, "bf16", 3),
    ]


def draw(rng):
    levels = rng.choice((0, 1, 1, 1, 2, 2, 2, 3))
    unit = 1 << levels
    area = math.exp(rng.uniform(math.log(64 * 64), math.log(3840 * 2160)))
    aspect = rng.uniform(1.0, 1.8)
    width = max(unit, round(math.sqrt(area * aspect) / unit) * unit)
    height = max(unit, round(math.sqrt(area / aspect) / unit) * unit)
    g = math.exp(rng.uniform(math.log(20), math.log(512)))
    gt = max(16, round(g * rng.uniform(0.8, 1.2)))
    gs = gt if rng.random() < 0.5 else max(16, round(g * rng.uniform(0.8, 1.2)))
    low = (width >> levels) * (height >> levels)
    lowpass = "tikhonov" if rng.random() < 0.12 else "bayes"
    # at most 3e7 pixels a call and a third of the largest listed posterior
    most = min(16, int(3.0e7 / (width * height)))
    if lowpass == "bayes":
        while low * gt * gs > 4e10:
            gt, gs = max(16, gt * 3 // 4), max(16, gs * 3 // 4)
        most = min(most, int(4e10 / (low * gt * gs)))
    batch = max(1, min(most, rng.choice((1, 1, 2, 3, 4, 8, 16))))
    return _case(None, width, height, levels, gt, gs, rng.choice(("f32", "f16", "bf16")), batch,
                 sigma=round(math.exp(rng.uniform(math.log(0.008), math.log(0.02))), 4), lowpass=lowpass,
                 illumination=lowpass == "bayes" and rng.random() < 0.15,
                 maps=rng.choice(("all", "all", "all", "thb", "thb+so2")),
                 call="graph" if rng.random() < 0.2 else "estimate")


def _fields(case, seed):
    """True THb and SO2, float64 [batch][H][W]: blob fields under a slow rigid motion."""
    W, H, n = case["width"], case["height"], case["batch"]
    rng = np.random.default_rng(1000 + seed)
    m = min(H, W)
    motion = synth.make_motion(seed, W)
    yy, xx = torch.meshgrid(torch.arange(H, device="cuda", dtype=torch.float64),
                            torch.arange(W, device="cuda", dtype=torch.float64), indexing="ij")
    out = []
    for _ in range(2):
        cy, cx = rng.uniform(0, H, 8), rng.uniform(0, W, 8)
        sd, amp = rng.uniform(0.08, 0.25, 8) * m, rng.uniform(0.3, 1.0, 8)

        def raw(y, x):
            v = torch.zeros_like(y)
            for b in range(8):
                v += amp[b] * torch.exp(((y - cy[b]) ** 2 + (x - cx[b]) ** 2) * (-0.5 / sd[b] ** 2))
            return v

        still = raw(yy, xx)
        lo, hi = still.min(), still.max()
        frames = []
        for f in range(n):
            th, tx, ty = motion.at(18 * f)
            c, s = math.cos(th), math.sin(th)
            dy, dx = yy - 0.5 * (H - 1), xx - 0.5 * (W - 1)
            v = raw(0.5 * (H - 1) + c * dy - s * dx - ty, 0.5 * (W - 1) + s * dy + c * dx - tx)
            frames.append(((v - lo) / (hi - lo)).clamp(0.0, 1.0))
        out.append(torch.stack(frames))
    return THB_MIN + (THB_MAX - THB_MIN) * out[0], SO2_MIN + (SO2_MAX - SO2_MIN) * out[1]


def _frames(case, seed):
    """Stored RGB frames [batch][H][W][3] on the GPU."""
    sp = synth.spectra()
    dev = "cuda"
    resp = torch.tensor((sp.response / sp.response.sum(axis=1, keepdims=True)).T.copy(), device=dev)   # [n][3]
    eps = torch.tensor(np.stack([sp.eps_hb, sp.eps_hbo2]), device=dev)                                  # [2][n]
    thb, so2 = _fields(case, seed)
    conc = torch.stack([thb * (1.0 - so2), thb * so2], dim=-1).reshape(-1, 2)
    del thb, so2
    gen = torch.Generator(device=dev).manual_seed(seed)
    out = torch.empty((conc.shape[0], 3), device=dev, dtype=DTYPES[case["dtype"]])
    step = 1 << 21
    for i in range(0, conc.shape[0], step):
        c = conc[i:i + step]
        clean = torch.exp(-sp.path_length_cm * (c @ eps)) @ resp
        noise = torch.randn(clean.shape, generator=gen, device=dev, dtype=torch.float64)
        out[i:i + step] = (clean + synth.NOISE_SIGMA * noise).to(out.dtype)
    return out.reshape(case["batch"], case["height"], case["width"], 3)


def prepare(case, seed):
    frames = _frames(case, seed)
    n, H, W = case["batch"], case["height"], case["width"]
    desc = hb.make_desc(W, H, levels=case["levels"], dtype=case["dtype"], max_batch=n, grid_thb=case["grid_thb"],
                        grid_so2=case["grid_so2"], thb_min=THB_MIN, thb_max=THB_MAX, so2_min=SO2_MIN,
                        so2_max=SO2_MAX, lam=LAMBDA, sigma=case["sigma"], intensity_floor=FLOOR, thb_eps=THB_EPS,
                        lowpass=hb.HB_LOWPASS_TIKHONOV if case["lowpass"] == "tikhonov" else hb.HB_LOWPASS_BAYES,
                        illumination=int(case["illumination"]))
    plan = hb.Plan(desc, 0).set_forward_model(synth.spectra())
    maps = [torch.zeros((n, H, W), device="cuda", dtype=torch.float32) if k else None for k in MAPS[case["maps"]]]
    state = dict(plan=plan, frames=frames, maps=maps, noalloc=case["call"] == "noalloc", graph=None)
    if case["call"] == "graph":
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            plan.estimate(frames, maps)      # eager warm-up, then one graph for the lane
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            plan.estimate(frames, maps)
        state["graph"] = graph
    return state


def run(state):
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        state["plan"].estimate(state["frames"], state["maps"], noalloc=state["noalloc"])
    return [m for m in state["maps"] if m is not None]


def work(case):
    pixels = case["batch"] * case["width"] * case["height"]
    item = 4 if case["dtype"] == "f32" else 2
    out = {"bytes": pixels * (3 * item + 4 * sum(MAPS[case["maps"]])), "flops": 0}
    if case["lowpass"] == "bayes":
        # per node: squared distance (8), scale, reference, three moments
        out["flops"] = 15 * NODE_SHARE * (pixels >> (2 * case["levels"])) * case["grid_thb"] * case["grid_so2"]
    return out


def exact(case, seed):
    """The maps in 64 bits: log-attenuation, block means, the linear inverse of what deviates from them, and
    the posterior mean (or the linear inverse) of the means.  With an orthonormal Haar transform the inverted
    directional coefficients recompose to M (y - block mean of y)."""
    sp = synth.spectra()
    dev, f64 = "cuda", torch.float64
    n, H, W, B = case["batch"], case["height"], case["width"], 1 << case["levels"]
    resp = torch.tensor((sp.response / sp.response.sum(axis=1, keepdims=True)).T.copy(), device=dev)
    eps = torch.tensor(np.stack([sp.eps_hb, sp.eps_hbo2]), device=dev)
    L = sp.path_length_cm

    def attenuation(conc):
        return -torch.log(torch.exp(-L * (conc @ eps)) @ resp)

    ref_thb, ref_so2 = 0.5 * (THB_MIN + THB_MAX), 0.5 * (SO2_MIN + SO2_MAX)
    ref = torch.tensor([[ref_thb * (1 - ref_so2), ref_thb * ref_so2]], device=dev, dtype=f64)
    w = torch.exp(-L * (ref @ eps))[0][:, None] * resp                       # [n][3]
    E = L * (eps @ w / w.sum(0)).T                                           # [3][2]
    A = E.T @ E
    M = torch.linalg.solve(A + LAMBDA * 0.5 * torch.trace(A) * torch.eye(2, device=dev, dtype=f64), E.T)   # [2][3]

    thb = torch.linspace(THB_MIN, THB_MAX, case["grid_thb"], device=dev, dtype=f64)
    so2 = torch.linspace(SO2_MIN, SO2_MAX, case["grid_so2"], device=dev, dtype=f64)
    nodes = torch.stack([(thb[:, None] * (1 - so2)).reshape(-1), (thb[:, None] * so2).reshape(-1)], dim=1)
    mu0 = attenuation(ref)
    v = attenuation(nodes) - mu0
    if case["illumination"]:
        v = v - v.mean(dim=1, keepdim=True)
    scale = 1.0 / (2.0 * case["sigma"] ** 2)
    vt = (2.0 * scale) * v.T.contiguous()
    vv = -scale * (v * v).sum(dim=1)
    moments = torch.cat([torch.ones_like(nodes[:, :1]), nodes], dim=1)

    frames = _frames(case, seed)
    out = [torch.empty((n, H, W), device=dev, dtype=f64) for _ in range(4)]
    for f in range(n):
        y = -torch.log(frames[f].to(f64).clamp_min(float(np.float32(FLOOR))))
        blocks = y.reshape(H // B, B, W // B, B, 3)
        mean = blocks.mean(dim=(1, 3))                                       # [h][w][3]
        detail = (blocks - mean[:, None, :, None, :]) @ M.T
        z = mean.reshape(-1, 3) - mu0
        if case["lowpass"] == "tikhonov":
            est = ref + z @ M.T
        else:
            if case["illumination"]:
                z = z - z.mean(dim=1, keepdim=True)
            est = torch.empty((z.shape[0], 2), device=dev, dtype=f64)
            step = max(1, (1 << 29) // moments.shape[0])
            for i in range(0, z.shape[0], step):
                t = torch.addmm(vv, z[i:i + step], vt)
                t -= t.max(dim=1, keepdim=True).values
                s = t.exp_() @ moments
                est[i:i + step] = s[:, 1:] / s[:, :1]
        maps = (est.reshape(H // B, 1, W // B, 1, 2) + detail).reshape(H, W, 2)
        out[0][f], out[1][f] = maps[..., 0], maps[..., 1]
        out[2][f] = maps.sum(dim=-1)
        out[3][f] = torch.where(out[2][f] > THB_EPS, maps[..., 1] / out[2][f], math.nan)
    return [m for m, k in zip(out, MAPS[case["maps"]]) if k]
