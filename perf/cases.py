"""Performance cases: the work a user of the library has it do, through the
public entry points of paper_1209_6038_amd.rt.

    listed()            the cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs on the GPU, and what a program keeps (cloak
                        handles, render plans, a model)
    run(state)          one pass; returns its outputs whole
    work(case)          bytes and flops one pass cannot do without
    exact(case, seed)   the outputs in 64 bits, without this library, where a
                        closed form or plain torch gives them

Geometry and sizes are those of paper_1209_6038_amd.workloads, bench.py and
the tests: radii 1 and 2, the cloak of height 4 on the floor of the
checkerboard room, Dormand-Prince 5(4) at 1e-8 in FP64 for rays, a network of
6 -> 256 x 4 -> 5 units for the surrogate.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1209_6038_amd import rt
from paper_1209_6038_amd import workloads as W

DEV = "cuda"
HID, NIN, NOUT = 256, 6, 5


def listed():
    return [
        # a handful of rays, with all per-ray diagnostics (the call's
        # default): interactive use, unit tests; launches and the longest
        # ray's serial chain
        {"name": "trace_256", "do": "trace", "axis": 1, "pol": 1, "n": 256, "trans": False},
        # a serving-size batch with the Eq. (12) intensity weights
        {"name": "trace_weights_50k", "do": "trace", "axis": 0, "pol": 1, "n": 50_001, "trans": True},
        # the weighted bundle of the weights benchmark
        {"name": "trace_weights_1m", "do": "trace", "axis": 1, "pol": 0, "n": 1 << 20, "trans": True},
        # the paper's own scheme (fixed-step RK4, h = 1e-3) on the 2-D
        # in-plane bundle: 16,384 impact parameters x 8 angles
        {"name": "inplane_rk4", "do": "inplane", "n": 16384, "angles": 8, "h": 1e-3},
        # one small preview image of one cloak, both branches
        {"name": "preview_200x150", "do": "render", "w": 200, "h": 150, "spp": 1, "views": 1, "ncl": 1, "aux": ""},
        # the 3-D render workload: both cloaks x 4 elevations x 1024^2 x
        # both branches, replayed from a plan (HIP graph)
        {"name": "plan_1024_x4", "do": "plan", "w": 1024, "h": 1024, "spp": 1, "views": 4, "ncl": 2},
        # one frame of the large render: both cloaks, 4096^2 x 4 samples
        {"name": "frame_4096_4spp", "do": "render", "w": 4096, "h": 4096, "spp": 4, "views": 1, "ncl": 2, "aux": ""},
        # the paper's figures: unpolarized, goggle and reflection images
        # (odd size, 4 samples per pixel)
        {"name": "figures_501x377", "do": "render", "w": 501, "h": 377, "spp": 4, "views": 1, "ncl": 2,
         "aux": "reflections"},
        # labelling surrogate training data: exact transits and their targets
        {"name": "label_1m", "do": "label", "n": 1 << 20},
        # network inference on a million entries
        {"name": "forward_1m", "do": "forward", "n": 1 << 20},
        # one optimization step at the training benchmark's batch, and at
        # a small ragged one
        {"name": "train_65536", "do": "train", "n": 65536},
        {"name": "train_1000", "do": "train", "n": 1000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["trace", "trace", "inplane", "render", "render", "plan", "label", "forward", "train", "train"])
    if do == "trace":
        return {"do": do, "axis": rng.randint(0, 1), "pol": rng.randint(0, 1), "n": _log_int(rng, 64, 1 << 20),
                "trans": rng.random() < 0.5}
    if do == "inplane":
        return {"do": do, "n": _log_int(rng, 100, 16384), "angles": rng.randint(1, 8),
                "h": rng.choice([1e-3, 2e-3, 4e-3])}
    if do in ("render", "plan"):
        big = do == "plan"
        w, h = _log_int(rng, 64, 1024), _log_int(rng, 64, 1024)
        c = {"do": do, "w": w, "h": h, "spp": rng.choice([1, 1, 4]), "views": rng.randint(1, 4),
             "ncl": rng.randint(1, 2)}
        if not big:
            c["aux"] = rng.choice(["", "", "tof", "unpolarized", "goggles", "reflections"])
        return c
    if do == "label":
        return {"do": do, "n": _log_int(rng, 1000, 1 << 20)}
    if do == "forward":
        return {"do": do, "n": _log_int(rng, 100, 1 << 20)}
    return {"do": do, "n": _log_int(rng, 100, 65536)}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _bundle(case, seed):
    """The in-plane bundle, turned by an angle of the seed. float64 (6, n)."""
    b = W.inplane_bundle(case["n"], case["angles"])
    a = np.random.default_rng(seed).uniform(0.0, 2.0 * math.pi)
    c, s = math.cos(a), math.sin(a)
    out = b.copy()
    for i in (0, 3):
        out[i], out[i + 1] = c * b[i] - s * b[i + 1], s * b[i] + c * b[i + 1]
    return out


def _cams(case, seed):
    """Views of one elevation each (0 to 45 degrees as in the 3-D render
    workload; a single view at 30), at an azimuth of the seed."""
    az = np.random.default_rng(seed).uniform(0.0, 2.0 * math.pi)
    el = [30.0] if case["views"] == 1 else [0.0, 15.0, 30.0, 45.0][: case["views"]]
    return [W.orbit_camera(az, e, case["w"], case["h"], case["spp"], seed=seed) for e in el]


def _params(seed):
    """FP32 parameters (weights uniform in +-1/sqrt(fan_in)), drawn here so
    that exact() knows them."""
    r = np.random.default_rng(seed + 77)
    sizes = [(NIN, HID), (HID, HID), (HID, HID), (HID, HID), (HID, NOUT)]
    return [r.uniform(-1.0 / math.sqrt(a), 1.0 / math.sqrt(a), k).astype(np.float32)
            for a, b in sizes for k in ((a, b), (b,))]


# standardization of (k_theta, k_z, alpha, beta, bits) for uniform entries,
# and the spread of the training targets
_SCALING = np.array([0.0, 0.0, 0.0, 0.0, 0.5, 0.5, 2.0, 1.414, 1.103, 1.103, 2.0, 2.0,
                     0.0, 0.0, 0.0, 0.0, 0.0, 2e-3, 2e-3, 1e-3, 1e-3, 2e-3], dtype=np.float32)


def _entries(n, seed):
    return torch.from_numpy(W.surrogate_features(n, seed))


def _targets(x6, seed):
    """Smooth residual targets of the transits with some scatter, and row
    weights with one row in eight unlabelled."""
    g = torch.Generator().manual_seed(seed + 5)
    al, be = x6[2], x6[3]
    base = torch.stack([torch.sin(2 * al) * torch.cos(be), torch.sin(be) * torch.cos(al), al * be * 0.4,
                        torch.cos(3 * be) * (0.5 - x6[4]), torch.cos(al + be) * (0.5 - x6[5])])
    t = (base + 0.1 * torch.randn(base.shape, generator=g)) * torch.from_numpy(_SCALING[17:22])[:, None]
    w = (torch.rand(x6.shape[1], generator=g) >= 0.125).float()
    return t, w


def _model(seed):
    m = rt.Surrogate(seed=0)
    m.set_params(np.concatenate([p.reshape(-1) for p in _params(seed)]))
    m.set_scaling(_SCALING)
    return m


def prepare(case, seed):
    do, s = case["do"], {"case": case}
    if do == "trace":
        s["cloak"] = rt.Cloak(W.cloak(case["axis"], height=W.HEIGHT))
        s["rays"] = torch.from_numpy(W.random_rays(case["n"], seed)).to(DEV)
        s["opts"] = W.opts_dp45()
    elif do == "inplane":
        s["cloak"] = rt.Cloak(W.cloak(W.RADIAL))
        s["rays"] = torch.from_numpy(_bundle(case, seed)).to(DEV)
        s["opts"] = W.opts_rk4(case["h"])
    elif do in ("render", "plan"):
        s["cloaks"] = [rt.Cloak(W.cloak(a, height=W.HEIGHT)) for a in (1, 0)[: case["ncl"]]]
        s["room"], s["opts"], s["cams"] = W.room(), W.render_opts(), _cams(case, seed)
        if do == "plan":
            s["plan"] = rt.RenderPlan(s["cloaks"], s["opts"], s["room"], s["cams"], 3)
        else:
            s["rgb"] = torch.empty((case["ncl"], case["views"], 2, case["h"], case["w"], 3), device=DEV)
    elif do == "label":
        s["cloaks"] = [rt.Cloak(W.cloak(a)) for a in (W.RADIAL, W.AZIMUTHAL)]
        s["x6"] = _entries(case["n"], seed).to(DEV)
        s["opts"] = W.opts_dp45(1e-8, r_out=W.R2)
    else:
        x = _entries(case["n"], seed)
        s["x6"] = x.to(DEV)
        s["model"] = _model(seed)
        if do == "train":
            t, w = _targets(x, seed)
            s["t5"], s["w"] = t.to(DEV), w.to(DEV)
    return s


def run(s):
    c = s["case"]
    do = c["do"]
    if do == "trace":
        return rt.trace_batch(s["cloak"], s["opts"], c["pol"], s["rays"], with_trans=c["trans"])
    if do == "inplane":
        return rt.trace_batch(s["cloak"], s["opts"], W.EXTRAORDINARY, s["rays"], with_aux=False)
    if do == "plan":
        s["plan"].launch()
        return s["plan"].rgb
    if do == "render":
        a = c["aux"]
        return rt.render_multi(s["cloaks"], s["opts"], s["room"], s["cams"], 3, out=s["rgb"],
                               aux=("tof",) if a == "tof" else False,
                               unpolarized=a in ("unpolarized", "goggles", "reflections"),
                               goggles=a in ("goggles", "reflections"), reflections=a == "reflections")
    if do == "label":
        y5, st = rt.transit_exact(s["cloaks"], s["opts"], s["x6"])
        t5, w = rt.surrogate_encode(s["cloaks"], s["x6"], y5, st)
        return {"y5": y5, "status": st, "t5": t5, "w": w}
    if do == "forward":
        return s["model"].forward(s["x6"])
    g, loss = s["model"].grad(s["x6"], s["t5"], s["w"], huber=0.01)
    s["model"].step(g, lr=1e-4)
    return {"grad": g, "loss": loss}


# ---------------------------------------------------------------------------
# work: bytes in and out of one pass, and its flops. Rays: step attempts per
# entering ray (measured means) x flops per attempt (FMA = 2).
# ---------------------------------------------------------------------------
DP45_FLOPS, RK4_FLOPS = 437 + 6 * 34, 123 + 4 * 35
ATTEMPTS = 36.0           # DP45 at 1e-8, per entering ray
MLP_FLOPS = 2 * (NIN * HID + 3 * HID * HID + HID * NOUT)
NPARAM = NIN * HID + 3 * HID * HID + HID * NOUT + 4 * HID + NOUT


def work(case):
    do = case["do"]
    if do == "trace":
        n = case["n"]
        return {"bytes": n * (48 + 48 + 8 + 4 + 12 + (8 if case["trans"] else 0)),
                "flops": 0.46 * n * ATTEMPTS * DP45_FLOPS}
    if do == "inplane":
        n = case["n"] * case["angles"]
        return {"bytes": n * (48 + 48 + 8 + 4), "flops": n * (2.0 / 3.0) * (math.pi / case["h"]) * RK4_FLOPS}
    if do in ("render", "plan"):
        samples = case["w"] * case["h"] * case["spp"] * case["views"]
        images = case["ncl"] * 2 * case["w"] * case["h"] * case["views"] * 12
        a = case.get("aux", "")
        if a == "tof":
            images += images // 3
        images += {"unpolarized": images // 2, "goggles": 3 * images // 2, "reflections": 3 * images // 2}.get(a, 0)
        per = 2.0 if a == "reflections" else 1.0
        hit = 0.22 * min(1.0, case["h"] / case["w"])
        return {"bytes": images, "flops": samples * (100 + hit * case["ncl"] * 2 * per * ATTEMPTS * DP45_FLOPS)}
    n = case["n"]
    if do == "label":
        return {"bytes": n * (24 + 20 + 4 + 20 + 4), "flops": n * 70.0 * DP45_FLOPS}
    if do == "forward":
        return {"bytes": n * (24 + 20) + NPARAM * 4, "flops": n * MLP_FLOPS}
    # forward and backward; parameters, gradient and the two moments
    return {"bytes": n * (24 + 20 + 4) + NPARAM * 4 * 7, "flops": 3.0 * n * MLP_FLOPS}


# ---------------------------------------------------------------------------
# exact: closed form (in-plane cloaking) and plain float64 torch (the network)
# ---------------------------------------------------------------------------
def _mlp64(params, x6):
    al, be = x6[2].double(), x6[3].double()
    f = torch.stack([torch.cos(be) * torch.sin(al), torch.sin(be), al, be, x6[4].double(), x6[5].double()], 1)
    sc = torch.from_numpy(_SCALING).double().to(f.device)
    h = (f - sc[:6]) * sc[6:12]
    for k in range(4):
        z = h @ params[2 * k] + params[2 * k + 1]
        h = z * torch.sigmoid(z)
    return h @ params[8] + params[9]


def exact(case, seed):
    do = case["do"]
    if do == "inplane":
        # A cloaked in-plane ray leaves on its incident line after the
        # vacuum's optical path, and so does one that misses. The fixed step
        # does not resolve rays aimed next to the axis, and the last states
        # of those that diverge there have no exact value, so only the
        # optical path is given.
        r = _bundle(case, seed)
        b = r[0] * r[3] + r[1] * r[4]
        p2 = (r[0] - b * r[3]) ** 2 + (r[1] - b * r[4]) ** 2
        return {"out": None, "opl": np.sqrt(np.maximum(9.0 - p2, 0.0)) - b, "status": None}
    if do not in ("forward", "train"):
        return None
    dev = DEV if torch.cuda.is_available() else "cpu"
    params = [torch.from_numpy(p).double().to(dev) for p in _params(seed)]
    x = _entries(case["n"], seed)
    if do == "forward":
        sc = torch.from_numpy(_SCALING).double().to(dev)
        xd = x.to(dev)
        out = [_mlp64(params, xd[:, i:i + (1 << 16)]) for i in range(0, case["n"], 1 << 16)]
        return (torch.cat(out) * sc[17:22] + sc[12:17]).T.contiguous()
    t, w = _targets(x, seed)
    t, w, n = t.double().to(dev), w.double().to(dev), case["n"]
    sc = torch.from_numpy(_SCALING).double().to(dev)
    for p in params:
        p.requires_grad_(True)
    d = _mlp64(params, x.to(dev)) - ((t - sc[12:17, None]) / sc[17:22, None]).T
    a = d.abs()
    rho = torch.where(a <= 0.01, d * d, 0.02 * a - 1e-4)
    loss = (rho * w[:, None]).sum() / n
    loss.backward()
    return {"grad": torch.cat([p.grad.reshape(-1) for p in params]), "loss": loss.detach().reshape(1)}
