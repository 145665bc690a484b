"""The work a user of this generator has it do, as cases that can be timed.

Every case goes through the public entry points of ``paper_2512_09664_amd``:

* ``eager``    seed -> advect -> render_pair calls with kept buffers;
* ``plan``     the same path as one captured plan, replayed;
* ``sampler``  ``make(config)`` and ``next(sampler)``;
* ``model``    the full particle model (second diameter, rho, frame-2 variation,
  hiding, the Remark 1 sheet, out-of-plane motion), eager;
* ``fit``      one step of a fit to recorded images: advect, render, and the
  backward of the mean squared difference;
* ``autograd`` the same step through ``render_images`` and torch's autograd.

``sizes`` lists the pairs as ``HxW*count`` terms; a pair's flow grid has one
node per ``grid_div`` pixels and axis.  ``exact`` restates the path in float64
with plain torch (counter-based draws included), without the library.
"""

import math

import numpy as np
import torch

import paper_2512_09664_amd as sp
from paper_2512_09664_amd import sampler as smp

DEV = "cuda"
D_CLIP = (1.0, 5.0)                 # clip of a normal diameter, pixels
I0_RANGE, Z_RANGE, SHEET = (0.8, 1.0), (-1.0, 1.0), 0.5
MODEL = {"hide_p": 0.1, "jitter": (0.1, 0.05, 0.02), "sheet_law": "remark1", "sheet_dz0": 1.0, "sheet_shape": 2.0}
RHO = (-0.5, 0.5)
W_SCALE = 0.02                      # out-of-plane velocity, sheet units per frame


def _case(kind, sizes, ppp, d, **kw):
    c = {"kind": kind, "sizes": sizes, "ppp_lo": ppp[0], "ppp_hi": ppp[1], "d_dist": d[0], "d_a": d[1], "d_b": d[2],
         "flow": "vortex", "grid_div": 4, "disp": 8.0, "integrator": "rk4", "substeps": 4, "blur": 1,
         "blur_sigma": 0.7, "noise": 0.01, "bits": 12}
    c.update(kw)
    return c


def listed():
    normal, tiny, wide = ("normal", 2.5, 0.5), ("uniform", 0.8, 1.2), ("uniform", 2.0, 6.0)
    menu = "256x256*13,512x512*13,768x1024*13,1024x1280*13,2048x2048*12"
    return [
        # one small pair at a time, as an interactive or serving loop asks for it: latency
        _case("eager", "256x256*1", (0.02, 0.02), ("uniform", 1.5, 3.0), name="pair_256", flow="uniform", disp=2.8,
              integrator="euler", substeps=1, blur=0, noise=0.0, bits=0),
        # a handful of cropped, odd-sized pairs with 8-bit codes
        _case("eager", "97x131*1,240x321*2,333x250*2,480x642*1,601x777*1,719x1021*1", (0.005, 0.1),
              ("uniform", 1.0, 5.0), name="ragged_8", bits=8),
        # one pair of a 4-megapixel camera, raw intensities
        _case("eager", "2048x2048*1", (0.05, 0.05), normal, name="camera_2048", bits=0),
        # a training batch at the usual estimator input size, from the sampler front end
        _case("sampler", "512x512*64", (0.06, 0.06), tiny, name="sampler_512", fields=1, keep=1 << 20, model=False,
              integrator="euler", substeps=1, blur=0, noise=0.0, bits=0),
        # the same front end with the full model and codes adjusted to a histogram
        _case("sampler", "512x512*64", (0.06, 0.06), tiny, name="sampler_model_512", fields=1, keep=1 << 20,
              model=True, integrator="euler", substeps=1),
        # the throughput workload: 64 pairs of 1024^2, replayed as one plan
        _case("plan", "1024x1024*64", (0.05, 0.05), normal, name="plan_1024"),
        # uneven sizes and densities in one plan
        _case("plan", menu, (0.005, 0.1), ("uniform", 1.0, 5.0), name="plan_uneven"),
        # dense stress: large images, large particles, long trajectories
        _case("plan", "2048x2048*32", (0.1, 0.1), wide, name="plan_dense_2048", flow="modes", disp=12.0, substeps=8,
              blur=2, blur_sigma=1.0, noise=0.02),
        # full particle model with out-of-plane motion
        _case("model", "1024x1024*16", (0.05, 0.05), normal, name="model_1024"),
        # a fit step over a batch of recorded pairs
        _case("fit", "512x512*64", (0.05, 0.05), normal, name="fit_512", flow="modes", disp=6.0, noise=0.0, bits=0),
        # a fit step on large dense images
        _case("fit", "2048x2048*4", (0.1, 0.1), wide, name="fit_dense_2048", flow="modes", disp=12.0, substeps=8,
              blur=2, blur_sigma=1.0, noise=0.0, bits=0),
        # a small fit through torch's autograd: latency
        _case("autograd", "120x160*2", (0.05, 0.05), normal, name="autograd_120", flow="modes", disp=4.0, substeps=2,
              noise=0.0, bits=0),
    ]


def draw(rng):
    kind = rng.choice(["eager", "eager", "plan", "plan", "plan", "sampler", "model", "fit", "fit", "autograd"])
    budget = {"eager": 1 << 23, "plan": 1 << 26, "sampler": 1 << 24, "model": 1 << 24, "fit": 1 << 24,
              "autograd": 1 << 21}[kind]
    total = math.exp(rng.uniform(math.log(1 << 15), math.log(budget)))       # pixels of one frame of every pair

    def side():
        s = int(math.exp(rng.uniform(math.log(96), math.log(2048))))
        return s if rng.random() < 0.5 else (s + 31) // 32 * 32

    terms, left = [], total
    for _ in range(1 if kind == "sampler" else rng.randint(1, 4)):
        h, w = side(), side()
        n = max(1, min(64, int(left / (h * w) * rng.uniform(0.3, 1.0))))
        if terms and n * h * w > left:
            break
        terms.append("%dx%d*%d" % (h, w, n))
        left -= n * h * w
    if kind == "sampler":
        fields = rng.choice([1, 2])
        terms[0] = terms[0].split("*")[0] + "*%d" % (fields * max(1, int(terms[0].split("*")[1]) // fields))
    # a fit needs particles on its flow nodes: no sparse seeding there
    lo = math.exp(rng.uniform(math.log(0.03 if kind in ("fit", "autograd") else 0.005), math.log(0.06)))
    hi = lo if rng.random() < 0.6 or kind in ("fit", "autograd") else min(0.1, lo * rng.uniform(1.5, 8.0))
    a = rng.uniform(0.8, 2.5)
    d = ("normal", rng.uniform(2.0, 3.0), 0.5) if rng.random() < 0.5 else ("uniform", a, a + rng.uniform(0.3, 3.5))
    blur = rng.choice([0, 1, 1, 2])
    rk = rng.random() < 0.7
    grad = kind in ("fit", "autograd")
    model = kind == "sampler" and rng.random() < 0.5
    c = _case(kind, ",".join(terms), (lo, hi), d, flow=rng.choice(["vortex", "modes"]), grid_div=rng.choice([4, 4, 8]),
              disp=rng.uniform(1.0, 10.0), integrator="rk4" if rk else "euler",
              substeps=rng.choice([1, 2, 3, 4, 8]) if rk else rng.choice([1, 1, 4]), blur=blur,
              blur_sigma=rng.uniform(0.5, 1.2), noise=0.0 if grad else rng.choice([0.0, 0.01, 0.02]),
              bits=0 if grad else 12 if model else rng.choice([0, 8, 10, 12, 16]))
    if kind == "sampler":
        c.update(fields=fields, keep=1 << 20, model=model)
    return c


# ---------------------------------------------------------------- inputs

def _sizes(c):
    out = []
    for term in c["sizes"].split(","):
        hw, n = term.split("*")
        h, w = hw.split("x")
        out += [(int(h), int(w))] * int(n)
    return out


def _grid(c, h, w):
    return max(h // c["grid_div"], 2), max(w // c["grid_div"], 2)


def _counts(c):
    return [int(math.floor(float(h) * w * c["ppp_hi"] + 0.5)) for h, w in _sizes(c)]


def _d_max(c):
    return c["d_b"] if c["d_dist"] == "uniform" else D_CLIP[1]


def _gen(seed, salt):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 16 + salt)


def _flow(c, h, w, gh, gw, g):
    """One pair's (u, v) grid [gh, gw, 2], float32, of peak speed ``disp``."""
    r = torch.rand(32, generator=g, device=DEV, dtype=torch.float64)
    if c["flow"] == "uniform":
        a = 2 * math.pi * r[0]
        return (c["disp"] * torch.stack([torch.cos(a), torch.sin(a)])).float().expand(gh, gw, 2).contiguous()
    X = (torch.arange(gw, device=DEV, dtype=torch.float64) + 0.5) * (w / gw)
    Y = (torch.arange(gh, device=DEV, dtype=torch.float64) + 0.5) * (h / gh)
    if c["flow"] == "vortex":           # eight Lamb-Oseen vortices
        r = r.view(4, 8, 1, 1)
        dx, dy = X[None, None, :] - r[0] * w, Y[None, :, None] - r[1] * h
        r2 = (dx * dx + dy * dy).clamp_min(1e-12)
        gam = torch.where(r[3] < 0.5, -1.0 + r[3], r[3])
        f = -gam / r2 * torch.expm1(-r2 / (20.0 + 60.0 * r[2]) ** 2)
        uv = torch.stack([(-f * dy).sum(0), (f * dx).sum(0)], -1)
    else:                               # divergence-free modes with a k^(-5/3) energy spectrum
        kmax = max(1, min(gh, gw) // 8)
        ky = torch.fft.fftfreq(gh, 1.0 / gh, device=DEV, dtype=torch.float64)[:, None]
        kx = torch.fft.fftfreq(gw, 1.0 / gw, device=DEV, dtype=torch.float64)[None, :]
        kk = torch.sqrt(kx * kx + ky * ky)
        half = (ky > 0) | ((ky == 0) & (kx > 0))
        amp = torch.where(half & (kk <= kmax), kk.clamp_min(1.0) ** (-7.0 / 3.0), torch.zeros_like(kk))
        ph = 2 * math.pi * torch.rand(gh, gw, generator=g, device=DEV, dtype=torch.float64)
        C = torch.polar(amp, ph)
        uv = torch.stack([torch.fft.ifft2(C * (1j * ky / h)).real, torch.fft.ifft2(-C * (1j * kx / w)).real], -1)
    return (uv * (c["disp"] / uv.norm(dim=-1).amax())).float()


def _flows(c, seed, count=None):
    g = _gen(seed, 1)
    sizes = _sizes(c) if count is None else _sizes(c)[:1] * count
    return [_flow(c, h, w, *_grid(c, h, w), g) for h, w in sizes]


def _table(c):
    """Per-particle int64 columns (H, W, Gh, Gw, first flow node, pair, index) of the packed batch."""
    rows, node = [], 0
    for h, w in _sizes(c):
        gh, gw = _grid(c, h, w)
        rows.append((h, w, gh, gw, node))
        node += gh * gw
    if c["kind"] == "sampler":
        per = len(rows) // c["fields"]
        rows = [(h, w, gh, gw, (p // per) * gh * gw) for p, (h, w, gh, gw, _) in enumerate(rows)]
    n = torch.tensor(_counts(c), device=DEV)
    pair = torch.repeat_interleave(torch.arange(len(rows), device=DEV), n)
    first = torch.cumsum(n, 0) - n
    index = torch.arange(pair.numel(), device=DEV) - first[pair]
    cols = torch.tensor(rows, device=DEV, dtype=torch.int64)[pair].unbind(1)
    return (*cols, pair, index)


def _particles(c, seed):
    """Particles a fitting program has in hand (float32)."""
    H, W = _table(c)[:2]
    g = _gen(seed, 2)
    u = torch.rand(5, H.numel(), generator=g, device=DEV)
    d = c["d_a"] + (c["d_b"] - c["d_a"]) * u[3] if c["d_dist"] == "uniform" else \
        (c["d_a"] + c["d_b"] * torch.randn(H.numel(), generator=g, device=DEV)).clamp(*D_CLIP)
    return {"x1": u[0] * W, "y1": u[1] * H, "z": -1.0 + 2.0 * u[2], "d": d, "I0": 0.8 + 0.2 * u[4]}


def _target(c, seed, P, flow):
    """Recorded images: the particles under a flow 30% off, darker than the model's by a fifth."""
    off = flow + 0.3 * flow.square().mean().sqrt() * torch.randn(flow.shape, generator=_gen(seed, 3), device=DEV)
    Q = {k: v.double() for k, v in P.items()}
    x2, y2 = _advect64(c, off.double(), Q["x1"], Q["y1"])
    A = 0.8 * Q["I0"] * torch.exp(-Q["z"] ** 2 / (2 * SHEET ** 2))
    return _images64(c, [(Q["x1"], Q["y1"]), (x2, y2)], A, Q["d"]).float()


def _params(c, seed):
    d = (c["d_a"], c["d_b"]) if c["d_dist"] == "uniform" else (c["d_a"], c["d_b"], *D_CLIP)
    s = sp.seed_params((c["ppp_lo"], c["ppp_hi"]), c["d_dist"], d, I0_RANGE, Z_RANGE)
    a = sp.advect_params(1.0, c["substeps"], c["integrator"])
    r = sp.render_params(SHEET, _d_max(c), c["blur"], c["blur_sigma"], c["noise"], c["bits"], seed, 1.0,
                         c["substeps"], c["integrator"], **(MODEL if c["kind"] == "model" else {}))
    return s, a, r


def prepare(case, seed):
    c = dict(case)
    st = {"c": c, "seed": seed}
    sizes = _sizes(c)
    if c["kind"] == "sampler":
        grids = torch.stack(_flows(c, seed, c["fields"])).cpu().numpy()
        d = {"dist": "uniform", "range": [c["d_a"], c["d_b"]]} if c["d_dist"] == "uniform" else \
            {"dist": "normal", "mean": c["d_a"], "std": c["d_b"], "clip": list(D_CLIP)}
        cfg = {"image_shape": sizes[0], "batch_size": len(sizes), "flows_per_batch": c["fields"],
               "batches_per_flow": c["keep"], "seeding_density": (c["ppp_lo"], c["ppp_hi"]), "diameter": d,
               "integrator": c["integrator"], "substeps": c["substeps"], "noise_sigma": c["noise"],
               "bits": c["bits"], "blur": {"radius": c["blur"], "sigma": c["blur_sigma"]}, "seed": seed,
               "flow": {"fn": lambda epoch, f, h, w: grids}}
        if c["model"]:
            cfg.update(rho=RHO, jitter=(0.05, 0.05, 0.02), hide_p=0.05, histogram=[1] * (1 << c["bits"]),
                       sheet={"law": "remark1", "dz0": 1.0, "shape": 2.0})
        st["sampler"] = smp.make(cfg)
        return st
    grids = [_grid(c, h, w) for h, w in sizes]
    b = st["batch"] = sp.PairBatch.build(sizes, grids, _counts(c), device=DEV)
    st["flow"] = torch.cat([f.reshape(-1) for f in _flows(c, seed)])
    st["sprm"], st["aprm"], st["rprm"] = _params(c, seed)
    n = max(b.n_particles, 1)

    def buffers(*names):
        return {k: torch.empty(n, dtype=torch.float32, device=DEV) for k in names}

    images = torch.empty(b.n_pixels, dtype=sp.api.U16 if c["bits"] else torch.float32, device=DEV)
    if c["kind"] == "plan":
        st["io"] = {**buffers("x1", "y1", "x2", "y2", "z", "d", "I0"), "flow": st["flow"], "images": images,
                    "n_active": torch.empty(b.n_pairs, dtype=torch.int32, device=DEV),
                    "ppp": torch.empty(b.n_pairs, dtype=torch.float64, device=DEV)}
        st["plan"] = sp.Plan(b, st["sprm"], seed, st["aprm"], st["rprm"], st["io"])
    elif c["kind"] in ("eager", "model"):
        st["P"] = {**buffers("x", "y", "z", "d", "I0"),
                   "n_active": torch.empty(b.n_pairs, dtype=torch.int32, device=DEV),
                   "ppp": torch.empty(b.n_pairs, dtype=torch.float64, device=DEV)}
        st["Q"] = buffers("x2", "y2", *(("z2", "dy", "rho") if c["kind"] == "model" else ()))
        st["images"] = images
        st["ws"] = sp.alloc_workspace(b, st["rprm"])
        if c["kind"] == "model":
            st["w"] = W_SCALE * torch.randn(st["flow"].numel() // 2, generator=_gen(seed, 4), device=DEV)
    else:
        st["P"] = _particles(c, seed)
        st["T"] = _target(c, seed, st["P"], st["flow"])
        if c["kind"] == "fit":
            st["x2"], st["y2"] = buffers("x2", "y2").values()
            st["images"] = images
            st["ws"] = sp.alloc_workspace(b, st["rprm"])
            st["bws"] = sp.alloc_workspace(b, st["rprm"], backward="mse")
        else:
            st["sheet"] = torch.tensor(SHEET, device=DEV, requires_grad=True)
            st["leaf"] = {k: v.clone().requires_grad_(True) for k, v in {"flow": st["flow"], **st["P"]}.items()}
    return st


def _codes(t):
    return t.view(torch.int16) if t.dtype == sp.api.U16 else t


def run(st):
    c, seed = st["c"], st["seed"]
    if c["kind"] == "sampler":
        b = next(st["sampler"])
        return {"images1": _codes(b.images1), "images2": _codes(b.images2), "flow_fields": b.flow_fields,
                "ppp": b.params["seeding_densities"], "n_active": b.params["n_active"]}
    batch, flow, rp = st["batch"], st["flow"], st["rprm"]
    if c["kind"] == "plan":
        st["plan"].launch()
        return {k: _codes(v) for k, v in st["io"].items() if k != "flow"}
    P = st.get("P")
    if c["kind"] == "eager":
        Q = st["Q"]
        sp.seed(batch, st["sprm"], seed, out=P)
        sp.advect(batch, flow, st["aprm"], P["x"], P["y"], Q["x2"], Q["y2"], st["ws"])
        sp.render_pair(batch, P["x"], P["y"], Q["x2"], Q["y2"], P["z"], P["d"], P["I0"], rp, None, st["images"],
                       st["ws"])
        return {**P, **Q, "images": _codes(st["images"])}
    if c["kind"] == "model":
        Q = st["Q"]
        sp.seed(batch, st["sprm"], seed, out=P)
        sp.seed_shape(batch, st["sprm"], RHO, seed, out=(Q["dy"], Q["rho"]))
        sp.advect(batch, flow, st["aprm"], P["x"], P["y"], Q["x2"], Q["y2"], wflow=st["w"], z1=P["z"], z2=Q["z2"])
        sp.render_pair(batch, P["x"], P["y"], Q["x2"], Q["y2"], P["z"], P["d"], P["I0"], rp, None, st["images"],
                       st["ws"], dy=Q["dy"], rho=Q["rho"], z2=Q["z2"])
        return {**P, **Q, "images": _codes(st["images"])}
    if c["kind"] == "fit":
        x2, y2 = sp.advect(batch, flow, st["aprm"], P["x1"], P["y1"], st["x2"], st["y2"], st["ws"])
        J = sp.render_pair(batch, P["x1"], P["y1"], x2, y2, P["z"], P["d"], P["I0"], rp, None, st["images"],
                           st["ws"])
        g = sp.render_pair_backward_mse(batch, flow, P["x1"], P["y1"], P["z"], P["d"], P["I0"], rp, J, st["T"],
                                        loss=True, workspace=st["bws"], x2=x2, y2=y2)
        return {**g, "images": J}
    leaf = st["leaf"]
    J = sp.render_images(batch, leaf["flow"], leaf["x1"], leaf["y1"], leaf["z"], leaf["d"], leaf["I0"], st["sheet"],
                         rp)
    loss = (J - st["T"]).square().mean()
    g = torch.autograd.grad(loss, [*leaf.values(), st["sheet"]])
    return {**dict(zip([*leaf, "sheet_total"], g)), "loss": loss.detach(), "images": J.detach()}


# ---------------------------------------------------------------- necessary work

def work(case):
    c = case
    px = sum(2 * h * w for h, w in _sizes(c))
    mid = 0.5 * (c["ppp_lo"] + c["ppp_hi"]) / c["ppp_hi"]
    n = sum(_counts(c))
    live = mid * n
    d2 = c["d_a"] ** 2 + c["d_b"] ** 2 if c["d_dist"] == "normal" else \
        (c["d_a"] ** 2 + c["d_a"] * c["d_b"] + c["d_b"] ** 2) / 3.0
    foot = 2 * live * 9.0 * d2                              # footprint pixels of both frames
    fields = c.get("fields", len(_sizes(c)))
    nodes = sum(gh * gw for gh, gw in [_grid(c, h, w) for h, w in _sizes(c)][:fields])
    elem = 2 if c["bits"] else 4
    samples = live * c["substeps"] * (4 if c["integrator"] == "rk4" else 1)
    flops = samples * 26 + 2 * live * 2 * 3 * math.sqrt(d2) * 12 + foot * 2 + px * 4 * (2 * c["blur"] + 1) * (
        c["blur"] > 0) + px * 20 * (c["noise"] > 0)
    if c["kind"] == "sampler":
        return {"bytes": nodes * 8 + px * elem + px * 4, "flops": flops}
    if c["kind"] in ("eager", "plan"):
        return {"bytes": nodes * 8 + n * 28 + px * elem, "flops": flops}
    if c["kind"] == "model":
        return {"bytes": nodes * 12 + n * 40 + px * elem, "flops": flops + foot * 12}
    # fit, autograd: particles, flow and target read, images and every gradient written
    return {"bytes": nodes * 16 + n * 40 + px * 8, "flops": 2 * flops + samples * 60 + foot * 8}


# ---------------------------------------------------------------- the path in float64

M32 = 0xFFFFFFFF


def _philox(index, stream, pid, seed):
    """Philox4x32-10 words of counter (index, stream, pid, 0) and key seed (int64 tensors)."""
    a, b = index & M32, torch.full_like(index, stream)
    c, d = (pid & M32).expand_as(index), (pid >> 32).expand_as(index)
    k0, k1 = seed & M32, seed >> 32
    for _ in range(10):
        p0, p1 = a * 0xD2511F53, c * 0xCD9E8D57
        a, b, c, d = ((p1 >> 32) & M32) ^ b ^ k0, p1 & M32, ((p0 >> 32) & M32) ^ d ^ k1, p0 & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return a, b, c, d


def _u(w):
    return (w >> 8).double() * 2.0 ** -24


def _normal(w1, w2, trig=torch.cos):
    return torch.sqrt(-2.0 * torch.log(((w1 >> 8) + 1).double() * 2.0 ** -24)) * trig(2.0 * math.pi * _u(w2))


def _seed64(c, seed):
    H, W, _, _, _, pair, index = _table(c)
    pid = torch.arange(len(_sizes(c)), device=DEV)
    w = _philox(torch.zeros_like(pid), 5, pid, seed)
    ppp = c["ppp_lo"] + (c["ppp_hi"] - c["ppp_lo"]) * _u(w[0])
    hw = torch.tensor([float(h * w) for h, w in _sizes(c)], device=DEV, dtype=torch.float64)
    active = torch.minimum(torch.floor(hw * ppp + 0.5), torch.tensor(_counts(c), device=DEV).double())
    gw, hw = _philox(index, 0, pair, seed), _philox(index, 1, pair, seed)
    d = c["d_a"] + (c["d_b"] - c["d_a"]) * _u(gw[3]) if c["d_dist"] == "uniform" else \
        (c["d_a"] + c["d_b"] * _normal(hw[1], hw[2])).clamp(*D_CLIP)
    I0 = torch.where(index < active[pair], 0.8 + 0.2 * _u(hw[0]), torch.zeros_like(d))
    return {"x": _u(gw[0]) * W, "y": _u(gw[1]) * H, "z": -1.0 + 2.0 * _u(gw[2]), "d": d, "I0": I0, "ppp": ppp}


def _sample64(grid, px, py, H, W, gh, gw, node):
    """Bilinear, clamped, cell-centred sample; grid: float64 [nodes, k]."""
    gx = (px * (gw.double() / W) - 0.5).clamp_min(0.0).minimum(gw.double() - 1)
    gy = (py * (gh.double() / H) - 0.5).clamp_min(0.0).minimum(gh.double() - 1)
    j = gx.detach().floor().long().minimum(gw - 2)
    i = gy.detach().floor().long().minimum(gh - 2)
    fx, fy = (gx - j)[:, None], (gy - i)[:, None]
    k = node + i * gw + j
    top = grid[k] + fx * (grid[k + 1] - grid[k])
    bot = grid[k + gw] + fx * (grid[k + gw + 1] - grid[k + gw])
    return top + fy * (bot - top)


def _advect64(c, flow, x, y, w=None, z=None):
    H, W, gh, gw, node, _, _ = _table(c)
    grid = flow.view(-1, 2) if w is None else torch.cat([flow.view(-1, 2), w[:, None]], 1)
    h = 1.0 / c["substeps"]

    def f(px, py):
        return _sample64(grid, px, py, H, W, gh, gw, node)

    for _ in range(c["substeps"]):
        k = f(x, y)
        if c["integrator"] == "rk4":
            k2 = f(x + 0.5 * h * k[:, 0], y + 0.5 * h * k[:, 1])
            k3 = f(x + 0.5 * h * k2[:, 0], y + 0.5 * h * k2[:, 1])
            k4 = f(x + h * k3[:, 0], y + h * k3[:, 1])
            k = (k + 2.0 * k2 + 2.0 * k3 + k4) / 6.0
        x, y = x + h * k[:, 0], y + h * k[:, 1]
        if w is not None:
            z = z + h * k[:, 2]
    return (x, y) if w is None else (x, y, z)


def _taps(c):
    b = c["blur"]
    g = [math.exp(-k * k / (2.0 * float(np.float32(c["blur_sigma"])) ** 2)) for k in range(-b, b + 1)]
    return [v / sum(g) for v in g]


def _blur64(c, packed):
    """Zero-padded separable blur of every image of a packed buffer."""
    b, out, o = c["blur"], [], 0
    if b == 0:
        return packed
    for h, w in _sizes(c):
        im = torch.nn.functional.pad(packed[o:o + 2 * h * w].view(2, h, w), (b, b, b, b))
        t = _taps(c)
        im = sum(t[k] * im[:, :, k:k + w] for k in range(2 * b + 1))
        out.append(sum(t[k] * im[:, k:k + h] for k in range(2 * b + 1)).reshape(-1))
        o += 2 * h * w
    return torch.cat(out)


def _windows(c, f, x, y, d, sl):
    """Footprints of particles ``sl`` in frame f: separable factors [n, K] and pixel numbers [n, K, K]."""
    H, W, _, _, _, pair, _ = (t[sl] for t in _table(c))
    px = torch.tensor([h * w for h, w in _sizes(c)], device=DEV)
    base = 2 * (torch.cumsum(px, 0) - px)[pair] + f * px[pair]
    K = int(3 * _d_max(c)) + 2
    k = torch.arange(K, device=DEV)

    def axis(p, n):
        q = torch.ceil((p - 1.5 * d).detach() - 0.5).long()[:, None] + k
        t = q + 0.5 - p[:, None]
        on = (t.detach().abs() <= 1.5 * d.detach()[:, None]) & (q >= 0) & (q < n[:, None])
        return torch.where(on, torch.exp(-8.0 * t * t / (d * d)[:, None]), torch.zeros_like(t)), \
            q.clamp_min(0).minimum(n[:, None] - 1)

    gx, cx = axis(x, W)
    gy, cy = axis(y, H)
    return gx, gy, base[:, None, None] + cy[:, :, None] * W[:, None, None] + cx[:, None, :]


def _chunks(n):
    return [slice(i, min(n, i + (1 << 18))) for i in range(0, n, 1 << 18)]


def _images64(c, frames, A, d):
    """Float images of every pair, summed in 2^-40 steps (the order of the sums does not matter)."""
    out = torch.zeros(sum(2 * h * w for h, w in _sizes(c)), device=DEV, dtype=torch.int64)
    for f, (x, y) in enumerate(frames):
        for sl in _chunks(x.numel()):
            gx, gy, at = _windows(c, f, x[sl], y[sl], d[sl], sl)
            v = (A[sl, None, None] * gy[:, :, None] * gx[:, None, :] * 2.0 ** 40).round().long()
            out.index_add_(0, at.view(-1), v.view(-1))
    return _blur64(c, out.double() * 2.0 ** -40)


def _noise64(c, packed, seed):
    if not c["noise"]:
        return packed
    out, o = [], 0
    for p, (h, w) in enumerate(_sizes(c)):
        wq = (w + 3) // 4
        at = torch.arange(h * wq, device=DEV)
        for f in range(2):
            q = _philox(at, 3 + f, torch.tensor(p, device=DEV), seed)
            v = torch.stack([_normal(q[2 * k], q[2 * k + 1], t) for k in (0, 1) for t in (torch.cos, torch.sin)], 1)
            out.append(packed[o:o + h * w] + c["noise"] * v.view(h, 4 * wq)[:, :w].reshape(-1))
            o += h * w
    return torch.cat(out)


def _fields64(c, flow):
    h, w = _sizes(c)[0]
    gh, gw = _grid(c, h, w)
    y, x = torch.meshgrid(torch.arange(h, device=DEV), torch.arange(w, device=DEV), indexing="ij")
    one = torch.ones(h * w, device=DEV, dtype=torch.int64)
    per = [_sample64(f.double().view(-1, 2), x.reshape(-1) + 0.5, y.reshape(-1) + 0.5, one * h, one * w, one * gh,
                     one * gw, 0 * one).view(h, w, 2) for f in flow]
    n = len(_sizes(c)) // len(flow)
    return torch.stack([f for f in per for _ in range(n)])


def _gradients64(c, flow, P, T):
    """Images, loss and gradients of the mean squared difference to T."""
    flow = flow.double().requires_grad_(True)
    Q = {k: v.double() for k, v in P.items()}
    x1, y1 = Q["x1"].requires_grad_(True), Q["y1"].requires_grad_(True)
    x2, y2 = _advect64(c, flow, x1, y1)
    s = torch.full((len(_sizes(c)),), SHEET, device=DEV, dtype=torch.float64)
    pair = _table(c)[5]
    with torch.no_grad():
        A = Q["I0"] * torch.exp(-Q["z"] ** 2 / (2 * SHEET ** 2))
        J = _images64(c, [(x1, y1), (x2, y2)], A, Q["d"])
        e = J - T.double()
        E = _blur64(c, 2.0 / e.numel() * e)
    g = {k: torch.zeros_like(Q["z"]) for k in ("x1", "y1", "x2", "y2", "z", "d", "I0")}
    g["sheet"] = torch.zeros_like(s)
    for f, (x, y) in enumerate([(x1, y1), (x2, y2)]):
        for sl in _chunks(x.numel()):
            leaf = [t.detach()[sl].requires_grad_(True) for t in (x, y, Q["z"], Q["d"], Q["I0"], s[pair])]
            gx, gy, at = _windows(c, f, leaf[0], leaf[1], leaf[3], sl)
            A = leaf[4] * torch.exp(-leaf[2] ** 2 / (2 * leaf[5] ** 2))
            got = torch.autograd.grad((A * ((E[at] * gx[:, None, :]).sum(2) * gy).sum(1)).sum(), leaf)
            for k, v in zip(("x2" if f else "x1", "y2" if f else "y1", "z", "d", "I0"), got):
                g[k][sl] += v
            g["sheet"].index_add_(0, pair[sl], got[5])
    gf, gx, gy = torch.autograd.grad([x2, y2], [flow, x1, y1], [g.pop("x2"), g.pop("y2")])
    g["x1"], g["y1"], g["flow"] = g["x1"] + gx, g["y1"] + gy, gf
    g["sheet_total"] = g["sheet"].sum()
    return {**g, "loss": e.square().mean(), "images": J.detach()}


def exact(case, seed):
    c = dict(case)
    if c["kind"] == "sampler":
        flow = _flows(c, seed, c["fields"])
        P = _seed64(c, seed)
        out = {"images1": None, "images2": None, "flow_fields": _fields64(c, flow), "ppp": P["ppp"], "n_active": None}
        if not c["bits"]:
            x2, y2 = _advect64(c, torch.cat([f.reshape(-1) for f in flow]).double(), P["x"], P["y"])
            A = P["I0"] * torch.exp(-P["z"] ** 2 / (2 * SHEET ** 2))
            J = _noise64(c, _images64(c, [(P["x"], P["y"]), (x2, y2)], A, P["d"]), seed)
            J = J.view(len(_sizes(c)), 2, *_sizes(c)[0])
            out["images1"], out["images2"] = J[:, 0], J[:, 1]
        return out
    flow = torch.cat([f.reshape(-1) for f in _flows(c, seed)])
    if c["kind"] in ("fit", "autograd"):
        P = _particles(c, seed)
        g = _gradients64(c, flow, P, _target(c, seed, P, flow))
        if c["kind"] == "autograd":
            del g["sheet"]
        return g
    P = _seed64(c, seed)
    flow = flow.double()
    if c["kind"] == "model":
        w = (W_SCALE * torch.randn(flow.numel() // 2, generator=_gen(seed, 4), device=DEV)).double()
        x2, y2, z2 = _advect64(c, flow, P["x"], P["y"], w, P["z"])
        pair, index = _table(c)[5:]
        q = _philox(index, 6, pair, seed)
        dy = c["d_a"] + (c["d_b"] - c["d_a"]) * _u(q[0]) if c["d_dist"] == "uniform" else \
            (c["d_a"] + c["d_b"] * _normal(q[1], q[2])).clamp(*D_CLIP)
        return {**P, "n_active": None, "x2": x2, "y2": y2, "z2": z2, "dy": dy,
                "rho": RHO[0] + (RHO[1] - RHO[0]) * _u(q[3]), "images": None}
    # a plan leaves masked candidates where they are
    x2, y2 = _advect64(c, flow, P["x"], P["y"])
    J = None
    if not c["bits"]:
        A = P["I0"] * torch.exp(-P["z"] ** 2 / (2 * SHEET ** 2))
        J = _noise64(c, _images64(c, [(P["x"], P["y"]), (x2, y2)], A, P["d"]), seed)
    if c["kind"] == "plan":
        still = P["I0"] == 0
        x2, y2 = torch.where(still, P["x"], x2), torch.where(still, P["y"], y2)
        P["x1"], P["y1"] = P.pop("x"), P.pop("y")
    return {**P, "x2": x2, "y2": y2, "images": J, "n_active": None}
