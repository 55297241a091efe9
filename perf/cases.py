"""The calls this library is used for, as cases to time and to compare.

A case is a dict of plain values.  kind says which entry point it takes:

  map      one magnification map into a device tensor (irs_shoot_map), by the
           direct sum in FP64 or FP32, the three-level interpolation or the
           learned interpolant; the plan is made beforehand
  deflect  deflections and pixels of a range of rays (irs_deflect_grid)
  batch    several interpolated maps in one graph launch (irs_batch_run)
  field    a new lens field from host arrays to a host map: plan, map, release
  grad     loss and gradient of the learned interpolant's network on a batch of
           sample records (irs_mlp_loss_grad)

Lenses are uniform in the plan's rectangle, their number by the lens-count rule
round(kappa_* I_x I_y / pi), masses equal or Salpeter on [0.1, 1] M_sun.
"""
import math

import numpy as np
import torch

import paper_2204_10871_amd as irs
import synth

MIN_LAMBDA = 0.05        # maps closer to a critical line have no bounded rectangle
MAX_RAYS = 4.0e9         # of a drawn map
N_PARAM, N_FREQ = irs.IRS_LEARN_NPARAMS, 64
HID, N_OUT = 128, 16


def _map(name, method, precision, kappa_star, kappa_c, gamma, side, npix, rpp=0.0, n_rays=0,
         mass="unit", mult=0.0, kind="map", **more):
    return dict(name=name, kind=kind, method=method, precision=precision, kappa_star=kappa_star,
                kappa_c=kappa_c, gamma=gamma, source_side=side, npix=npix, rays_per_pixel=rpp,
                n_rays=n_rays, mass=mass, level2_ray_multiple=mult, **more)


def listed():
    return [
        # the brute-force FP64 map every other path is checked against: 2048^2
        # rays, 105 lenses
        _map("direct64_map", "direct", "fp64", 0.3, 0.0, 0.3, 10.0, 256, n_rays=2048 * 2048),
        # a direct FP32 map at one ray per pixel, 4450 lenses: a quick look at a field
        _map("direct32_map", "direct", "fp32", 0.45, 0.05, 0.45, 25.0, 1024, rpp=1.0),
        # the direct FP32 sum at 1e5 lenses (the rate a full-size direct map sees)
        _map("direct32_n1e5", "direct", "fp32", 0.45, 0.05, 0.45, 168.69, 1024, n_rays=2_000_003),
        # the smallest interpolated map: a parameter scan's first look, all latency
        _map("interp_tiny", "interp", "fp64", 0.45, 0.05, 0.45, 4.0, 64, n_rays=120_001),
        # an ordinary map: 1024^2 pixels, 100 rays per pixel, 5133 lenses
        _map("interp_1k", "interp", "fp64", 0.36, 0.0, 0.36, 100.0, 1024, rpp=100.0),
        # 4096^2 pixels, 1e5 lenses, coarse grid at 16 ray spacings
        _map("interp_n1e5", "interp", "fp64", 0.45, 0.05, 0.45, 168.69, 4096, rpp=100.0,
             mult=16.0),
        # the benchmark's map: 1e6 Salpeter lenses, 10000^2 pixels, 1e11 rays
        _map("interp_n1e6", "interp", "fp64", 0.6, 0.0, 0.6, 1007.8, 10000, rpp=1000.0,
             mass="salpeter"),
        # deflections along part of a trajectory's rows: a ragged ray range
        _map("deflect_interp", "interp", "fp64", 0.45, 0.05, 0.45, 25.0, 1000, rpp=100.0,
             kind="deflect", first=12_345_679, count=300_007),
        # sampling lens-model parameters: maps of different fields at once
        dict(name="batch_12", kind="batch", maps=12, npix_lo=256, npix_hi=1024, side_lo=8.0,
             side_hi=80.0, rays_per_pixel=100.0, draw_seed=4),
        # a new field each time, host arrays in, host map out
        _map("field_2k", "interp", "fp64", 0.3, 0.0, 0.25, 90.0, 768, rpp=64.0, kind="field"),
        # the learned interpolant with an installed network
        _map("learned_map", "learned", "fp64", 0.5, 0.05, 0.5, 40.0, 1024, rpp=100.0, coarse=16),
        # one training batch of its network, forward and backward
        dict(name="mlp_grad_8k", kind="grad", count=8192),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _physics(rng):
    """kappa_*, kappa_c, gamma as the batched workload draws them."""
    while True:
        ks, g = round(rng.uniform(0.1, 0.8), 4), round(rng.uniform(0.1, 0.8), 4)
        kc = rng.choice((0.0, 0.2))
        if min(abs(1 - ks - kc - g), abs(1 - ks - kc + g)) >= MIN_LAMBDA:
            return ks, kc, g


def _counts(c):
    """(lenses, rays) of a map by the geometry rules."""
    k = c["kappa_star"] + c["kappa_c"]
    w = c["source_side"] + 20.0 * math.sqrt(c["kappa_star"])
    area = w / abs(1 - k - c["gamma"]) * w / abs(1 - k + c["gamma"])
    rays = c["n_rays"] or c["rays_per_pixel"] * c["npix"] ** 2    # of the whole rectangle
    return round(c["kappa_star"] * area / math.pi), rays


def draw(rng):
    kind = rng.choice(("direct64", "direct32", "interp", "interp", "interp", "deflect", "batch",
                       "field", "learned", "grad"))
    if kind == "grad":
        return dict(kind="grad", count=int(_log(rng, 200, 70_000)))
    if kind == "batch":
        return dict(kind="batch", maps=rng.randint(2, 16), npix_lo=rng.randint(64, 256),
                    npix_hi=rng.randint(257, 1100), side_lo=6.0, side_hi=_log(rng, 12.0, 90.0),
                    rays_per_pixel=round(_log(rng, 20.0, 200.0), 1),
                    draw_seed=rng.randrange(1, 1 << 20))
    while True:
        ks, kc, g = _physics(rng)
        mass = rng.choice(("unit", "salpeter"))
        if kind == "direct64":
            c = _map("", "direct", "fp64", ks, kc, g, round(_log(rng, 4, 40), 3),
                     int(_log(rng, 64, 600)), n_rays=int(_log(rng, 2e4, 4.2e6)), mass=mass)
            most_l, most = 20_000, 1e10
        elif kind == "direct32":
            c = _map("", "direct", "fp32", ks, kc, g, round(_log(rng, 5, 180), 3),
                     int(_log(rng, 128, 2048)), n_rays=int(_log(rng, 1e5, 4e6)), mass=mass)
            most_l, most = 200_000, 2.5e11
        elif kind == "deflect":
            method, precision = rng.choice((("interp", "fp64"), ("interp", "fp64"),
                                            ("direct", "fp32"), ("direct", "fp64")))
            c = _map("", method, precision, ks, kc, g, round(_log(rng, 4, 60), 3),
                     int(_log(rng, 100, 1200)), rpp=round(_log(rng, 4, 100), 1), kind="deflect",
                     mass=mass)
            rays = 0.98 * c["rays_per_pixel"] * c["npix"] ** 2
            c["count"] = int(_log(rng, 1, min(1e6, rays / 2)))
            c["first"] = rng.randrange(0, int(rays / 2) - c["count"] + 1 or 1)
            most_l, most = 20_000, math.inf
        elif kind == "learned":
            c = _map("", "learned", "fp64", ks, kc, g, round(_log(rng, 6, 120), 3),
                     int(_log(rng, 128, 2048)), rpp=round(_log(rng, 10, 100), 1), mass=mass,
                     coarse=rng.choice((8, 12, 16)))
            most_l, most = 100_000, math.inf
        elif kind == "field":
            c = _map("", "interp", "fp64", ks, kc, g, round(_log(rng, 4, 150), 3),
                     int(_log(rng, 64, 1500)), rpp=round(_log(rng, 10, 150), 1), kind="field",
                     mass=mass)
            most_l, most = 100_000, math.inf
        else:
            c = _map("", "interp", "fp64", ks, kc, g, round(_log(rng, 2.5, 500), 3),
                     int(_log(rng, 48, 5000)), rpp=round(_log(rng, 10, 1000), 1), mass=mass,
                     mult=rng.choice((0.0, 0.0, 16.0)))
            most_l, most = 600_000, math.inf
        lenses, rays = _counts(c)
        if 0 < lenses <= most_l and rays <= MAX_RAYS and lenses * rays <= most:
            del c["name"]
            return c


# ---- inputs ----------------------------------------------------------------------

def _params(c):
    return irs.make_params(c["kappa_star"], c["kappa_c"], c["gamma"], c["source_side"], c["npix"],
                           rays_per_pixel=c["rays_per_pixel"], n_rays=c["n_rays"],
                           method=c["method"], precision=c["precision"],
                           level2_ray_multiple=c["level2_ray_multiple"])


def _lenses(c, p, seed):
    g = irs.geometry(p, 0)
    return synth.uniform_lenses(g["n_stars_expected"], (g["a1"], g["a2"], g["b1"], g["b2"]),
                                1_000_003 * seed + 17, mass=c["mass"])


def _plan(c, seed):
    p = _params(c)
    L = _lenses(c, p, seed)
    return irs.Plan(p, L.x, L.y, L.m, stream=torch.cuda.current_stream().cuda_stream), L


def _new_counts(npix):
    return torch.zeros(npix * npix, dtype=torch.int32, device="cuda:0")


def _network(rx, ry):
    """A network for squares of sides (rx, ry) in units of their mean: its
    hidden layers are a random He initialisation, its head is fitted to the
    weights of the degree-7 polynomial through A and A' at the corners."""
    freqs = synth.network.fourier_frequencies()
    # the polynomial: rows A(z_c), A'(z_c), columns z^n about the centre
    zc = np.array([0, rx, 1j * ry, rx + 1j * ry]) - 0.5 * (rx + 1j * ry)
    n = np.arange(8)
    V = np.concatenate([zc[:, None] ** n, n * zc[:, None] ** np.maximum(n - 1, 0)])
    a, b = np.meshgrid(np.linspace(0, 1, 33), np.linspace(0, 1, 33))
    h = np.stack([a.ravel(), b.ravel()], 1)
    z = (h[:, 0] * rx + 1j * h[:, 1] * ry) - 0.5 * (rx + 1j * ry)
    card = (z[:, None] ** n) @ np.linalg.inv(V)                  # of A_c, then of A'_c
    w = np.stack([(1 - h[:, 0]) * (1 - h[:, 1]), h[:, 0] * (1 - h[:, 1]),
                  (1 - h[:, 0]) * h[:, 1], h[:, 0] * h[:, 1]], 1)
    Lk = np.concatenate([card[:, 4:] - w * (z[:, None] - zc), card[:, :4] - w], 1)
    target = np.stack([Lk.real, Lk.imag], 2).reshape(len(h), N_OUT)
    rng = np.random.default_rng(11)
    ph = 2 * np.pi * (h - 0.5) @ freqs.T.astype(np.float64)
    act, theta = np.concatenate([np.sin(ph), np.cos(ph)], 1), []
    for _ in range(4):
        W = rng.normal(size=(HID, HID)) * math.sqrt(2.0 / HID)
        bias = rng.normal(size=HID) * 0.1
        act = np.maximum(act @ W.T + bias, 0.0)
        theta += [W.ravel(), bias]
    F = np.concatenate([act, np.ones((len(h), 1))], 1)
    X = np.linalg.solve(F.T @ F + 1e-4 * np.eye(HID + 1), F.T @ target)
    theta += [X[:HID].T.ravel(), X[HID]]
    return freqs, np.concatenate(theta).astype(np.float32)


def _records(count, seed):
    """Sample records as irs_learn_samples writes them: offsets, unit-size
    local data, targets."""
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    f = torch.zeros(irs.IRS_LEARN_FIELDS, count, device="cuda:0")
    f[0:2] = torch.rand(2, count, device="cuda:0", generator=g)
    f[2:18] = 0.5 * torch.randn(16, count, device="cuda:0", generator=g)
    f[18:20] = 0.3 * torch.randn(2, count, device="cuda:0", generator=g)
    f[20] = 1.0
    return f


def prepare(case, seed):
    kind = case["kind"]
    if kind == "grad":
        freqs = synth.network.fourier_frequencies()
        theta = synth.network.random_parameters(seed, 0.1)
        return dict(kind=kind, freqs=freqs, theta=theta, count=case["count"],
                    records=_records(case["count"], seed))
    if kind == "field":
        p = _params(case)
        L = _lenses(case, p, seed)
        return dict(kind=kind, params=p, lenses=L)
    if kind == "batch":
        import random
        rng = random.Random(case["draw_seed"])
        plans, counts = [], []
        for k in range(case["maps"]):
            c = None
            while c is None or _counts(c)[0] > 30_000:
                ks, kc, g = _physics(rng)
                c = _map("", "interp", "fp64", ks, kc, g,
                         round(_log(rng, case["side_lo"], case["side_hi"]), 3),
                         int(_log(rng, case["npix_lo"], case["npix_hi"])),
                         rpp=case["rays_per_pixel"])
            plans.append(_plan(c, 64 * seed + k)[0])
            counts.append(_new_counts(c["npix"]))
        return dict(kind=kind, batch=irs.Batch(plans), counts=counts)
    plan, L = _plan(case, seed)
    st = dict(kind=kind, plan=plan)
    if kind == "deflect":
        st["first"], n = case["first"], case["count"]
        st["out"] = [torch.empty(n, dtype=torch.float64, device="cuda:0") for _ in range(2)]
        st["out"].append(torch.empty(n, dtype=torch.int64, device="cuda:0"))
        return st
    if case["method"] == "learned":
        g = plan.geometry
        sx, sy = g["ix"] / g["n1x"], g["iy"] / g["n1y"]
        freqs, theta = _network(2 * sx / (sx + sy), 2 * sy / (sx + sy))
        # an installed network is kept whatever the tolerance would say of it
        plan.learn_set(freqs, theta, irs.learn_params(coarse=case["coarse"], n_val=2000,
                                                      train_rows=2, tol_mean=1e3, tol_p9999=1e3))
    st["counts"] = _new_counts(case["npix"])
    return st


def run(state):
    kind = state["kind"]
    if kind == "map":
        st = state["plan"].shoot_map_device(state["counts"])
        return {"counts": state["counts"], "landed": st["rays_landed"]}
    if kind == "deflect":
        a1, a2, px = state["out"]
        state["plan"].deflect_grid_device(state["first"], a1.numel(), a1, a2, px)
        return {"alpha1": a1, "alpha2": a2, "pixel": px}
    if kind == "batch":
        st = state["batch"].run(state["counts"])
        return {"counts": state["counts"], "landed": [s["rays_landed"] for s in st]}
    if kind == "field":
        L = state["lenses"]
        with irs.Plan(state["params"], L.x, L.y, L.m) as plan:
            counts, st = plan.shoot_map()
        return {"counts": counts.view(np.int32), "landed": st["rays_landed"]}
    loss, grad = irs.mlp_loss_grad(state["freqs"], state["theta"], state["records"],
                                   state["count"])
    return {"loss": float(loss), "grad": grad}


def work(case):
    """Operations and bytes a pass cannot do without: a direct sum 11 flops a
    ray and lens; the other paths 46 a ray and 10 for each of the about nine
    lenses in the 3 x 3 cells around it (a cell holds one lens on average);
    bytes: the lenses once (24 each) and the counts or per-ray results once."""
    kind = case["kind"]
    if kind == "grad":
        n = case["count"]
        fwd = 2 * (4 * HID * HID + HID * N_OUT)
        return {"flops": n * (2 * fwd + 2 * (3 * HID * HID + HID * N_OUT)),
                "bytes": 80.0 * n + 8.0 * N_PARAM}
    if kind == "batch":
        npix = math.sqrt(case["npix_lo"] * case["npix_hi"])
        rays = case["maps"] * case["rays_per_pixel"] * npix ** 2
        return {"flops": 136.0 * rays, "bytes": 4.0 * case["maps"] * npix ** 2}
    lenses, rays = _counts(case)
    out = 4.0 * case["npix"] ** 2
    if kind == "deflect":
        rays = case["count"]
        out = 24.0 * rays
    per = 11.0 * lenses if case["method"] == "direct" else 136.0
    return {"flops": per * rays, "bytes": 24.0 * lenses + out}


# ---- 64-bit values ---------------------------------------------------------------

def _exact_deflect(case, seed):
    """The direct sum (Eq. 6) of the case's rays in 64 bits: every lens, the
    macro term, the negative sheet over the rectangle."""
    p = _params(case)
    L = _lenses(case, p, seed)
    g = irs.geometry(p, L.n)
    dev = "cuda:0" if torch.cuda.is_available() else "cpu"
    lx, ly = (torch.tensor(v, device=dev) for v in (L.x, L.y))
    lm = torch.tensor(L.masses(), device=dev)
    a1, a2 = (torch.empty(case["count"], dtype=torch.float64, device=dev) for _ in range(2))
    kpg, kmg = g["kappa"] + case["gamma"], g["kappa"] - case["gamma"]
    step = max(1, 40_000_000 // max(1, L.n))
    for r0 in range(0, case["count"], step):
        r = torch.arange(r0, min(case["count"], r0 + step), device=dev) + case["first"]
        i, j = r % g["nx"], torch.div(r, g["nx"], rounding_mode="floor")
        x = g["a1"] + (i.double() + 0.5) * g["ray_dx"]
        y = g["b1"] + (j.double() + 0.5) * g["ray_dy"]
        dx, dy = x[:, None] - lx, y[:, None] - ly
        r2 = dx * dx + dy * dy
        w = torch.where(r2 > 0, lm / r2, torch.zeros_like(r2))
        s1, s2 = (w * dx).sum(1), (w * dy).sum(1)
        i1, i2 = torch.zeros_like(x), torch.zeros_like(x)
        for a, b, sg in ((g["a1"], g["b1"], 1), (g["a2"], g["b1"], -1), (g["a2"], g["b2"], 1),
                         (g["a1"], g["b2"], -1)):
            u, v = x - a, y - b
            lr = torch.log(u * u + v * v)
            i1 += sg * (0.5 * v * lr + u * torch.atan(v / u))
            i2 += sg * (0.5 * u * lr + v * torch.atan(u / v))
        f = -case["kappa_star"] / math.pi
        a1[r - case["first"]] = kpg * x + s1 + f * i1
        a2[r - case["first"]] = kmg * y + s2 + f * i2
    return {"alpha1": a1, "alpha2": a2, "pixel": None}


def _exact_grad(case, seed):
    st = prepare(case, seed)
    rec = st["records"].double()
    th = torch.tensor(st["theta"], dtype=torch.float64, device=rec.device, requires_grad=True)
    fr = torch.tensor(st["freqs"], dtype=torch.float64, device=rec.device)
    ph = 2 * math.pi * (rec[0:2].T - 0.5) @ fr.T
    a, o = torch.cat([torch.sin(ph), torch.cos(ph)], 1), 0
    for l in range(5):
        m = HID if l < 4 else N_OUT
        W, b = th[o:o + m * HID].reshape(m, HID), th[o + m * HID:o + m * HID + m]
        o += m * HID + m
        a = a @ W.T + b
        if l < 4:
            a = torch.relu(a)
    y, D = torch.view_as_complex(a.reshape(-1, 8, 2)), torch.complex(rec[2:18:2].T, rec[3:18:2].T)
    d = (y * D).sum(1) - torch.complex(rec[18], rec[19])
    loss = (d.real ** 2 + d.imag ** 2).mean()
    loss.backward()
    return {"loss": float(loss.detach()), "grad": th.grad}


def exact(case, seed):
    if case["kind"] == "deflect":
        return _exact_deflect(case, seed)
    if case["kind"] == "grad":
        return _exact_grad(case, seed)
    return None                                  # whole numbers only
