"""Timed cases of the reconstruction library: its operators, the TV prox and
whole solves, called through the package's public entry points.

Each listed case stands for a call that a user's program makes; draw() gives
more of the same ranges.  A case is a dict of plain values: "op" (what is
called), the scan and grid (mm), and the op's own settings.
"""

import math

import numpy as np
import torch

import paper_1002_3675_amd as cb

SAD, SDD = 1000.0, 1500.0


def _scan(n, h, det, pitch, views, arc=360.0, u_off=0.0, off=(0.0, 0.0, 0.0)):
    return {"nx": n[0], "ny": n[1], "nz": n[2], "hx": h[0], "hy": h[1], "hz": h[2],
            "nu": det[0], "nv": det[1], "au": pitch, "av": pitch, "views": views, "arc": arc,
            "u_off": u_off, "x_off": off[0], "y_off": off[1], "z_off": off[2]}


def _head(views):
    return _scan((512, 512, 70), (0.88, 0.88, 2.5), (512, 384), 0.776, views)


def _thick(views):
    return _scan((256, 256, 64), (1.0, 1.0, 2.5), (256, 192), 1.552, views)


def _cube128(views):
    return _scan((128, 128, 128), (1.5, 1.5, 1.5), (256, 192), 1.6, views)


def _tiny(views):
    return _scan((64, 64, 64), (2.0, 2.0, 2.0), (128, 96), 1.6, views)


def _fd(views):
    return _scan((32, 32, 32), (6.0, 6.0, 6.0), (64, 48), 6.4, views)


def _grid(n, h):
    return {"nx": n[0], "ny": n[1], "nz": n[2], "hx": h[0], "hy": h[1], "hz": h[2]}


def listed():
    return [
        # the projector at the size of the paper's experiment: simulating a
        # scan, or one half of an iteration of a solve
        {"name": "project_head40", "op": "project", **_head(40)},
        # Step 1 of an iteration, g = f - tau P^T r, on a thick-slice volume
        # of the serving mix; the larger half of a solve's time
        {"name": "update_thick60", "op": "update", **_thick(60)},
        # one training step through the differentiable projector (forward
        # and backward) at the isotropic size its tests use
        {"name": "train_cube60", "op": "train", **_cube128(60)},
        # the energy of a small volume (residual, its square sum, E1): the
        # smallest float32 calls, where launches and latency count
        {"name": "energy_tiny16", "op": "energy", **_tiny(16)},
        # transpose on an odd-sized region off the axis seen by a shifted
        # (half-fan) detector over a short scan
        {"name": "transpose_halffan_odd", "op": "transpose",
         **_scan((157, 141, 67), (1.1, 1.1, 1.75), (219, 139), 1.4, 31, 200.0, 38.0,
                 (21.0, -12.5, 6.3))},
        # both operators in float64 at the finite-difference size of the
        # derivative checks
        {"name": "double_fd60", "op": "double", **_fd(60)},
        # the paper's Eq. (2) gradient at the head size: the cheap mode
        {"name": "eq2_head40", "op": "eq2", **_head(40)},
        # TV prox of one outer iteration at the head's fine level
        {"name": "prox_head", "op": "prox", "n_inner": 65,
         **_grid((512, 512, 70), (0.88, 0.88, 2.5))},
        # the same on a small odd grid (rows not a multiple of 4 voxels), a
        # chain of short launches
        {"name": "prox_odd_small", "op": "prox", "n_inner": 60,
         **_grid((91, 83, 29), (2.0, 2.0, 2.25))},
        # counts of a head scan to line integrals, with a flat field
        {"name": "log_head40", "op": "log", "nu": 512, "nv": 384, "views": 40},
        # a whole small reconstruction, one level of 10 iterations
        {"name": "solve_tiny16", "op": "solve", "coarse": 0, "fine": 10, **_tiny(16)},
        # a whole head reconstruction, two levels of 20 iterations: the
        # headline workload
        {"name": "solve_head40", "op": "solve", "coarse": 20, "fine": 20, **_head(40)},
    ]


def _log_uniform(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def _draw_grid(rng, most):
    """Grid of 24^3 to about `most` voxels, odd sizes among them."""
    nxy = _log_uniform(rng, 24, 400)
    nx, ny = nxy, max(16, int(nxy * rng.uniform(0.75, 1.1)))
    nz = max(8, min(_log_uniform(rng, 12, 160), most // (nx * ny)))
    if rng.random() < 0.5:  # rows of whole 16-byte groups, as most volumes have
        nx += -nx % 4
    fov = rng.uniform(130.0, 360.0)  # mm across
    h = round(fov / max(nx, ny), 3)
    hz = round(h * rng.choice((1.0, 1.0, 1.25, 2.0, 2.8)), 3)
    return _grid((nx, ny, max(8, min(nz, int(300.0 / hz)))), (h, h, hz))


def draw(rng):
    op = rng.choice(("project", "update", "transpose", "train", "energy", "eq2", "prox", "prox",
                     "double", "log", "solve"))
    if op == "log":
        return {"op": op, "nu": _log_uniform(rng, 60, 800), "nv": _log_uniform(rng, 45, 600),
                "views": rng.randint(1, 40)}
    if op == "prox":
        return {"op": op, "n_inner": rng.randint(1, 100), **_draw_grid(rng, 12000000)}
    small = op in ("double", "solve")
    g = _draw_grid(rng, 400000 if small else 6000000)
    if small and g["nx"] > 100:
        f = 100.0 / g["nx"]
        g = {**g, "nx": 100, "ny": max(16, int(g["ny"] * f)), "hx": round(g["hx"] / f, 3),
             "hy": round(g["hy"] / f, 3)}
    ext = max(g["nx"] * g["hx"], g["ny"] * g["hy"])
    # pixels near the voxel size at the axis, the detector a little wider
    # than the grid's shadow, or half of it shifted sideways
    pitch = round(1.5 * g["hx"] * rng.uniform(0.55, 1.1), 3)
    half = rng.random() < 0.25
    nu = int(min(512, (0.62 if half else 1.25) * 1.5 * ext / pitch))
    nv = int(min(384, 1.3 * 1.5 * g["nz"] * g["hz"] / pitch)) + 3
    odd = rng.random() < 0.3
    case = {"op": op, **g, "nu": max(8, nu), "nv": max(6, nv), "au": pitch, "av": pitch,
            "views": _log_uniform(rng, 6, 20 if small else 60),
            "arc": rng.choice((360.0, 360.0, 200.0)),
            "u_off": round(0.4 * nu * pitch, 2) if half else 0.0,
            "x_off": round(rng.uniform(-25, 25), 2) if odd else 0.0,
            "y_off": round(rng.uniform(-25, 25), 2) if odd else 0.0,
            "z_off": round(rng.uniform(-8, 8), 2) if odd else 0.0}
    if op == "solve":
        case.update(coarse=rng.choice((0, 6)), fine=rng.randint(4, 10))
    return case


# ------------------------------------------------------------ inputs ----

def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _geometry(c):
    angles = None
    if c["arc"] != 360.0:
        angles = tuple(math.radians(c["arc"]) * k / c["views"] for k in range(c["views"]))
    return cb.Geometry(c["nx"], c["ny"], c["nz"], c["hx"], c["hy"], c["hz"], c["nu"], c["nv"],
                       c["au"], c["av"], SAD, SDD, c["views"], angles, 0.0, c["u_off"], 0.0,
                       c["x_off"], c["y_off"], c["z_off"])


def _angles(c):
    return [math.radians(c["arc"]) * k / c["views"] for k in range(c["views"])]


def _axis(n, h, off, dev):
    return (torch.arange(n, dtype=torch.float64, device=dev) - 0.5 * (n - 1)) * h + off


def _phantom(c, seed):
    """Ellipsoids (centre, semi-axes, density): a shell, its inside and
    small inserts, so that values lie between 0 and about 0.04 / mm."""
    rng = np.random.default_rng(seed)
    o = np.array([c.get("x_off", 0.0), c.get("y_off", 0.0), c.get("z_off", 0.0)])
    e = 0.5 * np.array([c["nx"] * c["hx"], c["ny"] * c["hy"], c["nz"] * c["hz"]])
    parts = [(o, 0.85 * e, 0.04), (o, 0.78 * e, -0.02)]
    for _ in range(10):
        parts.append((o + rng.uniform(-0.45, 0.45, 3) * e, rng.uniform(0.05, 0.2, 3) * e,
                      rng.choice([-0.02, -0.005, 0.005, 0.02])))
    return parts


def _volume(c, seed):
    dev = _dev()
    x = _axis(c["nx"], c["hx"], c.get("x_off", 0.0), dev)[None, None, :]
    y = _axis(c["ny"], c["hy"], c.get("y_off", 0.0), dev)[None, :, None]
    z = _axis(c["nz"], c["hz"], c.get("z_off", 0.0), dev)[:, None, None]
    f = torch.zeros((c["nz"], c["ny"], c["nx"]), dtype=torch.float32, device=dev)
    for m, a, rho in _phantom(c, seed):
        inside = ((x - m[0]) / a[0]) ** 2 + ((y - m[1]) / a[1]) ** 2 + ((z - m[2]) / a[2]) ** 2 <= 1
        f += rho * inside.to(torch.float32)
    gen = torch.Generator(device=dev).manual_seed(seed)
    f += 0.002 * torch.randn(f.shape, generator=gen, device=dev)
    return f.clamp_(min=0.0)


def _rays(c, th, dev):
    """Source (3 numbers) and unit directions [nv][nu] x 3 of one view."""
    s = (SAD * math.sin(th), -SAD * math.cos(th), 0.0)
    u = _axis(c["nu"], c["au"], c["u_off"], dev)[None, :]
    v = _axis(c["nv"], c["av"], 0.0, dev)[:, None]
    inv = 1.0 / torch.sqrt(u * u + v * v + SDD * SDD)
    return s, ((u * math.cos(th) - SDD * math.sin(th)) * inv,
               (u * math.sin(th) + SDD * math.cos(th)) * inv, v * inv)


def _line_integrals(c, seed, i0):
    """Exact chords through the phantom with the noise of i0 photons."""
    dev = _dev()
    out = torch.empty((c["views"], c["nv"], c["nu"]), dtype=torch.float64, device=dev)
    parts = _phantom(c, seed)
    for k, th in enumerate(_angles(c)):
        s, d = _rays(c, th, dev)
        out[k] = 0.0
        for m, a, rho in parts:
            al, be, ga = 0.0, 0.0, -1.0
            for t in range(3):
                q, w = (s[t] - m[t]) / a[t], d[t] / a[t]
                al, be, ga = al + w * w, be + q * w, ga + q * q
            out[k] += rho * 2.0 * torch.sqrt((be * be - al * ga).clamp(min=0.0)) / al
    gen = torch.Generator(device=dev).manual_seed(seed + 1)
    sd = torch.exp(0.5 * out) / math.sqrt(i0)
    return (out + sd * torch.randn(out.shape, generator=gen, device=dev)).to(torch.float32)


def _residual(c, seed):
    """Signed data, as P f - Y is during a solve: the difference of two
    scans with noise."""
    return _line_integrals(c, 2 * seed + 1000003, 5e4) - _line_integrals(c, 2 * seed + 2000003, 5e4)


def _prox_settings(c):
    # eps as the solver's default; beta as its rule gives it for a head scan
    return (c["hx"], c["hy"], c["hz"]), 535.0, 1e-3


def prepare(case, seed):
    c = dict(case)
    op = c["op"]
    st = {"op": op, "case": c}
    if op == "log":
        dev = _dev()
        gen = torch.Generator(device=dev).manual_seed(seed)
        shape = (c["views"], c["nv"], c["nu"])
        st["flat"] = 5e4 * (1 + 0.05 * torch.randn(shape, generator=gen, device=dev))
        p = 4.0 * torch.rand(shape, generator=gen, device=dev)
        st["counts"] = torch.poisson(st["flat"] * torch.exp(-2.5 * p), generator=gen)
        return st
    if op == "prox":
        st["z0"] = _volume(c, seed)
        gen = torch.Generator(device=_dev()).manual_seed(seed + 2)
        st["g"] = st["z0"] + 0.004 * torch.randn(st["z0"].shape, generator=gen, device=_dev())
        return st
    st["plan"] = cb.Plan(_geometry(c))
    if op in ("project", "energy", "update", "train", "double"):
        st["f"] = _volume(c, seed)
    if op in ("energy", "train", "solve"):
        st["Y"] = _line_integrals(c, seed, 5e4)
    if op in ("update", "transpose", "eq2", "double"):
        st["r"] = _residual(c, seed)
    if op == "train":
        st["f"].requires_grad_()
    if op == "double":
        st["f"], st["r"] = st["f"].double(), st["r"].double()
    if op == "energy":
        st["sumsq"] = torch.zeros(1, dtype=torch.float64, device=_dev())
    if op == "solve":
        iters = (c["coarse"], c["fine"]) if c["coarse"] else (c["fine"],)
        st["params"] = cb.FbsParams(mu=1e-3, iters=iters, trace_energy="final")
    return st


def run(st):
    op, c = st["op"], st["case"]
    if op == "log":
        return cb.log_counts(st["counts"], flat=st["flat"])
    if op == "prox":
        h, beta, eps = _prox_settings(c)
        return cb.tv_prox(st["g"], st["z0"], h, beta, eps, c["n_inner"])
    plan = st["plan"]
    if op == "project":
        return plan.project(st["f"])
    if op == "transpose":
        return plan.backproject(st["r"])
    if op == "update":
        return plan.backproject_update(st["r"], st["f"], 1e-3)
    if op == "eq2":
        return plan.backproject_eq2(st["r"])
    if op == "double":
        return plan.project(st["f"]), plan.backproject(st["r"])
    if op == "energy":
        r = plan.project_residual(st["f"], st["Y"], sumsq=st["sumsq"])
        e1, e1_eps = cb.tv_energy(st["f"], (c["hx"], c["hy"], c["hz"]), 1e-3)
        return r, st["sumsq"], e1, e1_eps
    if op == "train":
        st["f"].grad = None
        loss = 0.5 * ((cb.Project.apply(st["f"], plan) - st["Y"]) ** 2).sum()
        loss.backward()
        return loss.detach(), st["f"].grad
    f, rep = cb.fbs_solve(plan, st["Y"], st["params"])
    return f, rep.E, rep.E1, rep.E2


# -------------------------------------------------------------- work ----

def _step(c):
    return 0.5 * min(c["hx"], c["hy"], c["hz"])


def _samples(c):
    """Ray samples of one projection: chords of the bordered grid over the
    step, from every third pixel each way."""
    half = [0.5 * (c["n" + a] + 1) * c["h" + a] for a in "xyz"]
    off = [c["x_off"], c["y_off"], c["z_off"]]
    total = 0.0
    for th in _angles(c):
        s, d = _rays(c, th, torch.device("cpu"))
        lo, hi = torch.zeros(()), torch.full((), 1e30)
        for a in range(3):
            da = d[a][::3, ::3] + torch.zeros_like(d[0][::3, ::3])
            da = torch.where(da.abs() < 1e-12, torch.full_like(da, 1e-12), da)
            t0, t1 = (off[a] - half[a] - s[a]) / da, (off[a] + half[a] - s[a]) / da
            lo, hi = torch.maximum(lo, torch.minimum(t0, t1)), torch.minimum(hi, torch.maximum(t0, t1))
        total += float((hi - lo).clamp(min=0).mean()) * c["nu"] * c["nv"]
    return total / _step(c)


def _half(c):
    d = dict(c)
    for k in ("nx", "ny", "nz", "nu", "nv"):
        d[k] = c[k] // 2
    for k in ("hx", "hy", "hz", "au", "av"):
        d[k] = 2 * c[k]
    return d


def work(case):
    c, op = case, case["op"]
    if op == "log":
        n = c["nu"] * c["nv"] * c["views"]
        return {"bytes": 12 * n, "flops": 12 * n}
    vox = c["nx"] * c["ny"] * c["nz"]
    if op == "prox":
        # z and g in, z out; about 60 operations a voxel and step
        return {"bytes": 12 * vox, "flops": 60 * vox * c["n_inner"]}
    meas = c["nu"] * c["nv"] * c["views"]
    if op == "eq2":
        return {"bytes": 4 * (vox + meas), "flops": 35 * vox * c["views"]}
    if op == "solve":
        # 34 operations a ray sample in each direction; 40 TV steps of 60
        # operations a voxel
        flops = 0
        for d, n in ((c, c["fine"]), (_half(c), c["coarse"])):
            if n:
                flops += n * (68 * _samples(d) + 40 * 60 * d["nx"] * d["ny"] * d["nz"])
        return {"bytes": 4 * (vox + meas), "flops": flops}
    n = 34 * _samples(c)
    return {"project": {"bytes": 4 * (vox + meas), "flops": n},
            "transpose": {"bytes": 4 * (vox + meas), "flops": n},
            "update": {"bytes": 4 * (2 * vox + meas), "flops": n},
            "energy": {"bytes": 4 * (vox + 2 * meas), "flops": n + 20 * vox},
            "train": {"bytes": 4 * (2 * vox + meas), "flops": 2 * n},
            "double": {"bytes": 16 * (vox + meas), "flops": 2 * n}}[op]


# -------------------------------------------------------- 64-bit values ----

def _sample_grids(c, k, th, rays_at_once):
    """Sampling positions of view k in grid_sample's coordinates, a block of
    detector rows at a time: (rows, [rays, samples, 1, 3])."""
    dev = _dev()
    s, d = _rays(c, th, dev)
    n = [c["nx"], c["ny"], c["nz"]]
    h = [c["hx"], c["hy"], c["hz"]]
    off = [c["x_off"], c["y_off"], c["z_off"]]
    step = _step(c)
    centre = math.sqrt((s[0] - off[0]) ** 2 + (s[1] - off[1]) ** 2 + off[2] ** 2)
    reach = 0.5 * math.sqrt(sum(((n[a] + 2) * h[a]) ** 2 for a in range(3)))
    idx = torch.arange(max(0, int((centre - reach) / step) - 1), int((centre + reach) / step) + 2,
                       dtype=torch.float64, device=dev)
    rows = max(1, int(rays_at_once // (c["nu"] * idx.numel())))
    for j in range(0, c["nv"], rows):
        q = torch.empty((min(rows, c["nv"] - j) * c["nu"], idx.numel(), 1, 3),
                        dtype=torch.float64, device=dev)
        for a in range(3):
            da = (d[a][j:j + rows] if d[a].shape[0] > 1 else d[a].expand(c["nv"], -1)[j:j + rows])
            da = da.expand(-1, c["nu"]).reshape(-1, 1)
            # index coordinate i -> (2 i + 1) / n - 1
            x = ((s[a] - off[a]) + idx * step * da) / h[a] + 0.5 * (n[a] - 1)
            q[:, :, 0, a] = (2 * x + 1) / n[a] - 1
        yield slice(j, j + rows), q


def _project64(c, f):
    y = torch.empty((c["views"], c["nv"], c["nu"]), dtype=torch.float64, device=f.device)
    f = f.double()[None, None]
    for k, th in enumerate(_angles(c)):
        for rows, q in _sample_grids(c, k, th, 2e8):
            v = torch.nn.functional.grid_sample(f, q[None], mode="bilinear", padding_mode="zeros",
                                                align_corners=False)
            y[k, rows] = _step(c) * v[0, 0, :, :, 0].sum(1).reshape(-1, c["nu"])
    return y


def _transpose64(c, y):
    f = torch.zeros((1, 1, c["nz"], c["ny"], c["nx"]), dtype=torch.float64, device=y.device)
    like = torch.zeros_like(f)
    for k, th in enumerate(_angles(c)):
        for rows, q in _sample_grids(c, k, th, 1e8):
            w = (_step(c) * y[k, rows].double()).reshape(1, 1, -1, 1, 1).expand(
                1, 1, -1, q.shape[1], 1).contiguous()
            f += torch.ops.aten.grid_sampler_3d_backward(w, like, q[None], 0, 0, False,
                                                         [True, False])[0]
    return f[0, 0]


def _eq2_64(c, y):
    dev = y.device
    x = _axis(c["nx"], c["hx"], c["x_off"], dev)[None, None, :]
    yy = _axis(c["ny"], c["hy"], c["y_off"], dev)[None, :, None]
    z = _axis(c["nz"], c["hz"], c["z_off"], dev)[:, None, None]
    out = torch.zeros((c["nz"], c["ny"], c["nx"]), dtype=torch.float64, device=dev)
    for k, th in enumerate(_angles(c)):
        cs, sn = math.cos(th), math.sin(th)
        wx, wy = x - SAD * sn, yy + SAD * cs
        d = wy * cs - wx * sn
        u, v = SDD * (wx * cs + wy * sn) / d, SDD * z / d
        i = (u - c["u_off"]) / c["au"] + 0.5 * (c["nu"] - 1)
        j = v / c["av"] + 0.5 * (c["nv"] - 1)
        q = torch.stack(torch.broadcast_tensors((2 * i + 1) / c["nu"] - 1, (2 * j + 1) / c["nv"] - 1),
                        -1).reshape(1, -1, 1, 2)
        r = torch.nn.functional.grid_sample(y[k].double()[None, None], q, mode="bilinear",
                                            padding_mode="zeros", align_corners=False)
        out += SDD * SDD * torch.sqrt(wx * wx + wy * wy + z * z) / d ** 3 * r.reshape(out.shape)
    return out * (c["hx"] * c["hy"] * c["hz"] / (c["au"] * c["av"]))


def _slopes(z, h):
    """Forward differences over the spacing (zero at the last index)."""
    g = []
    for a, s in zip((2, 1, 0), h):
        d = torch.zeros_like(z)
        m = z.shape[a] - 1
        d.narrow(a, 0, m).copy_((z.narrow(a, 1, m) - z.narrow(a, 0, m)) / s)
        g.append(d)
    return g


def _prox64(g, z, h, beta, eps, n_inner):
    g, z = g.double(), z.double()
    step = 1.0 / (beta + 4.0 * sum(s ** -2 for s in h) / eps)
    for _ in range(n_inner):
        p = _slopes(z, h)
        norm = torch.sqrt(p[0] ** 2 + p[1] ** 2 + p[2] ** 2 + eps * eps)
        grad = beta * (z - g)
        for a, s, pa in zip((2, 1, 0), h, p):
            pa = pa / norm / s
            m = z.shape[a] - 1
            grad = grad - pa
            grad.narrow(a, 1, m).add_(pa.narrow(a, 0, m))
        z = (z - step * grad).clamp(min=0.0)
    return z


def exact(case, seed):
    c, op = dict(case), case["op"]
    if op == "solve":
        return None  # dozens of iterations of the operators below
    st = prepare(case, seed)
    if op == "log":
        return torch.log(st["flat"].double() / st["counts"].double().clamp(min=1.0))
    if op == "prox":
        return _prox64(st["g"], st["z0"], *_prox_settings(c), c["n_inner"])
    if op == "project":
        return _project64(c, st["f"])
    if op == "transpose":
        return _transpose64(c, st["r"])
    if op == "update":
        return st["f"].double() - 1e-3 * _transpose64(c, st["r"])
    if op == "eq2":
        return _eq2_64(c, st["r"])
    if op == "double":
        return _project64(c, st["f"]), _transpose64(c, st["r"])
    if op == "energy":
        r = _project64(c, st["f"]) - st["Y"].double()
        p = _slopes(st["f"].double(), (c["hx"], c["hy"], c["hz"]))
        m = p[0] ** 2 + p[1] ** 2 + p[2] ** 2
        return (r, (r * r).sum().reshape(1), float(torch.sqrt(m).mean()),
                float(torch.sqrt(m + 1e-6).mean()))
    r = _project64(c, st["f"].detach()) - st["Y"].double()
    return 0.5 * (r * r).sum(), _transpose64(c, r)
