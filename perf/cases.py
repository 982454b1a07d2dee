"""The work that programs built on this package have it do, as cases to be timed.

A case names an operator or a whole call, its sizes and its storage type; `prepare` builds what a
program holds before the call (plan, inputs, network), `run` is one call through the public entry
points, `exact` the same result in FP64 from the formulas alone (plain torch and numpy), and `work`
the bytes and operations that the call cannot do without.

Kinds: project (H), backproject (H^T), fbp (Fourier deconvolution of the transducers' response,
then filtered backprojection), pls (PLS-TV reconstruction), sph_project and sph_backproject (the
spherical-voxel model), net (the learned preconditioner's forward pass), train (its gradients for
one training pair).
"""
import math

import numpy as np
import torch

from paper_1304_2017_amd import oat, precond, recon, synth

DEVICE = torch.device("cuda", 0)
GAMMA = 1.0
TYPES = {"f32": torch.float32, "bf16": torch.bfloat16}

# Measurement set-ups of the package's workloads: node spacing (mm), sampling interval and first
# sample (us), samples, speed of sound (mm/us), radius of the measurement sphere (mm).
SETUPS = {
    "small": dict(dx=0.5, dt=0.1, t0=0.0, nt=256, c0=1.5, rs=25.0, layout="sphere"),
    "medium": dict(dx=0.1, dt=0.05, t0=0.0, nt=512, c0=1.5, rs=25.0, layout="sphere"),
    "large": dict(dx=0.1, dt=0.05, t0=0.0, nt=1024, c0=1.5, rs=40.0, layout="hemisphere"),
    "rings": dict(dx=0.14, dt=0.05, t0=17.5, nt=1022, c0=1.54, rs=65.0, layout="rings"),
    "spherical": dict(dx=0.4, dt=0.05, t0=0.0, nt=1024, c0=1.5, rs=40.0, layout="hemisphere"),
}
F_CUT = 5.0          # MHz, the Hann window's cutoff
TV_EPS = 1e-3        # smoothing of the TV penalty


def _case(kind, setup, nx, ny, nz, q, **more):
    return dict(kind=kind, setup=setup, nx=nx, ny=ny, nz=nz, q=q, **more)


def _net(kind, d, h, w):
    return dict(kind=kind, nx=w, ny=h, nz=d)


def listed():
    return [
        # The smallest calls (the parity workload; interactive use): latency and launches.
        dict(_case("project", "small", 32, 32, 32, 64, dtype="f32", image="phantom"), name="project-32"),
        dict(_case("backproject", "small", 32, 32, 32, 64, dtype="f32"), name="backproject-32"),
        # An iteration's two operators at the training workload's size, ragged grids, BF16 storage.
        dict(_case("project", "medium", 128, 105, 117, 1024, dtype="bf16", image="iterate"),
             name="project-128-bf16"),
        dict(_case("backproject", "medium", 117, 128, 99, 1000, dtype="bf16"), name="backproject-128-bf16"),
        # The benchmark's workload: 256^3 nodes, 2048 transducers, 1024 samples.
        dict(_case("project", "large", 256, 256, 256, 2048, dtype="f32", image="phantom"), name="project-256"),
        dict(_case("backproject", "large", 256, 256, 256, 2048, dtype="f32"), name="backproject-256"),
        # Analytic reconstruction of measured data: deconvolution of the response, then FBP.
        dict(_case("fbp", "large", 256, 256, 256, 2048, dtype="f32", taps=64), name="deconvolve-fbp-256"),
        # A whole iterative reconstruction call: plan-resident PLS-TV, a few iterations.
        dict(_case("pls", "medium", 96, 96, 96, 512, iters=3), name="pls-tv-96"),
        # The spherical-voxel model, both directions: 64^3 voxels, 2048 transducers, 256 frequencies
        # in (0, 5] MHz; the forward direction on an iterate (every voxel set, as in reconstruction).
        dict(_case("sph_project", "spherical", 64, 64, 64, 2048, n_f=256, f_min=F_CUT / 256, faces=0,
                   dtype="f32", image="iterate"), name="sph-project-64"),
        dict(_case("sph_backproject", "spherical", 64, 64, 64, 2048, n_f=256, f_min=F_CUT / 256, faces=0,
                   dtype="f32"), name="sph-backproject-64"),
        # The learned preconditioner: its forward pass in a 256^3 reconstruction, and the gradients
        # of one training pair at the training workload's 128^3.
        dict(_net("net", 256, 256, 256), name="net-forward-256"),
        dict(_net("train", 128, 128, 128), name="net-gradients-128"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("project", "backproject", "project", "backproject", "fbp", "pls", "sph_project",
                       "sph_backproject", "net", "train"))
    if kind == "net":
        return _net(kind, *(rng.randint(40, 256) for _ in range(3)))
    if kind == "train":
        return _net(kind, *(rng.randint(40, 128) for _ in range(3)))
    if kind == "pls":
        n = [rng.randint(48, 96) for _ in range(3)]
        return _case(kind, "medium", *n, _log_int(rng, 128, 512), iters=rng.randint(2, 3))
    if kind in ("sph_project", "sph_backproject"):
        more = {"image": rng.choice(("phantom", "iterate"))} if kind == "sph_project" else {}
        while True:
            n = [_log_int(rng, 12, 64) for _ in range(3)]
            q, n_f, faces = _log_int(rng, 64, 2048), _log_int(rng, 16, 511), rng.choice((0, 0, 0, 2, 3, 4))
            if n[0] * n[1] * n[2] * q * n_f * max(1, faces) ** 2 <= 64 ** 3 * 2048 * 256:
                break
        f_min = rng.choice((0.0, F_CUT / n_f, round(rng.uniform(0.05, 1.0), 3)))
        return _case(kind, "spherical", *n, q, n_f=n_f, f_min=f_min, faces=faces,
                     dtype=rng.choice(("f32", "f32", "bf16")), **more)
    setup = rng.choice(("small", "medium", "large", "rings"))
    while True:
        if setup == "small":
            n, q = [rng.randint(9, 32) for _ in range(3)], _log_int(rng, 4, 64)
        elif setup == "medium":
            n, q = [rng.randint(33, 128) for _ in range(3)], _log_int(rng, 32, 1024)
        elif setup == "large":
            n, q = [_log_int(rng, 80, 256) for _ in range(3)], _log_int(rng, 128, 2048)
        else:
            n = [rng.randint(60, 210), rng.randint(60, 210), rng.randint(60, 440)]
            q = rng.randint(8, 32) * 45
        if _points(_case(kind, setup, *n, q)) <= _points(_case(kind, "large", 256, 256, 256, 2048)):
            break
    dtype = rng.choice(("f32", "bf16"))
    if kind == "fbp":
        return _case(kind, setup, *n, q, dtype=dtype, taps=rng.choice((0, rng.randint(16, 128))))
    if kind == "project":
        return _case(kind, setup, *n, q, dtype=dtype, image=rng.choice(("phantom", "iterate")))
    return _case(kind, setup, *n, q, dtype=dtype)


# --------------------------------------------------------------------------------------------------
# Geometry and inputs
# --------------------------------------------------------------------------------------------------
def _positions(case):
    """Transducer positions [Q][3] (mm) and FBP patch areas [Q] (mm^2)."""
    s, q = SETUPS[case["setup"]], case["q"]
    rs = s["rs"]
    i = np.arange(q, dtype=np.float64)
    if s["layout"] == "rings":          # rings of 45 views over the whole polar range
        n = q // 45
        th, ph = np.meshgrid((np.arange(n) + 0.5) * math.pi / n, 2 * math.pi * np.arange(45) / 45, indexing="ij")
        th, ph = th.ravel(), ph.ravel()
        xyz = rs * np.stack([np.sin(th) * np.cos(ph), np.sin(th) * np.sin(ph), np.cos(th)], 1)
        return xyz, rs * rs * (math.pi / n) * (2 * math.pi / 45) * np.sin(th)
    half = s["layout"] == "hemisphere"
    z = -(i + 0.5) / q if half else 1.0 - (2.0 * i + 1.0) / q
    ph = i * math.pi * (3.0 - math.sqrt(5.0))
    r = np.sqrt(np.maximum(0.0, 1.0 - z * z))
    xyz = rs * np.stack([r * np.cos(ph), r * np.sin(ph), z], 1)
    return xyz, np.full(q, (2.0 if half else 4.0) * math.pi * rs * rs / q)


def _origin(case):
    dx = SETUPS[case["setup"]]["dx"]
    return [-0.5 * (case[a] - 1) * dx for a in ("nx", "ny", "nz")]


def _support(case):
    """Radius of the ball that holds every point with a nonzero image value."""
    dx = SETUPS[case["setup"]]["dx"]
    return math.sqrt(sum((abs(o) + dx) ** 2 for o in _origin(case)))


def _plan(case):
    s = SETUPS[case["setup"]]
    xyz, area = _positions(case)
    x0, y0, z0 = _origin(case)
    return oat.Plan(synth.Geometry(case["nx"], case["ny"], case["nz"], s["dx"], x0, y0, z0, xyz, s["nt"], s["dt"],
                                   s["t0"], s["c0"], GAMMA, area), DEVICE.index)


def _taps(case):
    """A causal low-pass response t/tau^2 exp(-t/tau), tau = 0.1 us, sampled at dt."""
    dt = SETUPS[case["setup"]]["dt"]
    t = np.arange(case["taps"]) * dt
    return dt * t / 0.01 * np.exp(-t / 0.1)


def _axes(case, dtype=torch.float32):
    dx = SETUPS[case["setup"]]["dx"]
    return [o + dx * torch.arange(case[a], device=DEVICE, dtype=dtype)
            for o, a in zip(_origin(case), ("nx", "ny", "nz"))]


def _image(case, gen):
    """A phantom of 40 seeded ellipsoids, or an iterate: the phantom with small values everywhere."""
    x, y, z = _axes(case)
    g = np.random.default_rng(int(torch.randint(1 << 30, (1,), generator=gen)))
    span = [float(a[-1] - a[0]) for a in (x, y, z)]
    img = torch.zeros((case["nz"], case["ny"], case["nx"]), device=DEVICE)
    for _ in range(40):
        ax = g.uniform(0.012, 0.12, 3) * max(min(span), 1e-3)
        c = [g.uniform(-0.5, 0.5) * max(0.0, sp - 2 * ax.max()) for sp in span]
        rot, _ = np.linalg.qr(g.normal(size=(3, 3)))
        amp, r2 = g.uniform(0.0, 1.0), 0.0
        for k in range(3):
            r2 = r2 + (((x[None, None, :] - c[0]) * float(rot[0, k]) + (y[None, :, None] - c[1]) * float(rot[1, k])
                        + (z[:, None, None] - c[2]) * float(rot[2, k])) / float(ax[k])) ** 2
        img += float(amp) * (r2 <= 1.0)
    if case["image"] == "iterate":
        img += 0.02 * torch.randn(img.shape, device=DEVICE,
                                  generator=torch.Generator(DEVICE).manual_seed(int(g.integers(1 << 30))))
    return img.to(TYPES[case["dtype"]])


def _noise(case, gen, shape, dtype):
    dev = torch.Generator(DEVICE).manual_seed(int(torch.randint(1 << 30, (1,), generator=gen)))
    return torch.randn(shape, device=DEVICE, generator=dev).to(dtype)


def _pressure(case, gen, noise):
    """The pressure of 9 seeded uniform balls, p = (A Gamma / 2)(d - c0 t)/d for |d - c0 t| <= a, with
    white noise of `noise` times its largest value."""
    s = SETUPS[case["setup"]]
    g = np.random.default_rng(int(torch.randint(1 << 30, (1,), generator=gen)))
    xyz = torch.from_numpy(_positions(case)[0]).to(DEVICE)
    rho = s["c0"] * (s["t0"] + s["dt"] * torch.arange(s["nt"], device=DEVICE, dtype=torch.float64))
    half = 0.5 * s["dx"] * min(case["nx"], case["ny"], case["nz"])
    p = torch.zeros((case["q"], s["nt"]), device=DEVICE, dtype=torch.float64)
    for _ in range(9):
        a = g.uniform(0.06, 0.25) * half
        c = torch.from_numpy(g.uniform(-1, 1, 3) * (half - a) / math.sqrt(3.0)).to(DEVICE)
        d = torch.linalg.norm(xyz - c, dim=1)[:, None]
        p += torch.where((d - rho).abs() <= a, 0.5 * g.uniform(0.5, 1.0) * GAMMA * (d - rho) / d, 0.0)
    return p + noise * p.abs().max() * _noise(case, gen, p.shape, torch.float64)


def _network(case, seed):
    model = precond.Preconditioner(device=DEVICE.index, seed=seed)
    g = torch.Generator().manual_seed(seed + 1)
    for b in model.b:                    # a trained network's biases are not zero
        b.copy_(0.05 * torch.randn(b.shape, generator=g))
    return model


def _field(case, gen, dtype):
    """A volume of unit RMS like a normalised descent direction: smooth structure plus noise."""
    shape = (case["nz"], case["ny"], case["nx"])
    coarse = _noise(case, gen, (1, 1) + tuple((n + 7) // 8 for n in shape), torch.float32)
    v = torch.nn.functional.interpolate(coarse, size=shape, mode="trilinear", align_corners=False)[0, 0]
    v = v + 0.5 * _noise(case, gen, shape, torch.float32)
    return (v / v.square().mean().sqrt()).to(dtype).contiguous()


def _inputs(case, seed):
    """Everything random that the case's call takes, from the seed alone."""
    gen, kind = torch.Generator().manual_seed(int(seed)), case["kind"]
    if kind in ("net", "train"):
        if kind == "net":                # a reconstruction hands over an FP32 direction
            return {"x": _field(case, gen, torch.float32)}
        return {"x": _field(case, gen, torch.bfloat16), "t": _field(case, gen, torch.bfloat16)}
    shape = (case["q"], SETUPS[case["setup"]]["nt"])
    if kind in ("project", "sph_project"):
        return {"x": _image(case, gen)}
    if kind == "backproject":
        return {"y": _noise(case, gen, shape, TYPES[case["dtype"]])}
    if kind == "fbp":
        return {"u": _pressure(case, gen, 0.01).to(TYPES[case["dtype"]])}
    if kind == "pls":
        u = _pressure(case, gen, 0.02).float()
        n = case["nx"] * case["ny"] * case["nz"]
        return {"u": u, "mu": 1e-3 * float(u.double().square().sum()) / (n * TV_EPS)}
    u = _noise(case, gen, (case["q"], case["n_f"], 2), torch.float32)
    return {"u": torch.view_as_complex(u.contiguous())}


def prepare(case, seed):
    state = dict(_inputs(case, seed), case=case)
    if case["kind"] in ("net", "train"):
        state["model"] = _network(case, int(seed))
        return state
    plan = state["plan"] = _plan(case)
    if case.get("taps"):
        plan.set_eir(_taps(case))
    if case.get("faces"):
        plan.set_aperture(2.0, 2.0, case["faces"])
    return state


# --------------------------------------------------------------------------------------------------
# One pass
# --------------------------------------------------------------------------------------------------
def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "project":
        return state["plan"].project(state["x"])
    if kind == "backproject":
        return state["plan"].backproject(state["y"])
    if kind == "fbp":
        if not case["taps"]:
            return state["plan"].fbp(state["u"])
        p = state["plan"].deconvolve(state["u"], F_CUT)
        return p, state["plan"].fbp(p)
    if kind == "pls":
        r = recon.pls_tv(state["plan"], state["u"], state["mu"], TV_EPS, iters=case["iters"])
        return {"image": r.image, "residuals": r.residuals, "objective": r.objective}
    if kind == "sph_project":
        return state["plan"].sph_project(state["x"], case["n_f"], case["f_min"], F_CUT / case["n_f"])
    if kind == "sph_backproject":
        return state["plan"].sph_backproject(state["u"], case["f_min"], F_CUT / case["n_f"],
                                             out_dtype=TYPES[case["dtype"]])
    model = state["model"]
    if kind == "net":
        return model.forward(state["x"])
    z = model.forward(state["x"], keep=True)
    loss, dz = precond.mse(z, state["t"])
    return {"z": z, "loss": loss, "grads": model.backward(dz)}


# --------------------------------------------------------------------------------------------------
# What a pass cannot do without
# --------------------------------------------------------------------------------------------------
def _points(case):
    """Quadrature points of one H or H^T: one per cell volume of the shells that cross the image."""
    s = SETUPS[case["setup"]]
    cells = (case["nx"] + 1.0) * (case["ny"] + 1.0) * (case["nz"] + 1.0)
    return cells * case["q"] * s["dx"] / (s["c0"] * s["dt"])


def work(case):
    kind, n = case["kind"], float(case["nx"]) * case["ny"] * case["nz"]
    if kind in ("net", "train"):
        macs = 27.0 * (16 + 16 * 16 + 16) * n          # the three layers
        if kind == "net":
            return {"bytes": 6.0 * n, "flops": 2 * macs}
        return {"bytes": 6.0 * n, "flops": 2 * (2 * macs + 27.0 * (16 * 16 + 16) * n)}
    s, size = SETUPS[case["setup"]], 2.0 if case.get("dtype") == "bf16" else 4.0
    if kind in ("sph_project", "sph_backproject"):
        # a distance and one value of the transducer's band-limited time function per pair
        pairs = n * case["q"] * max(1, case["faces"]) ** 2
        return {"bytes": size * n + 8.0 * case["q"] * case["n_f"], "flops": 40 * pairs}
    data = float(case["q"]) * s["nt"]
    if kind == "fbp":
        return {"bytes": size * (n + (3 if case["taps"] else 1) * data), "flops": 25 * n * case["q"]}
    # position of a point (rotation of its segment), floor and fraction, trilinear weights: about 50
    if kind == "pls":
        ops = 2 * case["iters"] + 1
        return {"bytes": 4.0 * (n + data) * ops, "flops": 50 * _points(case) * ops}
    return {"bytes": size * (n + data), "flops": 50 * _points(case)}


# --------------------------------------------------------------------------------------------------
# The same results in FP64 from the formulas
# --------------------------------------------------------------------------------------------------
EXACT_POINTS = 1.2e10    # H or H^T evaluated point by point stays within seconds up to here


def _candidates(case):
    """Points that `_quadrature` lists: those in the ball that holds the image."""
    s = SETUPS[case["setup"]]
    return case["q"] * 4.19 * _support(case) ** 3 / (s["dx"] ** 2 * s["c0"] * s["dt"])


def _frames(xyz):
    """Rows e1, e2, e3 of each transducer's frame: polar, minus azimuthal, inward direction."""
    d = np.linalg.norm(xyz, axis=1)
    th, ph = np.arccos(xyz[:, 2] / d), np.arctan2(xyz[:, 1], xyz[:, 0])
    e1 = np.stack([np.cos(th) * np.cos(ph), np.cos(th) * np.sin(ph), -np.sin(th)], 1)
    e2 = np.stack([np.sin(ph), -np.cos(ph), np.zeros_like(ph)], 1)
    return np.stack([e1, e2, -xyz / d[:, None]], 1), d


def _quadrature(case):
    """For every shell k that meets the image: (k, points in the transducer frame [P][3], weights [P])."""
    s = SETUPS[case["setup"]]
    dx, rs, r_sup = s["dx"], s["rs"], _support(case)
    for k in range(s["nt"]):
        rho = s["c0"] * (s["t0"] + k * s["dt"])
        if not rho > 0 or abs(rho - rs) > r_sup:
            continue
        dth = dx / rho
        th_max = math.acos(max(-1.0, min(1.0, (rs * rs + rho * rho - r_sup * r_sup) / (2 * rs * rho))))
        i = torch.arange(min(math.ceil(math.pi / dth), math.ceil(th_max / dth) + 1), device=DEVICE, dtype=torch.float64)
        lo, hi = i * dth, ((i + 1) * dth).clamp(max=math.pi)
        th = 0.5 * (lo + hi)
        nj = torch.floor(2 * math.pi * rho * torch.sin(th) / dx + 0.5).clamp(min=1)
        w = 2 * math.pi * rho * rho * (torch.cos(lo) - torch.cos(hi)) / nj
        cnt = nj.long()
        ring = torch.repeat_interleave(torch.arange(len(cnt), device=DEVICE), cnt)
        j = torch.arange(len(ring), device=DEVICE) - (torch.cumsum(cnt, 0) - cnt)[ring]
        ph = 2 * math.pi * j.double() / nj[ring]
        st = rho * torch.sin(th)[ring]
        yield k, torch.stack([st * torch.cos(ph), st * torch.sin(ph), rho * torch.cos(th)[ring]], 1), w[ring]


def _cells(case, pts, xyz, frames):
    """The points that fall in the image's cells, for transducers (xyz, frames): their transducer and
    point numbers, the cell's index in the zero-padded image and the position in the cell."""
    s = SETUPS[case["setup"]]
    pos = (torch.matmul(pts, frames.reshape(-1, 3, 3).permute(1, 0, 2).reshape(3, -1)).reshape(len(pts), -1, 3)
           + (xyz - torch.tensor(_origin(case), device=DEVICE, dtype=torch.float64))) / s["dx"]
    c = torch.floor(pos)
    n = torch.tensor([case["nx"], case["ny"], case["nz"]], device=DEVICE, dtype=torch.float64)
    p, q = torch.nonzero(((c >= -1) & (c < n)).all(-1), as_tuple=True)
    c, f = c[p, q], (pos[p, q] - c[p, q])
    c = c.long() + 1
    return q, p, (c[:, 2] * (case["ny"] + 2) + c[:, 1]) * (case["nx"] + 2) + c[:, 0], f


def _corners(case, f):
    """(offset in the padded image, trilinear weight) of a cell's 8 nodes."""
    for z in (0, 1):
        for y in (0, 1):
            for x in (0, 1):
                w = (f[:, 0] if x else 1 - f[:, 0]) * (f[:, 1] if y else 1 - f[:, 1]) * (f[:, 2] if z else 1 - f[:, 2])
                yield (z * (case["ny"] + 2) + y) * (case["nx"] + 2) + x, w


def _batches(case):
    xyz = _positions(case)[0]
    frames = torch.from_numpy(_frames(xyz)[0]).to(DEVICE)
    xyz = torch.from_numpy(xyz).to(DEVICE)
    for k, pts, w in _quadrature(case):
        step = max(1, (1 << 24) // len(pts))
        for q0 in range(0, case["q"], step):
            yield k, w, q0, step, _cells(case, pts, xyz[q0:q0 + step], frames[q0:q0 + step])


def _times(case):
    s = SETUPS[case["setup"]]
    return s["t0"] + s["dt"] * torch.arange(s["nt"], device=DEVICE, dtype=torch.float64)


def _project64(case, img):
    """H img: sums over the quadrature, s = g / t, central difference."""
    s = SETUPS[case["setup"]]
    pad = torch.nn.functional.pad(img.double(), (1, 1, 1, 1, 1, 1)).reshape(-1)
    g = torch.zeros((s["nt"], case["q"]), device=DEVICE, dtype=torch.float64)
    for k, w, q0, step, (q, p, cell, f) in _batches(case):
        v = torch.zeros(len(q), device=DEVICE, dtype=torch.float64)
        for off, c in _corners(case, f):
            v += c * pad[cell + off]
        n = min(case["q"], q0 + step) - q0
        rows = torch.zeros(len(w) * n, device=DEVICE, dtype=torch.float64)
        rows[p * n + q] = v * w[p]
        g[k, q0:q0 + n] = rows.reshape(-1, n).sum(0)
    t = _times(case)[:, None]
    r = torch.nn.functional.pad(torch.where(t > 0, g / t, 0.0), (0, 0, 1, 1))
    return (GAMMA / (4 * math.pi * s["c0"] ** 2) * (r[2:] - r[:-2]) / (2 * s["dt"])).T.contiguous()


def _backproject64(case, y):
    """H^T y: the transposes of the difference and of the sums."""
    s = SETUPS[case["setup"]]
    r = torch.nn.functional.pad(y.double().T, (0, 0, 1, 1))
    t = _times(case)[:, None]
    g = torch.where(t > 0, GAMMA / (4 * math.pi * s["c0"] ** 2) * (r[:-2] - r[2:]) / (2 * s["dt"]) / t, 0.0)
    shape = (case["nz"] + 2, case["ny"] + 2, case["nx"] + 2)
    pad = torch.zeros(shape[0] * shape[1] * shape[2], device=DEVICE, dtype=torch.float64)
    for k, w, q0, _, (q, p, cell, f) in _batches(case):
        v = w[p] * g[k][q + q0]
        for off, c in _corners(case, f):
            pad.index_add_(0, cell + off, c * v)
    return pad.reshape(shape)[1:-1, 1:-1, 1:-1].contiguous()


def _deconvolve64(case, u):
    s, h = SETUPS[case["setup"]], _taps(case)
    n = 1 << (2 * s["nt"] - 1).bit_length()
    delayed = np.zeros(n)
    delayed[1:1 + len(h)] = h
    ht = torch.from_numpy(np.fft.fft(delayed)).to(DEVICE)
    f = torch.fft.fftfreq(n, s["dt"], device=DEVICE, dtype=torch.float64).abs()
    win = torch.where(f <= F_CUT, 0.5 * (1 - torch.cos(math.pi * (F_CUT - f) / F_CUT)), 0.0)
    return torch.fft.ifft(torch.fft.fft(u.double(), n, dim=1) * win / ht, dim=1).real[:, :s["nt"]].contiguous()


def _fbp64(case, p):
    s = SETUPS[case["setup"]]
    xyz, area = _positions(case)
    x, y, z = _axes(case, torch.float64)
    tau, nt = s["t0"] / s["dt"], s["nt"]
    pad = torch.nn.functional.pad(p, (1, 1))
    img = torch.zeros((case["nz"], case["ny"], case["nx"]), device=DEVICE, dtype=torch.float64)
    for q in range(case["q"]):
        a = [float(v) for v in xyz[q]]
        r2 = ((x - a[0]) ** 2)[None, None, :] + ((y - a[1]) ** 2)[None, :, None] + ((z - a[2]) ** 2)[:, None, None]
        kt = (torch.sqrt(r2) / s["c0"] - s["t0"]) / s["dt"]
        k = torch.floor(kt)
        i = k.clamp(-1, nt).long() + 1
        inv = 1.0 / (kt + tau)
        img += float(area[q] / np.linalg.norm(xyz[q])) * (
            ((k + 1 + tau) * inv - 1.5) * pad[q][i] + (1.5 - (k + tau) * inv) * pad[q][(i + 1).clamp(max=nt + 1)])
    return img * (-1.0 / (math.pi * GAMMA * s["c0"] * s["dt"]))


def _pls64(case, u, mu):
    """The recursion of recon.pls_tv on the operators above, FP64 throughout."""
    def diff(a):
        return [torch.nn.functional.pad(torch.diff(a, dim=d), (0, 0) * (2 - d) + (0, 1)) for d in (2, 1, 0)]

    def tv(a):
        g = diff(a)
        w = 1.0 / torch.sqrt(g[0] ** 2 + g[1] ** 2 + g[2] ** 2 + TV_EPS ** 2)
        grad = torch.zeros_like(a)
        for v, d in zip(g, (2, 1, 0)):
            v = (v * w).narrow(d, 0, a.shape[d] - 1)
            grad.narrow(d, 1, a.shape[d] - 1).add_(v)
            grad.narrow(d, 0, a.shape[d] - 1).sub_(v)
        return float((1.0 / w).sum()), grad, w

    def dot(a, b):
        return float((a * b).sum())

    u = u.double()
    a, r = torch.zeros((case["nz"], case["ny"], case["nx"]), device=DEVICE, dtype=torch.float64), u.clone()
    value, tg, w = tv(a)
    g = -2 * _backproject64(case, r) + mu * tg
    d, gg, un = -g, dot(g, g), dot(u, u) ** 0.5
    res, obj = [1.0], [un * un + mu * value]
    for _ in range(case["iters"]):
        hd = _project64(case, d)
        t = -dot(g, d) / (2 * dot(hd, hd) + mu * float((w * sum(v * v for v in diff(d))).sum()))
        a, r = a + t * d, r - t * hd
        value, tg, w = tv(a)
        new = -2 * _backproject64(case, r) + mu * tg
        ng = dot(new, new)
        d = -new + max(0.0, (ng - dot(new, g)) / gg) * d
        if dot(new, d) >= 0:
            d = -new
        g, gg = new, ng
        res.append(dot(r, r) ** 0.5 / un)
        obj.append(dot(r, r) + mu * value)
    return {"image": a, "residuals": res, "objective": obj}


def _faces(case):
    """(nodes [Q][m^2][3], weights [m^2]) of the transducer faces."""
    xyz = _positions(case)[0]
    m = case["faces"]
    if not m:
        return xyz[:, None, :], np.ones(1)
    e = _frames(xyz)[0]
    x, w = np.polynomial.legendre.leggauss(m)
    a, b = [v.ravel() for v in np.meshgrid(x, x, indexing="ij")]
    nodes = xyz[:, None, :] + a[None, :, None] * e[:, None, 0, :] + b[None, :, None] * e[:, None, 1, :]  # half of 2 mm
    return nodes, 0.25 * np.outer(w, w).ravel()


def _p0(case, f):
    s = SETUPS[case["setup"]]
    fs = f.clamp(min=1e-300)
    br = s["dx"] / (2 * s["c0"]) * torch.cos(math.pi * f * s["dx"] / s["c0"]) - \
        torch.sin(math.pi * f * s["dx"] / s["c0"]) / (2 * math.pi * fs)
    return torch.where(f > 0, torch.complex(torch.zeros_like(f), -GAMMA * s["c0"] / fs * br), 0.0)


def _turns(x):
    x = 2 * math.pi * (x - torch.round(x))
    return torch.complex(torch.cos(x), torch.sin(x))


def _spherical64(case, img, u):
    """The printed sums; frequencies l = 16 a + b, so that exp(j 2 pi f_l t) = A_a B_b."""
    s, n_f, df = SETUPS[case["setup"]], case["n_f"], F_CUT / case["n_f"]
    f = case["f_min"] + df * torch.arange(n_f, device=DEVICE, dtype=torch.float64)
    p0, na = _p0(case, f), (n_f + 15) // 16
    fa = (case["f_min"] + 16 * df * torch.arange(na, device=DEVICE, dtype=torch.float64))[:, None]
    fb = (df * torch.arange(16, device=DEVICE, dtype=torch.float64))[:, None]
    z, y, x = torch.meshgrid(*reversed(_axes(case, torch.float64)), indexing="ij")
    pos = [v.reshape(-1) for v in (x, y, z)]
    nodes, wts = _faces(case)
    if u is None:
        al = img.double().reshape(-1)
        keep = torch.nonzero(al)[:, 0]
        al, pos = al[keep], [v[keep] for v in pos]
        out = torch.zeros((case["q"], na * 16), device=DEVICE, dtype=torch.complex128)
    else:
        v = torch.zeros((case["q"], na * 16), device=DEVICE, dtype=torch.complex128)
        v[:, :n_f] = u.to(torch.complex128) * p0.conj()
        out = torch.zeros(len(pos[0]), device=DEVICE, dtype=torch.float64)
    for q in range(case["q"]):
        for r, w in zip(nodes[q], wts):
            d = torch.sqrt(sum((c - float(o)) ** 2 for c, o in zip(pos, r)))
            t = d / s["c0"]
            a, b, w = _turns(fa * t), _turns(fb * t), float(w) / (2 * math.pi * d)
            if u is None:
                a, b = [torch.nn.functional.pad(v.conj(), (0, -len(al) % 1024)).resolve_conj().reshape(len(v), -1, 1024)
                        for v in (a * (w * al), b)]          # the sum over voxels in runs of 1024
                out[q] += torch.bmm(a.transpose(0, 1).contiguous(), b.permute(1, 2, 0).contiguous()).sum(0).reshape(-1)
            else:
                out += w * (a * torch.matmul(v[q].reshape(na, 16), b)).sum(0).real
    return out[:, :n_f] * p0 if u is None else out.reshape(case["nz"], case["ny"], case["nx"])


def _conv64(x, w, b):
    """'Same' 3x3x3 convolution: x [C_in][D][H][W], w [C_out][C_in][27]."""
    _, d, h, wd = x.shape
    pad, y = torch.nn.functional.pad(x, (1, 1, 1, 1, 1, 1)), 0.0
    for t in range(27):
        dz, dy, dx = t // 9, t // 3 % 3, t % 3
        y = y + torch.matmul(w[:, :, t], pad[:, dz:dz + d, dy:dy + h, dx:dx + wd].reshape(x.shape[0], -1))
    return (y + b[:, None]).reshape(-1, d, h, wd)


def _network64(case, inputs, seed):
    model = _network(case, seed)
    train = case["kind"] == "train"
    ws, bs = [[v.double().requires_grad_(train) for v in g] for g in (model.w, model.b)]
    x = inputs["x"].to(torch.bfloat16).double()[None]
    with torch.set_grad_enabled(train):
        a = torch.relu(_conv64(x, ws[0], bs[0]))
        a = torch.relu(_conv64(a, ws[1], bs[1]))
        z = (x + _conv64(a, ws[2], bs[2]))[0]
        if not train:
            return z
        loss = (z - inputs["t"].double()).square().mean()
        grads = torch.autograd.grad(loss, ws + bs)
    return {"z": z.detach(), "loss": loss.detach().reshape(1), "grads": list(grads)}


def exact(case, seed):
    kind, inputs = case["kind"], _inputs(case, seed)
    if kind in ("project", "backproject", "pls"):
        if _candidates(case) * (2 * case["iters"] + 1 if kind == "pls" else 1) > EXACT_POINTS:
            return None
        if kind == "project":
            return _project64(case, inputs["x"])
        if kind == "backproject":
            return _backproject64(case, inputs["y"])
        return _pls64(case, inputs["u"], inputs["mu"])
    if kind == "fbp":
        if not case["taps"]:
            return _fbp64(case, inputs["u"].double())
        p = _deconvolve64(case, inputs["u"])
        return p, _fbp64(case, p)
    if kind in ("sph_project", "sph_backproject"):
        return _spherical64(case, inputs.get("x"), inputs.get("u"))
    return _network64(case, inputs, int(seed))
