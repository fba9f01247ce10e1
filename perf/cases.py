"""The work that a user of this library has it do, as cases that can be timed and compared.

Every case goes through the Python binding's public calls on a scanner geometry of the
library's own configurations (the 54/95 cm fan over a 51.2 cm field, the 0.5 cm parallel
beam) or of a generic size.  Measurements are Poisson counts of simulated luggage or of
three ellipses, with exact chords as line integrals.

  project, backproject   R and its transpose, called as operators
  cdm                    constrained per-ray decomposition (the projection-wise baseline)
  decompose              per-ray decomposition with the quadratic coupling of the ADMM
  fbp                    filtered backprojection of line integrals
  precondition           the ramp preconditioner of the x-update
  start                  counts -> measurements -> CDM -> FBP -> start image
  admm                   initial state and outer iterations of one slice
  lmcg                   counts -> the LM x CG baseline on one slice
  batch                  slices of several sizes advanced together

exact() is the same computation in plain torch, in double precision, from the geometry and
the formulas alone.
"""
import math

import numpy as np
import torch

from paper_1905_00934_amd import dect, synth

DEVICE = "cuda"
FOV = 51.2  # cm, side of the fan scanner's field
I0 = 2e5    # unattenuated counts


# ------------------------------------------------------------------ cases ---
def _case(name, kind, beam, nx, ny, views, bins, dtype="f32", **more):
    c = dict(name=name, kind=kind, beam=beam, nx=nx, ny=ny, views=views, bins=bins, dtype=dtype)
    c.update(more)
    return c


def listed():
    return [
        # The smallest call a program makes: one image of the tiny configuration, in double
        # precision, projected on its own (latency and launches).
        _case("project_tiny64_f64", "project", "parallel", 64, 64, 90, 95, "f64", ch=1),
        # One application of each operator on the headline slice's basis pair: what a user's
        # own solver calls in its loop.
        _case("project_fan512", "project", "fan", 512, 512, 720, 1024, ch=2),
        _case("backproject_fan512", "backproject", "fan", 512, 512, 720, 1024, ch=2),
        # An odd-sized parallel scan with a shifted detector: one image, no rotational
        # symmetry.
        _case("backproject_parallel_odd", "backproject", "parallel", 350, 301, 451, 481, ch=1,
              offset=-0.25),
        # The largest operator call: four images (a pair of slices) at twice the headline
        # resolution.
        _case("project_fan1024_4ch", "project", "fan", 1024, 1024, 1440, 2048, ch=4),
        # Filtered backprojection alone, as a user runs it on any line integrals.
        _case("fbp_parallel366", "fbp", "parallel", 366, 366, 540, 545, ch=2),
        # The projection-wise baseline and the start image of a slice, from raw counts.
        _case("start_fan512", "start", "fan", 512, 512, 720, 1024, iters=20),
        # The headline slice from its start image, advanced as far as a server's first check:
        # initial state and five outer iterations (UDM1-CG1, adaptive rho).
        _case("admm_fan512", "admm", "fan", 512, 512, 720, 1024, iters=5, lm=1, cg=1,
              precond=False, warm=True),
        # The preconditioned scheme, the transposes summing in double.
        _case("admm_pcg_fan256", "admm", "fan", 256, 256, 360, 512, iters=5, lm=1, cg=1,
              precond=True, warm=True, sums64=True),
        # The whole tiny configuration in double precision: 20 outer iterations.
        _case("admm_tiny64_f64", "admm", "parallel", 64, 64, 90, 95, "f64", iters=20, lm=1, cg=1,
              precond=False, warm=False),
        # The baseline scheme on the middle size of the uneven mix.
        _case("lmcg_fan384", "lmcg", "fan", 384, 384, 540, 768, iters=2, lm=1, cg=1),
        # A small stack of the uneven mix (256, 384 and 512 in turn), replayed from a graph.
        _case("batch_uneven9", "batch", "fan", 512, 512, 720, 1024, iters=5, lm=1, cg=1,
              slices=9),
    ]


def _log_size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any kind, sizes over the whole range, even, odd and ragged."""
    kind = rng.choice(["project", "project", "backproject", "backproject", "cdm", "decompose",
                       "fbp", "precondition", "start", "admm", "admm", "lmcg", "batch"])
    n = _log_size(rng, 48, 640)
    whole = kind in ("admm", "lmcg", "batch")
    if whole:
        n = min(n, 512)
    beam = rng.choice(["fan", "fan", "parallel"])
    ragged = kind != "batch" and rng.random() < 0.4
    if ragged:
        nx, ny = n, max(16, int(n * rng.uniform(0.7, 1.2)))
        views = max(5, int(n * rng.uniform(0.7, 1.5)) | 1)
        bins = max(9, int(n * rng.uniform(1.2, 2.1)) | 1)
        offset = rng.choice([0.0, 0.25, -0.25])
    else:
        n += n % 2
        nx = ny = n
        views = 4 * max(2, int(round(0.35 * n)))
        bins = int(n * (2 if beam == "fan" else 1.485)) + rng.randint(0, 3)
        offset = rng.choice([0.0, 0.0, 0.25])
    f64 = kind != "batch" and rng.random() < 0.25
    c = dict(kind=kind, beam=beam, nx=nx, ny=ny, views=views, bins=bins,
             dtype="f64" if f64 else "f32", offset=offset)
    if kind in ("project", "backproject"):
        c["ch"] = rng.choice([1, 2, 2, 4])
    elif kind == "fbp":
        c["ch"] = rng.choice([1, 2])
    elif kind in ("cdm", "start"):
        c["iters"] = rng.choice([5, 10, 20])
    elif kind == "decompose":
        c["iters"] = rng.choice([1, 2, 5])
    elif whole:
        c["lm"], c["cg"] = rng.choice([(1, 1), (1, 1), (1, 2), (2 if f64 else 1, 1)])
        c["iters"] = rng.choice([1, 2, 5])
        if kind == "admm":
            c["precond"] = rng.random() < 0.4
            c["warm"] = not f64 or rng.random() < 0.4
            c["sums64"] = rng.random() < 0.2 or c["precond"]
        if kind == "batch":
            c["slices"] = rng.choice([2, 3, 5])
            c["nx"] = c["ny"] = n = max(64, min(n, 384)) // 2 * 2
            c["views"], c["bins"] = 4 * max(2, int(round(0.35 * n))), 2 * n
    return c


# ----------------------------------------------------------------- inputs ---
def _geometry(c):
    nx, ny, V, D = c["nx"], c["ny"], c["views"], c["bins"]
    if c["beam"] == "fan":
        g = synth.fan_geometry_fov(max(nx, ny), V, D)
        g["nx"], g["ny"] = nx, ny
    else:
        pix = 32.0 / max(nx, ny)
        g = synth.geometry("parallel", nx, ny, pix, V, D, 1.05 * pix * math.hypot(nx, ny) / D)
    g["det_offset"] = float(c.get("offset", 0.0))
    return g


def _dtype(c):
    return torch.float64 if c["dtype"] == "f64" else torch.float32


def _phantom(geom, seed):
    fov = geom["pixel_cm"] * min(geom["nx"], geom["ny"])
    if geom["kind"] == "parallel":
        return synth.tiny_phantom(seed, fov)
    rng = np.random.default_rng([seed, 17])
    return synth.luggage_phantom(seed, int(rng.integers(10, 41)), int(rng.integers(0, 4)), fov)


def _line_integrals(geom, seed):
    """Exact (a_c, a_p) of the seed's phantom along every ray, [V, D, 2] (double)."""
    V, D = geom["n_views"], geom["n_det"]
    f = dict(dtype=torch.float64, device=DEVICE)
    th = geom["angle0"] + torch.arange(V, **f) * (geom["span"] / V)
    cs, sn = torch.cos(th)[:, None], torch.sin(th)[:, None]
    u = ((torch.arange(D, **f) - (D - 1) / 2.0 + geom["det_offset"]) * geom["det_cm"])[None, :]
    if geom["kind"] == "parallel":
        ox, oy, dx, dy = u * cs, u * sn, (-sn).expand(V, D), cs.expand(V, D)
    else:
        so, sd = geom["src_iso_cm"], geom["src_det_cm"]
        ox, oy = (so * cs).expand(V, D), (so * sn).expand(V, D)
        dx, dy = -(sd - so) * cs - u * sn - ox, -(sd - so) * sn + u * cs - oy
        nrm = torch.hypot(dx, dy)
        dx, dy = dx / nrm, dy / nrm
    out = torch.zeros(V, D, 2, **f)
    for s in _phantom(geom, seed).shapes:
        c, d = math.cos(s.rot), math.sin(s.rot)
        px, py = (ox - s.cx) * c + (oy - s.cy) * d, (oy - s.cy) * c - (ox - s.cx) * d
        qx, qy = dx * c + dy * d, dy * c - dx * d
        if s.kind == "ellipse":
            px, py, qx, qy = px / s.ax, py / s.ay, qx / s.ax, qy / s.ay
            qa, qb, qc = qx * qx + qy * qy, px * qx + py * qy, px * px + py * py - 1.0
            ln = 2.0 * torch.sqrt((qb * qb - qa * qc).clamp_min(0.0)) / qa
        else:
            tiny = 1e-12
            qx = torch.where(qx.abs() < tiny, torch.full_like(qx, tiny), qx)
            qy = torch.where(qy.abs() < tiny, torch.full_like(qy, tiny), qy)
            tx, wx, ty, wy = -px / qx, s.ax / qx.abs(), -py / qy, s.ay / qy.abs()
            ln = (torch.minimum(tx + wx, ty + wy) - torch.maximum(tx - wx, ty - wy)).clamp_min(0.0)
        out[..., 0] += s.xc * ln
        out[..., 1] += s.xp * ln
    return out


def _spectra_tensors():
    s = synth.default_spectra()
    t = [torch.tensor(np.asarray(v), dtype=torch.float64, device=DEVICE)
         for v in (s.s_high, s.s_low, s.f_kn, s.f_p)]
    return t[0] / t[0].sum(), t[1] / t[1].sum(), t[2], t[3]


def _counts(geom, seed, dtype):
    """Poisson counts (high, low) of the seed's phantom, [V, D]."""
    a = _line_integrals(geom, seed)
    wh, wl, kn, fp = _spectra_tensors()
    lam = torch.zeros(2, *a.shape[:2], dtype=torch.float64, device=DEVICE)
    for k in range(kn.numel()):
        t = torch.exp(-kn[k] * a[..., 0] - fp[k] * a[..., 1])
        lam[0] += wh[k] * t
        lam[1] += wl[k] * t
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    n = torch.poisson(I0 * lam, generator=gen)
    return n[0].to(dtype).contiguous(), n[1].to(dtype).contiguous()


def _image(geom, seed, ch, dtype):
    """The seed's phantom sampled at the pixel centres with a little noise, [ny, nx(, ch)]."""
    ny, nx, pix = geom["ny"], geom["nx"], geom["pixel_cm"]
    f = dict(dtype=torch.float64, device=DEVICE)
    X = ((torch.arange(nx, **f) - (nx - 1) / 2.0) * pix)[None, :]
    Y = ((torch.arange(ny, **f) - (ny - 1) / 2.0) * pix)[:, None]
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    out = 0.01 * torch.randn(ny, nx, ch, generator=gen, **f)
    for c in range(0, ch, 2):  # further pairs: further slices
        for s in _phantom(geom, seed + 101 * c).shapes:
            cs, sn = math.cos(s.rot), math.sin(s.rot)
            u = ((X - s.cx) * cs + (Y - s.cy) * sn) / s.ax
            v = ((Y - s.cy) * cs - (X - s.cx) * sn) / s.ay
            m = (u * u + v * v <= 1.0) if s.kind == "ellipse" else ((u.abs() <= 1) & (v.abs() <= 1))
            out[..., c] += s.xc * m
            if ch > 1:
                out[..., c + 1] += s.xp * m
    out = out.to(dtype)
    return (out[..., 0] if ch == 1 else out).contiguous()


def _sinogram(geom, seed, ch, dtype):
    """Line integrals of the seed's phantom with noise, [V, D(, ch)]."""
    a = torch.cat([_line_integrals(geom, seed + 101 * c) for c in range(0, ch, 2)], -1)[..., :ch]
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    a = a + 0.02 * torch.randn(a.shape, generator=gen, dtype=a.dtype, device=DEVICE)
    a = a.to(dtype)
    return (a[..., 0] if ch == 1 else a).contiguous()


def _params(c):
    return dect.AdmmParams(lm_iters=c["lm"], cg_iters=c["cg"],
                           precond=dect.PRECOND_RAMP if c.get("precond") else dect.PRECOND_NONE,
                           rt_sums=dect.RT_SUMS_F64 if c.get("sums64") else dect.RT_SUMS_PLAN)


def _batch_cases(c):
    """The slices of a batch: 1/2, 3/4 and the whole of the case's size in turn."""
    out = []
    for k in range(c["slices"]):
        f = (2, 3, 4)[k % 3]
        n, V, D = (v * f // 4 for v in (c["nx"], c["views"], c["bins"]))
        out.append(dict(c, nx=n // 2 * 2, ny=n // 2 * 2, views=V // 4 * 4, bins=D))
    return out


def prepare(case, seed):
    c = dict(case)
    kind, dtype = c["kind"], _dtype(c)
    spec = synth.default_spectra()
    s = dict(case=c)
    if kind == "batch":
        plans, slices = {}, []
        for k, cc in enumerate(_batch_cases(c)):
            key = (cc["nx"], cc["views"], cc["bins"])
            if key not in plans:
                plans[key] = dect.Plan(_geometry(cc), spec, dtype, device=DEVICE)
            plan = plans[key]
            h, l = _counts(plan.geom, seed + 1000 * k, dtype)
            slices.append((plan, list(plan.ingest(h, l, I0)), plan.new_state()))
        s["slices"], s["params"] = slices, _params(c)
        s["x0"] = [plan.cdm_fbp_start(meas)[2] for plan, meas, _ in slices]
        for (plan, meas, st), x0 in zip(slices, s["x0"]):
            plan.admm_init(meas, st, s["params"], x0)
        s["batch"] = dect.Batch(slices, s["params"], graph=True)
        return s
    geom = _geometry(c)
    plan = s["plan"] = dect.Plan(geom, spec, dtype, device=DEVICE)
    if kind in ("project", "precondition"):
        s["img"] = _image(geom, seed, c.get("ch", 2), dtype)
    elif kind in ("backproject", "fbp"):
        s["sino"] = _sinogram(geom, seed, c["ch"], dtype)
    else:
        s["counts"] = _counts(geom, seed, dtype)
    if kind in ("cdm", "decompose"):
        s["meas"] = plan.ingest(*s["counts"], I0)
    if kind == "cdm":
        s["cost"] = torch.empty(plan.V, plan.D, dtype=dtype, device=DEVICE)
    if kind == "decompose":
        # The a-update's setting: a near the measured line integrals, the coupling centre a
        # little off it.
        a = _line_integrals(geom, seed)
        gen = torch.Generator(device=DEVICE)
        gen.manual_seed(int(seed) + 1)
        noise = torch.randn(2, *a.shape, generator=gen, dtype=a.dtype, device=DEVICE)
        s["a0"] = (a * (1.0 + 0.05 * noise[0])).to(dtype).contiguous()
        s["v"] = (a + 0.05 * noise[1]).to(dtype).contiguous()
    if kind == "admm":
        s["meas"] = plan.ingest(*s["counts"], I0)
        s["x0"] = plan.cdm_fbp_start(s["meas"])[2] if c["warm"] else None
        s["state"], s["params"] = plan.new_state(), _params(c)
    if kind == "lmcg":
        s["state"], s["params"] = plan.new_lmcg_state(), _params(c)
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "batch":
        for (plan, meas, st), x0 in zip(s["slices"], s["x0"]):
            plan.admm_init(meas, st, s["params"], x0)
        s["batch"].iterate(c["iters"])
        return [dict(x=st.x, z=st.z, Rx=st.Rx) for _, _, st in s["slices"]]
    plan = s["plan"]
    if kind == "project":
        return plan.project(s["img"])
    if kind == "backproject":
        return plan.backproject(s["sino"])
    if kind == "precondition":
        return plan.precondition(s["img"])
    if kind == "fbp":
        return plan.fbp(s["sino"])
    if kind == "cdm":
        return plan.cdm(*s["meas"], lm_iters=c["iters"], cost=s["cost"]), s["cost"]
    if kind == "decompose":
        return plan.decompose_rays(*s["meas"], a=s["a0"].clone(), v=s["v"], rho=(1e-3, 1e-3),
                                   lm_iters=c["iters"])
    if kind == "admm":
        st = s["state"]
        plan.admm_init(s["meas"], st, s["params"], s["x0"])
        plan.admm_iterate(s["meas"], st, s["params"], c["iters"])
        return _admm_outputs(c, dict(x=st.x, z=st.z, Rx=st.Rx, y=st.y, a=st.a))
    meas = plan.ingest(*s["counts"], I0)
    if kind == "start":
        return dict(zip(("a", "fbp", "x0"), plan.cdm_fbp_start(meas, c["iters"])))
    st = s["state"]
    plan.lmcg_init(meas, st, s["params"])
    plan.lmcg_iterate(meas, st, s["params"], c["iters"])
    return dict(x=st.x, z=st.z, Rx=st.Rx)


def _admm_outputs(c, out):
    """The images and R x; in double precision the decomposition and the differences too (in
    single precision a ray whose accept test is a tie may move either way)."""
    return out if c["dtype"] == "f64" else {k: out[k] for k in ("x", "z", "Rx")}


# ------------------------------------------------------------------- work ---
def _samples(c):
    """Joseph samples of one application of R, nearly: lines times rays crossing each."""
    g = _geometry(c)
    delta = g["det_cm"] * (g["src_iso_cm"] / g["src_det_cm"] if g["kind"] == "fan" else 1.0)
    return 0.9 * c["views"] * c["nx"] * c["ny"] * g["pixel_cm"] / delta


def work(case):
    """Bytes of inputs and outputs once, and operations of the method: 2 taps x 2 per sample
    and channel for R and R^T, 16 per energy bin (110) and ray for both spectra, 8 per pixel,
    view and channel for the FBP gather, 5 P log2 P per FFT."""
    c = case
    kind = c["kind"]
    if kind == "batch":
        parts = [work(dict(cc, kind="admm", precond=False, warm=True)) for cc in _batch_cases(c)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    e = 8 if c["dtype"] == "f64" else 4
    N, M, ch = c["nx"] * c["ny"], c["views"] * c["bins"], c.get("ch", 2)
    op = 4.0 * _samples(c)  # per channel
    spec = 16.0 * 110 * M
    if kind in ("project", "backproject"):
        return {"bytes": e * ch * (N + M), "flops": op * ch}
    if kind == "precondition":
        P = 2 ** math.ceil(math.log2(2 * max(c["nx"], c["ny"])))
        return {"bytes": e * 4 * N, "flops": 4 * 5.0 * P * P * math.log2(P)}
    if kind == "fbp":
        return {"bytes": e * ch * (N + M), "flops": 8.0 * N * c["views"] * ch}
    if kind == "cdm":
        return {"bytes": e * 7 * M, "flops": spec * c["iters"]}
    if kind == "decompose":
        return {"bytes": e * 10 * M, "flops": spec * c["iters"]}
    if kind == "start":
        return {"bytes": e * (4 * M + 4 * N), "flops": spec * c["iters"] + 16.0 * N * c["views"]}
    m, n, k = c["lm"], c["cg"], c["iters"]
    if kind == "lmcg":
        return {"bytes": e * (4 * M + 8 * N), "flops": k * (4 * m * (n + 1) * op + 2 * m * spec)}
    start = 10 * spec + (4 if c["warm"] else 2) * op
    return {"bytes": e * (6 * M + 8 * N), "flops": start + k * (2 * (2 * n + 1) * op + m * spec)}


# ------------------------------------------------------------------ exact ---
class _Joseph:
    """R and R^T in double precision: per ray one linearly interpolated sample on every
    column (|dx| >= |dy|) or row it crosses, times the step.  For a fan over a full turn with
    quarter-turn symmetric views, view v + k V/4 is view v turned by k quarter turns."""

    def __init__(self, g):
        self.g = g
        V, D = g["n_views"], g["n_det"]
        self.sym = 4 if (g["kind"] == "fan" and abs(g["span"] - 2 * math.pi) < 1e-12
                         and V % 4 == 0 and g["nx"] == g["ny"] and g["nx"] % 2 == 0) else 1
        self.Vb = V // self.sym
        self.mat = None
        # Angles through numpy: the orientation of a 45 degree ray hangs on its last bit.
        th = g["angle0"] + np.arange(self.Vb) * g["span"] / V
        c, s = np.cos(th)[:, None], np.sin(th)[:, None]
        u = ((np.arange(D) - 0.5 * (D - 1) + g["det_offset"]) * g["det_cm"])[None, :]
        if g["kind"] == "parallel":
            ox, oy, dx, dy = u * c, u * s, -s + 0 * u, c + 0 * u
        else:
            so, sd = g["src_iso_cm"], g["src_det_cm"]
            ox, oy = so * c + 0 * u, so * s + 0 * u
            dx, dy = (-(sd - so) * c - u * s) - ox, (-(sd - so) * s + u * c) - oy
        cx, cy, pix = 0.5 * (g["nx"] - 1), 0.5 * (g["ny"] - 1), g["pixel_cm"]
        xs = np.abs(dx) >= np.abs(dy)
        with np.errstate(divide="ignore", invalid="ignore"):
            slope = np.where(xs, dy / dx, dx / dy)
            phi0 = np.where(xs, (oy - ox * slope) / pix - cx * slope + cy,
                            (ox - oy * slope) / pix - cy * slope + cx)
        step = pix * np.sqrt(1.0 + slope * slope)
        up = lambda a: torch.tensor(a.reshape(-1), device=DEVICE)
        self.parts = []
        for want in (True, False):
            sel = torch.nonzero(up(xs == want)).reshape(-1)
            self.parts.append((sel, up(phi0)[sel], up(slope)[sel], up(step)[sel]))

    def _taps(self, phi0, slope, k, n):
        phi = phi0 + slope * k
        j = torch.floor(phi)
        al = (phi - j)[:, None]
        return (j.clamp(-1, n) + 1).long(), (j.clamp(-2, n - 1) + 2).long(), al

    def project(self, img):  # [ny, nx, ch] -> [V, D, ch]
        ny, nx, ch = img.shape
        stack = torch.cat([torch.rot90(img, k, (0, 1)) for k in range(self.sym)], -1)
        out = torch.zeros(self.Vb * self.g["n_det"], stack.shape[-1], dtype=img.dtype, device=DEVICE)
        for (sel, phi0, slope, step), im in zip(self.parts, (stack.transpose(0, 1), stack)):
            steps, n = im.shape[0], im.shape[1]
            pad = torch.zeros(steps, n + 3, im.shape[2], dtype=img.dtype, device=DEVICE)
            pad[:, 1:n + 1] = im
            acc = torch.zeros(sel.numel(), im.shape[2], dtype=img.dtype, device=DEVICE)
            for k in range(steps):
                j0, j1, al = self._taps(phi0, slope, k, n)
                acc += (1.0 - al) * pad[k][j0] + al * pad[k][j1]
            out[sel] = acc * step[:, None]
        out = out.reshape(self.Vb, -1, self.sym, ch).permute(2, 0, 1, 3)
        return out.reshape(self.sym * self.Vb, -1, ch).contiguous()

    def _matrix(self):
        """R^T of the base views as a sparse matrix [pixels, base rays]."""
        g, pix, ray, val = self.g, [], [], []
        nx, ny = g["nx"], g["ny"]
        for (sel, phi0, slope, step), xstep in zip(self.parts, (True, False)):
            for k in range(nx if xstep else ny):
                phi = phi0 + slope * k
                j = torch.floor(phi)
                for jj, w in ((j, 1.0 - (phi - j)), (j + 1, phi - j)):
                    on = torch.nonzero((jj >= 0) & (jj < (ny if xstep else nx))).reshape(-1)
                    q = jj[on].int()
                    pix.append(q * nx + k if xstep else k * nx + q)
                    ray.append(sel[on].int())
                    val.append((w * step)[on])
        pix, order = torch.sort(torch.cat(pix))
        rows = torch.searchsorted(pix, torch.arange(nx * ny + 1, device=DEVICE, dtype=pix.dtype))
        return torch.sparse_csr_tensor(rows.int(), torch.cat(ray)[order], torch.cat(val)[order],
                                       (nx * ny, self.Vb * g["n_det"]))

    def transpose(self, sino):  # [V, D, ch] -> [ny, nx, ch]
        g = self.g
        ny, nx, ch = g["ny"], g["nx"], sino.shape[-1]
        rows = sino.reshape(self.sym, self.Vb, -1, ch).permute(1, 2, 0, 3).reshape(
            -1, self.sym * ch)
        if self.mat is None:
            self.mat = self._matrix()
        im = (self.mat @ rows.contiguous()).reshape(ny, nx, self.sym, ch)
        return sum(torch.rot90(im[:, :, k], -k, (0, 1)) for k in range(self.sym)).contiguous()


class _Spectral:
    """f_s(a) = -ln sum_k w_k exp(-f_KN a_c - f_p a_p) of both spectra and their gradients."""

    def __init__(self):
        wh, wl, kn, fp = _spectra_tensors()
        self.s = [(torch.log(w[w > 0]), kn[w > 0], fp[w > 0]) for w in (wh, wl)]
        self.mean = [((w * kn).sum().item(), (w * fp).sum().item()) for w in (wh, wl)]

    def eval(self, a):  # [R, 2] -> f [R, 2 spectra], grad [R, 2 spectra, 2 bases]
        f, g = [], []
        for lw, kn, fp in self.s:
            fs, gs = [], []
            for part in a.split(1 << 16):
                e = lw - part[:, :1] * kn - part[:, 1:] * fp
                fs.append(-torch.logsumexp(e, 1))
                q = torch.softmax(e, 1)
                gs.append(torch.stack([q @ kn, q @ fp], 1))
            f.append(torch.cat(fs))
            g.append(torch.cat(gs))
        return torch.stack(f, 1), torch.stack(g, 1)

    def linearised(self, m):
        (hc, hp), (lc, lp) = self.mean
        det = hc * lp - hp * lc
        return torch.stack([(lp * m[:, 0] - hp * m[:, 1]) / det,
                            (hc * m[:, 1] - lc * m[:, 0]) / det], 1)

    def lm(self, m, w, a, iters, v=None, rho=(0.0, 0.0), mu0=1e-3, nonneg=False):
        """Levenberg-Marquardt with Marquardt scaling per ray (x10 on rejection, /10 on
        acceptance); nonneg: projected onto a >= 0, an outward coordinate at 0 held there."""
        rho = torch.tensor(rho, dtype=torch.float64, device=DEVICE)
        v = torch.zeros_like(a) if v is None else v
        phi_of = lambda f, a: 0.5 * (w * (f - m) ** 2).sum(1) + 0.5 * (rho * (a - v) ** 2).sum(1)
        f, g = self.eval(a)
        phi, mu = phi_of(f, a), torch.full_like(a[:, 0], mu0)
        for _ in range(iters):
            G = ((w * (f - m))[..., None] * g).sum(1) + rho * (a - v)
            Hc = (w * g[..., 0] ** 2).sum(1) + rho[0]
            Hp = (w * g[..., 1] ** 2).sum(1) + rho[1]
            X = (w * g[..., 0] * g[..., 1]).sum(1)
            Dc, Dp = (1.0 + mu) * Hc, (1.0 + mu) * Hp
            det = Dc * Dp - X * X
            d = torch.stack([-(Dp * G[:, 0] - X * G[:, 1]) / det,
                             -(Dc * G[:, 1] - X * G[:, 0]) / det], 1)
            bad = ~((det > 0) & torch.isfinite(det))
            stop = torch.zeros_like(bad)
            if nonneg:
                fix = (a == 0) & (G > 0)
                one = torch.stack([-G[:, 0] / Dc, -G[:, 1] / Dp], 1)
                any_fix = fix.any(1)
                d = torch.where(any_fix[:, None], torch.where(fix, torch.zeros_like(d), one), d)
                bad = torch.where(any_fix, ~((torch.where(fix[:, 0], Dp, Dc) > 0)), bad)
                stop = fix.all(1)
            t = a + d
            if nonneg:
                t = t.clamp_min(0.0)
            t = torch.where((bad | stop)[:, None], a, t)
            ft, gt = self.eval(t)
            pt = phi_of(ft, t)
            ok = (pt < phi) & ~bad & ~stop
            a = torch.where(ok[:, None], t, a)
            f = torch.where(ok[:, None], ft, f)
            g = torch.where(ok[:, None, None], gt, g)
            phi = torch.where(ok, pt, phi)
            mu = torch.where(stop, mu, torch.where(ok, 0.1 * mu, 10.0 * mu))
        return a, phi


def _fbp_exact(g, sino):  # [V, D, ch] -> [ny, nx, ch]
    V, D, ch = sino.shape
    P = 1
    while P < 2 * D:
        P *= 2
    fan = g["kind"] == "fan"
    delta = g["det_cm"] * (g["src_iso_cm"] / g["src_det_cm"] if fan else 1.0)
    f = dict(dtype=torch.float64, device=DEVICE)
    h = torch.zeros(P, **f)
    n = torch.arange(1, P // 2 + 1, 2, **f)
    h[0] = 1.0 / (4.0 * delta * delta)
    h[1:P // 2 + 1:2] = -1.0 / (math.pi ** 2 * n * n * delta * delta)
    h[P // 2 + 1:] = h[1:P // 2].flip(0)
    so = g["src_iso_cm"]
    if fan:
        u = (torch.arange(D, **f) - 0.5 * (D - 1) + g["det_offset"]) * delta
        sino = sino * (so / torch.sqrt(so * so + u * u))[None, :, None]
    q = torch.fft.irfft(torch.fft.rfft(sino, P, dim=1) * torch.fft.rfft(h)[None, :, None], P,
                        dim=1)[:, :D] * (delta * (0.5 if fan else 1.0))
    pad = torch.zeros(V, D + 3, ch, **f)
    pad[:, 1:D + 1] = q
    X = ((torch.arange(g["nx"], **f) - 0.5 * (g["nx"] - 1)) * g["pixel_cm"])[None, :]
    Y = ((torch.arange(g["ny"], **f) - 0.5 * (g["ny"] - 1)) * g["pixel_cm"])[:, None]
    img = torch.zeros(g["ny"], g["nx"], ch, **f)
    for v in range(V):
        t = g["angle0"] + v * g["span"] / V
        c, s = math.cos(t), math.sin(t)
        L = so - (X * c + Y * s) if fan else None
        b = (so * (Y * c - X * s) / L if fan else X * c + Y * s) / delta
        b = b + (0.5 * (D - 1) - g["det_offset"])
        k = torch.floor(b)
        al = (b - k)[..., None]
        val = (1.0 - al) * pad[v][(k.clamp(-1, D) + 1).long()] + \
            al * pad[v][(k.clamp(-2, D - 1) + 2).long()]
        img += val * ((so / L) ** 2)[..., None] if fan else val
    return img * (g["span"] / V)


def _ramp(img):  # [ny, nx, 2]
    ny, nx = img.shape[:2]
    py, px = (2 ** math.ceil(math.log2(2 * n)) for n in (ny, nx))
    f = dict(dtype=torch.float64, device=DEVICE)
    w = torch.sqrt(torch.fft.fftfreq(py, **f)[:, None] ** 2 + torch.fft.rfftfreq(px, **f) ** 2)
    w = w.clamp_min(1.0 / max(px, py))[..., None]
    z = torch.fft.irfft2(torch.fft.rfft2(img, (py, px), dim=(0, 1)) * w, (py, px), dim=(0, 1))
    return z[:ny, :nx].contiguous()


def _grad(x):  # [ny, nx, 2] -> horizontal and vertical forward differences, [ny, nx, 2, 2]
    d = torch.zeros(*x.shape[:2], 2, 2, dtype=x.dtype, device=DEVICE)
    d[:, :-1, 0] = x[:, 1:] - x[:, :-1]
    d[:-1, :, 1] = x[1:] - x[:-1]
    return d


def _grad_t(y):
    s = torch.zeros(*y.shape[:2], 2, dtype=y.dtype, device=DEVICE)
    h, v = y[:, :-1, 0], y[:-1, :, 1]
    s[:, :-1] -= h
    s[:, 1:] += h
    s[:-1] -= v
    s[1:] += v
    return s


def _measurements(counts):
    n = torch.stack([t.double().reshape(-1) for t in counts], 1)
    return torch.log(I0 / n.clamp_min(1.0)), n / I0


def _start_exact(g, S, m, w, iters):
    V, D = g["n_views"], g["n_det"]
    a, _ = S.lm(m, w, S.linearised(m).clamp_min(0.0), iters, nonneg=True)
    img = _fbp_exact(g, a.reshape(V, D, 2))
    tot = a.sum(0)
    x0 = torch.stack([img[..., 0], img[..., 0] * (tot[1] / tot[0])], -1)
    return a.reshape(V, D, 2), img, x0


def _admm_exact(c, counts):
    """The splitting scheme's outer iterations (Eqs. (9)-(13)) with residual balancing."""
    g, S = _geometry(c), _Spectral()
    J = _Joseph(g)
    V, D, ny, nx = g["n_views"], g["n_det"], g["ny"], g["nx"]
    m, w = _measurements(counts)
    lam, mu, tau = 1e-5, 10.0, 2.0
    rho = torch.full((2,), 1e-3, dtype=torch.float64, device=DEVICE)
    zero = lambda *s: torch.zeros(*s, 2, dtype=torch.float64, device=DEVICE)
    a = S.lm(m, w, S.linearised(m), 10)[0].reshape(V, D, 2)
    x, Rx, ua, y, uy, z, uz = (zero(ny, nx), zero(V, D), zero(V, D), zero(ny, nx, 2),
                               zero(ny, nx, 2), zero(ny, nx), zero(ny, nx))
    if c["warm"]:
        x = _start_exact(g, S, m, w, 20)[2]
        z, Rx, y = x.clone(), J.project(x), _grad(x)
    dot = lambda p, q: (p * q).sum((0, 1))
    M = _ramp if c["precond"] else (lambda t: t)
    soft = lambda t, h: torch.sign(t) * (t.abs() - h).clamp_min(0.0)
    for _ in range(c["iters"]):
        r = J.transpose(a + ua - Rx) + _grad_t(y + uy - _grad(x)) + z + uz - x
        zz = M(r)
        p, gam = zz.clone(), dot(r, zz)
        for _ in range(c["cg"]):
            Rp = J.project(p)
            q = J.transpose(Rp) + _grad_t(_grad(p)) + p
            al = gam / dot(p, q)
            x, Rx, r = x + al * p, Rx + al * Rp, r - al * q
            zz = M(r)
            new = dot(r, zz)
            p, gam = zz + (new / gam) * p, new
        a1 = S.lm(m, w, a.reshape(-1, 2), c["lm"], (Rx - ua).reshape(-1, 2),
                  tuple(rho.tolist()))[0].reshape(V, D, 2)
        Dx = _grad(x)
        y1, z1 = soft(Dx - uy, lam / rho), (x - uz).clamp_min(0.0)
        ua, uy, uz = ua + a1 - Rx, uy + y1 - Dx, uz + z1 - x
        s = J.transpose(a1 - a) + _grad_t(y1 - y) + (z1 - z)
        a, y, z = a1, y1, z1
        rn = torch.sqrt(dot(a - Rx, a - Rx) + (y - Dx).square().sum((0, 1, 2))
                        + dot(z - x, z - x))
        sn = rho * torch.sqrt(dot(s, s))
        new = torch.where(rn > mu * sn, rho * tau, torch.where(sn > mu * rn, rho / tau, rho))
        ua, uy, uz, rho = ua * (rho / new), uy * (rho / new), uz * (rho / new), new
    return dict(x=x, z=z, y=y.reshape(ny, nx, 4), Rx=Rx, a=a)


def _lmcg_exact(c, counts):
    """The baseline's outer iterations (Eqs. (7)-(8) by LM(m) x CG(n), then (9)-(11))."""
    g, S = _geometry(c), _Spectral()
    J = _Joseph(g)
    V, D, ny, nx = g["n_views"], g["n_det"], g["ny"], g["nx"]
    m, w = _measurements(counts)
    lam, bal, tau = 1e-5, 10.0, 2.0
    rho = torch.full((2,), 1e-3, dtype=torch.float64, device=DEVICE)
    zero = lambda *s: torch.zeros(*s, dtype=torch.float64, device=DEVICE)
    x, Rx, z, uz = zero(ny, nx, 2), zero(V * D, 2), zero(ny, nx, 2), zero(ny, nx, 2)
    y, uy = zero(ny, nx, 2, 2), zero(ny, nx, 2, 2)
    f, gr = S.eval(Rx)
    R1 = lambda t: J.project(t[..., None]).reshape(-1)
    T1 = lambda t: J.transpose(t.reshape(V, D, 1))[..., 0]
    G1 = lambda t: _grad(torch.stack([t, t], -1))[..., 0]
    GT1 = lambda t: _grad_t(torch.stack([t, t], -1))[..., 0]
    data = lambda f: 0.5 * (w * (f - m) ** 2).sum()
    for _ in range(c["iters"]):
        for b in range(2):
            damp, rb = 1e-3, rho[b]
            yb, uyb, zb, uzb = y[..., b], uy[..., b], z[..., b], uz[..., b]
            pen = lambda t: 0.5 * rb * (((yb - G1(t) + uyb) ** 2).sum()
                                        + ((zb - t + uzb) ** 2).sum())
            for _ in range(c["lm"]):
                xb, Jb = x[..., b], gr[..., b]
                W = (w * Jb ** 2).sum(1)
                grad = T1((w * (f - m) * Jb).sum(1)) + rb * (GT1(G1(xb)) + xb - GT1(yb + uyb)
                                                            - zb - uzb)
                d, r = torch.zeros_like(xb), -grad
                p, rr, kappa = r.clone(), (r * r).sum(), None
                for _ in range(c["cg"]):
                    Hp = T1(W * R1(p)) + rb * (GT1(G1(p)) + p)
                    kappa = (p * Hp).sum() / (p * p).sum() if kappa is None else kappa
                    q = Hp + damp * kappa * p
                    al = rr / (p * q).sum()
                    d, r = d + al * p, r - al * q
                    new = (r * r).sum()
                    p, rr = r + (new / rr) * p, new
                t = xb + d
                at = Rx.clone()
                at[:, b] = R1(t)
                ft, gt = S.eval(at)
                if data(ft) + pen(t) < data(f) + pen(xb):
                    x = x.clone()
                    x[..., b] = t
                    Rx, f, gr, damp = at, ft, gt, damp / 10.0
                else:
                    damp *= 10.0
        Dx = _grad(x)
        v = Dx - uy
        y1, z1 = torch.sign(v) * (v.abs() - lam / rho).clamp_min(0.0), (x - uz).clamp_min(0.0)
        uy, uz = uy + y1 - Dx, uz + z1 - x
        rn = torch.sqrt((y1 - Dx).square().sum((0, 1, 2)) + (z1 - x).square().sum((0, 1)))
        sn = rho * torch.sqrt((_grad_t(y1 - y) + z1 - z).square().sum((0, 1)))
        y, z = y1, z1
        new = torch.where(rn > bal * sn, rho * tau, torch.where(sn > bal * rn, rho / tau, rho))
        uy, uz, rho = uy * (rho / new), uz * (rho / new), new
    planes = lambda t: t.permute(2, 0, 1).contiguous()
    return dict(x=planes(x), z=planes(z),
                Rx=Rx.reshape(V, D, 2).permute(2, 0, 1).contiguous())


def exact(case, seed):
    c = dict(case)
    kind, dtype = c["kind"], _dtype(c)
    if kind == "batch":
        outs = []
        for k, cc in enumerate(_batch_cases(c)):
            cc = dict(cc, precond=False, warm=True)
            counts = _counts(_geometry(cc), seed + 1000 * k, dtype)
            outs.append(_admm_outputs(cc, _admm_exact(cc, counts)))
        return outs
    g = _geometry(c)
    if kind in ("project", "precondition"):
        img = _image(g, seed, c.get("ch", 2), dtype).double()
        if kind == "precondition":
            return _ramp(img)
        out = _Joseph(g).project(img[..., None] if img.dim() == 2 else img)
        return out[..., 0].contiguous() if img.dim() == 2 else out
    if kind in ("backproject", "fbp"):
        sino = _sinogram(g, seed, c["ch"], dtype).double()
        s3 = sino[..., None] if sino.dim() == 2 else sino
        out = _Joseph(g).transpose(s3) if kind == "backproject" else _fbp_exact(g, s3)
        return out[..., 0].contiguous() if sino.dim() == 2 else out
    counts = _counts(g, seed, dtype)
    if kind == "admm":
        return _admm_outputs(c, _admm_exact(c, counts))
    if kind == "lmcg":
        return _lmcg_exact(c, counts)
    S = _Spectral()
    m, w = _measurements(counts)
    if kind == "start":
        return dict(zip(("a", "fbp", "x0"), _start_exact(g, S, m, w, c["iters"])))
    if kind == "cdm":
        a, phi = S.lm(m, w, S.linearised(m).clamp_min(0.0), c["iters"], nonneg=True)
        return a.reshape(g["n_views"], g["n_det"], 2), phi.reshape(g["n_views"], g["n_det"])
    s = prepare(c, seed)
    a, _ = S.lm(m, w, s["a0"].double().reshape(-1, 2), c["iters"],
                s["v"].double().reshape(-1, 2), (1e-3, 1e-3))
    return a.reshape(g["n_views"], g["n_det"], 2)
