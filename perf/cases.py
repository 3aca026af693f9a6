"""Timed workloads of the Dirac solvers, through the public Python and C entry points.

A pass is one solve as a user's program runs it on a solver it keeps: set the
initial spinor (a complex128 device tensor), advance the case's steps, copy the
state to a pinned host buffer the program keeps, and, for plain FP64 solves, read
the observables.  The solver (tables, schedules), the initial spinor and the host
buffer are what the program has in hand before the pass.  FP32 states come back as
float32 (the C call widens them exactly).

Families: "solve2" one 2-D Scheme II solve (plain, corrected second-order or with
time-dependent potentials), "scheme1" Crank-Nicolson by GMRES, "solve3" the 3-D
4-spinor solve, "batch" many 2-D FP32 solves of mixed sizes in one batch run.
"""
import ctypes
import math

import numpy as np
import torch

from paper_1909_02894_amd import dirac as D

FLAT, BUMP, EXP3 = D.METRIC_FLAT, D.METRIC_GAUSS_BUMP, D.METRIC_PAPER_EXP3
SPIN_NONE, SPIN_PAPER, SPIN_2P1 = D.SPIN_NONE, D.SPIN_PAPER, D.SPIN_2P1

# ---------------------------------------------------------------- the cases


def _solve2(name, n1, n2, steps, metric, prec, layer=True, tuned=False, form="plain"):
    return {"name": name, "family": "solve2", "n1": n1, "n2": n2, "steps": steps, "metric": metric, "prec": prec,
            "layer": layer, "tuned": tuned, "form": form}


def listed():
    return [
        # the flat packet solve, the smallest call: launches and latency count
        _solve2("flat_64_f64", 64, 64, 100, "flat", "f64", layer=False),
        # the curved bump solve with its absorbing layer at full length, tuned as a long run is
        _solve2("curved_512_f64_tuned", 512, 512, 2000, "bump", "f64", tuned=True),
        # a rectangular FP32 curved solve as created, without tuning
        _solve2("curved_1024x256_f32", 1024, 256, 200, "bump", "f32"),
        # the precision study's large flat grid in FP32, tuned
        _solve2("flat_2048_f32_tuned", 2048, 2048, 200, "flat", "f32", layer=False, tuned=True),
        # a large curved FP64 solve of the paper's metric with a layer, as created
        _solve2("curved_2048_f64", 2048, 2048, 100, "exp3", "f64"),
        # the largest curved grid, beyond the Infinity Cache
        _solve2("curved_4096_f32", 4096, 4096, 60, "bump", "f32"),
        # the corrected second-order step
        _solve2("step2bis_512_f64", 512, 512, 400, "bump", "f64", form="step2bis"),
        # time-dependent potentials (static V, pulsed A)
        _solve2("potentials_512_f64", 512, 512, 400, "bump", "f64", form="potentials"),
        # Scheme I: a Crank-Nicolson solve by GMRES on the device each step
        {"name": "scheme1_512_f64", "family": "scheme1", "n1": 512, "n2": 512, "steps": 40, "metric": "bump"},
        # 3-D, the paper's metric with a layer, FP64
        {"name": "curved3d_128_f64", "family": "solve3", "n1": 128, "n2": 128, "n3": 128, "steps": 50,
         "metric": "exp3", "prec": "f64", "layer": True},
        # 3-D flat FP32, beyond the Infinity Cache
        {"name": "flat3d_256x256x128_f32", "family": "solve3", "n1": 256, "n2": 256, "n3": 128, "steps": 50,
         "metric": "flat", "prec": "f32", "layer": False},
        # the batch of mixed curved solves, tuned: every solve the same number of steps
        {"name": "batch64_f32_tuned", "family": "batch", "count": 64, "steps": 200, "lo": 128, "hi": 512,
         "tuned": True, "ragged": False},
    ]


# a drawn case moves at most this many bytes (work())
_MOST = 6.0e10


def draw(rng):
    def pow2(lo, hi):
        return 1 << rng.randint(lo.bit_length() - 1, hi.bit_length() - 1)

    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["solve2", "solve2", "solve2", "step2bis", "potentials", "scheme1", "solve3", "batch"])
    while True:
        if kind == "solve2":
            prec = rng.choice(["f64", "f32"])
            metric = rng.choice(["flat", "bump", "exp3"])
            c = {"family": "solve2", "n1": pow2(32, 4096), "n2": pow2(32, 4096),
                 "steps": logint(15, 1000 if prec == "f64" else 150), "metric": metric, "prec": prec,
                 "layer": metric != "flat" or rng.random() < 0.3, "tuned": rng.random() < 0.3, "form": "plain"}
        elif kind in ("step2bis", "potentials"):
            prec = rng.choice(["f64", "f64", "f32"])
            c = {"family": "solve2", "n1": pow2(64, 2048), "n2": pow2(64, 2048), "steps": logint(15, 150),
                 "metric": "bump", "prec": prec, "layer": True, "tuned": False, "form": kind}
        elif kind == "scheme1":
            c = {"family": "scheme1", "n1": pow2(64, 1024), "n2": pow2(64, 1024), "steps": logint(5, 30),
                 "metric": "bump"}
        elif kind == "solve3":
            prec = rng.choice(["f64", "f32"])
            metric = rng.choice(["flat", "exp3"])
            c = {"family": "solve3", "n1": pow2(32, 256), "n2": pow2(32, 256), "n3": pow2(32, 256),
                 "steps": logint(10, 60), "metric": metric, "prec": prec,
                 "layer": metric != "flat" or rng.random() < 0.3}
        else:
            lo = pow2(64, 256)
            c = {"family": "batch", "count": rng.randint(5, 64), "steps": logint(30, 200), "lo": lo,
                 "hi": max(lo, pow2(128, 512)), "tuned": rng.random() < 0.5, "ragged": rng.random() < 0.5}
        if 2e7 < work(c)["bytes"] <= _MOST:
            return c


# ---------------------------------------------------------------- inputs (from the seed alone)


def _packet(rng, half, spatial):
    """Momentum, start and width of a Gaussian packet that crosses the domain's centre."""
    scale = half / 20.0
    k = rng.uniform(1.0, 4.0) / (scale if scale < 1 else 1.0)
    v = rng.standard_normal(spatial)
    v /= np.linalg.norm(v)
    return {"k0": (k * v).tolist(), "x0": (-0.4 * half * v).tolist(), "width": 2.0 * scale * rng.uniform(0.9, 1.4)}


def _spec2(c, rng):
    metric = c["metric"]
    half = 5.0 if metric == "exp3" else 20.0
    s = {"n1": c["n1"], "n2": c["n2"], "a1": half, "a2": half, "c": 1.0,
         "dt": 1.14e-4 if metric == "exp3" else 0.01, "m": 0.0 if metric == "bump" else 1.0,
         "kind": {"flat": FLAT, "bump": BUMP, "exp3": EXP3}[metric],
         "spin": {"flat": SPIN_NONE, "bump": SPIN_2P1, "exp3": SPIN_PAPER}[metric],
         "A": float(rng.uniform(0.5, 2.0)), "s": float(rng.uniform(2.0, 6.0)),
         "width_pts": min(c["n1"], c["n2"]) // 16 if c.get("layer", True) else 0}
    s.update(_packet(rng, half, 2))
    return s


def _spec3(c, rng):
    exp3 = c["metric"] == "exp3"
    half = 5.0 if exp3 else 10.0
    s = {"n": (c["n1"], c["n2"], c["n3"]), "a": (half,) * 3, "c": 1.0, "m": 1.0, "dt": 1e-3 if exp3 else 0.01,
         "kind": EXP3 if exp3 else FLAT, "spin": SPIN_PAPER if exp3 else SPIN_NONE,
         "width_pts": min(c["n1"], c["n2"], c["n3"]) // 16 if c["layer"] else 0}
    s.update(_packet(rng, half, 3))
    return s


def _grid(n, a, dev):
    return -a + (2.0 * a / n) * torch.arange(n, dtype=torch.float64, device=dev)


def _packet_axis(x, x0, k0, width):
    return torch.exp(torch.complex(-(x - x0) ** 2 / (2.0 * width * width), k0 * x))


def _psi2(s, dev):
    """[n2][n1][2] complex128."""
    fx = _packet_axis(_grid(s["n1"], s["a1"], dev), s["x0"][0], s["k0"][0], s["width"])
    fy = _packet_axis(_grid(s["n2"], s["a2"], dev), s["x0"][1], s["k0"][1], s["width"])
    psi = torch.empty(s["n2"], s["n1"], 2, dtype=torch.complex128, device=dev)
    psi[..., 0] = fy[:, None] * fx[None, :]
    psi[..., 1] = 0.5j * psi[..., 0]
    return psi


def _psi3(s, dev):
    """[n3][n2][n1][4] complex128."""
    f = [_packet_axis(_grid(n, a, dev), x, k, s["width"]) for n, a, x, k in zip(s["n"], s["a"], s["x0"], s["k0"])]
    g = f[2][:, None, None] * f[1][None, :, None] * f[0][None, None, :]
    return torch.stack([g, 0.5 * g, 0.0 * g, 0.2j * g], dim=-1).contiguous()


def _potentials(s):
    """A static scalar potential and a uniform pulsed A_x."""
    x = -s["a1"] + (2.0 * s["a1"] / s["n1"]) * np.arange(s["n1"])
    y = -s["a2"] + (2.0 * s["a2"] / s["n2"]) * np.arange(s["n2"])
    V = 0.5 * np.exp(-(x[None, :] ** 2 + y[:, None] ** 2) / 50.0)
    return {"V": V, "Ax": np.full_like(V, 0.8), "Ay": 0.3 * np.tanh(y / 5.0)[:, None] * np.ones_like(V), "charge": 1.0,
            "env_V": (1.0, 0.0, 0.0, 0.0, 0.0, 0.0), "env_A": (0.0, 1.0, 3.0, 0.0, 1.0, 0.7)}


def _batch_specs(c, seed):
    rng = np.random.default_rng(seed)
    sizes = [n for n in (64, 128, 256, 512) if c["lo"] <= n <= c["hi"]]
    specs, steps = [], []
    for i in range(c["count"]):
        # the sizes in equal shares, whatever the seed, so that every state is the same work
        n = sizes[i % len(sizes)]
        specs.append(_spec2({"n1": n, "n2": n, "metric": "bump"}, rng))
        steps.append(max(1, c["steps"] * (1 + i % 4) // 4) if c["ragged"] else c["steps"])
    return specs, steps


# ---------------------------------------------------------------- state and pass


def _solver2(s, prec, **kw):
    return D.Solver(s["n1"], s["n2"], s["a1"], s["a2"], s["dt"], s["c"], s["m"],
                    D.FP64 if prec == "f64" else D.FP32, s["kind"], s["spin"], s["A"], s["s"],
                    pml_width=s["width_pts"], **kw)


def _host(numel):
    return torch.empty(numel, dtype=torch.float64, pin_memory=True)


def prepare(case, seed):
    dev = torch.device("cuda")
    fam = case["family"]
    rng = np.random.default_rng(seed)
    st = {"family": fam, "steps": case["steps"]}
    if fam in ("solve2", "scheme1"):
        s = _spec2(case, rng)
        form = case.get("form", "plain")
        kw = {}
        if fam == "scheme1":
            kw = {"scheme": D.SCHEME_CN_GMRES, "gmres_restart": 20, "gmres_rtol": 1e-12}
        elif form == "step2bis":
            kw = {"scheme": D.SCHEME_EXP_SPLIT_2BIS}
        elif form == "potentials":
            kw = {"potentials": _potentials(s)}
        prec = case.get("prec", "f64")
        sv = _solver2(s, prec, **kw)
        st.update(solver=sv, psi=_psi2(s, dev), host=_host(4 * s["n1"] * s["n2"]), prec=prec,
                  shape=(s["n2"], s["n1"], 2, 2), obs=fam == "solve2" and form == "plain" and prec == "f64")
        if case.get("tuned"):
            sv.set_initial_spinor_device(st["psi"])
            sv.autotune(50)
    elif fam == "solve3":
        s = _spec3(case, rng)
        sv = D.Solver3(*s["n"], *s["a"], s["dt"], s["c"], s["m"], D.FP64 if case["prec"] == "f64" else D.FP32,
                       s["kind"], s["spin"], pml_width=s["width_pts"])
        st.update(solver=sv, psi=_psi3(s, dev), host=_host(8 * math.prod(s["n"])), prec=case["prec"],
                  shape=s["n"][::-1] + (4, 2))
    else:
        specs, steps = _batch_specs(case, seed)
        b = D.Batch(precision=D.FP32, capacity=case["count"])
        st.update(batch=b, members=[], steps=steps)
        off = 0
        for s in specs:
            sv, psi = _solver2(s, "f32"), _psi2(s, dev)
            sv.set_initial_spinor_device(psi)
            b.add(sv)
            n = 4 * s["n1"] * s["n2"]
            st["members"].append((sv, psi, off, n))
            off += n
        st["host"] = _host(off)
        if case["tuned"]:
            b.autotune(3)
    torch.cuda.synchronize()
    return st


def _fetch(status):
    if status != 0:
        raise D.DiracError(status, D.last_error())


def _host_ptr(t, off=0):
    return ctypes.cast(t.data_ptr() + 8 * off, ctypes.POINTER(ctypes.c_double))


def run(st):
    fam = st["family"]
    if fam == "batch":
        for sv, psi, _, _ in st["members"]:
            sv.set_initial_spinor_device(psi)
        st["batch"].run(st["steps"])
        st["batch"].sync()
        for sv, _, off, _ in st["members"]:
            _fetch(D.lib.dirac_get_spinor(sv.h, _host_ptr(st["host"], off)))
        return st["host"].to(torch.float32)
    sv = st["solver"]
    sv.set_initial_spinor_device(st["psi"])
    sv.step_n(st["steps"])
    get = D.lib.dirac3_get_spinor if fam == "solve3" else D.lib.dirac_get_spinor
    if not st.get("obs"):
        _fetch(get(sv.h, _host_ptr(st["host"])))
        out = st["host"].view(st["shape"])
        return out if st["prec"] == "f64" else out.to(torch.float32)
    o = sv.observables()
    _fetch(get(sv.h, _host_ptr(st["host"])))
    return {"psi": st["host"].view(st["shape"]), "step": o["step"],
            "obs": np.array([o[k] for k in ("norm_l2", "norm_w", "energy_re", "energy_im", "x_mean", "y_mean")])}


# ---------------------------------------------------------------- work


def work(case):
    """Per step a direction pass reads and writes the state once (a line transform needs
    every point of its line, and the next direction's lines cross all of them) and reads
    its per-point tables; per pass the initial spinor is read and the result written.
    Flops: 5 n log2 n per complex transform of length n, plus the pointwise stages."""
    fam = case["family"]
    if fam == "batch":
        specs, steps = _batch_specs(case, 0)
        by = fl = 0.0
        for s, k in zip(specs, steps):
            npts, lg = s["n1"] * s["n2"], math.log2(s["n1"] * s["n2"])
            by += npts * (88.0 * k + 64.0)
            fl += npts * (20.0 * lg + 100.0) * k
        return {"bytes": by, "flops": fl}
    k = case["steps"]
    r = 8.0 if case.get("prec", "f64") == "f64" else 4.0
    if fam == "solve3":
        npts = case["n1"] * case["n2"] * case["n3"]
        tables = 8.0 * r if case["metric"] != "flat" else 0.0          # 5 reals of E, a per direction
        return {"bytes": npts * ((48.0 * r + tables) * k + 128.0),
                "flops": npts * (40.0 * math.log2(npts) + 250.0) * k}
    npts = case["n1"] * case["n2"]
    lg = math.log2(npts)
    if fam == "scheme1":
        # a step is at least: right-hand side, first residual and four Krylov products and
        # their vectors read once each
        return {"bytes": npts * (32.0 * (2 * 3 + 4 * 4 + 6) * k + 64.0), "flops": npts * (20.0 * lg + 60.0) * 6 * k}
    tables = 0.0 if case["metric"] == "flat" else 6.0 * r              # 4 reals of E, a per direction
    if case["form"] == "step2bis":
        tables += 2.0 * r                                             # d a along each direction
    elif case["form"] == "potentials":
        tables = 8.0 * r                                              # six reals of the record, a per direction
    inv = {"step2bis": 4.0}.get(case["form"], 2.0)                     # transforms per direction and component
    return {"bytes": npts * ((16.0 * r + tables) * k + 64.0), "flops": npts * (10.0 * lg * inv + 100.0) * k}


# ---------------------------------------------------------------- 64-bit values in plain torch


def _xi(n, a, dev):
    q = torch.arange(n, dtype=torch.float64, device=dev)
    return torch.where(q < n // 2, q, q - n) * math.pi / a


def _inv_stretch(n, a, width, dev):
    """1/S of the type I layer, sigma0 = 1: S = 1 + (|x| - L*)^2 on the width points next to the seam."""
    k = torch.arange(n, dtype=torch.float64, device=dev)
    dk = torch.minimum(k, n - k)
    sig = ((width - dk) * (2.0 * a / n)) ** 2
    return torch.where(dk <= width, 1.0 / (1.0 + sig), torch.ones_like(sig)) if width > 0 else torch.ones_like(k)


def _cosh_pair(s2):
    """cosh r and sinh r / r of r^2 = s2 (complex)."""
    r = torch.sqrt(s2)
    small = s2.abs() < 1e-4
    rs = torch.where(small, torch.ones_like(r), r)
    C = torch.where(small, 1 + s2 / 2 + s2 ** 2 / 24 + s2 ** 3 / 720 + s2 ** 4 / 40320, torch.cosh(rs))
    D_ = torch.where(small, 1 + s2 / 6 + s2 ** 2 / 120 + s2 ** 3 / 5040 + s2 ** 4 / 362880, torch.sinh(rs) / rs)
    return C, D_


class _Plain2:
    """The 2-D scheme from its definitions; spinors as (psi_0, psi_1) of shape [n2][n1]."""

    def __init__(self, s, dev, form="plain"):
        self.s, self.dev, self.form = s, dev, form
        n1, n2 = s["n1"], s["n2"]
        x, y = _grid(n1, s["a1"], dev)[None, :], _grid(n2, s["a2"], dev)[:, None]
        self.x, self.y = x, y
        z = torch.zeros(n2, n1, dtype=torch.float64, device=dev)
        r2 = x * x + y * y
        phi = px = py = psi = qx = qy = z
        if s["kind"] == BUMP:
            w2 = s["s"] ** 2
            h = s["A"] * torch.exp(-r2 / w2)
            hx, hy = -2 / w2 * h * x, -2 / w2 * h * y
            hxx, hyy = h * (4 * x * x / w2 ** 2 - 2 / w2), h * (4 * y * y / w2 ** 2 - 2 / w2)
            hxy = h * (4 * x * y / w2 ** 2)
            g = hx * hx + hy * hy
            psi = 0.25 * torch.log1p(g)
            qx = 0.5 * (hx * hxx + hy * hxy) / (1 + g)
            qy = 0.5 * (hx * hxy + hy * hyy) / (1 + g)
        elif s["kind"] == EXP3:
            phi, psi = torch.exp(-0.01 * r2), torch.exp(-0.005 * r2)
            px, py = -0.02 * x * phi, -0.02 * y * phi
            qx, qy = -0.01 * x * psi, -0.01 * y * psi
        chi, cx, cy = {SPIN_NONE: (z, z, z), SPIN_PAPER: (phi, px, py),
                       SPIN_2P1: (phi + psi, px + qx, py + qy)}[s["spin"]]
        self.a = torch.exp(phi - psi)
        self.da = (self.a * (px - qx), self.a * (py - qy))
        self.chi = (cx, cy)
        self.V = s["m"] * s["c"] ** 2 * torch.exp(phi)
        self.w = torch.exp(chi - phi + psi)
        self.xi = (_xi(n1, s["a1"], dev)[None, :], _xi(n2, s["a2"], dev)[:, None])
        self.inv_s = (_inv_stretch(n1, s["a1"], s["width_pts"], dev)[None, :],
                      _inv_stretch(n2, s["a2"], s["width_pts"], dev)[:, None])
        self.em = _potentials(s) if form == "potentials" else None
        if self.em:
            self.planes = [torch.from_numpy(np.ascontiguousarray(self.em[k])).to(dev) for k in ("V", "Ax", "Ay")]
        self.E0 = None if self.em else self.exponential(0.0)

    def exponential(self, t):
        s = self.s
        dt, c = s["dt"], s["c"]
        ux = (-(dt / 4) * c * self.a * self.chi[0]).to(torch.complex128)
        uy = (-(dt / 4) * c * self.a * self.chi[1]).to(torch.complex128)
        uz = -0.5j * dt * self.V
        ph = 1.0
        if self.em:
            e = self.em["charge"]
            fV, fA = (c0 + c1 * math.sin(om * t + p) * (math.exp(-((t - t0) / tau) ** 2) if tau > 0 else 1.0)
                      for c0, c1, om, p, t0, tau in (self.em["env_V"], self.em["env_A"]))
            ux = ux + 0.5j * dt * e * c * fA * self.a * self.planes[1]
            uy = uy + 0.5j * dt * e * c * fA * self.a * self.planes[2]
            ph = torch.exp(0.5j * dt * e * fV * self.planes[0])
        C, D_ = _cosh_pair(ux * ux + uy * uy + uz * uz)
        return ph * (C + D_ * uz), ph * D_ * (ux - 1j * uy), ph * D_ * (ux + 1j * uy), ph * (C - D_ * uz)

    @staticmethod
    def mul(E, p):
        return E[0] * p[0] + E[1] * p[1], E[2] * p[0] + E[3] * p[1]

    @staticmethod
    def sigma(d, p):
        return (p[1], p[0]) if d == 0 else (-1j * p[1], 1j * p[0])

    def direction(self, d, p):
        s, xi, dim = self.s, self.xi[d], 1 - d
        b = self.a * self.inv_s[d]
        h = [torch.fft.fft(q, dim=dim) for q in p]
        th = s["c"] * s["dt"] * xi
        g = self.sigma(d, h)
        out = []
        for k in range(2):
            v = torch.fft.ifft(torch.cos(th) * h[k] - 1j * torch.sin(th) * g[k], dim=dim)
            o = b * v + (1 - b) * p[k]
            if self.form == "step2bis":
                hh = 0.5 * (s["c"] * s["dt"]) ** 2
                o = o + hh * (b * (1 - b) * torch.fft.ifft(xi ** 2 * h[k], dim=dim)
                              + b * self.da[d] * self.inv_s[d] * torch.fft.ifft(1j * xi * h[k], dim=dim))
            out.append(o)
        return tuple(out)

    def step(self, n, p):
        E = self.E0 or self.exponential((n + 0.5) * self.s["dt"])
        p = self.mul(E, p)
        for d in range(2):
            p = self.direction(d, p)
        return self.mul(E, p)

    def transport(self, p):
        """A p = c (b_x sigma_x d_x + b_y sigma_y d_y) p."""
        out = [0, 0]
        for d in range(2):
            b = self.s["c"] * self.a * self.inv_s[d]
            g = self.sigma(d, [torch.fft.ifft(1j * self.xi[d] * torch.fft.fft(q, dim=1 - d), dim=1 - d) for q in p])
            out = [o + b * v for o, v in zip(out, g)]
        return out

    def scheme1_step(self, p):
        p = self.mul(self.E0, p)
        h = 0.5 * self.s["dt"]
        rhs = [q - h * v for q, v in zip(p, self.transport(p))]
        x, top, last = rhs, sum(float(q.abs().square().sum()) for q in rhs), math.inf
        for _ in range(400):                       # x <- rhs - (dt/2) A x, to rounding
            y = [r - h * v for r, v in zip(rhs, self.transport(x))]
            off = sum(float((u - v).abs().square().sum()) for u, v in zip(x, y))
            x = y
            if off <= 1e-32 * top or (off >= last and off < 1e-26 * top):
                return self.mul(self.E0, x)
            last = off
        return None

    def observables(self, p):
        dA = (2 * self.s["a1"] / self.s["n1"]) * (2 * self.s["a2"] / self.s["n2"])
        dens = p[0].abs().square() + p[1].abs().square()
        n = dens.sum()
        c = self.s["c"]
        H = [self.V * p[0], -self.V * p[1]]
        for d in range(2):
            g = [torch.fft.ifft(1j * self.xi[d] * torch.fft.fft(q, dim=1 - d), dim=1 - d) + 0.5 * self.chi[d] * q
                 for q in p]
            H = [u - 1j * c * self.a * v for u, v in zip(H, self.sigma(d, g))]
        e = dA * (self.w * (p[0].conj() * H[0] + p[1].conj() * H[1])).sum()
        return np.array([float(dA * n), float(dA * (self.w * dens).sum()), float(e.real), float(e.imag),
                         float((self.x * dens).sum() / n), float((self.y * dens).sum() / n)])


def _exact3(s, steps, dev):
    n, a = s["n"], s["a"]
    shape = lambda d: [1, 1, n[0]] if d == 0 else [1, n[1], 1] if d == 1 else [n[2], 1, 1]  # noqa: E731
    X = [_grid(n[d], a[d], dev).view(shape(d)) for d in range(3)]
    r2 = X[0] ** 2 + X[1] ** 2 + X[2] ** 2
    z = torch.zeros_like(r2)
    phi = torch.exp(-0.01 * r2) if s["kind"] == EXP3 else z
    psi = torch.exp(-0.005 * r2) if s["kind"] == EXP3 else z
    al = torch.exp(phi - psi)
    w = 0.5 * s["dt"] * s["m"] * s["c"] ** 2 * torch.exp(phi)
    g = [-(s["dt"] / 4) * s["c"] * al * (-0.02 * X[d] * phi if s["spin"] == SPIN_PAPER else z) for d in range(3)]
    C, D_ = _cosh_pair((g[0] ** 2 + g[1] ** 2 + g[2] ** 2 - w ** 2).to(torch.complex128))

    def sig(d, p):
        return ((p[1], p[0]), (-1j * p[1], 1j * p[0]), (p[0], -p[1]))[d]

    def half(p):
        up, lo = p[:2], p[2:]
        gs = lambda q: [sum(g[d] * sig(d, q)[k] for d in range(3)) for k in range(2)]  # noqa: E731
        gu, gl = gs(lo), gs(up)
        return [C * up[k] + D_ * (-1j * w * up[k] + gu[k]) for k in range(2)] + \
               [C * lo[k] + D_ * (1j * w * lo[k] + gl[k]) for k in range(2)]

    psi0 = _psi3(s, dev)
    p = [psi0[..., k].contiguous() for k in range(4)]
    del psi0
    for _ in range(steps):
        p = half(p)
        for d in range(3):
            dim = 2 - d
            th = s["c"] * s["dt"] * _xi(n[d], a[d], dev).view(shape(d))
            b = al * _inv_stretch(n[d], a[d], s["width_pts"], dev).view(shape(d))
            h = [torch.fft.fft(q, dim=dim) for q in p]
            m = list(sig(d, h[2:])) + list(sig(d, h[:2]))
            p = [b * torch.fft.ifft(torch.cos(th) * u - 1j * torch.sin(th) * v, dim=dim) + (1 - b) * q
                 for u, v, q in zip(h, m, p)]
        p = half(p)
    return torch.view_as_real(torch.stack(p, dim=-1))


def exact(case, seed):
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    fam, rng = case["family"], np.random.default_rng(seed)
    if fam == "solve3":
        return _exact3(_spec3(case, rng), case["steps"], dev)
    form = case.get("form", "plain")
    specs, steps = _batch_specs(case, seed) if fam == "batch" else ([_spec2(case, rng)], [case["steps"]])
    outs = []
    for s, k in zip(specs, steps):
        m = _Plain2(s, dev, form)
        psi = _psi2(s, dev)
        p = (psi[..., 0].contiguous(), psi[..., 1].contiguous())
        for n in range(k):
            p = m.scheme1_step(p) if fam == "scheme1" else m.step(n, p)
            if p is None:
                return None
        outs.append(torch.view_as_real(torch.stack(p, dim=-1)))
    if fam == "batch":
        return torch.cat([o.reshape(-1) for o in outs])
    if fam == "solve2" and form == "plain" and case["prec"] == "f64":
        return {"psi": outs[0], "step": None, "obs": m.observables(p)}
    return outs[0]
