"""Performance cases of the library: what its users run, from the smallest box to the largest.

Each kind of case is one thing a program does with the library:

  run        a segment of a stratified Taylor-Green run: (optionally) resume from a
             checkpoint, advance k steps with diagnostic records, drain the records and
             read the populations back (the next checkpoint)
  learned    the same with the network attached (64^3 to 256^3 boxes)
  train      one training step of the network: gradient over a batch, Adam, packing
  infer      the network on a batch of feature rows
  normalise  the normalisation of a training set
  snapshot   one teacher snapshot: restrict, four fine steps, restrict, the coarse step,
             training pairs
  spectrum   the kinetic-energy spectrum of the current state
  monitor    a record and the fields of the current state, as a run's monitor asks for them

Initial states are Taylor-Green equilibria with seeded perturbations of the density
anomaly and (`rough` > 0) of the velocity and the non-equilibrium populations, at the
sizes a developed flow has.  `exact` restates the method in FP64 (torch only).
"""
import itertools
import math
import os

import numpy as np
import torch

from paper_2605_14505_amd import learned, stgv

DEV = "cuda:0" if torch.cuda.is_available() else "cpu"
ELEM = {"fp32": 4, "fp16": 2, "bf16": 2}
DTYPE = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}
PAIRS = ((27, 19), (27, 7), (19, 7), (27, 27), (19, 19), (19, 15), (15, 7), (7, 27))
U0, SC, G_OVER_N = 0.05, 0.7, 0.02


def _run(n, steps, name=None, q_f=27, q_g=19, forcing="shift", storage="fp32", compute="fp32", layout="aa",
         diag_every=16, fr=1.0):
    c = dict(kind="run", n=n, steps=steps, q_f=q_f, q_g=q_g, forcing=forcing, storage=storage,
             compute=compute, layout=layout, diag_every=diag_every, fr=fr, rough=0.0)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the parity-size box: launches and latency, not bytes
        _run(32, 64, "run_32_guo", forcing="guo"),
        # the coarse run of the learned form, plain step; fits the last-level cache
        _run(64, 64, "run_64"),
        # a ragged box (rows not a multiple of the wavefront) on the smaller scalar lattice, FP16
        _run(90, 32, "run_90_fp16_27x7", q_g=7, storage="fp16"),
        # the 128^3 velocity-shift run at Fr 0.5, BF16 storage
        _run(128, 32, "run_128_bf16", storage="bf16", fr=0.5),
        # the headline: 256^3 D3Q27xD3Q19, FP32, a record every 16 steps
        _run(256, 32, "run_256"),
        # the largest regular run: 512^3 with FP16 populations
        _run(512, 8, "run_512_fp16", storage="fp16", fr=0.5, diag_every=100),
        # the deployed learned run at its coarse grid
        dict(name="learned_64", kind="learned", n=64, steps=32, forcing="shift", diag_every=16, fr=0.6, gain=0.1),
        # a training step at the trainer's batch
        dict(name="train_16384", kind="train", batch=16384, rows=262144),
        # network output for every node of a 64^3 grid
        dict(name="infer_64cubed", kind="infer", rows=262144),
        # normalisation over four 64^3 snapshots
        dict(name="normalise_4_snapshots", kind="normalise", rows=1048576),
        # a 256^3 -> 64^3 teacher snapshot
        dict(name="snapshot_256", kind="snapshot", n=256, forcing="shift", fr=0.6, rough=5e-3),
        # the spectrum of the headline box
        dict(name="spectrum_256", kind="spectrum", n=256, storage="fp32", rough=5e-3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _segment(n):
    """Even number of steps of one segment: more on small boxes."""
    return 64 if n <= 64 else (32 if n <= 128 else 8)


def draw(rng):
    """One more case of the listed ranges."""
    kind = rng.choice(("run", "run", "run", "run", "learned", "train", "infer", "normalise", "snapshot",
                       "spectrum", "monitor"))
    forcing = rng.choice(("shift", "shift", "guo", "edm", "hcz"))
    fr = rng.choice((0.3, 0.5, 0.6, 1.0, 3.0))
    if kind == "run":
        n = _log_int(rng, 8, 320)
        if rng.random() < 0.4:
            n = max(32, n // 32 * 32)
        q_f, q_g = rng.choice(((27, 19),) * 5 + PAIRS)
        storage = rng.choice(("fp32", "fp32", "fp16", "bf16"))
        compute = "fp64" if storage == "fp32" and rng.random() < 0.15 else "fp32"
        return _run(n, _segment(n), q_f=q_f, q_g=q_g, forcing=forcing, storage=storage, compute=compute,
                    layout="ab" if rng.random() < 0.15 else "aa", diag_every=rng.choice((0, 4, 16)), fr=fr)
    if kind == "learned":
        n = rng.choice((64, 64, 128, 192))
        return dict(kind=kind, n=n, steps=rng.choice((8, 16, 24, 32)), forcing=rng.choice(("shift", "guo")),
                    diag_every=rng.choice((0, 4, 16)), fr=fr, gain=rng.choice((0.05, 0.1)))
    if kind == "train":
        return dict(kind=kind, batch=_log_int(rng, 64, 65536), rows=_log_int(rng, 20000, 300000))
    if kind == "infer":
        return dict(kind=kind, rows=_log_int(rng, 64, 1000000))
    if kind == "normalise":
        return dict(kind=kind, rows=_log_int(rng, 500, 1500000))
    if kind == "snapshot":
        return dict(kind=kind, n=4 * _log_int(rng, 8, 64), forcing=rng.choice(("shift", "guo")), fr=fr, rough=5e-3)
    n = _log_int(rng, 12, 256)
    if rng.random() < 0.4:
        n = max(16, n // 16 * 16)
    storage = rng.choice(("fp32", "fp32", "fp16", "bf16"))
    if kind == "spectrum":
        return dict(kind=kind, n=n, storage=storage, rough=5e-3)
    return dict(kind=kind, n=n, storage=storage, fr=fr, rough=5e-3)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _physics(c):
    # Re grows with the box, so that the relaxation times are those of the 256^3 run
    return dict(n=c["n"], forcing=c.get("forcing", "shift"), u0=U0, re=6.25 * c["n"], fr=c.get("fr", 1.0), sc=SC,
                g_over_n=G_OVER_N, noise_amp=0.0, seed=0)


def _simulation(c):
    return stgv.Simulation(device=DEV, q_f=c.get("q_f", 27), q_g=c.get("q_g", 19), storage=c.get("storage", "fp32"),
                           compute=c.get("compute", "fp32"), layout=c.get("layout", "aa"),
                           diag_every=c.get("diag_every", 0), **_physics(c))


def _lattice(q):
    """Velocities in the library's order (rest, faces, edges, corners, opposite pairs), weights, c_s^2."""
    e, w, cs2 = stgv.lbm_stencil_info(q)
    return e, w, cs2


def _patches(n, gen):
    """Seeded standard-normal values constant on blocks of 8^3 nodes: [z, y, x]."""
    m = (n + 7) // 8
    r = torch.randn((m, m, m), generator=gen, dtype=torch.float32, device=DEV)
    for axis in range(3):
        r = r.repeat_interleave(8, dim=axis)
    return r[:n, :n, :n]


def _state(c, seed):
    """Natural-order FP32 deviations (q, n, n, n) of a perturbed Taylor-Green equilibrium."""
    n, rough = c["n"], c.get("rough", 0.0)
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    h = 2.0 * math.pi / n * torch.arange(n, dtype=torch.float32, device=DEV)
    x, y, z = h[None, None, :], h[None, :, None], h[:, None, None]
    u = [U0 * torch.sin(x) * torch.cos(y) * torch.cos(z), -U0 * torch.cos(x) * torch.sin(y) * torch.cos(z),
         torch.zeros((n, n, n), dtype=torch.float32, device=DEV)]
    if rough:
        u = [v + 20.0 * rough * U0 * _patches(n, gen) for v in u]
    (ef, wf, cf), (eg, wg, cg) = _lattice(c.get("q_f", 27)), _lattice(c.get("q_g", 19))
    drho = U0 * U0 / 16.0 * (torch.cos(2 * x) + torch.cos(2 * y)) * (torch.cos(2 * z) + 2.0) / cf
    rho_p = (10.0 * rough + 1e-3) * _patches(n, gen)
    usq = sum(v * v for v in u)
    out = torch.empty((len(ef) + len(eg), n, n, n), dtype=torch.float32, device=DEV)
    k = 0
    for es, ws, cs2, first, scale in ((ef, wf, cf, drho, 1.0 + drho), (eg, wg, cg, rho_p, 1.0 + rho_p)):
        for e, w in zip(es, ws):
            eu = sum(s * v for s, v in zip(e, u))
            out[k] = w * (first + scale * (eu / cs2 + eu * eu / (2 * cs2 * cs2) - usq / (2 * cs2)))
            if rough:
                out[k] += w * rough * _patches(n, gen)
            k += 1
    return out


def _feature_scales():
    with np.load(os.path.join(os.path.dirname(os.path.abspath(stgv.__file__)), "data", "learned64.npz"),
                 allow_pickle=False) as f:
        return f["theta"].astype(np.float32), f["norm"].astype(np.float32)


def _rows(rows, seed):
    """Feature rows [rows][47] and target rows [rows][41] with the trained columns' means and spreads."""
    _, norm = _feature_scales()
    norm = torch.tensor(norm, device=DEV)
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    iscale = norm[47:94]
    std = torch.where(iscale > 0, 1.0 / iscale.clamp_min(1e-30), torch.zeros_like(iscale))
    x = torch.randn((rows, 47), generator=gen, device=DEV) * std + norm[:47]
    y = torch.randn((rows, 41), generator=gen, device=DEV) * norm[94:]
    return x, y


def _network(gain=1.0, seed=None):
    """The shipped network with its correction scaled by `gain`, or with seeded changes of its weights."""
    theta, norm = _feature_scales()
    norm = norm.copy()
    norm[94:] *= gain
    if seed is not None:
        theta = theta + 0.02 * np.random.default_rng(seed).standard_normal(theta.size).astype(np.float32)
    return learned.Network(theta, norm, device=DEV)


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"case": c}
    if kind in ("run", "learned"):
        s["start"] = _state(c, seed)
        s["sim"] = _simulation(c)
        s["sim"].load(s["start"], step=0)
        if kind == "learned":
            s["net"] = _network(c["gain"])
            s["sim"].set_mlp(s["net"].packed)
        if c["n"] >= 256:          # a long run goes on from where it is
            s["start"] = None
    elif kind == "train":
        s["net"] = _network(seed=seed)
        s["x"], s["y"] = _rows(c["rows"], seed)
        gen = torch.Generator(device=DEV).manual_seed(int(seed) + 1)
        s["idx"] = torch.randint(0, c["rows"], (c["batch"],), generator=gen, dtype=torch.int64, device=DEV)
        s["grad"] = torch.empty(stgv.MLP_PARAMS, dtype=torch.float32, device=DEV)
        s["loss"] = torch.empty(1, dtype=torch.float64, device=DEV)
        s["work"] = torch.empty(stgv.lbm_mlp_grad_work_bytes(c["batch"]), dtype=torch.uint8, device=DEV)
    elif kind == "infer":
        s["net"] = _network(seed=seed)
        s["x"], _ = _rows(c["rows"], seed)
        s["y"] = torch.empty((c["rows"], 41), dtype=torch.float32, device=DEV)
    elif kind == "normalise":
        s["x"], s["y"] = _rows(c["rows"], seed)
        s["norm"] = torch.empty(stgv.MLP_NORM, dtype=torch.float32, device=DEV)
        s["work"] = torch.empty(stgv.lbm_mlp_norm_work_bytes(), dtype=torch.uint8, device=DEV)
    elif kind == "snapshot":
        s["fine"] = _simulation(c)
        s["fine"].load(_state(c, seed), step=0)
        s["coarse"] = _simulation(dict(c, n=c["n"] // 4))
        n3 = (c["n"] // 4) ** 3
        s["x"] = torch.empty((n3, 47), dtype=torch.float32, device=DEV)
        s["y"] = torch.empty((n3, 41), dtype=torch.float32, device=DEV)
    else:
        s["sim"] = _simulation(c)
        s["sim"].load(_state(c, seed), step=0)
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
RECORD = ("ek", "ep", "eps_k", "eps_p", "umax")


def _records(recs):
    out = {k: np.array([r[k] for r in recs]) for k in RECORD}
    out["budget"] = np.array([[r["mass"], r["scalar"], *r["mom"]] for r in recs])
    return out


def run(state):
    s, kind = state, state["case"]["kind"]
    if kind in ("run", "learned"):
        sim = s["sim"]
        if s["start"] is not None:
            sim.load(s["start"], step=0)
        sim.step(s["case"]["steps"])
        return {"records": _records(sim.diagnostics()), "populations": sim.populations()}
    if kind == "train":
        net, stream = s["net"], torch.cuda.current_stream().cuda_stream
        stgv.lbm_mlp_grad(net.packed, s["x"], s["y"], s["idx"], s["case"]["batch"], s["grad"], s["loss"], s["work"],
                          stream)
        net.t += 1
        stgv.lbm_mlp_adam(net.theta, net.m, net.v, s["grad"], net.t, 2e-4, stream)
        net.pack()
        return {"grad": s["grad"], "loss": s["loss"], "theta": net.theta, "m": net.m, "v": net.v}
    if kind == "infer":
        stgv.lbm_mlp_forward(s["net"].packed, s["x"], s["case"]["rows"], s["y"],
                             torch.cuda.current_stream().cuda_stream)
        return s["y"]
    if kind == "normalise":
        stgv.lbm_mlp_norm(s["x"], s["y"], s["case"]["rows"], s["norm"], s["work"],
                          torch.cuda.current_stream().cuda_stream)
        return {"mean": s["norm"][:47], "iscale": s["norm"][47:94], "y_scale": s["norm"][94:]}
    if kind == "snapshot":
        fine, coarse = s["fine"], s["coarse"]
        a = fine.restrict_to(coarse)
        fine.step(4)
        b = fine.restrict_to(coarse)
        coarse.load(a, step=0)
        coarse.step(1)
        c = coarse.populations()
        stgv.lbm_training_pairs(coarse.ctx, a, b, c, s["x"], s["y"])
        return {"a": a, "b": b, "c": c, "x": s["x"], "y": s["y"]}
    if kind == "spectrum":
        return s["sim"].spectrum()
    s["sim"].sample()
    return {"records": _records(s["sim"].diagnostics()), "fields": s["sim"].fields()}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
NETWORK_FLOPS = 2 * (47 * 64 + 64 * 64 + 64 * 41)


def work(case):
    c, kind = case, case["kind"]
    if kind in ("train", "infer", "normalise"):
        if kind == "train":
            return {"bytes": c["batch"] * (88 * 4 + 8) + 8 * 4 * stgv.MLP_PARAMS,
                    "flops": 3 * NETWORK_FLOPS * c["batch"]}
        if kind == "infer":
            return {"bytes": c["rows"] * 88 * 4 + 4 * stgv.MLP_PARAMS, "flops": NETWORK_FLOPS * c["rows"]}
        return {"bytes": c["rows"] * 88 * 4, "flops": c["rows"] * (3 * 47 + 2 * 41)}
    q, n3, b = c.get("q_f", 27) + c.get("q_g", 19), c["n"] ** 3, ELEM[c.get("storage", "fp32")]
    node_flops = 16 * q                                  # moments, equilibria and relaxation of q populations
    if kind in ("run", "learned"):
        records = len(range(0, c["steps"], c["diag_every"])) if c["diag_every"] else 0
        moved = c["steps"] * 2 * q * b + q * (b + 4) + records * 32
        flops = c["steps"] * node_flops
        if c["n"] < 256:
            moved += q * (b + 4)
        if kind == "learned":
            flops += c["steps"] * NETWORK_FLOPS
        return {"bytes": n3 * moved, "flops": n3 * flops}
    if kind == "snapshot":
        coarse = n3 // 64
        return {"bytes": n3 * 4 * q * (2 + 2 * 4) + coarse * 4 * (q * (2 + 2 + 2 + 2 + 3) + 88),
                "flops": n3 * node_flops * 6 + coarse * (node_flops + 4 * (47 * 46 + 46 * 46))}
    if kind == "spectrum":
        return {"bytes": n3 * q * b, "flops": 3 * 2.5 * n3 * math.log2(n3) + 2 * q * n3}
    return {"bytes": n3 * (2 * q * b + 20), "flops": n3 * (4 * q + 40)}


# ---------------------------------------------------------------------------
# the method in FP64
# ---------------------------------------------------------------------------
class _Model:
    """Populations as FP64 deviations from the weights, (q, n, n, n), stepped in place."""

    def __init__(self, c, dev64):
        self.c, self.n = c, c["n"]
        (self.ef, self.wf, self.cf), (self.eg, self.wg, self.cg) = _lattice(c.get("q_f", 27)), _lattice(c.get("q_g", 19))
        p = _physics(c)
        self.length = self.n / (2.0 * math.pi)
        self.nu = U0 * self.length / p["re"]
        self.diff = self.nu / SC
        self.tau_f, self.tau_g = self.nu / self.cf + 0.5, self.diff / self.cg + 0.5
        nb = U0 / (p["fr"] * self.length)
        self.gravity, self.beta = G_OVER_N * nb, -nb * nb / (G_OVER_N * nb)
        self.forcing = p["forcing"]
        self.d = dev64

    def f(self):
        return self.d[:len(self.ef)]

    def g(self):
        return self.d[len(self.ef):]

    def macro(self):
        f, g = self.f(), self.g()
        self.drho, self.sig = f.sum(0), g.sum(0)
        self.rho = 1.0 + self.drho
        self.j = [sum(e[k] * f[i] for i, e in enumerate(self.ef) if e[k]) for k in range(3)]
        up = [j / self.rho for j in self.j]
        self.s = -self.beta * up[2]
        self.rho_p = self.sig + 0.5 * self.s
        self.force = -self.gravity * self.rho_p
        self.u = [up[0], up[1], up[2] + 0.5 * self.force / self.rho]
        if self.forcing == "shift":
            self.ueq = [up[0], up[1], up[2] + self.tau_f * self.force / self.rho]
        else:
            self.ueq = up if self.forcing == "edm" else self.u
        self.uth = self.ueq if self.forcing == "shift" else self.u

    @staticmethod
    def poly1(e, u, cs2):
        """e.u/c^2 + (e.u)^2/(2 c^4) - u^2/(2 c^2)."""
        eu = sum(k * v for k, v in zip(e, u) if k) if any(e) else 0.0
        return eu / cs2 + eu * eu / (2 * cs2 * cs2) - sum(v * v for v in u) / (2 * cs2)

    def feq(self, i, u):
        return self.wf[i] * (self.drho + self.rho * self.poly1(self.ef[i], u, self.cf))

    def geq(self, j, u):
        return self.wg[j] * (self.rho_p + (1.0 + self.rho_p) * self.poly1(self.eg[j], u, self.cg))

    def collide(self, extra=None):
        self.macro()
        f, g, c2 = self.f(), self.g(), self.cf
        for i, (e, w) in enumerate(zip(self.ef, self.wf)):
            eq = self.feq(i, self.ueq)
            new = f[i] - (f[i] - eq) / self.tau_f
            if self.forcing in ("guo", "hcz"):
                half = (1.0 - 0.5 / self.tau_f) * self.force
                if self.forcing == "guo":
                    eu = sum(k * v for k, v in zip(e, self.u))
                    new += half * w * ((e[2] - self.u[2]) / c2 + eu * e[2] / (c2 * c2))
                else:
                    new += half * (e[2] - self.u[2]) / (self.rho * c2) * (w + eq)
            elif self.forcing == "edm":
                up = self.ueq
                new += self.feq(i, [up[0], up[1], up[2] + self.force / self.rho]) - eq
            f[i] = new
        for j, w in enumerate(self.wg):
            eq = self.geq(j, self.uth)
            g[j] = g[j] - (g[j] - eq) / self.tau_g + (1.0 - 0.5 / self.tau_g) * w * self.s
        if extra is not None:
            self.d += extra

    def stream(self):
        for k, e in enumerate([*self.ef, *self.eg]):
            if any(e):
                self.d[k] = torch.roll(self.d[k], (e[2], e[1], e[0]), (0, 1, 2))

    def record(self):
        """Energies, dissipation rates and budgets of the current state, in the paper's units."""
        self.macro()
        n3 = self.n ** 3

        def diff(a, axis):
            return 0.5 * (torch.roll(a, -1, axis) - torch.roll(a, 1, axis))
        u, x, y, z = self.u, 2, 1, 0
        curl = [diff(u[2], y) - diff(u[1], z), diff(u[0], z) - diff(u[2], x), diff(u[1], x) - diff(u[0], y)]
        grad = sum(diff(self.rho_p, a).square().sum() for a in (x, y, z))
        usq = sum(v * v for v in u)
        e_scale, eps_scale = 1.0 / (n3 * U0 * U0), self.length / (n3 * U0 ** 3)
        mom = [self.j[0].sum(), self.j[1].sum(), (self.j[2] + 0.5 * self.force).sum()]
        return dict(ek=0.5 * float(usq.sum()) * e_scale,
                    ep=0.5 * float((G_OVER_N * self.rho_p).square().sum()) * e_scale,
                    eps_k=self.nu * float(sum(w.square().sum() for w in curl)) * eps_scale,
                    eps_p=self.diff * G_OVER_N ** 2 * float(grad) * eps_scale,
                    umax=math.sqrt(float(usq.max())), mass=n3 + float(self.drho.sum()),
                    scalar=n3 + float(self.sig.sum()), mom=[float(m) for m in mom])

    def advance(self, steps, diag_every, extra=None):
        recs = []
        for k in range(steps):
            if diag_every and k % diag_every == 0:
                recs.append(self.record())
            self.collide(extra() if extra else None)
            self.stream()
        return recs


def _moments(q):
    """Monomial moments of D3Q27 or D3Q19, conserved slots first, and the inverse matrix."""
    every = list(itertools.product(range(3), repeat=3))
    keep = every if q == 27 else [t for t in every if min(t) == 0]
    head = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1)] if q == 27 else [(0, 0, 0)]
    e = np.array(_lattice(q)[0], dtype=np.float64)
    m = np.stack([e[:, 0] ** a * e[:, 1] ** b * e[:, 2] ** c for a, b, c in head + [t for t in keep if t not in head]])
    return (torch.tensor(m, dtype=torch.float64, device=DEV),
            torch.tensor(np.linalg.inv(m), dtype=torch.float64, device=DEV), len(head))


def _features(m):
    """(47, nodes) non-equilibrium moments of a _Model whose macro() is current, and rho'."""
    mf, mg = _moments(27)[0], _moments(19)[0]
    nf = torch.stack([m.f()[i] - m.feq(i, m.ueq) for i in range(27)]).reshape(27, -1)
    ng = torch.stack([m.g()[j] - m.geq(j, m.uth) for j in range(19)]).reshape(19, -1)
    x = torch.cat([mf @ nf, mg @ ng, m.rho_p.reshape(1, -1)])
    x[:3] = 0.0
    x[3] = (m.j[2] - m.rho * m.ueq[2]).reshape(-1)
    x[27] = (m.sig - m.rho_p).reshape(-1)
    return x


def _layers(theta):
    t = torch.as_tensor(theta, device=DEV).double()
    sizes = ((64, 47), (64,), (64, 64), (64,), (41, 64), (41,))
    return [p.reshape(s) for p, s in zip(t.split([math.prod(s) for s in sizes]), sizes)]


def _forward(theta, xn):
    w1, b1, w2, b2, w3, b3 = _layers(theta)
    h1 = torch.tanh(xn @ w1.T + b1)
    h2 = torch.tanh(h1 @ w2.T + b2)
    return h2 @ w3.T + b3, h1, h2


def _split_norm(norm):
    v = torch.as_tensor(norm, device=DEV).double()
    return v[:47], v[47:94], v[94:]


def _restricted(m, coarse):
    """The fine state of a _Model on the coarse grid: (46, nc, nc, nc)."""
    m.macro()

    def filtered(a):
        for axis in (0, 1, 2):
            a = sum(w * torch.roll(a, -k, axis) for k, w in zip(range(-2, 3), (0.125, 0.25, 0.25, 0.25, 0.125)))
        return a[::4, ::4, ::4]
    out = []
    for pops, eq, tau_f, tau_c, q in ((m.f(), m.feq, m.tau_f, coarse.tau_f, 27), (m.g(), m.geq, m.tau_g, coarse.tau_g, 19)):
        kept = torch.stack([filtered(p) for p in pops]).reshape(q, -1)
        rest = torch.stack([filtered(p - eq(i, m.u)) for i, p in enumerate(pops)]).reshape(q, -1)
        mat, inv, head = _moments(q)
        mom = mat @ rest
        mom[:head] = 0.0
        out.append(kept + (4.0 * tau_c / tau_f - 1.0) * (inv @ mom))
    nc = coarse.n
    return torch.cat(out).reshape(46, nc, nc, nc)


def _exact_snapshot(c, seed):
    fine = _Model(c, _state(c, seed).double())
    cc = dict(c, n=c["n"] // 4)
    coarse = _Model(cc, None)
    a = _restricted(fine, coarse)
    fine.advance(4, 0)
    b = _restricted(fine, coarse)
    coarse.d = a.clone()
    coarse.macro()
    x = _features(coarse)
    coarse.advance(1, 0)
    back = torch.stack([torch.roll(r, (-e[2], -e[1], -e[0]), (0, 1, 2))
                        for r, e in zip(b - coarse.d, [*coarse.ef, *coarse.eg])]).reshape(46, -1)
    (mf, _, hf), (mg, _, hg) = _moments(27), _moments(19)
    y = torch.cat([(mf @ back[:27])[hf:], (mg @ back[27:])[hg:]])
    return {"a": a, "b": b, "c": coarse.d, "x": x.T, "y": y.T}


def _exact_spectrum(c, seed):
    n = c["n"]
    m = _Model(c, _state(c, seed).to(DTYPE[c["storage"]]).double())
    m.macro()
    k = torch.fft.fftfreq(n, d=1.0 / n, device=DEV, dtype=torch.float64)
    shell = torch.floor(torch.sqrt(k[:, None, None] ** 2 + k[None, :, None] ** 2 + k[None, None, :] ** 2) + 0.5)
    shell = shell.long().reshape(-1)
    out = torch.zeros(int(math.floor(math.sqrt(3.0) * n / 2.0 + 0.5)) + 1, dtype=torch.float64, device=DEV)
    for v in m.u:
        power = (torch.fft.fftn(v / U0) / n ** 3).abs().square().reshape(-1)
        out.index_add_(0, shell, 0.5 * power)
    return out


def _exact_train(c, seed):
    net = _network(seed=seed)
    theta = net.theta.double()
    mean, iscale, scale = _split_norm(net.norm)
    x, y = _rows(c["rows"], seed)
    gen = torch.Generator(device=DEV).manual_seed(int(seed) + 1)
    idx = torch.randint(0, c["rows"], (c["batch"],), generator=gen, dtype=torch.int64, device=DEV)
    xn, yn = (x[idx].double() - mean) * iscale, y[idx].double() / scale
    o, h1, h2 = _forward(theta, xn)
    _, _, w2, _, w3, _ = _layers(theta)
    r = o - yn
    do = 2.0 * r / r.numel()
    d2 = (do @ w3) * (1.0 - h2 * h2)
    d1 = (d2 @ w2) * (1.0 - h1 * h1)
    grad = torch.cat([p.reshape(-1) for p in (d1.T @ xn, d1.sum(0), d2.T @ h1, d2.sum(0), do.T @ h2, do.sum(0))])
    m, v = 0.1 * grad, 0.001 * grad * grad
    theta = theta - 2e-4 * (m / 0.1) / (torch.sqrt(v / 0.001) + 1e-8)
    return {"grad": grad, "loss": r.square().mean().reshape(1), "theta": theta, "m": m, "v": v}


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("run", "learned"):
        m = _Model(c, _state(c, seed).to(DTYPE[c.get("storage", "fp32")]).double())
        extra = None
        if kind == "learned":
            net = _network(c["gain"])
            mean, iscale, scale = _split_norm(net.norm)
            (_, inv_f, hf), (_, inv_g, hg) = _moments(27), _moments(19)

            def extra():
                m.macro()
                dm = (_forward(net.theta, (_features(m).T - mean) * iscale)[0] * scale).T
                return torch.cat([inv_f[:, hf:] @ dm[:27 - hf], inv_g[:, hg:] @ dm[27 - hf:]]).reshape(m.d.shape)
        recs = m.advance(c["steps"], c["diag_every"], extra)
        return {"records": _records(recs), "populations": m.d}
    if kind == "train":
        return _exact_train(c, seed)
    if kind == "infer":
        net = _network(seed=seed)
        mean, iscale, scale = _split_norm(net.norm)
        return _forward(net.theta, (_rows(c["rows"], seed)[0].double() - mean) * iscale)[0] * scale
    if kind == "normalise":
        x, y = (a.double() for a in _rows(c["rows"], seed))
        std = x.std(0, unbiased=False)
        flat = (x == x[0]).all(0)
        return {"mean": x.mean(0), "iscale": torch.where(flat, torch.zeros_like(std), 1.0 / std),
                "y_scale": y.square().mean(0).sqrt()}
    if kind == "snapshot":
        return _exact_snapshot(c, seed)
    if kind == "spectrum":
        return _exact_spectrum(c, seed)
    m = _Model(c, _state(c, seed).to(DTYPE[c["storage"]]).double())
    rec = m.record()
    return {"records": _records([rec]), "fields": torch.stack([m.drho, *m.u, m.rho_p])}
