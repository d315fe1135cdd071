"""The dose engine's performance workloads.

Each case is one call that a program of this framework makes: the dose of one
field or of a whole VMAT plan (forward), a plan-optimisation step (forward and
the adjoint, through autograd), the learned large-kernel correction, one training
step of its network, and the assessment of a plan's dose.

    listed()            the named cases
    draw(rng)           another case of the same ranges
    prepare(case, seed) inputs on the GPU and the engine a program keeps
    run(state)          one pass; its outputs
    work(case)          bytes and operations no implementation can do without
    exact(case, seed)   the outputs in 64 bits from plain torch
"""
from __future__ import annotations

import math
import os

import numpy as np
import torch

import paper_2512_18863_amd
from paper_2512_18863_amd import engine as E
from paper_2512_18863_amd import inputs, learned, plan_eval

WEIGHTS = os.path.join(os.path.dirname(paper_2512_18863_amd.__file__), "data", "learned_c4.npz")

PLAN = dict(kind="plan", direction="step", nx=128, ny=128, nz=128, spacing=3.0, phantom="pelvis", n_cp=180,
            two_arcs=True, taps=61, jaw_x=40.0, jaw_y=40.0, limit=40.0, n_leaf=60, leaf_width=5.0, conv="fp32",
            cache="", project=False, corrections=False, collimator=False, central_axis=False, noalloc=False)


def _plan(name, **kw):
    return dict(PLAN, name=name, **kw)


def listed():
    return [
        # One static open field on a water phantom: the smallest call, where launches and latency count.
        _plan("static_field_forward", direction="forward", nx=32, ny=32, nz=32, spacing=5.0, phantom="water", n_cp=1,
              two_arcs=False, taps=7, jaw_x=50.0, jaw_y=50.0, limit=50.0, n_leaf=40, leaf_width=10.0),
        # The output calibration's field: one control point on a fine 30 cm water cube of odd size with the
        # full kernel.
        _plan("calibration_field_forward", direction="forward", nx=151, ny=151, nz=151, spacing=2.0, phantom="water",
              n_cp=1, two_arcs=False, jaw_x=50.0, jaw_y=50.0, limit=50.0),
        # A single-arc plan with a narrow kernel: an early stage of coarse-to-fine optimisation.
        _plan("arc_narrow_kernel_step", nz=96, n_cp=90, two_arcs=False, taps=15),
        # The optimisation loop: projection to machine limits, then forward and adjoint on the plan's FP32
        # geometry cache (two arcs, 31 x 31 kernel).
        _plan("optimise_cached_step", nx=192, ny=192, spacing=2.5, taps=31, limit=50.0, cache="fp32", project=True),
        # The dose of a finished plan with the full 61 x 61 kernel: forward only.
        _plan("plan_forward", direction="forward"),
        # The same plan's optimisation step in FP32 and with the BF16 convolution.
        _plan("plan_step"),
        _plan("plan_step_bf16", conv="bf16"),
        # The published timing shape: 105 x 224 x 224, 180 control points, kernel 55.
        _plan("fine_grid_step", nx=224, ny=224, nz=105, spacing=2.0, taps=55),
        # Source penumbra, head scatter, off-axis factor and collimator rotation on: what a commissioned
        # machine model asks for.
        _plan("corrected_collimator_step", n_cp=90, two_arcs=False, corrections=True, collimator=True),
        # The learned 9 x 9 -> 61 x 61 correction in an optimisation step.
        dict(_plan("learned_step", taps=61), kind="learned"),
        # One training step of the correction's network (forward, loss, all gradients).
        dict(name="network_training_step", kind="train", nx=128, ny=128, nz=128, quantile=0.0),
        # A plan's assessment: objective with gradient, DVH report and Dice of six structures.
        dict(name="plan_assessment", kind="assess", nx=192, ny=192, nz=128, spacing=2.5, n_struct=6, bin_width=0.01),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_plan(rng, kind="plan"):
    c = dict(PLAN, kind=kind)
    c["spacing"] = rng.choice([2.0, 2.5, 3.0, 4.0, 5.0, round(rng.uniform(2.0, 5.0), 2)])
    c["nx"], c["ny"] = (int(_log_uniform(rng, 32, 225)) for _ in range(2))
    c["nz"] = int(_log_uniform(rng, 16, 160))
    if kind == "learned":
        c["nx"], c["ny"], c["nz"] = (4 * rng.randint(14, 32) for _ in range(3))
        c["spacing"] = 3.0
    c["n_cp"] = max(1, int(_log_uniform(rng, 1, 181)))
    c["two_arcs"] = c["n_cp"] > 120
    c["taps"] = 61 if kind == "learned" else 2 * int(_log_uniform(rng, 1.5, 36)) + 1
    c["jaw_x"], c["jaw_y"] = round(rng.uniform(12.0, 60.0), 1), round(rng.uniform(12.0, 60.0), 1)
    c["limit"] = max(c["jaw_x"], c["jaw_y"]) if rng.random() < 0.5 else 60.0
    c["phantom"] = "pelvis" if kind == "learned" or rng.random() < 0.7 else "water"
    if kind == "plan":
        c["direction"] = rng.choice(["step", "step", "forward"])
        c["conv"] = rng.choice(["fp32", "fp32", "bf16"])
        c["cache"] = rng.choice(["", "", "fp32", "bf16"])
        c["project"] = c["direction"] == "step" and rng.random() < 0.3
        c["corrections"] = rng.random() < 0.25
        c["collimator"] = rng.random() < 0.25
        c["central_axis"] = rng.random() < 0.15
        # (the allocation-free forward runs in small batches: it stands for moderate grids)
        c["noalloc"] = c["direction"] == "forward" and not c["cache"] and rng.random() < 0.25
    return c


def _cost(case):
    """A drawn case's size measures: operations and workspace elements."""
    if case["kind"] in ("plan", "learned"):
        g = _geometry(case)
        return work(case)["flops"], case["n_cp"] * g["nk"] * g["nu"] * g["nv"]
    return work(case)["flops"], 0


def draw(rng):
    r = rng.random()
    if r < 0.08:
        return dict(kind="train", nx=4 * rng.randint(8, 32), ny=4 * rng.randint(8, 32), nz=4 * rng.randint(8, 32),
                    quantile=rng.choice([0.0, 0.999]))
    if r < 0.16:
        return dict(kind="assess", nx=int(_log_uniform(rng, 32, 225)), ny=int(_log_uniform(rng, 32, 225)),
                    nz=int(_log_uniform(rng, 16, 160)), spacing=rng.choice([2.0, 2.5, 3.0]),
                    n_struct=rng.randint(1, 12), bin_width=rng.choice([0.01, 0.05]))
    kind = "learned" if r < 0.26 else "plan"
    top = _plan("top", nx=224, ny=224, nz=105, spacing=2.0, taps=55)  # the largest listed plan
    flops, elems = _cost(top)
    while True:
        c = _draw_plan(rng, kind)
        cf, ce = _cost(c)
        heavy = 3.0 if c["corrections"] or c["collimator"] else 1.0
        if c["noalloc"] and ce > 1.5e8:
            c["noalloc"] = False
        if heavy * cf <= flops and heavy * ce <= elems:
            return c


# --------------------------------------------------------------------------- inputs


def _geometry(case):
    """Beam-frame grid: rays, planes and the first plane, from the field limit and the kernel's reach."""
    d, h = case["spacing"], (case["taps"] - 1) // 2
    lim = case["limit"] * (math.sqrt(2.0) if case["collimator"] else 1.0)
    nu = 2 * math.ceil((lim + h * d) / d - 1e-9) + 1
    ox, oy = 0.5 * case["nx"] * d, 0.5 * case["ny"] * d
    r = math.hypot(ox, oy)
    return dict(nu=nu, nv=nu, nk=math.ceil(2.0 * r / d - 1e-9) + 1, R=r, h=h, d=d)


def _problem(case, seed):
    """The plan of a case: an inputs.Case whose arrays hold FP32 values, and the loss gradient dL/d dose."""
    shape, d, n = (case["nz"], case["ny"], case["nx"]), case["spacing"], case["n_cp"]
    m = inputs.Machine(n_leaf=case["n_leaf"], leaf_width=case["leaf_width"])
    if case["corrections"]:
        m = inputs.with_fluence_corrections(m)
    if case["phantom"] == "water":
        hu = np.zeros(shape, dtype=np.float32)
        origin = tuple(-(k - 1) / 2.0 * d for k in shape[::-1])
    else:
        hu, _, origin = inputs.pelvis_phantom(shape, d, seed=1000 * seed + 1)
    rng = np.random.default_rng(1000 * seed + 2)
    f32 = lambda a: np.asarray(a, dtype=np.float32).astype(np.float64)
    gantry = f32(inputs.arc_angles(n, case["two_arcs"]))
    leaves = f32(inputs.random_apertures(n, m.n_leaf, case["jaw_x"], seed=1000 * seed + 3))
    jaws = f32(inputs.jaws_square(n, case["jaw_x"], case["jaw_y"]) * rng.uniform(0.9, 1.0, size=(n, 4)))
    mu = f32(rng.uniform(1.0, 5.0, size=n))
    coll = f32(rng.uniform(-45.0, 45.0, size=n)) if case["collimator"] else None
    w = rng.random(shape, dtype=np.float32)
    mode = inputs.WEPL_CENTRAL_AXIS if case["central_axis"] else inputs.WEPL_PER_RAY
    c = inputs.Case("perf", hu, (d, d, d), origin, (0.0, 0.0, 0.0), gantry, leaves, jaws, mu, case["taps"],
                    (case["limit"], case["limit"]), m, wepl_mode=mode, collimator=coll)
    return c, w


def _dose_like(case, seed):
    """(dose, large-kernel dose, density, mask) of the network's training: crossing beams with exponential
    depth dose through an elliptic body, the larger kernel's dose a little higher towards the field edges."""
    rng = np.random.default_rng(1000 * seed + 5)
    ax = [(np.arange(case[k]) - (case[k] - 1) / 2.0) * 3.0 for k in ("nz", "ny", "nx")]
    Z, Y, X = np.meshgrid(*ax, indexing="ij")
    rho = np.where((X / 170.0) ** 2 + (Y / 110.0) ** 2 <= 1.0, 1.0, 0.0)
    rho = (rho * (1.0 + 0.02 * rng.standard_normal(rho.shape))).astype(np.float32)
    small, large = np.zeros(rho.shape), np.zeros(rho.shape)
    for a in rng.uniform(0.0, 2.0 * math.pi, size=9):
        t, s = np.cos(a) * Y - np.sin(a) * X, np.cos(a) * X + np.sin(a) * Y
        depth = np.exp(-0.0045 * (t + 200.0))
        prof = 1.0 / (1.0 + np.exp((np.abs(s) - rng.uniform(15, 45)) / 3.0)) \
            / (1.0 + np.exp((np.abs(Z) - rng.uniform(15, 45)) / 3.0))
        small += depth * prof
        large += depth * (1.02 * prof + 0.02 * np.exp(-(s ** 2 + Z ** 2) / 5000.0))
    small, large = (20.0 * v * (rho > 0.5) for v in (small, large))
    mask = (large >= 0.05 * large.max()).astype(np.float32)
    return small.astype(np.float32), large.astype(np.float32), rho, mask


def _assessment(case, seed):
    """(dose, structure masks, objective weights, targets) on a CT grid."""
    dose, _, _, _ = _dose_like(case, seed)
    dose = (dose * (78.0 / dose.max())).astype(np.float32)
    rng = np.random.default_rng(1000 * seed + 6)
    ax = [np.linspace(-1.0, 1.0, case[k]) for k in ("nz", "ny", "nx")]
    Z, Y, X = np.meshgrid(*ax, indexing="ij")
    masks = []
    for s in range(case["n_struct"]):
        c, r = rng.uniform(-0.3, 0.3, size=3), rng.uniform(0.1, 0.5 if s else 0.25, size=3)
        masks.append(((X - c[0]) / r[0]) ** 2 + ((Y - c[1]) / r[1]) ** 2 + ((Z - c[2]) / r[2]) ** 2 <= 1.0)
    weights = [100.0] + [10.0 ** rng.integers(-1, 2) for _ in range(case["n_struct"] - 1)]
    targets = [78.0] + [0.0] * (case["n_struct"] - 1)
    return dose, masks, [float(w) for w in weights], targets


LIMITS = {"leaf": 60.0, "jaw_x": 60.0, "jaw_y": 60.0, "w_min": 1.0, "mu_min": 0.22}


def prepare(case, seed):
    dev = torch.device("cuda")
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device=dev)
    if case["kind"] == "train":
        ds, dl, rho, mask = (t(a).reshape(-1) for a in _dose_like(case, seed))
        net = learned.Net3D.from_file(WEIGHTS, (case["nz"], case["ny"], case["nx"]))
        return dict(case=case, net=net, ds=ds, dl=dl, rho=rho, mask=mask, count=float(mask.sum()))
    if case["kind"] == "assess":
        dose, masks, weights, targets = _assessment(case, seed)
        return dict(case=case, dose=t(dose), ev=plan_eval.Evaluator(masks), weights=weights, targets=targets)
    c, w = _problem(case, seed)
    st = dict(case=case, leaves=t(c.leaves), jaws=t(c.jaws), mu=t(c.mu), w=t(w))
    if case["kind"] == "learned":
        net = learned.Net3D.from_file(WEIGHTS, c.shape)
        st["dose"] = learned.LearnedDose(net, c, small=9, large=case["taps"])
        return st
    st["engine"] = E.DoseEngine(c, conv=case["conv"])
    if case["cache"]:
        st["engine"].build_cache(case["cache"])
    if case["noalloc"]:
        st["out"] = torch.empty(c.shape, dtype=torch.float32, device=dev)
    if case["direction"] == "step":
        for k in ("leaves", "jaws", "mu"):
            st[k].requires_grad_(True)
    return st


def run(state):
    case = state["case"]
    if case["kind"] == "train":
        net = state["net"]
        net.forward(state["ds"], state["rho"])
        loss = net.train_loss(state["dl"], state["mask"], state["count"], quantile=case["quantile"])
        net.backward(net.gp, net.gr, weights=True)
        return loss, net.grads
    if case["kind"] == "assess":
        ev = state["ev"]
        loss, grad = ev.l1(state["dose"], state["weights"], state["targets"])
        report = ev.report(state["dose"], 78.0, case["spacing"] ** 3 / 1000.0, case["bin_width"])
        fields = ("N", "D98", "D50", "D2", "Dmean", "Dmax", "D2cc", "V50")
        table = np.array([[row.get(f, 0.0) for f in fields] for row in report.values()])
        return loss, grad, table, ev.dice(state["dose"], 0, 70.0)
    leaves, jaws, mu = state["leaves"], state["jaws"], state["mu"]
    if case["kind"] == "learned":
        dose = state["dose"].forward(leaves, jaws, mu)
        return (dose,) + tuple(state["dose"].backward(leaves, jaws, mu, state["w"]))
    eng = state["engine"]
    if case["noalloc"]:
        return eng.forward_noalloc(leaves, jaws, mu, state["out"])
    if case["direction"] == "forward":
        return eng.forward(leaves, jaws, mu)
    params = (leaves, jaws, mu)
    if case["project"]:
        dose = eng(*E.ProjectFunction.apply(leaves, jaws, mu, LIMITS, True))
    else:
        dose = eng(leaves, jaws, mu)
    return (dose,) + torch.autograd.grad(dose, params, state["w"])


# --------------------------------------------------------------------------- least work


def _net_flops(nvox):
    chans = [(16, 16, 1), (16, 16, 1), (16, 32, 8), (32, 32, 8), (32, 64, 64), (64, 64, 64), (96, 32, 8), (32, 32, 8),
             (48, 16, 1), (16, 16, 1)]
    return sum(2.0 * 27 * ci * co * nvox / f for ci, co, f in chans)


def work(case):
    nvox = case["nx"] * case["ny"] * case["nz"]
    if case["kind"] == "train":
        # forward, data gradient and weight gradient; dose, target, density and mask in, gradients out
        params = sum(27 * ci * co + co for ci, co in [(16, 16), (16, 16), (16, 32), (32, 32), (32, 64), (64, 64),
                                                      (96, 32), (32, 32), (48, 16), (16, 16)]) + 34
        return {"bytes": 16.0 * nvox + 8.0 * params, "flops": 3.0 * _net_flops(nvox)}
    if case["kind"] == "assess":
        return {"bytes": 12.0 * nvox, "flops": 2.0 * case["n_struct"] * nvox}
    g, n = _geometry(case), case["n_cp"]
    taps = 9 if case["kind"] == "learned" else case["taps"]
    rays = (2.0 * case["jaw_x"] / g["d"] + 1.0) * (2.0 * case["jaw_y"] / g["d"] + 1.0)
    dirs = 1 if case["kind"] == "plan" and case["direction"] == "forward" else 2
    # per control point: the aperture's samples (or cached factors) and taps at every plane, one trilinear
    # lookup per voxel, in each direction
    flops = dirs * n * (rays * g["nk"] * (2.0 * taps * taps + (2.0 if case["cache"] else 16.0)) + 16.0 * nvox)
    cached = {"": 0.0, "fp32": 4.0, "bf16": 2.0}[case["cache"]] * n * rays * g["nk"]
    nbytes = dirs * (4.0 * (nvox if case["cache"] else 2.0 * nvox) + cached + 4.0 * n * (2 * case["n_leaf"] + 5))
    if case["kind"] == "learned":
        flops += 2.0 * _net_flops(nvox)
    return {"bytes": nbytes, "flops": flops}


# --------------------------------------------------------------------------- the same in 64 bits


def _f64(a, dev):
    return torch.tensor(np.asarray(a, dtype=np.float64), dtype=torch.float64, device=dev)


def _sample(vol, *idx):
    """(Tri)linear samples of vol at continuous indices (one tensor per axis, first axis first), zero outside."""
    grid = torch.stack([(2.0 * i + 1.0) / n - 1.0 for i, n in zip(idx[::-1], vol.shape[::-1])], dim=-1)
    return torch.nn.functional.grid_sample(vol[None, None], grid[None], mode="bilinear", padding_mode="zeros",
                                           align_corners=False)[0, 0]


def _interp(x, xp, fp):
    """Piecewise-linear table lookup, clamped at both ends."""
    i = torch.clamp(torch.searchsorted(xp, x, right=True) - 1, 0, len(xp) - 2)
    f = torch.clamp((x - xp[i]) / (xp[i + 1] - xp[i]), 0.0, 1.0)
    return fp[i] + f * (fp[i + 1] - fp[i])


class _Exact:
    """The dose model of one plan in FP64, one control point at a time."""

    def __init__(self, c, geo, taps, dev):
        self.c, self.g, self.dev, self.m = c, geo, dev, c.machine
        self.rho = _interp(_f64(c.hu, dev), _f64(self.m.hu_pts, dev), _f64(self.m.rho_pts, dev))
        ax = lambda n: (torch.arange(n, dtype=torch.float64, device=dev) - (n - 1) / 2.0) * geo["d"]
        self.u, self.v = ax(geo["nu"]), ax(geo["nv"])
        self.e = -geo["R"] + geo["d"] * torch.arange(geo["nk"], dtype=torch.float64, device=dev)
        self.dk = self.m.sad + self.e
        nz, ny, nx = c.shape
        self.z, self.y, self.x = ax(nz), ax(ny), ax(nx)
        self.taps = taps
        dd = np.asarray(self.m.dd, dtype=np.float64)
        self.dd_x, self.dd = _f64(np.arange(len(dd)) * self.m.dd_step, dev), _f64(dd, dev)
        self.edges = _f64(self.m.leaf_edges, dev)

    def overlap(self, x, a, b):
        h = 0.5 * self.g["d"]
        return torch.clamp(torch.minimum(b, x + h) - torch.maximum(a, x - h), min=0.0) / self.g["d"]

    def _gauss(self, sigma, n):
        d = self.g["d"]
        r = math.ceil(3.0 * sigma / d - 1e-9) if sigma > 0.0 else 0
        w = np.array([math.exp(-(k * d) ** 2 / (2.0 * sigma * sigma)) if sigma > 0.0 else 1.0
                      for k in range(-r, r + 1)])
        w /= w.sum()
        m = np.zeros((n, n))
        for k in range(-r, r + 1):
            m += np.diag(np.full(n - abs(k), w[k + r]), k) if abs(k) < n else 0.0
        return _f64(m, self.dev)

    def fluence(self, b, leaves, jaws):
        m, u, v = self.m, self.u, self.v
        fx, fy = self.overlap(u, jaws[0], jaws[1]), self.overlap(v, jaws[2], jaws[3])
        w = self.overlap(v[None, :], self.edges[:-1, None], self.edges[1:, None])             # [L][Nv]
        f = self.overlap(u[:, None], leaves[0][None, :], leaves[1][None, :])                  # [Nu][L]
        F = fx[:, None] * fy[None, :] * (m.tau * w.sum(0)[None, :] + (1.0 - m.tau) * (f @ w))
        if m.fcorr:
            k = 2.0 * math.sqrt(2.0 * math.log(2.0))
            G = lambda s: self._gauss(s, len(u))
            F = G(m.pen_fwhm_u / k) @ F @ G(m.pen_fwhm_v / k)
            H = G(m.hs_sigma)
            r = torch.sqrt(u[:, None] ** 2 + v[None, :] ** 2)
            F = (1.0 + m.oar[0] * r + m.oar[1] * r * r) * (F + m.hs_amp * (H @ F @ H))
        if self.c.collimator is not None:
            a = math.radians(self.c.collimator[b])
            s, co = math.sin(a), math.cos(a)
            U, V = torch.meshgrid(u, v, indexing="ij")
            ctr, d = (len(u) - 1) / 2.0, self.g["d"]
            F = _sample(F, (co * U + s * V) / d + ctr, (-s * U + co * V) / d + ctr)
        return F

    def _density(self, q):
        d, o = self.c.spacing, self.c.origin
        return _sample(self.rho, *[(q[k] - o[k]) / d[k] for k in (2, 1, 0)])

    def plane_factors(self, b):
        """(G [Nk][Nu][Nv] with P = F G, taps [Nk][n][n]) of control point b."""
        a = math.radians(self.c.gantry[b])
        sn, cs, sad, d = math.sin(a), math.cos(a), self.m.sad, self.g["d"]
        e, mag = self.e[:, None, None], (self.dk / sad)[:, None, None]
        u, v = self.u[None, :, None], self.v[None, None, :]
        zero = torch.zeros((), dtype=torch.float64, device=self.dev)
        axis = torch.cumsum(self._density([x.expand(self.e.shape)[:, None, None] for x in
                                           (-self.e * sn, self.e * cs, zero)]).reshape(-1) * d, 0)
        if self.c.wepl_mode == inputs.WEPL_CENTRAL_AXIS:
            W = axis[:, None, None].expand(len(self.e), len(self.u), len(self.v))
        else:
            q = torch.broadcast_tensors(-e * sn + mag * u * cs, e * cs + mag * u * sn, mag * v)
            W = torch.cumsum(self._density(q) * d * torch.sqrt(1.0 + (u * u + v * v) / sad ** 2), 0)
        G = _interp(W.contiguous(), self.dd_x, self.dd) / mag ** 2
        zc = torch.clamp(axis, 0.0, self.m.kz_max)
        A, al, B, be = (sum(float(p[k]) * zc ** k for k in range(4))[:, None, None] for p in self.m.kpoly)
        delta, norm = mag * d, A / al + B / be
        h = (self.taps - 1) // 2
        t = torch.arange(-h, h + 1, dtype=torch.float64, device=self.dev)
        r = delta * torch.sqrt(t[:, None] ** 2 + t[None, :] ** 2)
        rs = torch.where(r > 0.0, r, delta)
        K = delta ** 2 * (A * torch.exp(-al * rs) + B * torch.exp(-be * rs)) / (2.0 * math.pi * rs * norm)
        r0 = delta / math.sqrt(math.pi)
        K[:, h, h] = (-(A / al * torch.expm1(-al * r0) + B / be * torch.expm1(-be * r0)) / norm)[:, 0, 0]
        return G, K

    def convolve(self, P, K):
        h, n = (self.taps - 1) // 2, [s + self.taps - 1 for s in P.shape[1:]]
        full = torch.fft.irfft2(torch.fft.rfft2(P, s=n) * torch.fft.rfft2(K, s=n), s=n)
        return full[:, h:h + P.shape[1], h:h + P.shape[2]]

    def voxels(self, b):
        """Continuous beam-frame indices (kappa, iota, jota) of every voxel."""
        a = math.radians(self.c.gantry[b])
        sn, cs, d = math.sin(a), math.cos(a), self.g["d"]
        z, y, x = self.z[:, None, None], self.y[None, :, None], self.x[None, None, :]
        e = -sn * x + cs * y
        q = self.m.sad / (self.m.sad + e)
        idx = ((e + self.g["R"]) / d, (cs * x + sn * y) * q / d + (len(self.u) - 1) / 2.0,
               z * q / d + (len(self.v) - 1) / 2.0)
        return torch.broadcast_tensors(*idx)

    def control_point(self, b, leaves, jaws):
        G, K = self.plane_factors(b)
        return _sample(self.convolve(self.fluence(b, leaves, jaws)[None] * G, K), *self.voxels(b))

    def params(self, b):
        return (_f64(self.c.leaves[b], self.dev), _f64(self.c.jaws[b], self.dev), float(self.c.mu[b]))

    def forward(self):
        with torch.no_grad():
            dose = torch.zeros(self.c.shape, dtype=torch.float64, device=self.dev)
            for b in range(self.c.n_cp):
                lv, jw, mu = self.params(b)
                dose += self.m.calib * mu * self.control_point(b, lv, jw)
        return dose

    def backward(self, w):
        """Gradients for dL/d dose = w (and the dose on the way)."""
        gl, gj, gm = [], [], []
        dose = torch.zeros(self.c.shape, dtype=torch.float64, device=self.dev)
        for b in range(self.c.n_cp):
            lv, jw, mu = self.params(b)
            lv.requires_grad_(True)
            jw.requires_grad_(True)
            d = self.m.calib * self.control_point(b, lv, jw)
            l = (d * w).sum()
            a, j = torch.autograd.grad(mu * l, (lv, jw))
            dose += mu * d.detach()
            gl.append(a)
            gj.append(j)
            gm.append(l.detach())
        return dose, torch.stack(gl), torch.stack(gj), torch.stack(gm)


def _project(c):
    """Centre / width projection of the plan's parameters (FP32 values in, FP64 out)."""
    def pair(a, b, lim):
        ctr, w = np.clip(0.5 * (a + b), -lim, lim), np.maximum(b - a, LIMITS["w_min"])
        return ctr - 0.5 * w, ctr + 0.5 * w
    l, r = pair(c.leaves[:, 0], c.leaves[:, 1], LIMITS["leaf"])
    j = np.empty_like(c.jaws)
    j[:, 0], j[:, 1] = pair(c.jaws[:, 0], c.jaws[:, 1], LIMITS["jaw_x"])
    j[:, 2], j[:, 3] = pair(c.jaws[:, 2], c.jaws[:, 3], LIMITS["jaw_y"])
    c.leaves, c.jaws, c.mu = np.stack([l, r], axis=1), j, np.maximum(c.mu, LIMITS["mu_min"])


def _net64(case, dev):
    """(parameters, forward function) of the correction network in FP64; volumes are [D][H][W][C]."""
    with np.load(WEIGHTS) as st:
        p = torch.tensor(st["params"].astype(np.float64), device=dev, requires_grad=True)
    off = 0
    layers = []
    for ci, co in [(16, 16), (16, 16), (16, 32), (32, 32), (32, 64), (64, 64), (96, 32), (32, 32), (48, 16), (16, 16)]:
        layers.append((off, ci, co))
        off += 27 * ci * co + co

    def conv(k, x):
        o, ci, co = layers[k]
        w, bias = p[o:o + 27 * ci * co].view(co, 27, ci), p[o + 27 * ci * co:o + 27 * ci * co + co]
        D, H, W, _ = x.shape
        xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
        y = bias.expand(D * H * W, co)
        for t in range(27):
            s = xp[t // 9:t // 9 + D, (t // 3) % 3:(t // 3) % 3 + H, t % 3:t % 3 + W].reshape(-1, ci)
            y = y + s @ w[:, t].T
        return torch.relu(y).view(D, H, W, co)

    def pool(x):
        D, H, W, C = x.shape
        return x.view(D // 2, 2, H // 2, 2, W // 2, 2, C).mean(dim=(1, 3, 5))

    def up(x):
        return x.repeat_interleave(2, 0).repeat_interleave(2, 1).repeat_interleave(2, 2)

    def forward(dose, rho, scale):
        x = torch.zeros(dose.shape + (16,), dtype=torch.float64, device=dev)
        x = torch.cat([(dose * scale)[..., None], rho[..., None], x[..., 2:]], dim=-1)
        s1 = conv(1, conv(0, x))
        s2 = conv(3, conv(2, pool(s1)))
        c2 = conv(7, conv(6, torch.cat([up(conv(5, conv(4, pool(s2)))), s2], dim=-1)))
        c1 = conv(9, conv(8, torch.cat([up(c2), s1], dim=-1)))
        hw, hb = p[off:off + 32].view(2, 16), p[off + 32:off + 34]
        return dose * scale + c1 @ hw[0] + hb[0], c1 @ hw[1] + hb[1]

    return p, forward


def exact(case, seed):
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    if case["kind"] == "train":
        ds, dl, rho, mask = (_f64(a, dev) for a in _dose_like(case, seed))
        p, net = _net64(case, dev)
        s = 1.0 / ds.max()
        pred, resid = net(ds, rho, s)
        e = pred - dl * s
        u = e.detach().abs() - resid
        q = case["quantile"]
        r = u * (q - (u < 0.0).to(u.dtype)) if q > 0.0 else u * u
        loss = (mask * (e * e + r)).sum() / max(1.0, float(mask.sum()))
        (g,) = torch.autograd.grad(loss, p)
        return loss.detach().reshape(1), g
    if case["kind"] == "assess":
        dose, masks, weights, targets = _assessment(case, seed)
        d = _f64(dose, dev)
        loss, grad = torch.zeros(1, dtype=torch.float64, device=dev), torch.zeros_like(d)
        for k, (w, t) in enumerate(zip(weights, targets)):
            mk = _f64(masks[k], dev)
            loss += w * (mk * (d - t).abs()).sum()
            grad += w * mk * torch.sign(d - t)
        return loss, grad, None, None
    c, w = _problem(case, seed)
    w = _f64(w, dev)
    if case["kind"] == "learned":
        small = dict(case, taps=9)
        ex = _Exact(c, _geometry(small), 9, dev)
        d9 = ex.forward().requires_grad_(True)
        _, net = _net64(case, dev)
        s = 1.0 / d9.max()
        pred, resid = net(d9, ex.rho, s)
        with torch.no_grad():
            top = pred.max()
            fallback = bool(resid[pred >= 0.1 * top].max() > 0.01 * top)
        if not fallback:
            (gd,) = torch.autograd.grad(((pred / s) * w).sum(), d9)
            return ((pred / s).detach(),) + ex.backward(gd)[1:]
        return _Exact(c, _geometry(case), case["taps"], dev).backward(w)
    if case["project"]:
        _project(c)
    ex = _Exact(c, _geometry(case), case["taps"], dev)
    return ex.forward() if case["direction"] == "forward" else ex.backward(w)
