"""The work a user has this library do, as timed cases.

Four kinds of case, each through the public entry points:

    grid    a resident grid stepped a fixed number of times (sc_lbm_create on
            the caller's own device buffers, sc_lbm_step): long runs between
            two outputs, on the automatic launch shape
    run     one whole run of an experiment: Sim, walls where it has them, steps
            with the steady-state check every `every` steps, observe, close
    sweep   one whole batched sweep (warmstart.steady_states): many droplets
            created, stepped with checks, their density fields read back
    train   one training step of the warm-start net: features, forward, loss,
            backward, Adam

No run reaches its steady state within the steps given, so every pass does
the same work.  exact() restates the method (Shan-Chen force, Guo or exact
difference forcing, SRT / MRT, pull streaming; the net's convolutions and
Adam) in plain 64-bit torch.
"""
import math

import numpy as np
import torch

from paper_1906_11027_amd import Sim
from paper_1906_11027_amd import sc_lbm as B
from paper_1906_11027_amd import warmstart as W

DEV = "cuda" if torch.cuda.is_available() else "cpu"

# Peng-Robinson set-up of the experiments (a = 2/49, b = 2/21, R = 1,
# omega = 0.344): T, alpha(T) and the Maxwell densities at T/Tc
PR = {
    0.85: dict(T=0.061981181597056186, alpha=1.1409491270952417, rv=0.3412375454535148, rl=6.62958997846167),
    0.90: dict(T=0.06562713345570656, alpha=1.0916312818634129, rv=0.5799723133759689, rl=5.908234645230209),
    0.95: dict(T=0.06927308531435691, alpha=1.0447105571509645, rv=1.012904503329191, rl=4.928660823075937),
}
EOS_A, EOS_B = 2.0 / 49.0, 2.0 / 21.0
C0 = 1.0 / 3.0
S_BULK = S_GHOST = 1.2
TOL = 1e-14            # below any change of max |u| these runs reach
RHO_L, RHO_V = 2.0, 0.15
LR = 2e-3


def _grid(name, lattice, shape, order, steps, precision="fp32", tau=1.0, collision="srt", tr=0.0, forcing="guo"):
    return dict(name=name, kind="grid", lattice=lattice, nx=shape[0], ny=shape[1],
                nz=shape[2] if len(shape) > 2 else 1, order=order, steps=steps, precision=precision, tau=tau,
                collision=collision, tr=tr, forcing=forcing)


def _run(name, lattice, shape, order, steps, every, tau=1.0, tr=0.0, forcing="guo", walls=False, precision="fp64"):
    return dict(name=name, kind="run", lattice=lattice, nx=shape[0], ny=shape[1], nz=1, order=order, steps=steps,
                every=every, precision=precision, tau=tau, collision="srt", tr=tr, forcing=forcing, walls=walls)


def listed():
    return [
        # the smallest: the 64^2 droplet with the check every 100 steps, one
        # of the per-droplet runs of a parameter study; latency of the calls
        _run("run_d2q9_e4_64_fp64", "D2Q9", (64, 64), 4, 1000, 100),
        # the 60^2 Peng-Robinson droplet of the spurious-current experiments
        _run("run_d2q13_e6_60_pr_fp64", "D2Q13", (60, 60), 6, 1000, 500, 11.0 / 12.0, 0.85, "edm"),
        # the droplet on a wall of a 200 x 100 channel (contact angles)
        _run("run_d2q25_e8_walls_200x100_pr_fp64", "D2Q25", (200, 100), 8, 1000, 500, 19.0 / 24.0, 0.90, "edm", True),
        # the 256^2 droplet, FP32 state: the everyday grid
        _grid("d2q9_e8_256", "D2Q9", (256, 256), 8, 400),
        # an odd, ragged grid with the widest stencil and the FP64 state
        _grid("d2q9_e10_1001x777_fp64", "D2Q9", (1001, 777), 10, 100, "fp64"),
        # the largest 2D grid: limited by memory traffic
        _grid("d2q9_e8_8192", "D2Q9", (8192, 8192), 8, 32),
        # the large-lattice 2D grid of the same size with the experiments' model
        _grid("d2q25_e8_pr_8192", "D2Q25", (8192, 8192), 8, 8, tau=19.0 / 24.0, tr=0.85, forcing="edm"),
        # 3D droplets, MRT: the everyday cube, the large one, and a ragged FP64 box
        _grid("d3q19_mrt_e8_128", "D3Q19", (128, 128, 128), 8, 64, collision="mrt"),
        _grid("d3q19_mrt_e8_320", "D3Q19", (320, 320, 320), 8, 16, collision="mrt"),
        _grid("d3q19_mrt_e8_200x181x150_fp64", "D3Q19", (200, 181, 150), 8, 16, "fp64", collision="mrt"),
        # a sweep over droplets of sides 64 to 512, as the warm start's data are made
        dict(name="sweep_24_droplets", kind="sweep", items=24, lo=64, hi=512, steps=300, every=100, precision="fp32"),
        # one mini-batch of the warm start's training at its own size
        dict(name="train_b16_256", kind="train", batch=16, side=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["grid2", "grid2", "grid3", "run", "sweep", "train"])
    if kind == "train":
        return dict(kind="train", batch=rng.choice([1, 4, 8, 16]), side=_log_int(rng, 33, 256))
    if kind == "sweep":
        lo = _log_int(rng, 48, 200)
        return dict(kind="sweep", items=_log_int(rng, 4, 24), lo=lo, hi=rng.randint(lo, 512), steps=300, every=100,
                    precision=rng.choice(["fp32", "fp64"]))
    if kind == "grid3":
        shape = tuple(_log_int(rng, 24, 320) for _ in range(3))
        n = shape[0] * shape[1] * shape[2]
        c = _grid("", "D3Q19", shape, rng.choice([4, 6, 8]), max(8, min(64, int(2e8 / n))),
                  rng.choice(["fp32", "fp32", "fp64"]), rng.choice([0.8, 1.0, 1.2]), rng.choice(["srt", "mrt"]))
    else:
        lattice = rng.choice(["D2Q9", "D2Q9", "D2Q13", "D2Q25"])
        pr = lattice != "D2Q9" or rng.random() < 0.3
        tr = rng.choice([0.85, 0.90, 0.95]) if pr else 0.0
        forcing = "edm" if pr else "guo"
        tau = {"D2Q9": 1.0 if pr else rng.choice([0.8, 1.0, 1.2]), "D2Q13": 11.0 / 12.0, "D2Q25": 19.0 / 24.0}[lattice]
        order = rng.choice([4, 6, 8, 10])
        if kind == "run":
            c = _run("", lattice, (_log_int(rng, 40, 256), _log_int(rng, 40, 200)), order, rng.choice([300, 700, 1000]),
                     rng.choice([100, 250, 500]), tau, tr, forcing, pr and rng.random() < 0.5)
        else:
            shape = (_log_int(rng, 64, 8192), _log_int(rng, 64, 4096))
            n = shape[0] * shape[1]
            c = _grid("", lattice, shape, order, max(8, min(400, int(4e8 / n))), rng.choice(["fp32", "fp32", "fp64"]),
                      tau, tr=tr, forcing=forcing)
    del c["name"]
    return c


# ------------------------------------------------------------- inputs ----

def _rng(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + salt)
    return g


def _droplet(shape, radius, rl, rv, width, jitter_seed, centre=None):
    """tanh droplet [z, y, x] (FP64, on the GPU) with a +-1e-3 jitter."""
    r2 = 0.0
    for ax, n in enumerate(shape):
        d = torch.arange(n, dtype=torch.float64, device=DEV) - (n // 2 if centre is None else centre[ax])
        d = (d + n / 2.0) % n - n / 2.0
        view = [1] * len(shape)
        view[len(shape) - 1 - ax] = n
        r2 = r2 + (d * d).reshape(view)
    rho = 0.5 * (rl + rv) - 0.5 * (rl - rv) * torch.tanh(2.0 * (r2.sqrt() - radius) / width)
    jit = torch.rand(rho.shape, generator=_rng(jitter_seed), dtype=torch.float64, device=DEV)
    return rho + (2.0 * jit - 1.0) * 1e-3


def _density(case, seed):
    shape = (case["nx"], case["ny"]) if case["nz"] == 1 else (case["nx"], case["ny"], case["nz"])
    rl, rv, width = (PR[case["tr"]]["rl"], PR[case["tr"]]["rv"], 4.0) if case["tr"] else (RHO_L, RHO_V, 2.0)
    if not case.get("walls"):
        return _droplet(shape, 0.2 * min(shape), rl, rv, width, seed)
    rho = _droplet(shape, 0.35 * shape[1], rl, rv, width, seed, (shape[0] / 2.0, 2.0))
    return torch.where(_solid(case), torch.full_like(rho, rv), rho)


def _solid(case):
    m = torch.zeros((case["ny"], case["nx"]), dtype=torch.bool, device=DEV)
    m[:2] = True
    m[-2:] = True
    return m


RHO_WALL = 2.5


def _model(case):
    kw = dict(order=case["order"], tau=case["tau"], collision=case["collision"], precision=case["precision"],
              forcing=case["forcing"], G=-5.0)
    if case["tr"]:
        e = PR[case["tr"]]
        kw.update(G=-1.0, psi="pr", eos=dict(a=EOS_A, b=EOS_B, R=1.0, T=e["T"], alpha=e["alpha"]))
    return kw


def _sides(case):
    """The droplets' box sides: spread evenly over the logarithm of the range."""
    n = case["items"]
    return [int(round(case["lo"] * (case["hi"] / case["lo"]) ** (k / max(1, n - 1)))) for k in range(n)]


def _sweep_items(case, seed):
    r = np.random.default_rng(seed)
    items = []
    for side in _sides(case):
        items.append(dict(side=side, R=float(r.uniform(0.17, 0.3) * side), G=float(r.uniform(-5.3, -4.8)),
                          tau=float(r.choice([0.8, 1.0, 1.2])), order=int(r.choice([4, 6, 8, 10])),
                          seed=int(r.integers(1 << 30))))
    return items


def _net_init(case, seed):
    """Inputs of a training step in mid-training: weights, biases, Adam moments, parameters, target."""
    g = _rng(seed, 7)

    def rnd(*s):
        return torch.randn(s, generator=g, dtype=torch.float32, device=DEV)

    layers = []
    for cin, cout in zip(W.CHANNELS[:-1], W.CHANNELS[1:]):
        layers.append(dict(W=rnd(cout, cin, 3, 3) / math.sqrt(9.0 * cin), b=0.05 * rnd(cout),
                           mW=1e-4 * rnd(cout, cin, 3, 3), mb=1e-4 * rnd(cout),
                           vW=1e-7 * (0.2 + rnd(cout, cin, 3, 3) ** 2), vb=1e-7 * (0.2 + rnd(cout) ** 2)))
    n, h = case["batch"], case["side"]
    u = torch.rand((n, 4), generator=g, dtype=torch.float32, device=DEV)
    prm = torch.stack([0.1 * h * (0.1 + 0.2 * u[:, 0]), 2.0 * u[:, 1] - 1.0, 2.0 * u[:, 2] - 1.0,
                       2.0 * u[:, 3] - 1.0], 1).contiguous()
    d = torch.arange(h, dtype=torch.float32, device=DEV) - h // 2
    r = (d[:, None] ** 2 + d[None, :] ** 2).sqrt() / W.SCALE_R
    ring = r[None] - prm[:, 0, None, None]
    tgt = (torch.exp(-(3.0 * ring) ** 2) * (1.0 + 0.1 * rnd(n, h, h)))[:, None].contiguous()
    return layers, prm, tgt


TRAIN_T = 200   # Adam steps already taken


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        layers, prm, tgt = _net_init(case, seed)
        net = W.WarmStartNet(case["side"], case["side"], case["batch"], seed=seed)
        for li, l in enumerate(layers):
            for dst, key in ((net.W, "W"), (net.b, "b"), (net.mW, "mW"), (net.vW, "vW"), (net.mb, "mb"),
                             (net.vb, "vb")):
                dst[li].copy_(l[key])
            net.Wb[li].copy_(l["W"].to(torch.bfloat16).view(torch.int16))
        net.t = TRAIN_T
        return dict(kind=kind, net=net, prm=prm, tgt=tgt)
    if kind == "sweep":
        items = [dict(rho0=_droplet((it["side"],) * 2, it["R"], RHO_L, RHO_V, 2.0, it["seed"]).cpu().numpy().T,
                      order=it["order"], G=it["G"], tau=it["tau"], precision=case["precision"])
                 for it in _sweep_items(case, seed)]
        return dict(kind=kind, items=items, case=case)
    rho = _density(case, seed).cpu().numpy()
    if kind == "run":
        solid = _solid(case).cpu().numpy().T if case["walls"] else None
        return dict(kind=kind, rho0=rho.T, solid=solid, case=case)
    shape = (case["nx"], case["ny"]) if case["nz"] == 1 else (case["nx"], case["ny"], case["nz"])
    p = B.make_params(case["lattice"], shape, **_model(case))
    dt = torch.float64 if case["precision"] == "fp64" else torch.float32
    q, n = B.Q[p.lattice], int(np.prod(shape))
    bufs = [torch.empty((q, n), dtype=dt, device=DEV) for _ in range(2)]
    h = B.sc_lbm_create(p, rho.ravel(), bufs[0].data_ptr(), bufs[1].data_ptr(), _stream().cuda_stream)
    return dict(kind=kind, handle=_Handle(h), bufs=bufs, steps=case["steps"])


_STREAM = []


def _stream():
    """The one stream the program steps its grids on, one after the other."""
    if not _STREAM:
        _STREAM.append(torch.cuda.Stream())
    return _STREAM[0]


class _Handle:
    """Destroys the grid with the state that holds it."""

    def __init__(self, h):
        self.h = h

    def __del__(self):
        if B is not None and self.h:
            B.sc_lbm_destroy(self.h)


def run(state):
    kind = state["kind"]
    if kind == "grid":
        h, bufs = state["handle"].h, state["bufs"]
        B.sc_lbm_step(h, state["steps"])
        return bufs[0] if B.sc_lbm_state_ptr(h) == bufs[0].data_ptr() else bufs[1]
    if kind == "train":
        net = state["net"]
        net.set_params(state["prm"])
        out = net.forward()
        net.loss_and_grad(state["tgt"])
        net.backward()
        net.adam(lr=LR)
        return dict(out=out, gW=net.gW, gb=net.gb, W=net.W, b=net.b, mW=net.mW, mb=net.mb, vW=net.vW, vb=net.vb)
    case = state["case"]
    if kind == "sweep":
        # the fields become the net's float32 training targets
        fields, steps, by, _ = W.steady_states(state["items"], tol=TOL, max_steps=case["steps"],
                                               obs_every=case["every"])
        dt = np.float64 if case["precision"] == "fp64" else np.float32
        return dict(fields=[np.ascontiguousarray(f, dtype=dt) for f in fields], steps=np.array(steps),
                    by=np.array(by))
    sim = Sim(state["rho0"], case["lattice"], obs_every=case["every"], **_model(case))
    if state["solid"] is not None:
        sim.set_walls(state["solid"], RHO_WALL)
    rc, steps = sim.step(case["steps"], tol=TOL)
    out = sim.observe()
    sim.close()
    o = out["obs"]
    return dict(rho=out["rho"], u=out["u"], steps=int(steps),
                obs=np.array([o[k] for k in ("mass", "max_u", "mean_u", "l2_u", "rho_in", "rho_out", "rho_min",
                                             "rho_max")]))


def _pairs(dim, order):
    """Neighbours of the force stencil."""
    return len(_stencil(dim, order))


def work(case):
    """One pass: the state read once and written once however many steps it
    takes (a run also reads its density and writes the fields), and the
    arithmetic of every step: 4 operations per force neighbour, 14 per
    population (sums, equilibrium, source, relaxation), 30 per population
    with MRT, 20 for psi and the velocity."""
    if case["kind"] == "train":
        px = case["batch"] * case["side"] ** 2
        # activations of four hidden layers and their gradients stored once and
        # read once, target in, output out; forward, data and weight gradients
        ch = list(zip(W.CHANNELS[:-1], W.CHANNELS[1:]))
        flops = sum(2 * 9 * a * b * (3 if k else 2) for k, (a, b) in enumerate(ch)) * px
        return dict(bytes=px * 4.0 * (2 * 4 * 32 * 2 + 2), flops=float(flops))
    if case["kind"] == "sweep":
        n = float(sum(side * side for side in _sides(case)))
        return dict(bytes=n * (8.0 + 8.0), flops=n * case["steps"] * (4 * 24 + 14 * 9 + 20))
    n = case["nx"] * case["ny"] * case["nz"]
    q, dim = B.Q[B.LATTICE[case["lattice"]]], 3 if case["nz"] > 1 else 2
    per = 4 * _pairs(dim, case["order"]) + (30 if case["collision"] == "mrt" else 14) * q + 20
    ts = 8 if case["precision"] == "fp64" else 4
    io = n * 8.0 * (1 + 1 + dim) if case["kind"] == "run" else 2.0 * n * q * ts
    return dict(bytes=io, flops=float(n) * case["steps"] * per)


# --------------------------------------------- the method in 64 bits ----

SHELLS = {
    (2, 4): {1: 1 / 3, 2: 1 / 12},
    (2, 6): {1: 4 / 15, 2: 1 / 10, 4: 1 / 120},
    (2, 8): {1: 4 / 21, 2: 4 / 45, 4: 1 / 60, 5: 2 / 315, 8: 1 / 5040},
    (2, 10): {1: 262 / 1785, 2: 93 / 1190, 4: 7 / 340, 5: 6 / 595, 8: 9 / 9520, 9: 2 / 5355, 10: 1 / 7140},
    (3, 4): {1: 1 / 6, 2: 1 / 12},
    (3, 6): {1: 2 / 15, 2: 1 / 15, 3: 1 / 60, 4: 1 / 120},
    (3, 8): {1: 4 / 45, 2: 1 / 21, 3: 2 / 105, 4: 5 / 504, 5: 1 / 315, 6: 1 / 630, 8: 1 / 5040},
}
Q13 = [(0, 0), (-1, 0), (0, -1), (0, 1), (1, 0), (-1, -1), (-1, 1), (1, -1), (1, 1), (-2, 0), (0, -2), (0, 2), (2, 0)]
VELOCITIES = {
    "D2Q9": [(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)],
    "D3Q19": [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (-1, -1, 0),
              (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 1, 1), (0, -1, -1),
              (0, 1, -1), (0, -1, 1)],
    "D2Q13": Q13,
    "D2Q25": Q13 + [(-2, -1), (-2, 1), (-1, -2), (-1, 2), (1, -2), (1, 2), (2, -1), (2, 1), (-2, -2), (-2, 2),
                    (2, -2), (2, 2)],
}
WEIGHTS = {
    "D2Q9": {0: 4 / 9, 1: 1 / 9, 2: 1 / 36},
    "D3Q19": {0: 1 / 3, 1: 1 / 18, 2: 1 / 36},
    "D2Q13": {0: 2 / 5, 1: 8 / 75, 2: 1 / 25, 4: 1 / 300},
    "D2Q25": {0: 72 / 245, 1: 16 / 147, 2: 16 / 315, 4: 1 / 105, 5: 8 / 2205, 8: 1 / 8820},
}
CS2 = {"D2Q9": 1 / 3, "D3Q19": 1 / 3, "D2Q13": 2 / 5, "D2Q25": 4 / 7}


def _stencil(dim, order):
    sh = SHELLS[dim, order]
    m = range(-3, 4)
    vecs = [(x, y, z) for x in m for y in m for z in (m if dim == 3 else (0,))]
    return [(v, sh[v[0] ** 2 + v[1] ** 2 + v[2] ** 2]) for v in vecs if v[0] ** 2 + v[1] ** 2 + v[2] ** 2 in sh]


def _shift(a, c):
    """a at x + c for arrays [..., y, x] or [..., z, y, x]."""
    d = len(c)
    return torch.roll(a, shifts=tuple(-v for v in c), dims=tuple(-1 - k for k in range(d)))


class _Exact:
    """The stepped fields f (pulled, pre-collision) of one grid."""

    def __init__(self, rho0, case, G, solid=None):
        self.v = VELOCITIES[case["lattice"]]
        self.d = len(self.v[0])
        self.w = [WEIGHTS[case["lattice"]][sum(c * c for c in v)] for v in self.v]
        self.cs2, self.case, self.G, self.solid = CS2[case["lattice"]], case, G, solid
        self.st = [(e, w) for e, w in _stencil(self.d, case["order"])
                   if next(c for c in e if c) > 0]          # one of each +-e pair
        self.f = [w * rho0 for w in self.w]

    def psi(self, rho):
        if not self.case["tr"]:
            return -torch.expm1(-rho)
        e = PR[self.case["tr"]]
        br = EOS_B * rho
        p = rho * e["T"] / (1.0 - br) - EOS_A * e["alpha"] * rho * rho / (1.0 + 2.0 * br - br * br)
        return torch.sqrt(torch.clamp(2.0 * (p - self.cs2 * rho) / (self.G * C0), min=0.0))

    def macro(self):
        rho = sum(self.f)
        psi = self.psi(rho)
        if self.solid is not None:
            wall = self.psi(torch.tensor(RHO_WALL, dtype=torch.float64, device=DEV))
            psi = torch.where(self.solid, wall, psi)
        F = [0.0] * self.d
        for e, w in self.st:
            c = e[:self.d]
            diff = w * (_shift(psi, c) - _shift(psi, tuple(-k for k in c)))
            F = [Fk + ck * diff if ck else Fk for Fk, ck in zip(F, c)]
        F = [-self.G * C0 * psi * Fk for Fk in F]
        j = []
        for k in range(self.d):
            j.append(sum(fb if v[k] == 1 else v[k] * fb for fb, v in zip(self.f, self.v) if v[k]))
        return rho, j, F

    def collide(self):
        rho, j, F = self.macro()
        case, cs2, om = self.case, self.cs2, 1.0 / self.case["tau"]
        dot = lambda c, a: sum(ck * ak for ck, ak in zip(c, a) if ck)                      # noqa: E731

        def feq(w, c, r, u, usq):
            cu = dot(c, u) if any(c) else 0.0
            return w * r * (1.0 + cu / cs2 + cu * cu / (2.0 * cs2 * cs2) - usq / (2.0 * cs2))

        if case["forcing"] == "edm":
            v = [jk / rho for jk in j]
            s = [vk + Fk / rho for vk, Fk in zip(v, F)]
            vsq, ssq = sum(k * k for k in v), sum(k * k for k in s)
            out = []
            for fb, w, c in zip(self.f, self.w, self.v):
                e0 = feq(w, c, rho, v, vsq)
                out.append(fb - om * (fb - e0) + feq(w, c, rho, s, ssq) - e0)
        else:
            u = [(jk + 0.5 * Fk) / rho for jk, Fk in zip(j, F)]
            usq, uF = sum(k * k for k in u), sum(a * b for a, b in zip(u, F))

            def source(w, c):
                if not any(c):
                    return -w * uF / cs2
                cu, cF = dot(c, u), dot(c, F)
                return w * ((cF - uF) / cs2 + cu * cF / (cs2 * cs2))

            if case["collision"] == "srt":
                out = [fb - om * (fb - feq(w, c, rho, u, usq)) + (1.0 - 0.5 * om) * source(w, c)
                       for fb, w, c in zip(self.f, self.w, self.v)]
            else:
                # BGK at the ghost rate, corrected on the bulk and the five shear moments
                mom = [[19 * sum(k * k for k in c) - 30 for c in self.v],
                       [2 * c[0] ** 2 - c[1] ** 2 - c[2] ** 2 for c in self.v],
                       [c[1] ** 2 - c[2] ** 2 for c in self.v], [c[0] * c[1] for c in self.v],
                       [c[1] * c[2] for c in self.v], [c[0] * c[2] for c in self.v]]
                rate = [S_BULK] + [om] * 5
                acc = [0.0] * 6
                out = []
                for b, (fb, w, c) in enumerate(zip(self.f, self.w, self.v)):
                    nb, ph = fb - feq(w, c, rho, u, usq), source(w, c)
                    out.append(fb - S_GHOST * nb + (1.0 - 0.5 * S_GHOST) * ph)
                    val = nb + 0.5 * ph
                    acc = [a + m[b] * val if m[b] else a for a, m in zip(acc, mom)]
                acc = [(S_GHOST - r) * a / sum(k * k for k in m) for a, m, r in zip(acc, mom, rate)]
                for b in range(len(out)):
                    out[b] = out[b] + sum(m[b] * a for a, m in zip(acc, mom) if m[b])
        if self.solid is not None:
            opp = [self.v.index(tuple(-k for k in c)) for c in self.v]
            out = [torch.where(self.solid, self.f[o], ob) for ob, o in zip(out, opp)]
        return out

    def step(self, n):
        """n steps; the post-collision values of the last are left in self.post."""
        for _ in range(n):
            self.post = self.collide()
            self.f = [_shift(g, tuple(-k for k in c)) for g, c in zip(self.post, self.v)]
        return self


def _median(rho):
    """Upper median of at most 2^20 evenly strided nodes (the storage shift)."""
    v = rho.reshape(-1)
    v = v[::max(1, v.numel() // (1 << 20))]
    return float(torch.kthvalue(v, v.numel() // 2 + 1).values)


def _exact_train(case, seed):
    layers, prm, tgt = _net_init(case, seed)
    n, h = case["batch"], case["side"]
    d = torch.arange(h, dtype=torch.float64, device=DEV) - h // 2
    p = prm.double()
    r = (d[:, None] ** 2 + d[None, :] ** 2).sqrt() / W.SCALE_R
    ones = torch.ones((n, h, h), dtype=torch.float64, device=DEV)
    x = torch.stack([r[None] - p[:, 0, None, None]] + [p[:, k, None, None] * ones for k in range(4)], 1)

    def conv(x, w):
        """sum over taps of W_t x(+d_t): [n, ci, h, h] -> [n, co, h, h]."""
        out = 0.0
        for k in range(9):
            xs = torch.roll(x, shifts=(1 - k // 3, 1 - k % 3), dims=(2, 3))
            out = out + torch.matmul(w[:, :, k // 3, k % 3].contiguous(), xs.reshape(n, x.shape[1], -1)).reshape(
                n, w.shape[0], h, h)
        return out

    wb = [l["W"].to(torch.bfloat16).double() for l in layers]
    acts = [x]
    for li, l in enumerate(layers):
        y = conv(acts[-1], wb[li]) + l["b"].double()[None, :, None, None]
        acts.append(torch.tanh(y) if li < 4 else y)
    g = 2.0 * (acts[5] - tgt.double()) / acts[5].numel()
    gW, gb = [None] * 5, [None] * 5
    for li in range(4, -1, -1):
        gb[li] = g.sum((0, 2, 3))
        rows = []
        for k in range(9):
            xs = torch.roll(acts[li], shifts=(1 - k // 3, 1 - k % 3), dims=(2, 3))
            a = g.transpose(0, 1).reshape(g.shape[1], -1)
            rows.append(torch.matmul(a, xs.transpose(0, 1).reshape(xs.shape[1], -1).t().contiguous()))
        gW[li] = torch.stack(rows, -1).reshape(layers[li]["W"].shape)
        if li:
            g = conv(g, wb[li].flip((2, 3)).transpose(0, 1)) * (1.0 - acts[li] ** 2)
    t = TRAIN_T + 1
    new = dict(out=acts[5], gW=gW, gb=gb, W=[], b=[], mW=[], mb=[], vW=[], vb=[])
    for li, l in enumerate(layers):
        for key, m, v, gr in (("W", "mW", "vW", gW[li]), ("b", "mb", "vb", gb[li])):
            mi = 0.9 * l[m].double() + 0.1 * gr
            vi = 0.999 * l[v].double() + 0.001 * gr * gr
            new[key].append(l[key].double() - LR * (mi / (1.0 - 0.9 ** t)) / (torch.sqrt(vi / (1.0 - 0.999 ** t)) + 1e-8))
            new[m].append(mi)
            new[v].append(vi)
    return new


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "sweep":
        fields = []
        for it in _sweep_items(case, seed):
            c = dict(lattice="D2Q9", order=it["order"], tau=it["tau"], tr=0.0, forcing="guo", collision="srt")
            rho0 = _droplet((it["side"],) * 2, it["R"], RHO_L, RHO_V, 2.0, it["seed"])
            fields.append(sum(_Exact(rho0, c, it["G"]).step(case["steps"]).f).cpu().numpy().T)
        return dict(fields=fields, steps=None, by=None)
    rho0 = _density(case, seed)
    solid = _solid(case) if case.get("walls") else None
    ex = _Exact(rho0, case, -1.0 if case["tr"] else -5.0, solid).step(case["steps"])
    if kind == "grid":
        ref = _median(rho0)
        return torch.stack([(g - w * ref).reshape(-1) for g, w in zip(ex.post, ex.w)])
    rho, j, F = ex.macro()
    u = torch.stack([(jk + 0.5 * Fk) / rho for jk, Fk in zip(j, F)])
    fluid = torch.ones_like(rho, dtype=torch.bool) if solid is None else ~solid
    u = u * fluid
    speed = (u * u).sum(0).sqrt()[fluid]
    obs = [rho.sum(), speed.max(), speed.mean(), (speed * speed).mean().sqrt(), rho[case["ny"] // 2, case["nx"] // 2],
           rho[0, 0], rho[fluid].min(), rho[fluid].max()]
    return dict(rho=rho.cpu().numpy().T, u=u.cpu().numpy().transpose(0, 2, 1), steps=None,
                obs=np.array([float(v) for v in obs]))
