"""The work that users of this library have it do, as cases whose speed and outputs are followed.

Every case goes through the public entry points of `paper_1410_2569_amd`. The kinds:

    steer       a few steps, then the observables: an interactive run or a parameter scan that
                looks at the droplet often (latency and launches count)
    forward     a run of many steps of one lattice, then its observables and density field
    spreading   dynamic wetting (wet-node walls, piecewise EOS): the contact line recorded on the
                device every few steps
    ensemble    many lattices together: an uneven sweep over wall forces and viscosity ratios, the
                static-angle points of one setup, or pillared surfaces given as solid masks
    gradient    one training step of the wetting objective: loss and dL/dG_w through autograd
    ens_grad    the same for an ensemble, with the library's own forward / loss / backward calls
    checkpoint  a state saved to the host and loaded back
    state_obs   observables of populations that the caller holds on the device

All arithmetic is binary64. `exact` states the model once more in plain torch on the CPU.
"""
import math

import numpy as np
import torch

import paper_1410_2569_amd as L
from paper_1410_2569_amd.autograd import lbm_run

# Carnahan-Starling fluid at density ratio 500 (configs/cs_ratio500.json) and the relaxation rates.
CS = dict(eos="cs", a=0.5, b=4.0, R=1.0, T=0.024461878423483633, sigma=0.11244,
          rho_l=0.445063267033785, rho_v=0.0008901265340675707)
# The paper's piecewise EOS (Eq. 15) at 500 : 1 with its spinodal densities.
PW = dict(eos="piecewise", th_v=0.64 / 3.0, th_m=-0.04 / 3.0, th_l=1.0 / 3.0, sigma=0.084,
          rho_l=500.0, rho_v=1.0, rho1=1.3585915514243099, rho2=481.04215601439284)
RATES = dict(s_rho=1.0, s_e=0.8, s_zeta=0.8, s_j=1.0, s_q=1.1, G=-1.0)
FORMS = ("rho", "psi", "modpsi")
# Bottom-wall G_w per force and EOS, inside the intervals that stay stable for long runs.
GW_CS = {"rho": (-0.12, 0.25), "psi": (-0.06, 0.02), "modpsi": (-0.15, 0.35)}
GW_PW = {"rho": (-0.4, 0.6), "psi": (-3.0, 4.0), "modpsi": (-0.5, 0.8)}
TWO_STEP = {"tile": 1, "schedule": 2}  # what the autotuner picks for filled-chip ensembles
FLOPS = 300.0                          # FP64 operations of one lattice update
FLOPS_ADJ = 1100.0                     # forward, its recomputation and the reverse step
OBS = ("rho_min", "rho_max", "umax", "umax_liquid", "mass", "theta_deg", "xc", "yc", "r")
EXACT_UPDATES = 2.7e7                  # lattice updates that `exact` can do in its time


def listed():
    return [
        # a scan that looks at the droplet every ten steps, on the paper's smallest lattice
        dict(name="steer_120x60", kind="steer", nx=120, ny=60, steps=10, form="psi", ratio=1.0),
        # one lattice too small to fill the GPU, an odd number of steps
        dict(name="forward_256x128", kind="forward", nx=256, ny=128, steps=501, form="modpsi",
             ratio=5.0),
        # the benchmark's sweep lattice
        dict(name="forward_1024x512", kind="forward", nx=1024, ny=512, steps=500, form="rho",
             ratio=1.0),
        # a large lattice of ragged size (no multiple of any tile), periodic in y
        dict(name="forward_1500x1001_periodic", kind="forward", nx=1500, ny=1001, steps=200,
             form="modpsi", ratio=15.0, walls=0),
        # dynamic wetting in the paper's setup, the contact line every ten steps
        dict(name="spreading_300x102", kind="spreading", nx=300, ny=102, steps=600, every=10,
             form="modpsi"),
        # the uneven 96-lattice sweep
        dict(name="ensemble_96_uneven", kind="ensemble", setup="uneven", count=96, nx=512,
             steps=400),
        # every static-angle point of the paper's setup at once
        dict(name="ensemble_20_paper_300x102", kind="ensemble", setup="paper", count=20, nx=300,
             ny=102, steps=300),
        # pillared surfaces (solid masks)
        dict(name="ensemble_4_pillars_300x150", kind="ensemble", setup="pillars", count=4, nx=300,
             ny=150, steps=140),
        # the largest lattices: chemically patterned walls, several droplets each
        dict(name="ensemble_8_striped_2048x1024", kind="ensemble", setup="striped", count=8,
             nx=2048, ny=1024, steps=300),
        # one optimisation step of a wall pattern
        dict(name="gradient_256x128", kind="gradient", nx=256, ny=128, steps=200, K=14,
             form="modpsi"),
        # gradients of an ensemble of large lattices
        dict(name="ens_grad_4_1536x768", kind="ens_grad", count=4, nx=1536, ny=768, steps=60, K=8),
        # a serving loop that asks for the observables of fields it holds itself
        dict(name="state_obs_1024x512", kind="state_obs", nx=1024, ny=512, form="modpsi"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["steer", "forward", "forward", "spreading", "ensemble", "ensemble",
                       "gradient", "ens_grad", "checkpoint", "state_obs"])
    form = rng.choice(FORMS)
    ratio = rng.choice([1.0, 5.0, 15.0])
    if kind == "steer":
        nx = _log(rng, 60, 500)
        return dict(kind=kind, nx=nx, ny=max(34, nx // 2 + rng.randint(0, 3)),
                    steps=rng.randint(1, 20), form=form, ratio=ratio)
    if kind == "forward":
        nx = _log(rng, 90, 2200)
        ny = max(40, nx // 2 + rng.randint(-3, 3))
        return dict(kind=kind, nx=nx, ny=ny, steps=max(60, min(1000, int(1.5e8 / (nx * ny)))) +
                    rng.randint(0, 1), form=form, ratio=ratio, walls=rng.choice([1, 1, 0]))
    if kind == "spreading":
        return dict(kind=kind, nx=rng.randint(200, 600), ny=rng.randint(80, 160),
                    steps=60 * rng.randint(2, 8), every=rng.choice([2, 5, 10, 20]), form=form)
    if kind == "ensemble":
        setup = rng.choice(["uneven", "paper", "pillars", "striped"])
        steps = rng.randint(60, 300)
        if setup == "uneven":
            return dict(kind=kind, setup=setup, count=_log(rng, 6, 120), nx=512, steps=steps)
        if setup == "striped":
            nx = _log(rng, 700, 2100)
            return dict(kind=kind, setup=setup, count=rng.randint(2, 6), nx=nx, ny=nx // 2,
                        steps=60 + rng.randint(0, 40))
        return dict(kind=kind, setup=setup, count=_log(rng, 2, 24), nx=rng.randint(250, 420),
                    ny=rng.randint(120, 180), steps=steps)
    if kind == "gradient":
        nx = _log(rng, 100, 1100)
        return dict(kind=kind, nx=nx, ny=max(60, nx // 2 + rng.randint(-2, 2)),
                    steps=rng.randint(40, 200), K=rng.randint(6, 20), form=form)
    if kind == "ens_grad":
        nx = _log(rng, 120, 1500)
        return dict(kind=kind, count=rng.randint(2, 4), nx=nx, ny=max(64, nx // 2),
                    steps=rng.randint(20, 60), K=rng.randint(4, 10))
    nx = _log(rng, 100, 1400)
    return dict(kind=kind, nx=nx, ny=max(50, nx // 2 + rng.randint(-3, 3)), form=form)


# ---- inputs ------------------------------------------------------------------------------------

def _params(case, **over):
    ratio = case.get("ratio", 1.0)
    p = dict(RATES, **CS, nx=case["nx"], ny=case["ny"], walls=case.get("walls", 1), ghost=1,
             wall_force=case.get("form", "modpsi"))
    # liquid viscosity 1/30 with a viscosity ratio, else the single tau of the paper
    p["tau_l"] = 1.1 if ratio == 1.0 else 0.6
    p["tau_v"] = 1.1 if ratio == 1.0 else 0.1 * ratio + 0.5
    p.update(over)
    return p


def _field(nx, ny, rho_l, rho_v, drops, width, seed, solid_rows):
    """Droplets (x0, y0, radius) with tanh edges in their vapour, jittered by 1e-3: (ny, nx)."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    y = torch.arange(ny, dtype=torch.float64, device=dev)[:, None]
    x = torch.arange(nx, dtype=torch.float64, device=dev)[None, :]
    rho = torch.full((ny, nx), -math.inf, dtype=torch.float64, device=dev)
    for x0, y0, r in drops:
        d = torch.sqrt((x - x0) ** 2 + (y - y0) ** 2)
        rho = torch.maximum(rho, 0.5 * (rho_l + rho_v) -
                            0.5 * (rho_l - rho_v) * torch.tanh(2.0 * (d - r) / width))
    g = torch.Generator(device="cpu").manual_seed(seed)
    u = torch.rand((ny, nx), dtype=torch.float64, generator=g).to(dev)
    rho = rho * (1.0 + 1e-3 * (2.0 * u - 1.0))
    if solid_rows:
        rho[0] = 0.0
        rho[-1] = 0.0
    return rho.cpu().numpy()


def _single(case, seed):
    """Parameters, G_w and initial density of one lattice."""
    r = np.random.RandomState(seed % (1 << 31))
    nx, ny = case["nx"], case["ny"]
    p = _params(case)
    gw = np.zeros((2, nx))
    if p["walls"]:
        lo, hi = GW_CS[p["wall_force"]]
        gw[0] = lo + (hi - lo) * r.rand()
        y0 = 0.5
    else:
        y0 = ny / 2.0
    rad = (0.15 + 0.12 * r.rand()) * min(nx, 2 * ny)
    return p, gw, _field(nx, ny, p["rho_l"], p["rho_v"], [(nx / 2.0, y0, rad)], 2.0, seed,
                         p["walls"] != 0)


def _paper(case, r, form):
    p = dict(RATES, **PW, nx=case["nx"], ny=case["ny"], walls=2, ghost=1, wall_force=form,
             tau_l=1.1, tau_v=1.1)
    lo, hi = GW_PW[form]
    gw = np.zeros((2, case["nx"]))
    gw[0] = lo + (hi - lo) * r.rand()
    return p, gw


def _smooth(nx, r, mean, amp):
    x = np.arange(nx)
    g = sum(r.uniform(0.5, 1.0) * np.sin(2 * np.pi * k * x / nx + r.uniform(0, 6.28))
            for k in range(1, 5))
    out = np.zeros((2, nx))
    out[0] = mean + amp * g / np.abs(g).max()
    return out


def _instances(case, seed):
    """(params, G_w, rho0, solid or None) of every instance of an ensemble."""
    r = np.random.RandomState(seed % (1 << 31))
    out = []
    for i in range(case["count"]):
        if case["kind"] == "ens_grad":
            nx, ny = case["nx"], case["ny"]
            p = _params(dict(case, form="modpsi"))
            rad = (0.12 + 0.1 * r.rand()) * nx
            out.append((p, _smooth(nx, r, -0.05, 0.05),
                        _field(nx, ny, p["rho_l"], p["rho_v"], [(nx / 2.0, 0.5, rad)], 2.0,
                               seed + i, True), None))
        elif case["setup"] == "uneven":
            # sizes cycle so that every seed is the same amount of work
            nx = (128, 192, 256, 384, 512)[(i * 7 + i // 5) % 5]
            c = dict(case, nx=nx, ny=nx // 2, form=FORMS[i % 3], ratio=(1.0, 5.0, 15.0)[i // 3 % 3])
            p, gw, rho = _single(c, seed + i)
            out.append((p, gw, rho, None))
        elif case["setup"] == "striped":
            nx, ny = case["nx"], case["ny"]
            p = _params(dict(case, form="modpsi"))
            gw = np.zeros((2, nx))
            gw[0] = np.where((np.arange(nx) // 64) % 2 == 0, -0.1, 0.2)
            drops = [((k + 0.5) * nx / 6.0, 0.5, (0.02 + 0.04 * r.rand()) * nx) for k in range(6)]
            out.append((p, gw, _field(nx, ny, p["rho_l"], p["rho_v"], drops, 2.0, seed + i, True),
                        None))
        elif case["setup"] == "paper":
            p, gw = _paper(case, r, FORMS[i % 3])
            out.append((p, gw, _field(case["nx"], case["ny"], 500.0, 1.0,
                                      [(case["nx"] / 2.0, 26.0, 30.0)], 4.0, seed + i, True), None))
        else:  # pillars 20 high and 6 wide, 3 apart, on a flat base
            nx, ny = case["nx"], case["ny"]
            solid = np.zeros((ny, nx), np.uint8)
            solid[0] = solid[-1] = 1
            solid[1:21, (np.arange(nx) % 9) < 6] = 1
            form = ("rho", "modpsi")[i % 2]
            gw = np.where(solid != 0, {"rho": -1.86, "modpsi": -2.76}[form] * (1 + 0.02 * r.rand()),
                          0.0)
            gw[-1] = 0.0
            rho = _field(nx, ny, 500.0, 1.0, [(nx / 2.0, 50.5, 30.0)], 4.0, seed + i, False)
            rho[solid != 0] = 0.0
            p = dict(RATES, **PW, nx=nx, ny=ny, walls=3, ghost=0, wall_force=form, tau_l=1.1,
                     tau_v=1.1)
            out.append((p, gw, rho, solid))
    return out


def _spreading(case, seed):
    r = np.random.RandomState(seed % (1 << 31))
    p, gw = _paper(case, r, case["form"])
    return p, gw, _field(case["nx"], case["ny"], 500.0, 1.0, [(case["nx"] / 2.0, 33.0, 30.0)], 4.0,
                         seed, True)


def _gradient(case, seed):
    r = np.random.RandomState(seed % (1 << 31))
    nx, ny = case["nx"], case["ny"]
    p = _params(case)
    mean, amp = {"rho": (-0.05, 0.03), "psi": (-0.03, 0.02), "modpsi": (-0.1, 0.05)}[case["form"]]
    return p, _smooth(nx, r, mean, amp), _field(nx, ny, p["rho_l"], p["rho_v"],
                                                [(nx / 2.0, 0.5, 0.16 * nx)], 2.0, seed, True)


def _held_state(case, seed):
    """Populations near equilibrium that a caller holds: t_a rho with small random currents."""
    p, gw, rho = _single(case, seed)
    g = torch.Generator(device="cpu").manual_seed(seed + 1)
    t = torch.tensor([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4, dtype=torch.float64)[:, None, None]
    f = t * torch.from_numpy(rho) * (1 + 1e-3 * (torch.rand((9,) + rho.shape, dtype=torch.float64,
                                                          generator=g) - 0.5))
    return p, gw, f


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("steer", "forward", "checkpoint"):
        return case, L.Sim(*_single(case, seed))
    if kind == "spreading":
        return case, L.Sim(*_spreading(case, seed))
    if kind == "ensemble":
        ps, gws, rhos, solids = zip(*_instances(case, seed))
        return case, L.Batch(list(ps), list(gws), list(rhos), tune=TWO_STEP,
                             solids=list(solids) if solids[0] is not None else None)
    if kind == "gradient":
        p, gw, rho = _gradient(case, seed)
        sim = L.Sim(p, gw, rho)
        return case, sim, sim.save_state(), torch.tensor(gw, device="cuda", requires_grad=True)
    if kind == "ens_grad":
        ps, gws, rhos, _ = zip(*_instances(case, seed))
        b = L.Batch(list(ps), list(gws), list(rhos), tune=TWO_STEP)
        return case, b, b.adjoint_workspace(case["steps"], case["K"])
    p, gw, f = _held_state(case, seed)
    return case, L.make_params(p), f.cuda(), torch.from_numpy(gw).cuda()


def _obs(o):
    return {k: float(o[k]) for k in OBS}


def _obs_table(obs):
    return np.array([[o[k] for k in OBS] for o in obs])


def _read_out(case):
    """Instances whose populations a pass reads out."""
    return [0] if case["setup"] == "striped" else [0, case["count"] - 1]


def run(state):
    case = state[0]
    kind = case["kind"]
    if kind in ("steer", "forward"):
        sim = state[1]
        sim.step(case["steps"])
        return {"obs": _obs(sim.observables()), "rho": sim.rho()}
    if kind == "spreading":
        line = state[1].record_contact_line(case["steps"], case["every"])
        return {"line": line, "rho": state[1].rho()}
    if kind == "ensemble":
        b = state[1]
        b.step(case["steps"])
        return {"obs": _obs_table(b.observables()), "f": [b.f(i) for i in _read_out(case)]}
    if kind == "gradient":
        _, sim, blob, gw = state
        gw.grad = None
        loss = lbm_run(gw, sim, blob, case["steps"], case["K"])
        loss.backward()
        return {"loss": loss, "grad": gw.grad}
    if kind == "ens_grad":
        _, b, ws = state
        b.forward_ckpt(case["steps"], case["K"], ws)
        return {"loss": b.loss(), "grad": b.backward(case["steps"], case["K"], ws)}
    if kind == "checkpoint":
        sim = state[1]
        blob = sim.save_state()
        sim.load_state(blob)
        return {"state": np.frombuffer(blob, dtype=np.float64, offset=32),
                "rho": sim.rho()}
    _, q, f, gw = state
    return {"obs": _obs(L.observables_of_state(q, f, gw))}


def work(case):
    """One pass: each lattice's state read once and written once and the outputs written once;
    the operations of every lattice update."""
    kind = case["kind"]
    if kind == "ensemble" and case["setup"] == "uneven":
        sizes = [(128, 192, 256, 384, 512)[(i * 7 + i // 5) % 5] for i in range(case["count"])]
        sizes = [n * (n // 2) for n in sizes]
    else:
        sizes = [case["nx"] * case["ny"]] * case.get("count", 1)
    nodes = sum(sizes)
    if kind in ("steer", "forward", "spreading"):
        return {"bytes": 152.0 * nodes, "flops": FLOPS * nodes * case["steps"]}
    if kind == "ensemble":
        read = sum(sizes[i] for i in _read_out(case))
        return {"bytes": 144.0 * nodes + 72.0 * read, "flops": FLOPS * nodes * case["steps"]}
    if kind == "gradient":
        return {"bytes": 72.0 * nodes, "flops": FLOPS_ADJ * nodes * case["steps"]}
    if kind == "ens_grad":
        return {"bytes": 144.0 * nodes, "flops": FLOPS_ADJ * nodes * case["steps"]}
    if kind == "checkpoint":
        return {"bytes": 296.0 * nodes, "flops": 8.0 * nodes}
    return {"bytes": 72.0 * nodes, "flops": 80.0 * nodes}


# ---- the model in plain torch, on the CPU --------------------------------------------------------

EX = (0, 1, 0, -1, 0, 1, -1, -1, 1)
EY = (0, 0, 1, 0, -1, 1, 1, -1, -1)
OPP = (0, 3, 4, 1, 2, 7, 8, 5, 6)
WC = (0.0,) + (1 / 3,) * 4 + (1 / 12,) * 4
MAT = torch.tensor([[1, 1, 1, 1, 1, 1, 1, 1, 1], [-4, -1, -1, -1, -1, 2, 2, 2, 2],
                    [4, -2, -2, -2, -2, 1, 1, 1, 1], [0, 1, 0, -1, 0, 1, -1, -1, 1],
                    [0, -2, 0, 2, 0, 1, -1, -1, 1], [0, 0, 1, 0, -1, 1, 1, -1, -1],
                    [0, 0, -2, 0, 2, 1, 1, -1, -1], [0, 1, -1, 1, -1, 0, 0, 0, 0],
                    [0, 0, 0, 0, 0, 1, -1, 1, -1]], dtype=torch.float64)
MINV = torch.linalg.inv(MAT)


def _shift(v, dx, dy):
    """v(x + dx, y + dy), periodic."""
    return torch.roll(v, shifts=(-dy, -dx), dims=(-2, -1))


class _Model:
    """One lattice: the time step of the method on pre-collision populations (9, ny, nx)."""

    def __init__(self, p, gw, solid=None):
        self.p = p
        ny, nx = p["ny"], p["nx"]
        self.rows = p["walls"] in (1, 2)
        if solid is None:
            solid = np.zeros((ny, nx), bool)
            if self.rows:
                solid[0] = solid[-1] = True
        self.solid = torch.from_numpy(np.asarray(solid) != 0)
        self.from_solid = [_shift(self.solid, -EX[a], -EY[a]) for a in range(9)]
        gw = torch.as_tensor(gw, dtype=torch.float64)
        if self.rows:
            mid = torch.zeros((ny - 2, nx), dtype=torch.float64)
            gw = torch.cat([gw[:1], mid, gw[1:]], 0)
        elif p["walls"] == 0:
            gw = torch.zeros((ny, nx), dtype=torch.float64)
        gs = torch.where(self.solid, gw, torch.zeros_like(gw))
        self.ax = sum(WC[a] / 3 * EX[a] * _shift(gs, EX[a], EY[a]) for a in range(1, 9))
        self.ay = sum(WC[a] / 3 * EY[a] * _shift(gs, EX[a], EY[a]) for a in range(1, 9))

    def rest(self, rho0):
        rho = torch.where(self.solid, torch.zeros((), dtype=torch.float64), torch.from_numpy(rho0))
        return torch.stack([(4 / 9 if a == 0 else 1 / 9 if a < 5 else 1 / 36) * rho
                            for a in range(9)])

    def pressure(self, rho):
        p = self.p
        if p["eos"] == "cs":
            e = p["b"] * rho / 4
            return (rho * p["R"] * p["T"] * (1 + e + e * e - e ** 3) / (1 - e) ** 3 -
                    p["a"] * rho * rho)
        p1 = p["rho1"] * p["th_v"]
        p2 = p1 + (p["rho2"] - p["rho1"]) * p["th_m"]
        return torch.where(rho <= p["rho1"], rho * p["th_v"],
                           torch.where(rho <= p["rho2"], p1 + (rho - p["rho1"]) * p["th_m"],
                                       p2 + (rho - p["rho2"]) * p["th_l"]))

    def forces(self, F):
        p, S = self.p, self.solid
        one = torch.full((), 0.5 * (p["rho_l"] + p["rho_v"]), dtype=torch.float64)
        rho = torch.where(S, one, F.sum(0))
        psi = torch.sqrt(2 * (self.pressure(rho) - rho / 3) / p["G"])
        psi = torch.where(S, torch.zeros((), dtype=torch.float64), psi)
        nb = torch.cat([psi[1:2], psi[1:-1], psi[-2:-1]], 0) if self.rows and p["ghost"] else psi
        sx = sum(WC[a] * EX[a] * _shift(nb, EX[a], EY[a]) for a in range(1, 9) if EX[a])
        sy = sum(WC[a] * EY[a] * _shift(nb, EX[a], EY[a]) for a in range(1, 9) if EY[a])
        pre = {"rho": rho, "psi": psi, "modpsi": psi * psi}[p["wall_force"]]
        fx, fy = -p["G"] * psi * sx - pre * self.ax, -p["G"] * psi * sy - pre * self.ay
        vx = ((F[1] - F[3]) + (F[5] + F[8]) - (F[6] + F[7]) + fx / 2) / rho
        vy = ((F[2] - F[4]) + (F[5] + F[6]) - (F[7] + F[8]) + fy / 2) / rho
        return rho, fx, fy, vx, vy, p["G"] ** 2 * (sx * sx + sy * sy)

    def step(self, F):
        p = self.p
        rho, fx, fy, vx, vy, s2 = self.forces(F)
        v2, vF = vx * vx + vy * vy, vx * fx + vy * fy
        m = torch.tensordot(MAT, F, 1)
        meq = torch.stack([rho, rho * (-2 + 3 * v2), rho * (1 - 3 * v2), rho * vx, -rho * vx,
                           rho * vy, -rho * vy, rho * (vx * vx - vy * vy), rho * vx * vy])
        nl, nv = (p["tau_l"] - 0.5) / 3, (p["tau_v"] - 0.5) / 3
        phi = torch.clamp((rho - p["rho_v"]) / (p["rho_l"] - p["rho_v"]), 0.0, 1.0)
        snu = 1 / (3 * (nv + phi * (nl - nv)) + 0.5)
        o = torch.ones_like(rho)
        s = torch.stack([p["s_rho"] * o, p["s_e"] * o, p["s_zeta"] * o, p["s_j"] * o, p["s_q"] * o,
                         p["s_j"] * o, p["s_q"] * o, snu, snu])
        c = 12 * p["sigma"] * s2
        src = torch.stack([0 * rho, 6 * vF + c / (1 / p["s_e"] - 0.5),
                           -6 * vF - c / (1 / p["s_zeta"] - 0.5), fx, -fx, fy, -fy,
                           2 * (vx * fx - vy * fy), vx * fy + vy * fx])
        fs = torch.tensordot(MINV, m - s * (m - meq) + (1 - s / 2) * src, 1)
        out = [torch.where(self.from_solid[a], fs[OPP[a]], _shift(fs[a], -EX[a], -EY[a]))
               for a in range(9)]
        if p["walls"] == 2:  # non-slip wet nodes on the wall planes
            d13 = out[1] - out[3]
            bot, top = torch.zeros_like(self.solid), torch.zeros_like(self.solid)
            bot[1], top[-2] = True, True
            new = {2: out[4], 5: out[7] - d13 / 2 - (fx + fy) / 4,
                   6: out[8] + d13 / 2 + (fx - fy) / 4}
            for a, v in new.items():
                out[a] = torch.where(bot, v, out[a])
            new = {4: out[2], 7: out[5] + d13 / 2 + (fx + fy) / 4,
                   8: out[6] - d13 / 2 - (fx - fy) / 4}
            for a, v in new.items():
                out[a] = torch.where(top, v, out[a])
        zero = torch.zeros((), dtype=torch.float64)
        return torch.where(self.solid, zero, torch.stack(out))

    def run(self, F, n):
        for _ in range(n):
            F = self.step(F)
        return F

    def observables(self, F):
        p = self.p
        rho, _, _, vx, vy, _ = self.forces(F)
        fluid = ~self.solid
        r, u = rho.numpy(), torch.sqrt(vx * vx + vy * vy)
        mid = 0.5 * (p["rho_l"] + p["rho_v"])
        liquid = fluid & (rho >= mid)
        yw = 1.0 if p["walls"] == 2 else 0.5
        fl = fluid.numpy()
        X, Y = [], []
        for dy, dx in ((0, 1), (1, 0)):  # crossings on horizontal and vertical fluid edges
            a, b = r[:r.shape[0] - dy, :r.shape[1] - dx], r[dy:, dx:]
            on = fl[:r.shape[0] - dy, :r.shape[1] - dx] & fl[dy:, dx:] & ((a >= mid) != (b >= mid))
            yy, xx = np.nonzero(on)
            t = (mid - a[on]) / (b[on] - a[on])
            keep = yy + dy * t >= yw + 3.0
            X.append((xx + dx * t)[keep])
            Y.append((yy + dy * t)[keep])
        X, Y = np.concatenate(X) - 0.5 * p["nx"], np.concatenate(Y) - yw
        xc = yc = rad = theta = math.nan
        if len(X) >= 6:
            A = np.column_stack([X, Y, np.ones_like(X)])
            (D, E, H), *_ = np.linalg.lstsq(A, -(X * X + Y * Y), rcond=None)
            rad = math.sqrt(D * D / 4 + E * E / 4 - H)
            xc, yc = -D / 2 + 0.5 * p["nx"], -E / 2 + yw
            cth = (yw - yc) / rad
            theta = math.degrees(math.acos(cth)) if abs(cth) <= 1 else math.nan
        return {"rho_min": float(rho[fluid].min()), "rho_max": float(rho[fluid].max()),
                "umax": float(u[fluid].max()),
                "umax_liquid": float(u[liquid].max()) if bool(liquid.any()) else 0.0,
                "mass": float(rho[fluid].sum()), "theta_deg": theta, "xc": xc, "yc": yc, "r": rad}

    def contact_line(self, F, row=1):
        mid = 0.5 * (self.p["rho_l"] + self.p["rho_v"])
        r = F[:, row].sum(0).numpy()
        a, b = r[:-1], r[1:]
        x = np.arange(len(a)) + (mid - a) / np.where(a == b, 1.0, b - a)
        up, down = x[(a < mid) & (b >= mid)], x[(a >= mid) & (b < mid)]
        if not len(up) or not len(down) or up.min() >= down.max():
            return math.nan, math.nan
        return up.min(), down.max()

    def objective(self, F):
        p = self.p
        phi = (F[:, 1:-1].sum(0) - p["rho_v"]) / (p["rho_l"] - p["rho_v"])
        y = torch.arange(1, p["ny"] - 1, dtype=torch.float64)[:, None] - 0.5
        return (phi * y).sum() / phi.sum() + phi[0].sum()


def _loss_grad(p, gw, rho0, n):
    from torch.utils.checkpoint import checkpoint
    g = torch.tensor(gw, dtype=torch.float64, requires_grad=True)
    m = _Model(p, g)
    F = m.rest(rho0)
    for i in range(0, n, 10):
        F = checkpoint(m.run, F, min(10, n - i), use_reentrant=False)
    loss = m.objective(F)
    loss.backward()
    return loss.detach(), g.grad


def exact(case, seed):
    kind = case["kind"]
    nodes = case["nx"] * case.get("ny", case["nx"] // 2) * case.get("count", 1)
    if nodes * case.get("steps", 0) * (4 if kind == "gradient" else 8 if kind == "ens_grad" else 1) \
            > EXACT_UPDATES:
        return None
    if kind in ("steer", "forward"):
        p, gw, rho0 = _single(case, seed)
        m = _Model(p, gw)
        F = m.run(m.rest(rho0), case["steps"])
        return {"obs": m.observables(F), "rho": F.sum(0)}
    if kind == "spreading":
        p, gw, rho0 = _spreading(case, seed)
        m = _Model(p, gw)
        F = m.rest(rho0)
        line = [m.contact_line(F)]
        for _ in range(case["steps"] // case["every"]):
            F = m.run(F, case["every"])
            line.append(m.contact_line(F))
        return {"line": np.array(line), "rho": F.sum(0)}
    if kind == "ensemble":
        obs, fs = [], []
        for p, gw, rho0, solid in _instances(case, seed):
            m = _Model(p, gw, solid)
            fs.append(m.run(m.rest(rho0), case["steps"]))
            obs.append(m.observables(fs[-1]))
        return {"obs": _obs_table(obs), "f": [fs[i] for i in _read_out(case)]}
    if kind == "gradient":
        loss, grad = _loss_grad(*_gradient(case, seed), case["steps"])
        return {"loss": loss, "grad": grad}
    if kind == "ens_grad":
        got = [_loss_grad(p, gw, rho0, case["steps"]) for p, gw, rho0, _ in _instances(case, seed)]
        return {"loss": [float(x) for x, _ in got], "grad": [g for _, g in got]}
    if kind == "checkpoint":
        return {"state": None, "rho": _single(case, seed)[2]}
    p, gw, f = _held_state(case, seed)  # solid rows already hold 0
    return {"obs": _Model(p, gw).observables(f)}
