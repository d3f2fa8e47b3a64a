"""Timing cases of the finite-volume framework.

Each case is one piece of work that a user's program does through the public
binding (paper_2602_08670_amd.fv): plain and learned solves from the smallest
grids, where launches count, to the largest; the spherical solver; the network
pass; a training evaluation; a served stream of requests.

  listed()            the cases
  draw(rng)           one more case of the same ranges
  prepare(case, seed) inputs on the GPU (or host requests) and the handles a
                      program keeps
  run(state)          one pass; returns its outputs
  exact(case, seed)   what run returns, from plain torch in double precision
  work(case)          bytes and operations a pass cannot do without
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2602_08670_amd import fv

G, GAMMA = 9.81, 1.4
F64 = torch.float64

# Training step of the learned coarse solver: 32 steps of a 2048^2 run of the
# unit square (CFL 0.4 in the two-axis form, depth <= 1.6, margin 1.25), cells
# of width 1/64.
LEARNED_DT = 32 * 0.4 / (1.25 * 2.0 * math.sqrt(G * 1.6) * 2048)
# The same for the learned Euler solver: 8 steps of a 512^2 run (|u| + c <= 4.3).
EULER_DT = 8 * 0.4 / (1.25 * 2.0 * 4.3 * 512)

# Layers of the coefficient network, (input, output) channels.
SWE_NET = [(3, 32), (32, 32), (32, 32), (32, 32), (32, 72)]
EULER_NET = [(4, 32), (32, 32), (32, 32), (32, 32), (32, 96)]

FLUXES = {"hlle": fv.FV_FLUX_HLLE, "rusanov": fv.FV_FLUX_RUSANOV, "roe": fv.FV_FLUX_ROE}


def listed():
    return [
        # a small coarse solve, as a parameter study runs by the thousand:
        # every launch is short, the time is launches and latency
        {"name": "swe_bed_64", "kind": "plain", "eqn": "swe", "bed": True, "wall": True, "prec": "f32", "nx": 64,
         "ny": 64, "flux": "hlle", "recon": "minmod", "rk": 2, "steps": 32},
        # the benchmark's workload: shallow water over a bed between walls
        {"name": "swe_bed_1024", "kind": "plain", "eqn": "swe", "bed": True, "wall": True, "prec": "f32", "nx": 1024,
         "ny": 1024, "flux": "hlle", "recon": "minmod", "rk": 2, "steps": 16},
        # Euler quadrants between walls on a ragged grid (cut last tiles)
        {"name": "euler_1000x700", "kind": "plain", "eqn": "euler", "bed": False, "wall": True, "prec": "f32",
         "nx": 1000, "ny": 700, "flux": "hlle", "recon": "minmod", "rk": 2, "steps": 16},
        # double precision, the three-stage scheme and the Roe flux, as a
        # convergence study runs them
        {"name": "swe_roe_rk3_f64_250", "kind": "plain", "eqn": "swe", "bed": False, "wall": False, "prec": "f64",
         "nx": 250, "ny": 250, "flux": "roe", "recon": "minmod", "rk": 3, "steps": 16},
        # training data: a fine run at the fixed step, one coarse snapshot
        # (32 fine steps, 32x block averages)
        {"name": "fine_2048_coarsen32", "kind": "fine", "n": 2048, "factor": 32},
        # rollout of the learned coarse solver from an initial state
        {"name": "learned_64", "kind": "learned", "scheme": "learned", "nx": 64, "ny": 64, "steps": 64},
        # the same on a larger domain at the training resolution
        {"name": "learned_256", "kind": "learned", "scheme": "learned", "nx": 256, "ny": 256, "steps": 16},
        # learned Euler rollouts of a small ensemble
        {"name": "euler_learned_4x64", "kind": "euler_learned", "B": 4, "nx": 64, "ny": 64, "steps": 32},
        # coefficients of a batch of coarse states (analysis, dataset scoring)
        {"name": "network_256x64", "kind": "network", "B": 256, "nx": 64, "ny": 64},
        # one training evaluation: unrolled loss and its gradients
        {"name": "train_16x64_T8", "kind": "train", "scheme": "learned", "B": 16, "n": 64, "T": 8},
        # shallow water on the sphere
        {"name": "sphere_512", "kind": "sphere", "n": 512, "prec": "f32", "flux": "hlle", "rk": 2, "steps": 8},
        # a mixed stream of plain and learned requests through the server
        {"name": "serve_mixed_24", "kind": "serve", "requests": 24, "steps": 32, "largest": 512, "mix": 0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plain", "plain", "plain", "plain", "fine", "learned", "learned", "euler_learned", "network",
                       "train", "sphere", "serve"])
    if kind == "plain":
        eqn = rng.choice(["swe", "swe", "euler"])
        prec = rng.choice(["f32", "f32", "f32", "f64"])
        usual = rng.random() < 0.6  # the default scheme, else any flux, reconstruction and stages
        side = _log_int(rng, 24, 1400 if prec == "f32" else 700)
        return {"kind": kind, "eqn": eqn, "bed": eqn == "swe" and rng.random() < 0.6, "wall": rng.random() < 0.6,
                "prec": prec, "nx": side, "ny": max(16, int(side * rng.uniform(0.5, 1.1))),
                "flux": "hlle" if usual else rng.choice(sorted(FLUXES)),
                "recon": "minmod" if usual or rng.random() < 0.7 else "first",
                "rk": 2 if usual else rng.choice([1, 2, 3]), "steps": rng.randint(8, 32)}
    if kind == "fine":
        factor = rng.choice([8, 16, 32])
        return {"kind": kind, "n": factor * rng.randint(24, 64), "factor": factor}
    if kind == "learned":
        return {"kind": kind, "scheme": rng.choice(["learned", "learned", "direct", "blend"]),
                "nx": 16 * rng.randint(2, 16), "ny": 8 * rng.randint(4, 32), "steps": rng.randint(8, 24)}
    if kind == "euler_learned":
        return {"kind": kind, "B": rng.randint(1, 8), "nx": 16 * rng.randint(2, 6), "ny": 8 * rng.randint(3, 12),
                "steps": rng.randint(8, 32)}
    if kind == "network":
        return {"kind": kind, "B": _log_int(rng, 1, 256), "nx": 16 * rng.randint(2, 5), "ny": 8 * rng.randint(3, 8)}
    if kind == "train":
        return {"kind": kind, "scheme": rng.choice(["learned", "learned", "direct", "blend", "euler"]),
                "B": rng.randint(1, 16), "n": 16 * rng.randint(2, 4), "T": rng.randint(1, 8)}
    if kind == "sphere":
        prec = rng.choice(["f32", "f64"])
        return {"kind": kind, "n": _log_int(rng, 32, 640 if prec == "f32" else 360), "prec": prec,
                "flux": rng.choice(["hlle", "hlle", "rusanov", "roe"]), "rk": rng.choice([2, 2, 3]),
                "steps": rng.randint(4, 12)}
    return {"kind": kind, "requests": rng.randint(8, 24), "steps": rng.randint(16, 48),
            "largest": rng.choice([128, 256, 512]), "mix": rng.randint(1, 1 << 20)}


# ------------------------------------------------------------------- inputs

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _mesh(nx, ny):
    x = (torch.arange(nx, dtype=F64, device=_device()) + 0.5) / nx
    y = (torch.arange(ny, dtype=F64, device=_device()) + 0.5) / ny
    return x[None, :], y[:, None]


def _bumps(nx, ny, rng, count, amp, width, periodic, periods=(1.0, 1.0)):
    """Sum of `count` Gaussians: amplitude +-U(amp) if its lower end is
    positive, else U(amp); exp(-r^2 / w^2), w ~ U(width), r in units of
    1/periods of the domain."""
    x, y = _mesh(nx, ny)
    out = torch.zeros(ny, nx, dtype=F64, device=_device())
    for _ in range(count):
        a = rng.uniform(*amp) * (1.0 if amp[0] <= 0 or rng.random() < 0.5 else -1.0)
        w = rng.uniform(*width)
        dx, dy = (x - rng.random()).abs(), (y - rng.random()).abs()
        if periodic:
            dx, dy = torch.minimum(dx, 1.0 - dx), torch.minimum(dy, 1.0 - dy)
        out += a * torch.exp(-((dx * periods[0]) ** 2)[...] / w ** 2) * torch.exp(-((dy * periods[1]) ** 2) / w ** 2)
    return out


def _plain_input(eqn, bed, nx, ny, seed):
    """State (double) and bed (or None): a perturbed surface over Gaussian
    hills at rest, or Euler data in four quadrants."""
    rng = np.random.default_rng(seed)
    if eqn == "swe":
        b = _bumps(nx, ny, rng, 8, (0.0, 0.07), (0.03, 0.1), False) if bed else None
        eta = 1.0 + _bumps(nx, ny, rng, 16, (-0.05, 0.05), (0.03, 0.1), False)
        h = (eta if b is None else eta - b).clamp(min=0.05)
        return torch.stack([h, torch.zeros_like(h), torch.zeros_like(h)]), b
    x, y = _mesh(nx, ny)
    q = torch.zeros(4, ny, nx, dtype=F64, device=_device())
    for east in (True, False):
        for north in (True, False):
            rho, p = rng.uniform(0.3, 1.5, size=2)
            u, v = rng.uniform(-0.6, 0.6, size=2)
            m = ((x >= 0.5) == east) & ((y >= 0.5) == north)
            for k, val in enumerate((rho, rho * u, rho * v, p / (GAMMA - 1) + 0.5 * rho * (u * u + v * v))):
                q[k][m] = val
    return q, None


def _smooth_swe(nx, ny, rng):
    """Periodic humps over unit depth, cells of width 1/64."""
    h = 1.0 + _bumps(nx, ny, rng, int(rng.integers(2, 5)), (0.05, 0.15), (0.08, 0.14), True, (nx / 64, ny / 64))
    return torch.stack([h, torch.zeros_like(h), torch.zeros_like(h)])


def _smooth_euler(nx, ny, rng):
    """A uniform drift carrying periodic humps of density and pressure."""
    u, v = rng.uniform(-0.5, 0.5, size=2)
    k = int(rng.integers(2, 5))
    rho = 1.0 + _bumps(nx, ny, rng, k, (0.05, 0.15), (0.08, 0.14), True, (nx / 64, ny / 64))
    p = 1.0 + _bumps(nx, ny, rng, k, (0.05, 0.15), (0.08, 0.14), True, (nx / 64, ny / 64))
    return torch.stack([rho, rho * u, rho * v, p / (GAMMA - 1) + 0.5 * rho * (u * u + v * v)])


def _net_params(layers, seed):
    """Master weights and biases (float32): He-scaled, a small last layer (the
    coefficients stay near their base stencils, as in a trained network)."""
    rng = np.random.default_rng(seed)
    ws, bs = [], []
    for i, (ci, co) in enumerate(layers):
        last = i == len(layers) - 1
        ws.append((rng.standard_normal((co, ci, 3, 3)) * math.sqrt(2.0 / (9 * ci)) * (0.05 if last else 1.0))
                  .astype(np.float32))
        bs.append((rng.standard_normal(co) * 0.01).astype(np.float32))
    return ws, bs


SWE_NORM = ((1.0, 0.0, 0.0), (10.0, 10.0, 10.0))
EULER_NORM = ((1.0, 0.0, 0.0, 2.5), (8.0, 4.0, 4.0, 2.0))
TRAIN_SCALE = {"swe": (0.05, 0.05, 0.05), "euler": (0.1, 0.1, 0.1, 0.2)}


def _model(seed):
    return fv.Model(fv.params_to_vector(*_net_params(SWE_NET, seed)), fv.make_model_desc(*SWE_NORM))


def _batch_input(euler, B, nx, ny, seed):
    rng = np.random.default_rng(seed)
    return torch.stack([(_smooth_euler if euler else _smooth_swe)(nx, ny, rng) for _ in range(B)]).float()


def _train_targets(euler, q0, T):
    """Reference states after 1..T steps: the plain scheme in double."""
    ph = _Physics("euler" if euler else "swe", "hlle", 1 / 64, 1 / 64, False)
    q, out = q0.double(), []
    for _ in range(T):
        q = ph.heun(q, EULER_DT if euler else LEARNED_DT)
        out.append(q.float())
    return torch.stack(out)


def _requests(case, seed):
    """(kind, side, steps, state, bed) of a stream: half shallow water over a
    bed or Euler, half learned shallow water; sides up to case["largest"]."""
    mix = np.random.default_rng(case["mix"])
    out = []
    for k in range(case["requests"]):
        kind = ("swe", "learned", "euler", "learned")[int(mix.integers(0, 4))]
        sides = [n for n in ((32, 64, 128, 256) if kind == "learned" else (64, 128, 256, 512)) if n <= case["largest"]]
        n = sides[int(mix.integers(0, len(sides)))]
        steps = max(1, int(case["steps"] * mix.uniform(0.5, 1.5)))
        if kind == "learned":
            q, b = _smooth_swe(n, n, np.random.default_rng([seed, k])), None
        else:
            q, b = _plain_input(kind, kind == "swe", n, n, [seed, k])
        out.append((kind, n, steps, q.float().cpu().numpy(), None if b is None else b.float().cpu().numpy()))
    return out


# ---------------------------------------------------------- prepare and run

def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "plain":
        q, b = _plain_input(case["eqn"], case["bed"], case["nx"], case["ny"], seed)
        bc = fv.FV_BC_WALL if case["wall"] else fv.FV_BC_PERIODIC
        st["solver"] = fv.Solver(q.cpu().numpy(), None if b is None else b.cpu().numpy(),
                                 prec=fv.FV_F64 if case["prec"] == "f64" else fv.FV_F32, bc_x=bc, bc_y=bc,
                                 flux=FLUXES[case["flux"]], rk_stages=case["rk"],
                                 recon=fv.FV_RECON_MINMOD if case["recon"] == "minmod" else fv.FV_RECON_FIRST,
                                 lx=1.0, ly=case["ny"] / case["nx"])
    elif kind == "fine":
        n = case["n"]
        q = _smooth_swe(64, 64, np.random.default_rng(seed))  # drawn on the coarse grid's scale, refined below
        q = torch.nn.functional.interpolate(q[None], size=(n, n), mode="bilinear")[0]
        st["solver"] = fv.Solver(q.cpu().numpy(), prec=fv.FV_F32, dt_fixed=LEARNED_DT * 64 / n)
    elif kind == "learned":
        nx, ny = case["nx"], case["ny"]
        st["q0"] = _smooth_swe(nx, ny, np.random.default_rng(seed)).float().cpu().numpy()
        st["model"] = _model(seed)
        st["solver"] = fv.Solver(st["q0"], prec=fv.FV_F32, dt_fixed=LEARNED_DT, learned=1, h_ref=1.0, lx=nx / 64,
                                 ly=ny / 64)
    elif kind == "euler_learned":
        B, nx, ny = case["B"], case["nx"], case["ny"]
        st["q0"] = _batch_input(True, B, nx, ny, seed)
        st["q"] = st["q0"].clone()
        st["net"] = fv.EulerLearned(fv.params_to_vector(*_net_params(EULER_NET, seed)), B, nx, ny, EULER_DT,
                                    lx=nx / 64, ly=ny / 64, mean=EULER_NORM[0], inv_std=EULER_NORM[1])
    elif kind == "network":
        st["q"] = _batch_input(False, case["B"], case["nx"], case["ny"], seed)
        st["model"] = _model(seed)
    elif kind == "train":
        euler, B, n, T = case["scheme"] == "euler", case["B"], case["n"], case["T"]
        st["q0"] = _batch_input(euler, B, n, n, seed)
        st["targets"] = _train_targets(euler, st["q0"], T)
        if euler:
            st["net"] = fv.EulerLearned(fv.params_to_vector(*_net_params(EULER_NET, seed)), B, n, n, EULER_DT,
                                        lx=n / 64, ly=n / 64, mean=EULER_NORM[0], inv_std=EULER_NORM[1])
            st["trainer"] = fv.EulerTrainer(st["net"], fv.make_euler_train_config(
                B, n, n, T, EULER_DT, lx=n / 64, ly=n / 64, scale=TRAIN_SCALE["euler"]))
        else:
            st["model"] = _model(seed)
            st["trainer"] = fv.Trainer(st["model"], fv.make_train_config(
                B, n, n, T, LEARNED_DT, lx=n / 64, ly=n / 64, scale=TRAIN_SCALE["swe"],
                direct=case["scheme"] == "direct", blend=case["scheme"] == "blend"))
    elif kind == "sphere":
        q = _sphere_input(case["n"], seed)
        st["solver"] = fv.SphereSolver(q.cpu().numpy(), prec=fv.FV_F64 if case["prec"] == "f64" else fv.FV_F32,
                                       flux=FLUXES[case["flux"]], rk_stages=case["rk"], g=1.0, omega=0.5)
    else:
        st["requests"] = _requests(case, seed)
        st["model"] = _model(seed)
        st["server"] = fv.Server(1 << 30, max_solves=64, steps_per_round=16, model=st["model"])
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("plain", "sphere"):
        state["solver"].run(case["steps"])
        return state["solver"].q
    if kind == "fine":
        s = state["solver"]
        s.run(case["factor"])
        return {"q": s.q, "coarse": fv.coarsen(s.q, case["factor"])}
    if kind == "learned":
        s = state["solver"]
        s.set_state(state["q0"])
        step = {"learned": s.learned_step, "direct": s.direct_step, "blend": s.blend_step}[case["scheme"]]
        step(state["model"], case["steps"], want_stats=False)
        return s.q
    if kind == "euler_learned":
        state["q"].copy_(state["q0"])
        state["net"].step(state["q"], case["steps"])
        return state["q"]
    if kind == "network":
        return state["model"].forward(state["q"])
    if kind == "train":
        tr = state["trainer"]
        loss, _ = tr.step(state["q0"], state["targets"])
        return {"loss": loss, "grads": tr.grads}
    srv, ids = state["server"], []
    for what, n, steps, q, b in state["requests"]:
        kw = {"learned": True, "dt_fixed": LEARNED_DT, "lx": n / 64} if what == "learned" else {}
        ids.append(srv.submit(q, steps, bed=b, **kw))
    while srv.round() != (0, 0):
        pass
    out = []
    for rid, req in zip(ids, state["requests"]):
        out.append(srv.result(rid, req[3].shape))
        srv.release(rid)
    return out


# --------------------------------------------------------------------- work

def _net_flops(layers):
    return sum(2 * 9 * ci * co for ci, co in layers)


# Operations of one cell-update with two stages, an FMA as two, counted from
# the formulas (faces, divergence, stage combine, CFL rate).
STEP_FLOPS = {"swe": 470, "bed": 543, "euler": 715, "sphere": 1000}


def _plain_work(eqn, bed, cells, steps, rk, size):
    nv = 3 if eqn == "swe" else 4
    return {"bytes": cells * size * (2 * nv + (1 if bed else 0)) * steps,
            "flops": cells * steps * rk / 2 * STEP_FLOPS["bed" if bed else eqn]}


def work(case):
    kind = case["kind"]
    if kind == "plain":
        return _plain_work(case["eqn"], case["bed"], case["nx"] * case["ny"], case["steps"], case["rk"],
                           8 if case["prec"] == "f64" else 4)
    if kind == "fine":
        return _plain_work("swe", False, case["n"] ** 2, case["factor"], 2, 4)
    if kind == "sphere":
        cells, size = 2 * case["n"] ** 2, 8 if case["prec"] == "f64" else 4
        # state in and out, and the faces' frames and cells' geometry read once a step
        return {"bytes": cells * size * (8 + 28) * case["steps"],
                "flops": cells * case["steps"] * case["rk"] / 2 * STEP_FLOPS["sphere"]}
    if kind == "learned":
        cells = case["nx"] * case["ny"]
        return {"bytes": cells * 24 * case["steps"],
                "flops": cells * case["steps"] * (2 * _net_flops(SWE_NET) + 1200)}
    if kind == "euler_learned":
        cells = case["B"] * case["nx"] * case["ny"]
        return {"bytes": cells * 32 * case["steps"],
                "flops": cells * case["steps"] * (2 * _net_flops(EULER_NET) + 1800)}
    if kind == "network":
        cells = case["B"] * case["nx"] * case["ny"]
        return {"bytes": cells * (12 + 288), "flops": cells * _net_flops(SWE_NET)}
    if kind == "train":
        euler = case["scheme"] == "euler"
        nv, net = (4, EULER_NET) if euler else (3, SWE_NET)
        cells = case["B"] * case["n"] ** 2
        # states, targets, and each stage's activations written by the forward and read by the reverse pass
        return {"bytes": cells * case["T"] * (8 * nv + 2 * 2 * (4 * 64 + 4 * net[-1][1])),
                "flops": cells * case["T"] * 2 * 3 * _net_flops(net)}
    total = {"bytes": 0, "flops": 0}
    mix = np.random.default_rng(case["mix"])
    for _ in range(case["requests"]):
        what = ("swe", "learned", "euler", "learned")[int(mix.integers(0, 4))]
        sides = [n for n in ((32, 64, 128, 256) if what == "learned" else (64, 128, 256, 512)) if n <= case["largest"]]
        n = sides[int(mix.integers(0, len(sides)))]
        steps = max(1, int(case["steps"] * mix.uniform(0.5, 1.5)))
        if what == "learned":
            w = {"bytes": n * n * 24 * steps, "flops": n * n * steps * (2 * _net_flops(SWE_NET) + 1200)}
        else:
            w = _plain_work(what, what == "swe", n * n, steps, 2, 4)
        for key in total:
            total[key] += w[key]
    return total


# -------------------------------------------------- plain torch in 64 bits

def _minmod(a, b):
    return torch.where(a * b > 0, torch.where(a.abs() <= b.abs(), a, b), torch.zeros_like(a))


class _Physics:
    """The step on states [..., var, y, x] in double precision.  sphere:
    states in the frame of a face, (h, normal, two tangential momenta)."""

    def __init__(self, eqn, flux, dx, dy, wall, bed=None, recon="minmod", g=G):
        self.eqn, self.flux, self.d, self.wall, self.bed, self.recon, self.g = eqn, flux, (dx, dy), wall, bed, recon, g

    def pressure(self, r, mn, mt, E):
        return (GAMMA - 1) * (E - 0.5 * (mn * mn + mt * mt) / r)

    def numflux(self, L, R):
        """Flux of two normal-frame states, tuples (h, m_n, m_t...) or (rho, m_n, m_t, E)."""
        euler, g = self.eqn == "euler", self.g
        ul, ur = L[1] / L[0], R[1] / R[0]
        if euler:
            pl, pr = self.pressure(*L), self.pressure(*R)
            cl, cr = torch.sqrt(GAMMA * pl / L[0]), torch.sqrt(GAMMA * pr / R[0])
            fl = (L[1], L[1] * ul + pl, L[2] * ul, ul * (L[3] + pl))
            fr = (R[1], R[1] * ur + pr, R[2] * ur, ur * (R[3] + pr))
        else:
            cl, cr = torch.sqrt(g * L[0]), torch.sqrt(g * R[0])
            fl = (L[1], L[1] * ul + 0.5 * g * L[0] ** 2) + tuple(m * ul for m in L[2:])
            fr = (R[1], R[1] * ur + 0.5 * g * R[0] ** 2) + tuple(m * ur for m in R[2:])
        dq = [b - a for a, b in zip(L, R)]
        if self.flux == "rusanov":
            a = torch.maximum(ul.abs() + cl, ur.abs() + cr)
            return [0.5 * (x + y) - 0.5 * a * d for x, y, d in zip(fl, fr, dq)]
        wl, wr = torch.sqrt(L[0]), torch.sqrt(R[0])
        mean = lambda x, y: (wl * x + wr * y) / (wl + wr)  # noqa: E731
        ua = mean(ul, ur)
        if euler:
            va = mean(L[2] / L[0], R[2] / R[0])
            Ha = mean((L[3] + pl) / L[0], (R[3] + pr) / R[0])
            ca = torch.sqrt(((GAMMA - 1) * (Ha - 0.5 * (ua * ua + va * va))).clamp(min=0))
        else:
            ca = torch.sqrt(0.5 * g * (L[0] + R[0]))
        if self.flux == "hlle":
            sL = torch.minimum(ul - cl, ua - ca).clamp(max=0)
            sR = torch.maximum(ur + cr, ua + ca).clamp(min=0)
            return [(sR * a - sL * b + sL * sR * d) / (sR - sL) for a, b, d in zip(fl, fr, dq)]
        lo, mid, hi = (ua - ca).abs(), ua.abs(), (ua + ca).abs()
        if euler:
            w3 = dq[2] - va * dq[0]
            d5 = dq[3] - w3 * va
            w2 = (GAMMA - 1) / ca ** 2 * (dq[0] * (Ha - ua * ua) + ua * dq[1] - d5)
            w1 = (dq[0] * (ua + ca) - dq[1] - ca * w2) / (2 * ca)
            w4 = dq[0] - w1 - w2
            w1, w2, w3, w4 = lo * w1, mid * w2, mid * w3, hi * w4
            diss = [w1 + w2 + w4, w1 * (ua - ca) + w2 * ua + w4 * (ua + ca), (w1 + w2 + w4) * va + w3,
                    w1 * (Ha - ua * ca) + w2 * 0.5 * (ua * ua + va * va) + w3 * va + w4 * (Ha + ua * ca)]
        else:
            a1 = lo * ((ua + ca) * dq[0] - dq[1]) / (2 * ca)
            a3 = hi * (dq[1] - (ua - ca) * dq[0]) / (2 * ca)
            diss = [a1 + a3, a1 * (ua - ca) + a3 * (ua + ca)]
            for k in range(2, len(L)):
                v = mean(L[k] / L[0], R[k] / R[0])
                diss.append((a1 + a3) * v + mid * (dq[k] - v * dq[0]))
        return [0.5 * (x + y) - 0.5 * w for x, y, w in zip(fl, fr, diss)]

    def _ghosts(self, q, dim, axis, scalar=False):
        n = q.shape[dim]
        lo, hi = q.narrow(dim, n - 2, 2), q.narrow(dim, 0, 2)
        if self.wall:
            sign = torch.ones(() if scalar else (q.shape[-3], 1, 1), dtype=F64, device=q.device)
            if not scalar:
                sign[1 + axis] = -1.0
            lo, hi = q.narrow(dim, 0, 2).flip(dim) * sign, q.narrow(dim, n - 2, 2).flip(dim) * sign
        return torch.cat([lo, q, hi], dim)

    def states(self, p, dim):
        """Left and right states of the n + 1 faces of a line with two ghosts."""
        n = p.shape[dim] - 4
        m1, c0, c1, p2 = (p.narrow(dim, k, n + 1) for k in range(4))
        if self.recon == "first":
            return c0, c1
        return c0 + 0.5 * _minmod(c0 - m1, c1 - c0), c1 - 0.5 * _minmod(c1 - c0, p2 - c1)

    def admissible(self, Q):
        """Face states that may be used (the others take the cell average)."""
        if self.eqn != "euler":
            return Q[..., :1, :, :] > 0
        r, m, t, E = Q.unbind(-3)
        return ((r > 0) & (self.pressure(r, m, t, E) > 0)).unsqueeze(-3)

    def face_flux(self, L, R, axis):
        nm, tm = (1, 2) if axis == 0 else (2, 1)
        order = [0, nm, tm] + list(range(3, L.shape[-3]))
        F = self.numflux([L.select(-3, k) for k in order], [R.select(-3, k) for k in order])
        out = [None] * len(order)
        for k, f in zip(order, F):
            out[k] = f
        return torch.stack(out, -3)

    def rhs(self, q):
        out = torch.zeros_like(q)
        for axis, dim in ((0, -1), (1, -2)):
            n = q.shape[dim]
            p = self._ghosts(q, dim, axis)
            L, R = self.states(p, dim)
            nm, g = 1 + axis, self.g
            c0, c1 = p.narrow(dim, 1, n + 1), p.narrow(dim, 2, n + 1)
            L, R = torch.where(self.admissible(L), L, c0), torch.where(self.admissible(R), R, c1)
            if self.bed is None:
                F = self.face_flux(L, R, axis)
                out -= (F.narrow(dim, 1, n) - F.narrow(dim, 0, n)) / self.d[axis]
                continue
            eta = p.select(-3, 0) + self._ghosts(self.bed, dim, axis, scalar=True)
            el, er = self.states(eta, dim)
            hl, hr = L[..., 0, :, :], R[..., 0, :, :]
            zl, zr = el - hl, er - hr
            z = torch.maximum(zl, zr)
            sl, sr = (el - z).clamp(min=0), (er - z).clamp(min=0)
            F = self.face_flux(L * (sl / hl).unsqueeze(-3), R * (sr / hr).unsqueeze(-3), axis)
            Fl, Fr = F.clone(), F
            Fl[..., nm, :, :] += 0.5 * g * (hl ** 2 - sl ** 2)
            Fr[..., nm, :, :] += 0.5 * g * (hr ** 2 - sr ** 2)
            D = Fl.narrow(dim, 1, n) - Fr.narrow(dim, 0, n)
            a, b = (lambda t: t.narrow(dim, 0, n)), (lambda t: t.narrow(dim, 1, n))
            D[..., nm, :, :] += 0.5 * g * (a(hr) + b(hl)) * (b(zl) - a(zr))
            out -= D / self.d[axis]
        return out

    def rate(self, q):
        r = q[..., 0, :, :]
        if self.eqn == "euler":
            c = torch.sqrt(GAMMA * self.pressure(*q.unbind(-3)) / r)
        else:
            c = torch.sqrt(self.g * r)
        return float((((q[..., 1, :, :] / r).abs() + c) / self.d[0] + ((q[..., 2, :, :] / r).abs() + c) / self.d[1])
                     .max())

    def heun(self, q, dt):
        return _stages(q, dt, self.rhs, 2)


def _stages(q, dt, rhs, rk, after=lambda q: q):
    q1 = after(q + dt * rhs(q))
    if rk == 1:
        return q1
    if rk == 2:
        return after(0.5 * q + 0.5 * (q1 + dt * rhs(q1)))
    q2 = after(0.75 * q + 0.25 * (q1 + dt * rhs(q1)))
    return after(q / 3.0 + 2.0 / 3.0 * (q2 + dt * rhs(q2)))


class _Net:
    """The network and the learned step in double precision (periodic)."""

    def __init__(self, euler, params, scheme, dx, dy):
        self.nv, self.scheme = (4 if euler else 3), scheme
        mean, inv = EULER_NORM if euler else SWE_NORM
        dev = _device()
        self.mean, self.inv = (torch.tensor(np.float32(v).astype(np.float64), device=dev)[:, None, None]
                               for v in (mean, inv))
        self.w, self.b = ([torch.tensor(p, dtype=F64, device=dev, requires_grad=True) for p in ps] for ps in params)
        self.ph = _Physics("euler" if euler else "swe", "hlle", dx, dy, False)
        pos = torch.arange(6, dtype=F64, device=dev) - 2.5
        A = torch.stack([torch.ones_like(pos), pos])
        self.P = torch.eye(6, dtype=F64, device=dev) - A.T @ torch.linalg.inv(A @ A.T) @ A
        self.base = torch.tensor([[0, -0.25, 1, 0.25, 0, 0], [0, 0, 0.25, 1, -0.25, 0]], dtype=F64, device=dev)

    def coefficients(self, q):
        """Raw outputs [B, y, x, channels] of states [B, var, y, x]."""
        x = ((q - self.mean) * self.inv).permute(0, 2, 3, 1)
        for l, (w, b) in enumerate(zip(self.w, self.b)):
            B, H, W, ci = x.shape
            y = b
            for ky in range(3):
                for kx in range(3):
                    s = torch.roll(x, (1 - ky, 1 - kx), (1, 2)).reshape(-1, ci)
                    y = y + s @ w[:, :, ky, kx].t()
            x = y.reshape(B, H, W, -1)
            if l < len(self.w) - 1:
                x = torch.relu(x)
        return x

    def faces(self, q, z, axis):
        """States on both sides of the high face of every cell."""
        dim = -1 if axis == 0 else -2
        at = lambda k: torch.roll(q, -k, dim)  # noqa: E731
        if self.scheme == "direct":
            def side(f):
                zf = (z[..., 3 * f:3 * f + 3].permute(0, 3, 1, 2)) / self.inv
                h = q[:, :1] * torch.nn.functional.softplus(zf[:, :1] + math.log(math.e - 1.0))
                return torch.cat([h, q[:, 1:] + zf[:, 1:]], 1)
            lo, hi = (0, 1) if axis == 0 else (2, 3)
            return side(hi), torch.roll(side(lo), -1, dim)
        a = z.reshape(*z.shape[:3], 2, 2, self.nv, 6)[:, :, :, axis] @ self.P.t()
        out = []
        for s in (0, 1):
            al = (a[:, :, :, s] + self.base[s]).permute(0, 3, 4, 1, 2)
            out.append(sum(al[:, :, k] * at(k - 2) for k in range(6)))
        return out

    def rhs(self, q):
        z = self.coefficients(q)
        out = 0.0
        for axis, dim in ((0, -1), (1, -2)):
            L, R = self.faces(q, z, axis)
            F = self.ph.face_flux(L, R, axis)
            if self.scheme == "blend":
                up, down = torch.roll(q, -1, dim) - q, q - torch.roll(q, 1, dim)
                flat = up == 0
                phi = torch.where(flat, torch.zeros_like(up), down / torch.where(flat, torch.ones_like(up), up))
                phi = phi.clamp(0, 1).detach()
                low = self.ph.face_flux(q, torch.roll(q, -1, dim), axis)
                F = low - phi * (low - F)
            out = out - (F - torch.roll(F, 1, dim)) / self.ph.d[axis]
        return out

    def step(self, q, dt):
        return _stages(q, dt, self.rhs, 2)


def _f32(q):
    return q.float().double()


def _exact_plain(eqn, q, bed, nx, ny, wall, flux, recon, rk, steps, lx=1.0, ly=1.0):
    ph = _Physics(eqn, flux, lx / nx, ly / ny, wall, bed, recon)
    for _ in range(steps):
        q = _stages(q, 0.4 / ph.rate(q), ph.rhs, rk)
    return q


def exact(case, seed):
    kind = case["kind"]
    if kind == "plain":
        q, b = _plain_input(case["eqn"], case["bed"], case["nx"], case["ny"], seed)
        if case["prec"] == "f32":
            q, b = _f32(q), None if b is None else _f32(b)
        return _exact_plain(case["eqn"], q, b, case["nx"], case["ny"], case["wall"], case["flux"], case["recon"],
                            case["rk"], case["steps"], 1.0, case["ny"] / case["nx"])
    if kind == "fine":
        n, f = case["n"], case["factor"]
        q = _smooth_swe(64, 64, np.random.default_rng(seed))
        q = _f32(torch.nn.functional.interpolate(q[None], size=(n, n), mode="bilinear")[0])
        ph = _Physics("swe", "hlle", 1 / n, 1 / n, False)
        for _ in range(f):
            q = ph.heun(q, LEARNED_DT * 64 / n)
        return {"q": q, "coarse": q.reshape(3, n // f, f, n // f, f).mean((2, 4))}
    if kind == "learned":
        with torch.no_grad():
            q = _f32(_smooth_swe(case["nx"], case["ny"], np.random.default_rng(seed)))[None]
            net = _Net(False, _net_params(SWE_NET, seed), case["scheme"], 1 / 64, 1 / 64)
            for _ in range(case["steps"]):
                q = net.step(q, LEARNED_DT)
            return q[0]
    if kind == "euler_learned":
        with torch.no_grad():
            q = _batch_input(True, case["B"], case["nx"], case["ny"], seed).double()
            net = _Net(True, _net_params(EULER_NET, seed), "learned", 1 / 64, 1 / 64)
            for _ in range(case["steps"]):
                q = net.step(q, EULER_DT)
            return q
    if kind == "network":
        with torch.no_grad():
            q = _batch_input(False, case["B"], case["nx"], case["ny"], seed).double()
            return _Net(False, _net_params(SWE_NET, seed), "learned", 1 / 64, 1 / 64).coefficients(q)
    if kind == "train":
        euler = case["scheme"] == "euler"
        q0 = _batch_input(euler, case["B"], case["n"], case["n"], seed)
        targets = _train_targets(euler, q0, case["T"])
        net = _Net(euler, _net_params(EULER_NET if euler else SWE_NET, seed), case["scheme"], 1 / 64, 1 / 64)
        scale = torch.tensor(TRAIN_SCALE["euler" if euler else "swe"], dtype=F64, device=q0.device)[:, None, None]
        q, loss = q0.double(), 0.0
        for t in range(case["T"]):
            q = net.step(q, EULER_DT if euler else LEARNED_DT)
            loss = loss + (((q - targets[t].double()) / scale) ** 2).mean()
        loss.backward()
        grads = torch.cat([g.grad.reshape(-1) for pair in zip(net.w, net.b) for g in pair])
        return {"loss": float(loss.detach()), "grads": grads}
    if kind == "sphere":
        return _exact_sphere(case, seed)
    out = []
    for k, (what, n, steps, q, b) in enumerate(_requests(case, seed)):
        q = torch.tensor(q, dtype=F64, device=_device())
        if what == "learned":
            with torch.no_grad():
                net = _Net(False, _net_params(SWE_NET, seed), "learned", 1 / 64, 1 / 64)
                q = q[None]
                for _ in range(steps):
                    q = net.step(q, LEARNED_DT)
                out.append(q[0])
        else:
            bed = None if b is None else torch.tensor(b, dtype=F64, device=_device())
            out.append(_exact_plain(what, q, bed, n, n, True, "hlle", "minmod", 2, steps))
    return out


# ------------------------------------------------------------------- sphere

def _sphere_points(n, twice_i, twice_j):
    """Unit vectors [3, j, i] of the computational points (x, y) =
    ((twice_i - 3n) / n, (twice_j - n) / n): the disk mapping of [-1, 1]^2 (and
    of its reflection x -> -2 - x for the southern half), lifted."""
    x = (twice_i.to(F64) - 3 * n)[None, :] / n
    y = (twice_j.to(F64) - n)[:, None] / n
    x, y = torch.broadcast_tensors(x, y)
    north = x >= -1
    xd = torch.where(north, x, -2.0 - x)
    swap = y.abs() > xd.abs()
    a, b = torch.where(swap, y, xd), torch.where(swap, xd, y)
    D, across = a.abs() / math.sqrt(2.0), b / math.sqrt(2.0)
    along = (D - torch.sqrt(1 - D * D) + torch.sqrt(1 - across * across)) * torch.where(a < 0, -1.0, 1.0)
    xp, yp = torch.where(swap, across, along), torch.where(swap, along, across)
    r2 = xp * xp + yp * yp
    edge = torch.maximum(xd.abs(), y.abs()) >= 1
    r = torch.where(edge, torch.sqrt(r2), torch.ones_like(r2))
    z = torch.sqrt((1 - r2).clamp(min=0)) * torch.where(north, 1.0, -1.0)
    return torch.stack([xp / r, yp / r, torch.where(edge, torch.zeros_like(z), z)])


def _dot(a, b):
    return (a * b).sum(0)


def _unit(a):
    return a / torch.sqrt(_dot(a, a))


def _cross(a, b):
    return torch.cross(a, b, dim=0)


def _sphere_centres(n):
    dev = _device()
    return _sphere_points(n, 2 * torch.arange(2 * n, device=dev) + 1, 2 * torch.arange(n, device=dev) + 1)


def _sphere_input(n, seed):
    """A balanced eastward flow on the rotating sphere under Gaussian bumps."""
    rng = np.random.default_rng(seed)
    c = _sphere_centres(n)
    u0, omega = 0.3, 0.5
    h = 1.0 - (omega * u0 + 0.5 * u0 * u0) * c[2] ** 2
    for _ in range(4):
        a, w = rng.uniform(0.02, 0.08), rng.uniform(0.15, 0.35)
        p = rng.standard_normal(3)
        p /= np.linalg.norm(p)
        ang = torch.arccos((p[0] * c[0] + p[1] * c[1] + p[2] * c[2]).clamp(-1, 1))
        h = h + a * torch.exp(-(ang * ang) / (w * w))
    return torch.stack([h, -h * u0 * c[1], h * u0 * c[0], torch.zeros_like(h)])


def _exact_sphere(case, seed):
    n, dev = case["n"], _device()
    nx, ny = 2 * n, n
    p = _sphere_points(n, 2 * torch.arange(nx + 1, device=dev), 2 * torch.arange(ny + 1, device=dev))
    cen = _sphere_centres(n)

    def face(a, b, flip):
        t, r = _unit(b - a), _unit(a + b)
        c = _cross(a, b)
        return (_unit(_cross(r, t) if flip else _cross(t, r)), t, r,
                torch.atan2(torch.sqrt(_dot(c, c)), _dot(a, b)))

    def triangle(a, b, c):
        return 2 * torch.atan2(_dot(a, _cross(b, c)).abs(), 1 + _dot(a, b) + _dot(b, c) + _dot(c, a))

    fx = face(p[:, :-1, :], p[:, 1:, :], False)
    fy = face(p[:, :, :-1], p[:, :, 1:], True)
    p00, p10, p11, p01 = p[:, :-1, :-1], p[:, :-1, 1:], p[:, 1:, 1:], p[:, 1:, :-1]
    area = triangle(p00, p10, p11) + triangle(p00, p11, p01)
    perim = fx[3][:, :-1] + fx[3][:, 1:] + fy[3][:-1] + fy[3][1:]
    nsum = (fx[3] * fx[0])[:, :, 1:] - (fx[3] * fx[0])[:, :, :-1] + (fy[3] * fy[0])[:, 1:] - (fy[3] * fy[0])[:, :-1]
    omega, g = 0.5, 1.0
    ph = _Physics("swe", case["flux"], 1.0, 1.0, False, g=g)

    def flux(q, axis, f):
        if axis == 0:
            pad, dim = torch.cat([q[..., -2:], q, q[..., :2]], -1), -1
        else:  # across y = -1 and 1: the mirrored column of the same side
            pad, dim = torch.cat([q[:, :2].flip(1, 2), q, q[:, -2:].flip(1, 2)], 1), -2
        L, R = ph.states(pad, dim)
        turn = lambda s: [s[0]] + [_dot(s[1:], f[k]) for k in range(3)]  # noqa: E731
        F = ph.numflux(turn(L), turn(R))
        return torch.cat([F[0][None], F[1] * f[0] + F[2] * f[1] + F[3] * f[2]]) * f[3]

    def rhs(q):
        X, Y = flux(q, 0, fx), flux(q, 1, fy)
        m = q[1:]
        out = X[:, :, 1:] - X[:, :, :-1] + Y[:, 1:] - Y[:, :-1]
        out[1:] -= m * (_dot(m, nsum) / q[0]) + 0.5 * g * q[0] ** 2 * nsum
        out = -out / area
        out[1:] -= 2 * omega * cen[2] * _cross(cen, m)
        return out

    def tangent(q):
        return torch.cat([q[:1], q[1:] - _dot(q[1:], cen) * cen])

    q = _sphere_input(n, seed)
    if case["prec"] == "f32":
        q = _f32(q)
    for _ in range(case["steps"]):
        speed = torch.sqrt(_dot(q[1:], q[1:])) / q[0] + torch.sqrt(g * q[0])
        q = _stages(q, 0.4 / float((speed * perim / (2 * area)).max()), rhs, case["rk"], tangent)
    return q
