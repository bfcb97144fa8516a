"""The work that a user of this library has it do, as cases that can be timed.

Every case is one call (or one short sequence of calls) of the public binding
``paper_1403_7561_amd.qe`` / ``autograd`` on a Si/SiO2 gate stack or a doped
silicon block, from a 17x17x9 mesh to the 257x257x129 one: Poisson solves over
the statistics, charge models and precisions, the dot-charge gradient, the
batched voltage sweep, the eigenstates of a dot, and the single operators.
``listed()`` gives the fixed cases, ``draw(rng)`` another one of the same
ranges, ``exact()`` the same results from plain torch in 64 bits.
"""
import math
import os
import tempfile

import numpy as np
import torch

from paper_1403_7561_amd import autograd, qe

# geometry and materials of the stacks (nm, nm^-3, eV)
FOOTPRINT, SI, OX = 200.0, 90.0, 10.0
EPS_SI, EPS_OX = 11.7, 3.9
ACCEPTORS = 1e15 * 1e-21
GATES = ((10.0, 50.0, 80.0, 120.0), (150.0, 190.0, 80.0, 120.0), (10.0, 190.0, 150.0, 190.0),
         (80.0, 120.0, 80.0, 120.0), (10.0, 190.0, 10.0, 50.0))      # P1, P2, B1, B2, B3
DOTS = ((0.0, 60.0, 70.0, 130.0, 70.0, 90.0), (140.0, 200.0, 70.0, 130.0, 70.0, 90.0))
# Newton's tolerance where results are compared (the library's tests use it too)
ATOL = 1e-10


def listed():
    return [
        # the smallest solve: two gates on 17x17x9 nodes at T = 0; launches and latency
        {"name": "solve 17x17x9 tf", "kind": "solve", "nx": 17, "ny": 17, "nz": 9, "stat": "tf", "T": 0.0},
        # a p-n junction at room temperature: Boltzmann carriers of both signs, Ohmic contacts, graded mesh
        {"name": "junction 33x29x41 mb", "kind": "junction", "nx": 33, "ny": 29, "nz": 41, "stat": "mb", "T": 300.0},
        # one device of a gate-voltage sweep, solved by itself
        {"name": "solve 65x65x33 fd", "kind": "solve", "nx": 65, "ny": 65, "nz": 33, "stat": "fd", "T": 4.0},
        # holes and incompletely ionised acceptors at 4 K on a ragged mesh
        {"name": "full charge 97x81x49", "kind": "solve", "nx": 97, "ny": 81, "nz": 49, "stat": "fd", "T": 4.0,
         "full": True},
        # the double-dot stack that the library's benchmark solves: potential, density, dot electrons
        {"name": "solve 129x129x65 fd", "kind": "solve", "nx": 129, "ny": 129, "nz": 65, "stat": "fd", "T": 4.0},
        # the largest: a rough oxide on 8.5M nodes in mixed precision
        {"name": "solve 257x257x129 mixed", "kind": "solve", "nx": 257, "ny": 257, "nz": 129, "stat": "fd", "T": 4.0,
         "precision": "mixed", "rough": True},
        # dot charge with its gradient in the gate voltages and the permittivity (autograd, forward and backward)
        {"name": "gradient 129x129x65", "kind": "gradient", "nx": 129, "ny": 129, "nz": 65, "stat": "fd", "T": 4.0},
        # interface charge and charged gates (Robin faces)
        {"name": "charged gates 113x97x49", "kind": "solve", "nx": 113, "ny": 97, "nz": 49, "stat": "fd", "T": 4.0,
         "sheets": True},
        # the predictor step of a Schrodinger-Poisson loop with 16 states
        {"name": "predictor 65x65x33", "kind": "predictor", "nx": 65, "ny": 65, "nz": 33, "stat": "fd", "T": 4.0,
         "states": 16},
        # eight dot states on the benchmark's mesh
        {"name": "states 129x129x65", "kind": "states", "nx": 129, "ny": 129, "nz": 65, "states": 8},
        # the gate-voltage sweep: 256 devices of 33x33x17 to 65x65x33 nodes in one call
        {"name": "sweep of 256", "kind": "sweep", "n": 256, "lo": 32, "hi": 64, "cache": True},
        # single operators on a ragged mesh: residual and diagonal, Jacobian products, density, counts
        {"name": "operators 151x133x77", "kind": "operators", "nx": 151, "ny": 133, "nz": 77, "stat": "fd", "T": 77.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mesh(rng, lo, hi):
    """Node counts of a mesh of lo .. hi nodes, spread over the logarithm; the three are odd and even alike."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    ax, ay = rng.uniform(0.8, 1.25), rng.uniform(0.8, 1.25)
    nx = max(7, int((2.0 * n) ** (1.0 / 3.0) * ax))
    ny = max(7, int((2.0 * n) ** (1.0 / 3.0) * ay))
    return nx, ny, max(7, min(int(n / (nx * ny)), 160))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "solve", "junction", "gradient", "predictor", "states", "sweep",
                       "operators", "operators"])
    if kind == "sweep":
        if rng.random() < 0.5:   # tuned by each call: small devices
            lo = rng.randint(8, 14)
            return {"kind": kind, "n": _log_int(rng, 4, 64), "lo": lo, "hi": lo + rng.randint(2, 8), "cache": False}
        lo = rng.randint(12, 40)
        return {"kind": kind, "n": _log_int(rng, 6, 200), "lo": lo, "hi": lo + rng.randint(4, 20), "cache": True}
    if kind == "states":
        nx, ny, nz = _mesh(rng, 15000, 1100000)
        return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "states": rng.randint(2, 10)}
    c = {"kind": kind}
    if kind == "junction":
        c["nx"], c["ny"], c["nz"] = _mesh(rng, 2500, 400000)
        c["stat"], c["T"] = rng.choice([("mb", 300.0), ("fd", 300.0), ("mb", 200.0)])
    elif kind == "operators":
        c["nx"], c["ny"], c["nz"] = _mesh(rng, 2500, 4000000)
        c["stat"], c["T"] = rng.choice([("fd", 4.0), ("fd", 77.0), ("mb", 300.0), ("tf", 0.0)])
    elif kind == "solve":
        c["nx"], c["ny"], c["nz"] = _mesh(rng, 2500, 3000000)
        c["stat"], c["T"] = rng.choice([("fd", 4.0), ("fd", 4.0), ("fd", 77.0), ("tf", 0.0)])
        how = rng.choice(["", "", "full", "sheets", "mixed"])
        if how == "mixed":
            c["precision"] = "mixed"
        elif how == "sheets" or (how == "full" and c["stat"] == "fd"):
            c[how] = True
    else:
        c["nx"], c["ny"], c["nz"] = _mesh(rng, 4000, 1100000 if kind == "gradient" else 400000)
        c["stat"], c["T"] = "fd", 4.0
        if kind == "predictor":
            c["states"] = rng.randint(4, 24)
    return c


# ------------------------------------------------------------------ devices
class Device:
    """Host arrays of one device, as ``qe.Problem`` takes them."""

    def __init__(self, x, y, z, eps, semi, net, dir_id, dir_val, stat, T):
        self.x, self.y, self.z = x, y, z
        self.nx, self.ny, self.nz = x.size, y.size, z.size
        self.n_nodes, self.n_elems = x.size * y.size * z.size, (x.size - 1) * (y.size - 1) * (z.size - 1)
        self.eps_r, self.semi, self.net_doping = eps, semi, net
        self.dir_id, self.dir_val = dir_id, dir_val
        self.stat, self.T_K, self.m_eff, self.Ec0_eV = stat, T, 1.08, 0.56
        self.holes, self.ionization, self.donors, self.acceptors = False, "complete", None, None
        self.sheets, self.quantum = [], None


class Sheet:
    def __init__(self, plane, a0, a1, b0, b1, sigma, d=0.0, eps=0.0, phi0=0.0):
        self.axis, self.plane, self.a0, self.a1, self.b0, self.b1 = 2, plane, a0, a1, b0, b1
        self.sigma, self.robin_d, self.robin_eps, self.phi0 = sigma, d, eps, phi0


class States:
    def __init__(self, psi2, phi_k, E_i):
        self.psi2, self.phi_k, self.E_i = psi2, phi_k, E_i
        self.confinement, self.m_t, self.region = 3, 0.19, None


def _stack_z(n_ez):
    """Node heights with a plane on the Si/SiO2 interface, and the oxide's layers."""
    ox = max(1, int(round(n_ez * OX / (SI + OX))))
    return np.concatenate([np.linspace(0.0, SI, n_ez - ox + 1), np.linspace(SI, SI + OX, ox + 1)[1:]]), ox


def _gate_nodes(x, y, r):
    return (np.nonzero((x >= r[0] - 1e-9) & (x <= r[1] + 1e-9))[0], np.nonzero((y >= r[2] - 1e-9) & (y <= r[3] + 1e-9))[0])


def _stack(c, rng, volts=None):
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    x, y = np.linspace(0.0, FOOTPRINT, nx), np.linspace(0.0, FOOTPRINT, ny)
    z, _ = _stack_z(nz - 1)
    zc = 0.5 * (z[1:] + z[:-1])
    if c.get("rough"):   # +-1 nm of oxide thickness, bilinear between 20 nm control points
        ctrl = rng.uniform(-1.0, 1.0, (11, 11))
        xc, yc = 0.5 * (x[1:] + x[:-1]) / 20.0, 0.5 * (y[1:] + y[:-1]) / 20.0
        i, j = np.minimum(xc.astype(int), 9), np.minimum(yc.astype(int), 9)
        u, v = (xc - i)[None, :], (yc - j)[:, None]
        cc = ctrl.T   # [iy, ix]
        a, b = cc[np.ix_(j, i)], cc[np.ix_(j, i + 1)]
        d, e = cc[np.ix_(j + 1, i)], cc[np.ix_(j + 1, i + 1)]
        top = SI + (1 - v) * ((1 - u) * a + u * b) + v * ((1 - u) * d + u * e)
        oxide = zc[:, None, None] > top[None]
    else:
        oxide = np.broadcast_to((zc > SI)[:, None, None], (nz - 1, ny - 1, nx - 1))
    oxide = np.ascontiguousarray(oxide).ravel()
    # two plungers over the dots and three barriers
    v = np.concatenate([rng.uniform(1.15, 1.6, 2), rng.uniform(0.0, 2.0, 3)]) if volts is None else volts
    dir_id = np.full(nx * ny * nz, -1, dtype=np.int32)
    dir_id[: nx * ny] = len(GATES)
    topf = dir_id[(nz - 1) * nx * ny:].reshape(ny, nx)
    for g, r in enumerate(GATES):
        ii, jj = _gate_nodes(x, y, r)
        topf[np.ix_(jj, ii)] = g
    dev = Device(x, y, z, np.where(oxide, EPS_OX, EPS_SI), (~oxide).astype(np.uint8),
                 np.where(oxide, 0.0, -ACCEPTORS), dir_id, np.append(v, 0.0), c["stat"], c["T"])
    if c.get("full"):   # holes, the substrate's boron as a species; the contact at its neutral potential
        dev.holes, dev.ionization = True, "incomplete"
        dev.donors, dev.acceptors = np.zeros(oxide.size), np.where(oxide, 0.0, ACCEPTORS * rng.uniform(0.7, 1.4))
        dev.dir_val[-1] = _ohmic_p_incomplete(dev)
    if c.get("sheets"):   # interface charge; the plungers as charged gates 10 nm away through oxide
        k = int(np.argmin(np.abs(z - SI)))
        dev.sheets.append(Sheet(k, 0, nx - 1, 0, ny - 1, 1e-3 * rng.uniform(0.5, 1.5, (nx - 1) * (ny - 1))))
        for g in range(2):
            ii, jj = _gate_nodes(x, y, GATES[g])
            if ii.size < 2 or jj.size < 2:
                continue
            topf[np.ix_(jj, ii)] = -1
            dev.sheets.append(Sheet(nz - 1, int(ii[0]), int(ii[-1]), int(jj[0]), int(jj[-1]),
                                    np.full((ii.size - 1) * (jj.size - 1), -2e-3), 10.0, EPS_OX, float(v[g] + 0.6)))
    return dev


def _graded(L, n, g):
    t = np.linspace(0.0, 1.0, n)
    return L * (t + g * np.sin(2.0 * np.pi * t) / (2.0 * np.pi))


def _junction(c, rng):
    """A silicon block, boron below and phosphorus above a junction, Ohmic contacts on both faces."""
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    x, y, z = _graded(80.0, nx, 0.0), _graded(70.0, ny, 0.3), _graded(240.0, nz, 0.5)
    at = 120.0 + rng.uniform(-15.0, 15.0)
    zc = 0.5 * (z[1:] + z[:-1])
    na, nd = 1e-21 * 10.0 ** rng.uniform(16.3, 17.3, 2)
    up = np.repeat(zc > at, (nx - 1) * (ny - 1))
    net = np.where(up, nd, -na) * rng.uniform(0.9, 1.1, up.size)
    dir_id = np.full(nx * ny * nz, -1, dtype=np.int32)
    dir_id[: nx * ny], dir_id[(nz - 1) * nx * ny:] = 0, 1
    kT = _K * c["T"] / _Q
    v = [0.56 - 1.12 - kT * math.log(na / _dos(qe.SI_M_H, c["T"])), 0.56 + kT * math.log(nd / _dos(1.08, c["T"]))]
    dev = Device(x, y, z, np.full(up.size, EPS_SI), np.ones(up.size, dtype=np.uint8), net, dir_id,
                 np.array(v), c["stat"], c["T"])
    dev.holes = True
    return dev


def _potential(dev, rng, depth=0.25):
    """A smooth potential like a solution's: pulled up under two gates, falling towards the substrate."""
    x, y, z = dev.x[None, None, :], dev.y[None, :, None], dev.z[:, None, None]
    a, b = rng.uniform(0.30, 0.45, 2)
    xy = a * np.exp(-((x - 30.0) / 26.0) ** 2 - ((y - 100.0) / 33.0) ** 2) + \
        b * np.exp(-((x - 165.0) / 29.0) ** 2 - ((y - 95.0) / 36.0) ** 2)
    return ((depth + xy) * (z / (SI + OX)) ** 2).ravel()


def _box_states(dev, n, rng, phi_k):
    """Standing waves of a hard box in the first dot, with levels around the Fermi level."""
    lo, hi = np.array([8.0, 82.0, 72.0]), np.array([58.0, 122.0, 90.0])
    L = hi - lo
    modes = sorted(((i, j, k) for i in range(1, 7) for j in range(1, 7) for k in range(1, 4)),
                   key=lambda m: (m[0] / L[0]) ** 2 + (m[1] / L[1]) ** 2 + (m[2] / L[2]) ** 2)[:n]

    def wave(s, a, length, m):
        t = (s - a) / length
        return np.where((t >= 0) & (t <= 1), np.sin(np.pi * m * t) ** 2, 0.0)

    psi2 = np.empty((n, dev.nz, dev.ny, dev.nx))
    for s, (i, j, k) in enumerate(modes):
        psi2[s] = (8.0 / np.prod(L)) * wave(dev.z, lo[2], L[2], k)[:, None, None] * \
            wave(dev.y, lo[1], L[1], j)[None, :, None] * wave(dev.x, lo[0], L[0], i)[None, None, :]
    E = -0.003 + np.concatenate([[0.0], np.cumsum(0.0006 * rng.uniform(0.5, 1.5, n - 1))])
    return States(psi2.reshape(n, -1), phi_k, E)


def _dot_region(dev):
    """Inverse masses, band edges and the fixed nodes of a quantum region in the first dot."""
    box = (0.0, 66.0, 66.0, 134.0, 50.0, 100.0)
    ox = dev.semi == 0
    im = np.stack([np.where(ox, 2.0, 1.0 / m) for m in (0.19, 0.19, 0.98)])
    v0 = np.where(ox, 0.56 + 3.1, 0.56)
    inside = ((dev.z > box[4]) & (dev.z < box[5]))[:, None, None] & ((dev.y > box[2]) & (dev.y < box[3]))[None, :, None] \
        & ((dev.x > box[0]) & (dev.x < box[1]))[None, None, :]
    return im, v0, ~inside.ravel()


def _device(case, seed):
    rng = np.random.default_rng([7561, int(seed)])
    kind = case["kind"]
    if kind == "junction":
        return _junction(case, rng), rng
    if kind == "states":
        return _stack({**case, "stat": "fd", "T": 4.0}, rng), rng
    return _stack(case, rng), rng


def _sweep_devices(case, seed):
    # the sweep's meshes are the case's, its voltages the seed's
    ms = np.random.default_rng([7561, case["lo"], case["hi"]]).integers(case["lo"], case["hi"] + 1, size=case["n"])
    rng = np.random.default_rng([7561, int(seed)])
    barriers = rng.uniform(0.0, 2.0, 3)
    for k in range(case["n"]):
        m = int(ms[k])
        v = np.concatenate([rng.uniform(0.8, 1.6, 2), barriers])
        yield _stack({"nx": m + 1, "ny": m + 1, "nz": m // 2 + 1, "stat": "fd", "T": 4.0}, rng, v)


def prepare(case, seed):
    kind = case["kind"]
    opts = qe.qe_default_options(newton_atol=ATOL if case.get("nx", 0) * case.get("ny", 0) * case.get("nz", 0) < 4000000 else 1e-9,
                                 precision=case.get("precision", "fp64"))
    if kind == "sweep":
        probs = [qe.Problem(d) for d in _sweep_devices(case, seed)]
        return {"kind": kind, "probs": probs, "opts": opts, "boxes": list(DOTS),
                "ws": qe.Workspace(qe.qe_batch_workspace_bytes(probs, opts), probs[0].device),
                "cache": os.path.join(tempfile.gettempdir(), "qe_sweep_tune_%d.txt" % os.getuid()) if case["cache"] else None}
    dev, rng = _device(case, seed)
    s = {"kind": kind, "opts": opts, "boxes": list(DOTS)}
    if kind in ("predictor", "operators", "states"):
        phi = _potential(dev, rng)
    if kind == "predictor":
        dev.quantum = _box_states(dev, case["states"], rng, phi)
    s["prob"] = P = qe.Problem(dev)
    if kind == "gradient":
        s["box"] = DOTS[int(dev.dir_val[1] > dev.dir_val[0])]
    elif kind == "states":
        im, v0, fixed = _dot_region(dev)
        s.update(im=im, v0=v0, fixed=fixed, n=case["states"], phi=torch.as_tensor(phi, device=P.device))
        lib, c = qe.load_library(), P.c()
        s["ws"] = qe.Workspace(lib.qe_schrodinger_workspace_bytes(qe.ctypes.byref(c), case["states"]), P.device)
    else:
        s["ws"] = qe.workspace_for(P, opts)
    if kind == "operators":
        v = rng.standard_normal(dev.n_nodes)
        s.update(phi=torch.as_tensor(phi, device=P.device), v=torch.as_tensor(v, device=P.device),
                 v32=torch.as_tensor(v.astype(np.float32), device=P.device))
    return s


def run(s):
    kind, opts = s["kind"], s["opts"]
    if kind == "sweep":
        phis, counts, _ = qe.qe_solve_batch(s["probs"], opts=opts, boxes=s["boxes"], tune_cache=s["cache"], ws=s["ws"])
        return {"counts": counts, "phi": torch.cat(phis)}
    P = s["prob"]
    if kind == "gradient":
        V = P.dir_val[: P.n_dir].clone().requires_grad_(True)
        eps = P.eps_r.clone().requires_grad_(True)
        Q = autograd.dot_charge(P, s["box"], V, eps, opts)
        Q.backward()
        return {"Q": Q.detach(), "dV": V.grad, "deps": eps.grad}
    if kind == "states":   # the sign of psi is arbitrary; |psi|^2 is what the Poisson step takes
        E, _, psi2, _ = qe.qe_schrodinger_solve(P, s["im"], s["v0"], s["phi"], s["n"], fixed=s["fixed"], tol=1e-11,
                                                maxit=3000, ws=s["ws"])
        return {"E": E, "psi2": psi2}
    if kind == "operators":
        phi, ws = s["phi"], s["ws"]
        F, diag, _ = qe.qe_residual(P, phi, ws=ws)
        return {"F": F, "diag": diag, "Jv": qe.qe_jv(P, phi, s["v"], ws=ws), "Jv32": qe.qe_jv_f32(P, phi, s["v32"], ws=ws),
                "n": qe.qe_density(P, phi, ws=ws), "counts": qe.qe_count_electrons(P, phi, s["boxes"], ws=ws)}
    phi, n, _ = qe.qe_solve(P, opts=opts, ws=s["ws"])
    if kind == "junction":
        return {"phi": phi, "n": n}
    return {"phi": phi, "n": n, "counts": qe.qe_count_electrons(P, phi, s["boxes"], ws=s["ws"])}


def work(case):
    """Inputs read once, outputs written once; about one residual and one Jacobian product of arithmetic."""
    if case["kind"] == "sweep":
        m = 0.5 * (case["lo"] + case["hi"])
        n = case["n"] * (m + 1) ** 2 * (m / 2 + 1)
        return {"bytes": 30.0 * n, "flops": 600.0 * n}
    n = float(case["nx"] * case["ny"] * case["nz"])
    k = case["kind"]
    if k == "states":   # the states and their squares out; the masses, band edges and the potential in
        return {"bytes": n * (16.0 * case["states"] + 41.0), "flops": 300.0 * n * case["states"]}
    if k == "operators":   # phi, v, v32, eps, flags, doping, ids in; F, diag, Jv, Jv32, n out
        return {"bytes": n * (8 + 8 + 4 + 8 + 1 + 8 + 4 + 8 + 8 + 8 + 4 + 8), "flops": 900.0 * n}
    extra = 8.0 * case.get("states", 0) + (16.0 if case.get("full") else 0.0) + (16.0 if k == "gradient" else 0.0)
    return {"bytes": n * (21.0 + 16.0 + extra), "flops": 600.0 * n}


# ------------------------------------------------------------------ 64-bit reference
# CODATA 2018
_Q, _EPS0, _HBAR, _M0, _K = 1.602176634e-19, 8.8541878128e-12, 1.054571817e-34, 9.1093837015e-31, 1.380649e-23
_KAPPA = _Q / _EPS0 * 1e9


def _dos(m, T):
    return 2.0 * (m * _M0 * _K * T / (2.0 * math.pi * _HBAR ** 2)) ** 1.5 * 1e-27


def _ohmic_p_incomplete(dev):
    """Potential of a neutral p contact with incomplete ionisation."""
    kT = _K * dev.T_K / _Q
    na = float(dev.acceptors.max())
    lnK = math.log(na / _dos(qe.SI_M_H, dev.T_K)) + qe.SI_EA_EV / kT
    if lnK < 600.0:
        ln_y = math.log(2.0) + lnK - math.log1p(math.sqrt(1.0 + 16.0 * math.exp(lnK)))
    else:
        ln_y = 0.5 * (lnK - math.log(4.0))
    return 0.56 - 1.12 + qe.SI_EA_EV - kT * ln_y


def _kron3(c, b, a):
    return torch.kron(c, torch.kron(b, a))   # local corner dx + 2 dy + 4 dz


class _Plain:
    """The discrete problem in plain torch: gathers of the eight element corners and 8x8 element matrices."""

    def __init__(self, dev, device):
        t = lambda a: torch.as_tensor(np.ascontiguousarray(a), device=device, dtype=torch.float64)  # noqa: E731
        self.dev, self.device = dev, device
        self.shape, self.es = (dev.nz, dev.ny, dev.nx), (dev.nz - 1, dev.ny - 1, dev.nx - 1)
        hx, hy, hz = t(np.diff(dev.x))[None, None, :], t(np.diff(dev.y))[None, :, None], t(np.diff(dev.z))[:, None, None]
        eps = t(dev.eps_r).view(self.es)
        self.s = torch.stack([(eps * hy * hz / hx).reshape(-1), (eps * hx * hz / hy).reshape(-1), (eps * hx * hy / hz).reshape(-1)])
        self.s1 = self.s / eps.reshape(-1)
        semi = t(dev.semi).reshape(-1)
        self.vol = (hx * hy * hz).expand(self.es).reshape(-1)
        self.W = semi * self.vol * 0.125
        self.net = None if dev.net_doping is None else t(dev.net_doping)
        self.nd, self.na = (None, None) if dev.donors is None else (t(dev.donors), t(dev.acceptors))
        A = torch.tensor([[1.0, -1.0], [-1.0, 1.0]], dtype=torch.float64, device=device)
        M = torch.tensor([[2.0, 1.0], [1.0, 2.0]], dtype=torch.float64, device=device) / 6.0
        g1, g0 = 0.5 * (1 + 1 / math.sqrt(3.0)), 0.5 * (1 - 1 / math.sqrt(3.0))
        B = torch.tensor([[g1, g0], [g0, g1]], dtype=torch.float64, device=device)
        self.A, self.M = A, M
        self.K3 = torch.stack([_kron3(M, M, A), _kron3(M, A, M), _kron3(A, M, M)])
        self.B = _kron3(B, B, B)
        ids = torch.as_tensor(dev.dir_id, device=device).long()
        self.ids, self.free = ids, (ids < 0).to(torch.float64)
        self.vals = t(dev.dir_val)
        self.semi = semi
        if dev.quantum is not None:
            q = dev.quantum
            self.qE, self.phik = t(q.E_i), self.B @ self.corners(t(q.phi_k))
            self.psi2 = t(q.psi2)

    def corners(self, v):
        v = v.view(self.shape)
        c = [v[a: a + self.es[0], b: b + self.es[1], d: d + self.es[2]].reshape(-1)
             for a in (0, 1) for b in (0, 1) for d in (0, 1)]
        return torch.stack(c)

    def gather(self, f):
        out = torch.zeros(self.shape, dtype=torch.float64, device=self.device)
        k = 0
        for a in (0, 1):
            for b in (0, 1):
                for d in (0, 1):
                    out[a: a + self.es[0], b: b + self.es[1], d: d + self.es[2]] += f[k].view(self.es)
                    k += 1
        return out.view(-1)

    def stiff(self, u, s):
        return s[0] * (self.K3[0] @ u) + s[1] * (self.K3[1] @ u) + s[2] * (self.K3[2] @ u)

    def band(self, u, m):
        """Density of one band and its derivative, u = E_F - band edge."""
        d = self.dev
        if d.stat == "tf":
            C = (2.0 * m * _M0 * _Q) ** 1.5 / (3.0 * math.pi ** 2 * _HBAR ** 3) * 1e-27
            p = u.clamp(min=0.0)
            return C * p ** 1.5, 1.5 * C * p.sqrt()
        kT = _K * d.T_K / _Q
        N, e = _dos(m, d.T_K), u / kT
        if d.stat == "mb":
            f = torch.exp(e)
            return N * f, N * f / kT
        h = e.clamp(min=-50.0)
        g = torch.exp(-0.17 * (h + 1.0) ** 2)
        v = h ** 4 + 50.0 + 33.6 * h * (1.0 - 0.68 * g)
        dv = 4.0 * h ** 3 + 33.6 * (1.0 - 0.68 * g) + 33.6 * 0.68 * 0.34 * h * (h + 1.0) * g
        a = 0.75 * math.sqrt(math.pi)
        den = torch.exp(-h) + a * v ** -0.375
        low = e < -50.0
        ex = torch.exp(e.clamp(max=-50.0))
        return (N * torch.where(low, ex, 1.0 / den),
                N / kT * torch.where(low, ex, (torch.exp(-h) + 0.375 * a * v ** -1.375 * dv) / den ** 2))

    def electrons(self, pq):
        if self.dev.quantum is None:
            return self.band(pq - self.dev.Ec0_eV, self.dev.m_eff)
        kT = _K * self.dev.T_K / _Q
        n, dn = torch.zeros_like(pq), torch.zeros_like(pq)
        for i in range(self.qE.numel()):
            p = 4.0 * (self.B @ self.corners(self.psi2[i]))
            f = torch.sigmoid((pq - self.phik - self.qE[i]) / kT)
            n += p * f
            dn += p * f * torch.sigmoid(-(pq - self.phik - self.qE[i]) / kT) / kT
        return n, dn

    def charge(self, pq):
        """rho and -drho/dphi at the Gauss points."""
        d = self.dev
        n, dn = self.electrons(pq)
        rho, c = -n, dn
        if d.holes:
            p, dp = self.band(d.Ec0_eV - qe.SI_EG_EV - pq, qe.SI_M_H)
            rho, c = rho + p, c + dp
        if d.ionization == "incomplete":
            kT = _K * d.T_K / _Q
            a = (pq - d.Ec0_eV + qe.SI_ED_EV) / kT + math.log(2.0)
            b = (d.Ec0_eV - qe.SI_EG_EV - pq + qe.SI_EA_EV) / kT + math.log(4.0)
            rho = rho + self.nd * torch.sigmoid(-a) - self.na * torch.sigmoid(-b)
            c = c + (self.nd * torch.sigmoid(a) * torch.sigmoid(-a) + self.na * torch.sigmoid(b) * torch.sigmoid(-b)) / kT
        else:
            rho = rho + self.net
        return rho, c

    def faces(self, fn):
        """Adds the sheets' face terms: fn(sheet, corner values [4, nb, na], areas) gives values for the corners."""
        out = torch.zeros(self.shape, dtype=torch.float64, device=self.device)
        d = self.dev
        M2 = torch.kron(self.M, self.M)
        for sh in d.sheets:
            ha = torch.as_tensor(np.diff(d.x)[sh.a0: sh.a1], device=self.device)
            hb = torch.as_tensor(np.diff(d.y)[sh.b0: sh.b1], device=self.device)
            f = fn(sh, (hb[:, None] * ha[None, :]), M2)
            if f is None:
                continue
            k = 0
            for b in (0, 1):
                for a in (0, 1):
                    out[sh.plane, sh.b0 + b: sh.b1 + b, sh.a0 + a: sh.a1 + a] += f[k]
                    k += 1
        return out.view(-1)

    def plane(self, v, sh):
        v = v.view(self.shape)[sh.plane]
        return torch.stack([v[sh.b0 + b: sh.b1 + b, sh.a0 + a: sh.a1 + a] for b in (0, 1) for a in (0, 1)])

    def residual(self, phi, linear=False):
        """F with its Dirichlet rows, and the Gauss-point coefficients."""
        u = self.corners(phi)
        pq = self.B @ u
        if linear:
            rho = (self.net if self.dev.donors is None else self.nd - self.na).expand_as(pq)
            c = torch.zeros_like(pq)
        else:
            rho, c = self.charge(pq)
        F = self.gather(self.stiff(u, self.s) - _KAPPA * self.W * (self.B @ rho))
        if self.dev.sheets:
            def load(sh, area, M2):
                f = torch.zeros((4,) + tuple(area.shape), dtype=torch.float64, device=self.device)
                if sh.sigma is not None:
                    f -= _KAPPA * 0.25 * area * torch.as_tensor(sh.sigma, device=self.device).view(area.shape)
                if sh.robin_d > 0:
                    w = torch.einsum("ij,jba->iba", M2, self.plane(phi, sh) - sh.phi0)
                    f += sh.robin_eps / sh.robin_d * area * w
                return f
            F = F + self.faces(load)
        return F, _KAPPA * self.W * c

    def product(self, c, v, rows=False):
        """J v with v zero on Dirichlet nodes; rows: keep the Dirichlet rows' sums."""
        v = v * self.free
        u = self.corners(v)
        y = self.gather(self.stiff(u, self.s) + self.B @ (c * (self.B @ u)))
        if self.dev.sheets:
            def robin(sh, area, M2):
                if not sh.robin_d > 0:
                    return None
                return sh.robin_eps / sh.robin_d * area * torch.einsum("ij,jba->iba", M2, self.plane(v, sh))
            y = y + self.faces(robin)
        return y if rows else y * self.free

    def diagonal(self, c):
        d = sum(self.s[a] * torch.diagonal(self.K3[a])[:, None] for a in range(3)) + (self.B * self.B) @ c
        y = self.gather(d)
        if self.dev.sheets:
            def robin(sh, area, M2):
                if not sh.robin_d > 0:
                    return None
                return (sh.robin_eps / sh.robin_d * area)[None] * torch.diagonal(M2)[:, None, None]
            y = y + self.faces(robin)
        return y * self.free + (1.0 - self.free)

    def cg(self, c, b, rtol, most=6000):
        dinv = self.free / self.diagonal(c)
        x, r = torch.zeros_like(b), b * self.free
        z = dinv * r
        p, rz = z.clone(), torch.dot(r, z)
        stop = rtol * rtol * float(rz)
        for _ in range(most):
            y = self.product(c, p)
            a = rz / torch.dot(p, y)
            x += a * p
            r -= a * y
            z = dinv * r
            new = torch.dot(r, z)
            if float(new) <= stop:
                break
            p = z + (new / rz) * p
            rz = new
        return x

    def solve(self):
        phi = torch.where(self.ids >= 0, self.vals[self.ids.clamp(min=0)], torch.zeros_like(self.free))
        F, c = self.residual(phi, linear=True)
        phi = phi - self.cg(c, F, 1e-3)
        F, c = self.residual(phi)
        nrm = float((F * self.free).norm())
        for _ in range(80):
            d = self.cg(c, F, min(0.1, max(1e-6, 1e-3 * nrm)) if nrm > 1e-6 else 1e-5)
            lam = 1.0
            while lam > 1e-6:
                F2, c2 = self.residual(phi - lam * d)
                n2 = float((F2 * self.free).norm())
                if n2 <= (1.0 - 1e-4 * lam) * nrm:
                    break
                lam *= 0.5
            else:
                break
            phi = phi - lam * d
            gain, F, c, nrm = nrm / n2, F2, c2, n2
            if nrm < 1e-9 and (gain < 5.0 or nrm < 1e-12):
                break
        return phi, c

    def density(self, phi):
        touch = self.gather(self.semi.expand(8, -1)) > 0
        if self.dev.quantum is None:
            n, _ = self.band(phi - self.dev.Ec0_eV, self.dev.m_eff)
        else:
            kT = _K * self.dev.T_K / _Q
            pk = torch.as_tensor(self.dev.quantum.phi_k, device=self.device)
            n = sum(4.0 * self.psi2[i] * torch.sigmoid((phi - pk - self.qE[i]) / kT) for i in range(self.qE.numel()))
        return torch.where(touch, n, torch.zeros_like(n))

    def inside(self, box):
        d = self.dev
        m = [(a[1:] + a[:-1]) * 0.5 for a in (d.x, d.y, d.z)]
        m = [(a >= box[2 * k]) & (a <= box[2 * k + 1]) for k, a in enumerate(m)]
        return torch.as_tensor(m[2][:, None, None] & m[1][None, :, None] & m[0][None, None, :], device=self.device).reshape(-1)

    def count(self, phi, boxes):
        n, _ = self.electrons(self.B @ self.corners(phi))
        e = self.W * n.sum(0)
        return np.array([float(e[self.inside(b)].sum()) for b in boxes])

    def gradient(self, box):
        phi, c = self.solve()
        u = self.corners(phi)
        n, dn = self.electrons(self.B @ u)
        w = self.W * self.inside(box).to(torch.float64)
        g = self.gather(self.B @ (w * dn))
        lam = self.cg(c, g, 1e-13)
        r = g - self.product(c, lam, rows=True)
        dV = torch.zeros(self.dev.dir_val.size, dtype=torch.float64, device=self.device)
        at = self.ids >= 0
        dV.index_add_(0, self.ids[at], r[at])
        return {"Q": (w * n.sum(0)).sum(), "dV": dV, "deps": -(self.corners(lam) * self.stiff(u, self.s1)).sum(0)}


def _dense_states(dev, phi, n):
    """The lowest states from the dense matrices of the region's free nodes."""
    im, v0, fixed = _dot_region(dev)
    f = _Plain(dev, "cpu")
    free = np.nonzero(~fixed)[0]
    num = np.full(dev.n_nodes, -1)
    num[free] = np.arange(free.size)
    c = _HBAR ** 2 / (2.0 * _M0 * _Q) * 1e18
    k = (c * torch.as_tensor(im) * f.s1)
    pq = f.B @ f.corners(torch.as_tensor(phi))
    w = f.vol * 0.125 * (torch.as_tensor(v0) - pq)
    idx = f.corners(torch.arange(dev.n_nodes, dtype=torch.float64)).long().numpy()
    H, S = np.zeros((free.size, free.size)), np.zeros((free.size, free.size))
    m8 = _kron3(f.M, f.M, f.M)
    for i in range(8):
        for j in range(8):
            h = sum(f.K3[a][i, j] * k[a] for a in range(3)) + ((f.B[i] * f.B[j])[:, None] * w).sum(0)
            a, b = num[idx[i]], num[idx[j]]
            at = (a >= 0) & (b >= 0)
            np.add.at(H, (a[at], b[at]), h.numpy()[at])
            np.add.at(S, (a[at], b[at]), (m8[i, j] * f.vol).numpy()[at])
    L = np.linalg.cholesky(S)
    Li = np.linalg.inv(L)
    E, U = np.linalg.eigh(Li @ H @ Li.T)
    psi = np.zeros((n, dev.n_nodes))
    psi[:, free] = (Li.T @ U[:, :n]).T
    return {"E": E[:n], "psi2": torch.as_tensor(psi ** 2)}


def exact(case, seed):
    device = "cuda" if torch.cuda.is_available() else "cpu"
    kind = case["kind"]
    if kind == "sweep":
        if case["n"] * (case["hi"] + 1) ** 2 * (case["hi"] / 2 + 1) > 200000 or case["n"] > 12:
            return None
        phis, counts = [], []
        for d in _sweep_devices(case, seed):
            f = _Plain(d, device)
            phi, _ = f.solve()
            phis.append(phi)
            counts.append(f.count(phi, DOTS))
        return {"counts": np.array(counts), "phi": torch.cat(phis)}
    if case["nx"] * case["ny"] * case["nz"] > 2000000:
        return None
    dev, rng = _device(case, seed)
    if kind in ("predictor", "operators", "states"):
        phi = _potential(dev, rng)
    if kind == "states":
        return _dense_states(dev, phi, case["states"]) if int((~_dot_region(dev)[2]).sum()) <= 2500 else None
    if kind == "predictor":
        dev.quantum = _box_states(dev, case["states"], rng, phi)
    f = _Plain(dev, device)
    if kind == "gradient":
        return f.gradient(DOTS[int(dev.dir_val[1] > dev.dir_val[0])])
    if kind == "operators":
        v = rng.standard_normal(dev.n_nodes)
        p = torch.as_tensor(phi, device=device)
        F, c = f.residual(p)
        full = lambda w: f.product(c, w) + (1.0 - f.free) * w  # noqa: E731
        return {"F": F * f.free, "diag": f.diagonal(c), "Jv": full(torch.as_tensor(v, device=device)),
                "Jv32": full(torch.as_tensor(v.astype(np.float32), device=device).double()),
                "n": f.density(p), "counts": f.count(p, DOTS)}
    phi, _ = f.solve()
    if kind == "junction":
        return {"phi": phi, "n": f.density(phi)}
    return {"phi": phi, "n": f.density(phi), "counts": f.count(phi, DOTS)}
