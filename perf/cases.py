"""Timed cases of the library: what a user's program runs, over the range of sizes it runs.

Each case is a dict of plain values; ``prepare`` makes a program's inputs and
handles on the GPU, ``run`` is one pass through the public entry points,
``work`` the bytes and operations the pass cannot do without and ``exact`` the
same results from a plain torch transcription of the scheme in 64 bits.

Kinds of case:

* ``grid``     -- set an initial state on a handle, advance it by CFL steps chosen
                  on the device, optionally take the Fourier amplitudes (1-D tubes,
                  2-D periodic boxes and discs; FP64 or FP32; three schemes);
* ``host``     -- a host-stepped loop: read the CFL rate back, one step, repeat;
* ``grid3``    -- device-timed steps of the three-dimensional sweep;
* ``batch``    -- many uneven 1-D tubes in one launch;
* ``gradient`` -- a differentiable run and its backward pass to the initial state.
"""
from __future__ import annotations

import math
import os

import numpy as np
import torch

import paper_1210_5246_amd as csh
from paper_1210_5246_amd import autograd as cag

# the autotuner's choice is made anew by every program here, not taken from a file of an earlier one
os.environ.setdefault("CSH_TUNE_CACHE", "off")

CFL = 0.8
SEGMENT = 20  # steps between two checkpoints of the larger gradients


def listed():
    return [
        # one modified Sod tube to t = 0.2, the smallest problem anyone runs: 200 dependent steps of 256 cells
        {"name": "sod_256", "kind": "grid", "problem": "tube", "nx": 256, "ny": 1, "nsteps": 200, "t_end": 0.2,
         "scheme": "muscl", "dtype": "f64", "fourier": 0},
        # a program that looks at every step itself: rate back to the host, one step of a small odd grid, ten times
        {"name": "host_251x187", "kind": "host", "problem": "periodic", "nx": 251, "ny": 187, "nsteps": 10},
        # the mid-size periodic run of the CPU comparison
        {"name": "periodic_1024", "kind": "grid", "problem": "periodic", "nx": 1024, "ny": 1024, "nsteps": 100,
         "t_end": 0.0, "scheme": "muscl", "dtype": "f64", "fourier": 0},
        # the headline disc in its potential, with the spiral-growth diagnostic after the steps
        {"name": "disc_4096", "kind": "grid", "problem": "disc", "nx": 4096, "ny": 4096, "nsteps": 20,
         "t_end": 0.0, "scheme": "muscl", "dtype": "f64", "fourier": 6},
        # the FP32 twin of a disc run
        {"name": "disc_2048_f32", "kind": "grid", "problem": "disc", "nx": 2048, "ny": 2048, "nsteps": 20,
         "t_end": 0.0, "scheme": "muscl", "dtype": "f32", "fourier": 6},
        # the contact-resolving solver on a ragged outflow disc
        {"name": "hllc_1531x977", "kind": "grid", "problem": "disc", "nx": 1531, "ny": 977, "nsteps": 20,
         "t_end": 0.0, "scheme": "hllc", "dtype": "f64", "fourier": 0},
        # the central scheme on a periodic box
        {"name": "kt_1000x700", "kind": "grid", "problem": "periodic", "nx": 1000, "ny": 700, "nsteps": 20,
         "t_end": 0.0, "scheme": "kt", "dtype": "f64", "fourier": 0},
        # the full batch of shock tubes, workgroup size tuned once
        {"name": "tubes_512", "kind": "batch", "ntubes": 512, "nmin": 128, "nmax": 4096, "nsteps": 200,
         "tuned": True},
        # the three-dimensional benchmark box
        {"name": "box_256", "kind": "grid3", "nx": 256, "ny": 256, "nz": 256, "nsteps": 6},
        # a small ragged box: fewer planes than compute units, odd in every axis
        {"name": "box_61x47x33", "kind": "grid3", "nx": 61, "ny": 47, "nz": 33, "nsteps": 20},
        # the gradient of a 512^2 run of 200 steps, checkpointed
        {"name": "gradient_512", "kind": "gradient", "problem": "periodic", "nx": 512, "ny": 512, "nsteps": 200,
         "every": SEGMENT},
        # a small ragged gradient in the potential with open boundaries, every state kept
        {"name": "gradient_131x93", "kind": "gradient", "problem": "disc", "nx": 131, "ny": 93, "nsteps": 50,
         "every": 1},
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["tube", "grid", "grid", "grid", "host", "grid3", "batch", "gradient"])
    if kind == "tube":
        return {"kind": "grid", "problem": "tube", "nx": _size(rng, 64, 20000), "ny": 1,
                "nsteps": rng.randint(50, 300), "t_end": rng.choice([0.0, 0.2]),
                "scheme": rng.choice(["muscl", "muscl", "hllc", "kt"]), "dtype": rng.choice(["f64", "f64", "f32"]),
                "fourier": 0}
    if kind == "grid":
        nx, ny = _size(rng, 48, 4096), _size(rng, 48, 4096)
        cells = nx * ny
        return {"kind": "grid", "problem": rng.choice(["disc", "periodic"]), "nx": nx, "ny": ny,
                "nsteps": max(4, min(rng.randint(10, 60), int(3.3e8 / cells))), "t_end": 0.0,
                "scheme": rng.choice(["muscl", "muscl", "hllc", "kt"]), "dtype": rng.choice(["f64", "f64", "f32"]),
                "fourier": rng.choice([0, 2, 6])}
    if kind == "host":
        return {"kind": "host", "problem": rng.choice(["disc", "periodic"]), "nx": _size(rng, 48, 1024),
                "ny": _size(rng, 48, 1024), "nsteps": rng.randint(4, 16)}
    if kind == "grid3":
        return {"kind": "grid3", "nx": _size(rng, 24, 200), "ny": _size(rng, 24, 200), "nz": _size(rng, 24, 200),
                "nsteps": rng.randint(4, 12)}
    if kind == "batch":
        return {"kind": "batch", "ntubes": _size(rng, 24, 512), "nmin": 128, "nmax": _size(rng, 300, 4096),
                "nsteps": rng.randint(50, 200), "tuned": rng.choice([True, False])}
    one_d = rng.random() < 0.25
    return {"kind": "gradient", "problem": "periodic" if one_d else rng.choice(["disc", "periodic"]),
            "nx": _size(rng, 60, 2000) if one_d else _size(rng, 48, 512), "ny": 1 if one_d else _size(rng, 48, 512),
            "nsteps": rng.randint(20, 80), "every": rng.choice([1, SEGMENT])}


# ---- inputs ------------------------------------------------------------------------------------

def _smooth(g, shape, device, scale=50.0):
    """A smooth periodic field of unit variance: random plane waves of about ``scale`` cells and more."""
    waves = 16
    f = torch.zeros(shape, dtype=torch.float64, device=device)
    for _ in range(waves):
        arg = 0.0
        for ax, n in enumerate(shape):
            k = int(round(g.standard_normal() * n / scale)) if n > 1 else 0
            line = (2.0 * math.pi * k / n) * torch.arange(n, dtype=torch.float64, device=device)
            arg = arg + line.view([-1 if a == ax else 1 for a in range(len(shape))])
        f += torch.cos(arg + 2.0 * math.pi * g.random())
    return f * math.sqrt(2.0 / waves)


def _uniform(f):
    """The standard normal's distribution function: a field of about uniform marginals."""
    return 0.5 * (1.0 + torch.erf(f / math.sqrt(2.0)))


def _periodic(g, shape, device, d):
    """Lognormal density, velocities of 0.1 and a positive-definite stress rho L L^T, smooth and random."""
    rho = torch.exp(0.3 * _smooth(g, shape, device))
    vel = [0.1 * _smooth(g, shape, device) for _ in range(d)]
    low = [[(0.5 + 0.5 * _uniform(_smooth(g, shape, device))) if i == j else
            (-0.2 + 0.4 * _uniform(_smooth(g, shape, device))) for j in range(i + 1)] for i in range(d)]
    stress = [rho * sum(low[i][k] * low[j][k] for k in range(min(i, j) + 1)) for i in range(d) for j in range(i, d)]
    return torch.stack([rho] + vel + stress)


def _disc(g, nx, ny, device):
    """An exponential disc in a flat-rotation-curve potential with a Toomre-stable, anisotropic stress."""
    h = 1.0 / max(nx, ny)
    x = ((torch.arange(nx, dtype=torch.float64, device=device) + 0.5) - 0.5 * nx) * h
    y = (((torch.arange(ny, dtype=torch.float64, device=device) + 0.5) - 0.5 * ny) * h)[:, None]
    r2 = x * x + y * y
    r = torch.sqrt(r2)
    phi = torch.atan2(y.expand_as(r2), x.expand_as(r2))
    vc, rc = 1.0, 0.02
    rho = torch.exp(-r / 0.1) * (1.0 + 0.01 * torch.cos(2.0 * phi + 0.1 * _smooth(g, (ny, nx), device)))
    vphi = vc * r / torch.sqrt(r2 + rc * rc)
    kappa = vc * torch.sqrt(2.0 * r2 + 4.0 * rc * rc) / (r2 + rc * rc)
    # a coarse grid cannot resolve a cold outer disc: its floor grows with the cell size
    sr = torch.clamp(3.36 * 1.5 * rho / kappa, min=0.02 + 10.0 * h)
    prr, ppp = rho * sr * sr, rho * (0.7 * sr) ** 2
    c, s = torch.cos(phi), torch.sin(phi)
    return torch.stack([rho, -vphi * s, vphi * c, prr * c * c + ppp * s * s, (prr - ppp) * s * c,
                        prr * s * s + ppp * c * c])


def _tube(g, n):
    """The modified Sod tube with its states varied by a few per cent, discontinuity in the middle."""
    W = np.zeros((6, n))
    left = (np.arange(n) + 0.5) / n < 0.5
    v = 1.0 + 0.03 * g.standard_normal(6)
    W[0] = np.where(left, v[0], 0.125 * v[1])
    W[3] = np.where(left, v[2], 0.1 * v[3])
    W[5] = np.where(left, v[4], 0.1 * v[5])
    return W


def _fields(case, seed, device):
    """Primitive fields, cell sizes, boundaries and potential (vc, rc, x0, y0) of a grid-shaped case."""
    g = np.random.Generator(np.random.PCG64(seed))
    nx, ny = case["nx"], case["ny"]
    if case["problem"] == "tube":
        W = torch.from_numpy(_tube(g, nx)).to(device)
        dx, dy, bc, pot = 1.0 / nx, 1.0, (1, 1), None
    elif case["problem"] == "disc":
        W = _disc(g, nx, ny, device)
        dx = dy = 1.0 / max(nx, ny)
        bc, pot = (1, 1), (1.0, 0.02, -0.5 * nx * dx, -0.5 * ny * dy)
    else:
        W = _periodic(g, (ny, nx), device, 2)
        dx, dy, bc, pot = 1.0 / nx, (1.0 / ny if ny > 1 else 1.0), (0, 0), None
        if ny == 1:
            W = W[:, 0]
    return W.contiguous().to(_dtype(case)), dx, dy, bc, pot


def _dtype(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.float64


def _tubes(case, seed, device):
    """Offsets and primitive fields of independent shock tubes of uneven length."""
    g = np.random.Generator(np.random.PCG64(seed))
    # the lengths belong to the case: the same program, other states
    lengths = np.random.Generator(np.random.PCG64(case["ntubes"])).integers(case["nmin"], case["nmax"],
                                                                            size=case["ntubes"], endpoint=True)
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    W = np.zeros((6, int(off[-1])))
    for k, n in enumerate(lengths):
        left = (np.arange(n) + 0.5) / n < 0.5
        a, b = ((g.uniform(0.1, 1.0), g.uniform(-0.5, 0.5), g.uniform(0.05, 1.0), g.uniform(0.05, 1.0))
                for _ in range(2))
        for f, i in ((0, 0), (1, 1), (3, 2), (5, 3)):
            W[f, off[k]:off[k + 1]] = np.where(left, a[i], b[i])
    return off, torch.from_numpy(W).to(device)


def _box(case, seed, device):
    g = np.random.Generator(np.random.PCG64(seed))
    shape = (case["nz"], case["ny"], case["nx"])
    return _periodic(g, shape, device, 3).contiguous(), tuple(1.0 / n for n in reversed(shape))


def prepare(case, seed):
    device = torch.device("cuda")
    kind = case["kind"]
    if kind == "batch":
        off, W = _tubes(case, seed, device)
        b = csh.Batch(W, off)
        if case["tuned"]:
            b.autotune()
        # a batch advances its own state: a pass starts again from the initial one
        return {"case": case, "b": b, "U0": b.U.clone()}
    if kind == "grid3":
        W, h = _box(case, seed, device)
        G = csh.Grid3(W, h)
        return {"case": case, "G": G, "U0": G.U.clone()}
    W, dx, dy, bc, pot = _fields(case, seed, device)
    if kind == "gradient":
        target = torch.exp(0.3 * _smooth(np.random.Generator(np.random.PCG64(seed + 1)),
                                         tuple(W.shape[1:]), device))
        return {"case": case, "W": W.requires_grad_(True), "dx": dx, "dy": dy, "bc": bc, "pot": pot, "target": target}
    g = csh.Grid(W, dx, dy, bc)
    if pot is not None:
        g.set_potential(*pot)
    if kind == "grid" and case["scheme"] != "muscl":
        g.set_scheme(case["scheme"])
    state = {"case": case, "g": g, "W": W, "pot": pot, "log": "f4" if W.dtype == torch.float32 else "f8"}
    if kind == "host":
        state["other"] = torch.empty_like(g.U)
    return state


# ---- one pass ----------------------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind, nsteps = case["kind"], case["nsteps"]
    if kind == "batch":
        b = state["b"]
        b.U.copy_(state["U0"])
        dts = b.run(nsteps, CFL)
        return {"U": b.U, "dts": dts}
    if kind == "grid3":
        G = state["G"]
        G.U.copy_(state["U0"])
        dts = G.run_cfl(nsteps, CFL)
        return {"U": G.U, "dts": dts}
    if kind == "gradient":
        W = state["W"]
        W.grad = None
        U, dts = cag.sweep(W, state["dx"], state["dy"], bc=state["bc"], nsteps=nsteps, checkpoint_every=case["every"],
                           cfl=CFL, potential=state["pot"])
        loss = 0.5 * state["dx"] * state["dy"] * (U[0] - state["target"]).square().sum()
        loss.backward()
        return {"U": U, "dts": dts, "grad": W.grad}
    g = state["g"]
    U = g.set_state(state["W"])
    if kind == "host":
        dts, V = [], state["other"]
        s = g.max_signal_speed(U)
        for k in range(nsteps):
            dts.append(CFL / s)
            g.step(dts[-1], U, out=V)
            s = g.last_signal_speed()
            U, V = V, U
        return {"U": U, "dts": np.array(dts), "rate": np.array([s])}
    # the logs of a run are kept in the precision of its state
    out = {"U": U, "dts": g.run_cfl(nsteps, CFL, case["t_end"]).to(U.dtype)}
    if case["fourier"]:
        x0, y0 = (state["pot"][2], state["pot"][3]) if state["pot"] else (-0.5, -0.5)
        out["A"] = np.array(g.fourier_amplitudes(x0, y0, case["fourier"]), dtype=state["log"])
    return out


# ---- what a pass cannot do without -------------------------------------------------------------

# operations of one cell-update as the scheme is written (slopes, limiters, tracing, fluxes, update, CFL rate)
_FLOPS = {"muscl": 640, "hllc": 700, "kt": 800, "1d": 360, "3d": 1900}


def work(case):
    kind, nsteps = case["kind"], case["nsteps"]
    item = 4 if case.get("dtype") == "f32" else 8
    if kind == "batch":
        n = int(np.random.Generator(np.random.PCG64(case["ntubes"])).integers(
            case["nmin"], case["nmax"], size=case["ntubes"], endpoint=True).sum())
        return {"bytes": 2 * 6 * 8 * n, "flops": _FLOPS["1d"] * n * nsteps}
    if kind == "grid3":
        n = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": 2 * 10 * 8 * n * nsteps, "flops": _FLOPS["3d"] * n * nsteps}
    n = case["nx"] * case["ny"]
    one = _FLOPS["1d"] if case["ny"] == 1 else _FLOPS[case.get("scheme", "muscl")]
    state = 6 * item * n
    if kind == "gradient":  # forward, the states again, and the reverse step (two forward steps' operations)
        steps = nsteps * (3 if case["every"] == 1 else 4)
        return {"bytes": 2 * state * steps, "flops": one * n * steps}
    # a 1-D state need not leave the chip between the steps
    return {"bytes": 2 * state * (1 if case["ny"] == 1 else nsteps), "flops": one * n * nsteps}


# ---- the same results from a plain transcription in 64 bits ------------------------------------
#
# States are lists of fields: density, d velocity (or momentum) components, the
# upper triangle of the stress.  Grids are padded by two mapped cells on each
# side; the neighbours come from rolls of the padded arrays, and the two outer
# cells, where a roll wraps, are cut off again.

def _tri(i, j, d):
    i, j = min(i, j), max(i, j)
    return 1 + d + i * d - i * (i - 1) // 2 + (j - i)


def _prim(U, d):
    u = [m / U[0] for m in U[1:1 + d]]
    return [U[0]] + u + [U[_tri(i, j, d)] - U[1 + i] * u[j] for i in range(d) for j in range(i, d)]


def _cons(W, d):
    m = [W[0] * u for u in W[1:1 + d]]
    return [W[0]] + m + [W[_tri(i, j, d)] + m[i] * W[1 + j] for i in range(d) for j in range(i, d)]


def _flux(W, n, d):
    """Moments of the flux along n: a conserved variable's advection plus the stress terms."""
    un, U = W[1 + n], _cons(W, d)
    F = [U[1 + n]] + [U[1 + i] * un + W[_tri(i, n, d)] for i in range(d)]
    for i in range(d):
        for j in range(i, d):
            F.append(U[_tri(i, j, d)] * un + W[_tri(i, n, d)] * W[1 + j] + W[_tri(j, n, d)] * W[1 + i])
    return F


def _jac(W, D, n, d):
    un, dn = W[1 + n], D[1 + n]
    out = [un * D[0] + W[0] * dn] + [un * D[1 + i] + D[_tri(i, n, d)] / W[0] for i in range(d)]
    for i in range(d):
        for j in range(i, d):
            out.append(un * D[_tri(i, j, d)] + W[_tri(i, j, d)] * dn + W[_tri(i, n, d)] * D[1 + j] +
                       W[_tri(j, n, d)] * D[1 + i])
    return out


def _mc(a, b):
    m = torch.minimum(torch.minimum(2.0 * a.abs(), 2.0 * b.abs()), 0.5 * (a + b).abs())
    return torch.where(a * b > 0, torch.sign(a) * m, torch.zeros_like(m))


def _slope(W, L, R, n, d):
    """Characteristic MC-limited slope along n from the one-sided differences L and R."""
    T = [t for t in range(d) if t != n]
    nn = _tri(n, n, d)
    rho, P = W[0], W[nn]
    c = torch.sqrt(P / rho)
    a = math.sqrt(3.0) * c
    q = {t: W[_tri(n, t, d)] / P for t in T}
    pairs = [(s, t) for i, s in enumerate(T) for t in T[i:]]

    def waves(D):
        s, h = D[nn] / (6 * P), D[1 + n] / (2 * a)
        out = [s - h, s + h, D[0] - rho * D[nn] / (3 * P)]
        for t in T:
            s, h = (D[_tri(n, t, d)] - q[t] * D[nn]) / (2 * P), (q[t] * D[1 + n] - D[1 + t]) / (2 * c)
            out += [s + h, s - h]
        for s, t in pairs:
            out.append(D[_tri(s, t, d)] - q[t] * D[_tri(n, s, d)] - q[s] * D[_tri(n, t, d)] +
                       (4 * q[s] * q[t] - W[_tri(s, t, d)] / P) * D[nn] / 3)
        return out

    m = [_mc(x, y) for x, y in zip(waves(L), waves(R))]
    S, D = m[0] + m[1], m[1] - m[0]
    sh = {t: (m[3 + 2 * k] + m[4 + 2 * k], m[4 + 2 * k] - m[3 + 2 * k]) for k, t in enumerate(T)}
    out = [None] * len(W)
    out[0] = rho * S + m[2]
    out[1 + n] = a * D
    out[nn] = 3 * P * S
    for t in T:
        out[1 + t] = a * q[t] * D + c * sh[t][1]
        out[_tri(n, t, d)] = 3 * W[_tri(n, t, d)] * S + P * sh[t][0]
    for k, (s, t) in enumerate(pairs):
        ps, pt = W[_tri(n, s, d)], W[_tri(n, t, d)]
        out[_tri(s, t, d)] = ((W[_tri(s, t, d)] + ps * q[t] + pt * q[s]) * S + ps * sh[t][0] + pt * sh[s][0] +
                              m[3 + 2 * len(T) + k])
    return out, a


def _hll(L, R, n, d):
    nn = _tri(n, n, d)
    al, ar = torch.sqrt(3 * L[nn] / L[0]), torch.sqrt(3 * R[nn] / R[0])
    sl = torch.clamp(torch.minimum(L[1 + n] - al, R[1 + n] - ar), max=0.0)
    sr = torch.clamp(torch.maximum(L[1 + n] + al, R[1 + n] + ar), min=0.0)
    return [(sr * f - sl * g + sl * sr * (v - u)) / (sr - sl)
            for f, g, u, v in zip(_flux(L, n, d), _flux(R, n, d), _cons(L, d), _cons(R, d))]


def _hllc(L, R, n, d):
    t, nn, nt, tt = 1 - n, _tri(n, n, d), _tri(0, 1, d), _tri(1 - n, 1 - n, d)
    al, ar = torch.sqrt(3 * L[nn] / L[0]), torch.sqrt(3 * R[nn] / R[0])
    sl, sr = torch.minimum(L[1 + n] - al, R[1 + n] - ar), torch.maximum(L[1 + n] + al, R[1 + n] + ar)
    dl, dr = L[0] * (sl - L[1 + n]), R[0] * (sr - R[1 + n])
    us = (R[nn] - L[nn] + dl * L[1 + n] - dr * R[1 + n]) / (dl - dr)
    vs = (R[nt] - L[nt] + dl * L[1 + t] - dr * R[1 + t]) / (dl - dr)
    left = us >= 0
    K = [torch.where(left, x, y) for x, y in zip(L, R)]
    sk, dk = torch.where(left, sl, sr), torch.where(left, dl, dr)
    skc = torch.where(left, torch.clamp(sl, max=0.0), torch.clamp(sr, min=0.0))
    pnn, pnt = K[nn] + dk * (us - K[1 + n]), K[nt] + dk * (vs - K[1 + t])
    zero = torch.zeros_like(us)
    star, side = [zero] * 6, [zero] * 6
    star[1 + n], star[1 + t], star[nn], star[nt], star[tt] = pnn, pnt, 2 * pnn * us, pnt * us + pnn * vs, 2 * pnt * vs
    side[1 + n], side[1 + t], side[nn], side[nt], side[tt] = (
        K[nn], K[nt], 2 * K[nn] * K[1 + n], K[nt] * K[1 + n] + K[nn] * K[1 + t], 2 * K[nt] * K[1 + t])
    return [f + skc / (sk - us) * (u * (us - K[1 + n]) + s - o)
            for f, u, s, o in zip(_flux(K, n, d), _cons(K, d), star, side)]


def _kt_flux(L, R, n, d):
    nn = _tri(n, n, d)
    a = torch.maximum(L[1 + n].abs() + torch.sqrt(3 * L[nn] / L[0]), R[1 + n].abs() + torch.sqrt(3 * R[nn] / R[0]))
    return [0.5 * (f + g) - 0.5 * a * (v - u)
            for f, g, u, v in zip(_flux(L, n, d), _flux(R, n, d), _cons(L, d), _cons(R, d))]


def _roll(fields, ax, by):
    return [torch.roll(f, by, -1 - ax) for f in fields]


class _Plain:
    """The scheme on one padded grid: axes (0 the last dimension), cell sizes, padding and cutting."""

    def __init__(self, d, axes, h, pad, cut, scheme="muscl", pot=None, centres=None):
        self.d, self.axes, self.h, self.pad, self.cut = d, axes, h, pad, cut
        self.scheme, self.pot, self.centres = scheme, pot, centres

    def rate(self, U):
        W = _prim(U, self.d)
        return sum((W[1 + n].abs() + torch.sqrt(3 * W[_tri(n, n, self.d)] / W[0])) / self.h[n] for n in self.axes)

    def _update(self, U, W, faces, flux, k):
        """U less dt/h times the difference of the face fluxes; k[n] = dt/h."""
        for n in self.axes:
            lo, hi = faces(W, n)
            F = flux(hi, _roll(lo, n, -1), n, self.d)
            U = [u - self.cut(k[n] * (f - g)) for u, f, g in zip(U, F, _roll(F, n, 1))]
        return U

    def step(self, U, dt):
        k = {n: dt / self.h[n] for n in self.axes}
        kp = {n: (self.pad(v) if torch.is_tensor(v) and v.dim() else v) for n, v in k.items()}
        d = self.d
        if self.scheme == "kt":
            def faces(W, n):
                s = [0.5 * _mc(w - l, r - w) for w, l, r in zip(W, _roll(W, n, 1), _roll(W, n, -1))]
                return [w - x for w, x in zip(W, s)], [w + x for w, x in zip(W, s)]

            def stage(V, f):
                W = _prim([self.pad(v) for v in V], d)
                return self._update(U, W, faces, _kt_flux, {n: f * x for n, x in kp.items()})
            V = stage(stage(U, 0.5), 1.0)
        else:
            W = _prim([self.pad(u) for u in U], d)
            slopes = {n: _slope(W, [w - l for w, l in zip(W, _roll(W, n, 1))],
                                [r - w for w, r in zip(W, _roll(W, n, -1))], n, d) for n in self.axes}
            base = W
            for n in self.axes:
                base = [b - 0.5 * kp[n] * x for b, x in zip(base, _jac(W, slopes[n][0], n, d))]

            def faces(W, n):
                s, a = slopes[n]
                up = 0.5 + 0.5 * kp[n] * torch.clamp(W[1 + n] + a, max=0.0)
                dn = 0.5 - 0.5 * kp[n] * torch.clamp(W[1 + n] - a, min=0.0)
                return [b - dn * x for b, x in zip(base, s)], [b + up * x for b, x in zip(base, s)]
            V = self._update(U, W, faces, _hllc if self.scheme == "hllc" else _hll, kp)
        if self.pot is not None:  # the velocity kick of the fixed field
            vc, rc = self.pot[:2]
            x, y = self.centres
            f = -dt * vc * vc / (x * x + y * y + rc * rc)
            W = _prim(V, d)
            V = _cons([W[0], W[1] + f * x, W[2] + f * y] + W[3:], d)
        return V


def _map(n, bc, device):
    i = torch.arange(-2, n + 2, device=device)
    return i % n if bc == 0 else i.clamp(0, n - 1)


def _plain_grid(shape, d, h, bc, scheme="muscl", pot=None, device="cuda"):
    """shape, in the order of the dimensions; h and bc along axes 0 (the last dimension), 1, ..."""
    axes = [n for n in range(len(shape)) if shape[-1 - n] > 1 or len(shape) == 1]
    maps = {n: _map(shape[-1 - n], bc[n], device) for n in axes}

    def pad(f):
        for n in axes:
            f = f.index_select(f.dim() - 1 - n, maps[n])
        return f

    def cut(f):
        for n in axes:
            f = f.narrow(f.dim() - 1 - n, 2, shape[-1 - n])
        return f

    centres = None
    if pot is not None:
        x = pot[2] + (torch.arange(shape[-1], dtype=torch.float64, device=device) + 0.5) * h[0]
        y = (pot[3] + (torch.arange(shape[-2], dtype=torch.float64, device=device) + 0.5) * h[1])[:, None]
        centres = (x, y)
    return _Plain(d, axes, h, pad, cut, scheme, pot, centres)


def _plain_run(p, U, nsteps, t_end=0.0):
    dts, t = [], 0.0
    for _ in range(nsteps):
        dt = CFL / p.rate(U).max().item()
        if t_end > 0:
            dt = 0.0 if t >= t_end else min(dt, t_end - t)
        U = p.step(U, dt)
        dts.append(dt)
        t += dt
    return U, dts


def exact(case, seed):
    device = torch.device("cuda")
    kind, nsteps = case["kind"], case["nsteps"]
    if kind == "batch":
        off, W = _tubes(case, seed, device)
        n = torch.from_numpy(np.diff(off)).to(device)
        tube = torch.repeat_interleave(torch.arange(len(n), device=device), n)
        starts = torch.from_numpy(off[:-1]).to(device)
        ptube = torch.repeat_interleave(torch.arange(len(n), device=device), n + 4)
        pos = torch.arange(len(ptube), device=device) - (starts + 4 * torch.arange(len(n), device=device))[ptube] - 2
        idx = starts[ptube] + pos.clamp(min=0).minimum(n[ptube] - 1)
        back = torch.arange(len(tube), device=device) + 4 * tube + 2
        p = _Plain(2, [0], {0: 1.0 / n[tube].double()}, lambda f: f[idx], lambda f: f[back])
        U, dts = _cons(list(W), 2), []
        for _ in range(nsteps):
            s = torch.zeros(len(n), dtype=torch.float64, device=device).scatter_reduce(0, tube, p.rate(U), "amax")
            dts.append(CFL / s)
            U = p.step(U, (CFL / s)[tube])
        return {"U": torch.stack(U), "dts": torch.stack(dts, dim=1)}
    if kind == "grid3":
        W, h = _box(case, seed, device)
        p = _plain_grid(tuple(W.shape[1:]), 3, h, (0, 0, 0))
        U, dts = _plain_run(p, _cons(list(W), 3), nsteps)
        return {"U": torch.stack(U), "dts": torch.tensor(dts, dtype=torch.float64)}
    W, dx, dy, bc, pot = _fields(case, seed, device)
    W = W.double()
    p = _plain_grid(tuple(W.shape[1:]), 2, (dx, dy), bc, case.get("scheme", "muscl"), pot)
    if kind == "gradient":
        states, dts = [_cons(list(W), 2)], []
        for _ in range(nsteps):
            dts.append(CFL / p.rate(states[-1]).max().item())
            states.append(p.step(states[-1], dts[-1]))
        target = torch.exp(0.3 * _smooth(np.random.Generator(np.random.PCG64(seed + 1)), tuple(W.shape[1:]), device))
        lam = [torch.zeros_like(f) for f in states[-1]]
        lam[0] = dx * dy * (states[-1][0] - target)
        for U, dt in zip(states[-2::-1], dts[::-1]):
            with torch.enable_grad():
                V = [f.detach().requires_grad_(True) for f in U]
                lam = torch.autograd.grad(p.step(V, dt), V, lam)
        with torch.enable_grad():
            V = W.detach().requires_grad_(True)
            grad, = torch.autograd.grad(_cons(list(V), 2), V, lam)
        return {"U": torch.stack(states[-1]), "dts": torch.tensor(dts, dtype=torch.float64), "grad": grad}
    U, dts = _plain_run(p, _cons(list(W), 2), nsteps, case.get("t_end", 0.0))
    out = {"U": torch.stack(U), "dts": torch.tensor(dts, dtype=torch.float64)}
    if kind == "host":
        return {"U": out["U"], "dts": out["dts"], "rate": p.rate(U).max().reshape(1)}
    if case["fourier"]:
        x0, y0 = (pot[2], pot[3]) if pot else (-0.5, -0.5)
        x = x0 + (torch.arange(case["nx"], dtype=torch.float64, device=device) + 0.5) * dx
        y = (y0 + (torch.arange(case["ny"], dtype=torch.float64, device=device) + 0.5) * dy)[:, None]
        phi = torch.atan2(y.expand(case["ny"], case["nx"]), x.expand(case["ny"], case["nx"]))
        on = (x * x + y * y > 0).double()
        rho = U[0] * on
        out["A"] = np.array([(torch.hypot((rho * torch.cos(m * phi)).sum(), (rho * torch.sin(m * phi)).sum()) /
                              U[0].sum()).item() for m in range(1, case["fourier"] + 1)])
    return out
