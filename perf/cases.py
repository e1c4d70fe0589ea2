"""Performance cases of the method-of-lines library: what a program that evolves patches
with it calls, over the range of sizes, systems and options it is used with.

`listed()` names the cases that are followed; `draw(rng)` gives another one from the same
ranges; `prepare` builds what such a program holds before the call (patchset, states, graph,
kept stage states); `run` is one pass through the public entry points; `work` the bytes and
operations of one pass that no implementation can do without; `exact` the same outputs from
plain torch in 64 bits, for the cases where the whole computation is short enough to restate.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1806_04182_amd import adjoint
from paper_1806_04182_amd import bh_runs
from paper_1806_04182_amd import fmr
from paper_1806_04182_amd import molamr as M
from paper_1806_04182_amd import synth

G = 3
SYSTEMS = {"wave": M.MOL_WAVE, "mhd": M.MOL_MHD, "glm": M.MOL_MHD_GLM, "ccz4": M.MOL_CCZ4}
RECON = {"weno5z": M.MOL_RECON_WENO5Z, "weno5js": M.MOL_RECON_WENO5JS, "weno3": M.MOL_RECON_WENO3}
FLUX = {"llf": M.MOL_FLUX_LLF, "hll": M.MOL_FLUX_HLL, "split": M.MOL_FLUX_SPLIT}
SIGMA, GAMMA, CH, KPSI = 0.1, 5.0 / 3.0, 1.0, 0.5
KZ = KC = 0.1
GD_G, GD_ETA = 0.75, 2.0


def listed():
    return [
        # the smallest evolution: launch latency decides (the 20-step wave runs)
        dict(name="wave_step_32", kind="step", system="wave", scheme="rk4", nx=32, ny=32, nz=32, cuts=1),
        # the largest single level: streaming memory traffic
        dict(name="wave_step_512", kind="step", system="wave", scheme="rk4", nx=512, ny=512, nz=512, cuts=1),
        # one CCZ4 patch of the size a refined level has, and the size runs are quoted on
        dict(name="ccz4_step_48", kind="step", system="ccz4", scheme="rk4", nx=48, ny=48, nz=48, cuts=1),
        dict(name="ccz4_step_96", kind="step", system="ccz4", scheme="rk4", nx=96, ny=96, nz=96, cuts=1),
        # MHD with its defaults, and the cleaned nine-field system on a ragged level of several patches
        dict(name="mhd_step_128", kind="step", system="mhd", scheme="ssprk3", recon="weno5z", flux="llf",
             nx=128, ny=128, nz=128, cuts=1),
        dict(name="glm_step_ragged", kind="step", system="glm", scheme="rk4", recon="weno3", flux="hll",
             nx=93, ny=61, nz=47, cuts=2),
        # whole coarse steps: the 200-patch hierarchy, the black hole's nested levels (open
        # domain, replayed graph) and the reflection channel, a chain of very small launches
        dict(name="amr_step_200", kind="amr", layout=0),
        dict(name="bh_step_5x32", kind="bh", levels=5, n=32),
        dict(name="channel_step_80", kind="channel", n=80, ratios=2),
        # gradients: one reverse CCZ4 step from kept stage states; the wave objective forward and back
        dict(name="ccz4_reverse_48", kind="reverse", system="ccz4", nx=48, ny=48, nz=48, cuts=1),
        dict(name="wave_gradient_64", kind="gradient", system="wave", n=64, steps=40),
        # the constraint monitors a run prints between steps
        dict(name="ccz4_monitor_ragged", kind="monitor", system="ccz4", nx=101, ny=58, nz=77, cuts=2),
    ]


def _size(rng, lo, hi):
    """Three extents around a common size spread over its logarithm, odd ones as often as even."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return {k: max(lo, min(hi, int(round(n * rng.uniform(0.75, 1.25))))) for k in ("nx", "ny", "nz")}


def draw(rng):
    kind = rng.choice(["wave", "ccz4", "ccz4", "mhd", "mhd", "reverse", "reverse", "gradient", "monitor", "bh", "channel"])
    if kind == "wave":
        return dict(kind="step", system="wave", scheme="rk4", cuts=rng.choice([1, 1, 2, 3]), **_size(rng, 20, 400))
    if kind == "ccz4":
        return dict(kind="step", system="ccz4", scheme="rk4", cuts=rng.choice([1, 1, 2, 3]), **_size(rng, 18, 128))
    if kind == "mhd":
        return dict(kind="step", system=rng.choice(["mhd", "mhd", "glm"]), scheme=rng.choice(["rk4", "ssprk3"]),
                    recon=rng.choice(["weno5z", "weno5z", "weno5js", "weno3"]),
                    flux=rng.choice(["llf", "llf", "hll", "split"]), cuts=rng.choice([1, 1, 2, 3]),
                    **_size(rng, 18, 144))
    if kind == "reverse":
        system = rng.choice(["ccz4", "ccz4", "wave"])
        return dict(kind="reverse", system=system, cuts=rng.choice([1, 1, 2]),
                    **_size(rng, 14, 64 if system == "ccz4" else 160))
    if kind == "gradient":
        system = rng.choice(["ccz4", "wave"])
        return dict(kind="gradient", system=system, n=rng.randint(20, 40 if system == "ccz4" else 96),
                    steps=rng.randint(2, 6) if system == "ccz4" else rng.randint(10, 40))
    if kind == "monitor":
        return dict(kind="monitor", system=rng.choice(["ccz4", "ccz4", "wave"]), cuts=rng.choice([1, 2]),
                    **_size(rng, 18, 128))
    if kind == "bh":
        return dict(kind="bh", levels=rng.randint(3, 5), n=2 * rng.randint(14, 24))
    return dict(kind="channel", n=40 * rng.randint(1, 4), ratios=rng.choice([2, 4, 22]))


# ------------------------------------------------------------------ set-up

def _dims(case):
    return case["nx"], case["ny"], case["nz"]


def _boxes(case):
    """The level's patches: the domain cut into `cuts` uneven parts per axis (2: 2x2x1 ...)."""
    n, c = _dims(case), case["cuts"]
    edges = []
    for d in range(3):
        parts = c if d < 2 else 1
        at = [0] + [(n[d] * (2 * p + 1)) // (2 * parts + 1) + p % 2 for p in range(1, parts)] + [n[d]]
        edges.append(at)
    return [((edges[0][i], edges[1][j], edges[2][k]),
             (edges[0][i + 1] - 1, edges[1][j + 1] - 1, edges[2][k + 1] - 1))
            for k in range(len(edges[2]) - 1) for j in range(len(edges[1]) - 1) for i in range(len(edges[0]) - 1)]


def _dx(case):
    return (1.0 if case["system"] in ("mhd", "glm") else 2.0) / max(_dims(case))


def _xlo(case):
    return (0.0,) * 3 if case["system"] in ("mhd", "glm") else (-1.0,) * 3


def _patchset(case):
    s = SYSTEMS[case["system"]]
    kw = dict(sigma=SIGMA) if s in (M.MOL_WAVE, M.MOL_CCZ4) else dict(
        sigma=0.0, gamma_ad=GAMMA, mhd_recon=RECON[case["recon"]], mhd_flux=FLUX[case["flux"]], mhd_ch=CH,
        mhd_kpsi=KPSI)
    return M.Patchset(M.Hierarchy(_dims(case), _xlo(case), _dx(case), [(1, _boxes(case))]), M.System(s, **kw))


def _views(ps, level, buf, nf):
    """(nf, nz, ny, nx) view of each patch's interior inside a level buffer (no copy)."""
    L, out = ps.layouts[level], []
    for (nx, ny, nz), px, fs, off in zip(L["dims"], L["pitches"], L["fstrides"], L["offsets"]):
        pz = px * (ny + 2 * G)
        out.append(buf.as_strided((nf, nz, ny, nx), (fs, pz, px, 1), off + G * (pz + px + 1)))
    return out


def _rng(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _grid(case):
    h, lo = _dx(case), _xlo(case)
    ax = [lo[d] + h * torch.arange(_dims(case)[d], dtype=torch.float64, device="cuda") for d in range(3)]
    return ax[0][None, None, :], ax[1][None, :, None], ax[2][:, None, None]


def _pulse(case, prm):
    """exp(-|x - c|^2 / w^2) times A with the nearest periodic image."""
    n, h = _dims(case), _dx(case)
    r2 = 0.0
    for x, c, m in zip(_grid(case), prm[2:], n):
        d = x - c
        d = d - m * h * torch.round(d / (m * h))
        r2 = r2 + d * d
    return prm[0] * torch.exp(-r2 / prm[1] ** 2)


def _initial(case, seed):
    """The level's interior state (nf, nz, ny, nx), from the seed."""
    g, n = _rng(seed), _dims(case)
    shape = tuple(reversed(n))
    rand = lambda *s: torch.rand(*s, dtype=torch.float64, device="cuda", generator=g)  # noqa: E731
    a = [float(v) for v in rand(8).cpu()]
    if case["system"] == "wave":
        # a pulse of width 0.2 at a random centre, as the runs use
        U = torch.zeros((2,) + shape, dtype=torch.float64, device="cuda")
        U[0] = _pulse(case, [0.5 + a[0], 0.2 + 0.2 * a[1]] + [0.6 * v - 0.3 for v in a[2:5]])
        return U
    if case["system"] == "ccz4":
        # a lapse pulse on flat space with small noise on every field: smooth, every term alive
        U = 1e-6 * (2.0 * rand(25, *shape) - 1.0)
        U += torch.tensor(synth.CCZ4_FLAT, device="cuda")[:, None, None, None]
        U[18] += _pulse(case, [0.05 + 0.1 * a[0], 0.3 + 0.3 * a[1]] + [0.6 * v - 0.3 for v in a[2:5]])
        return U
    # MHD: the smooth vortical state of the benchmarks with random phases
    x, y, z = _grid(case)
    h = _dx(case)
    x, y, z = ((v / (m * h) + p) * (2.0 * math.pi) for v, m, p in zip((x, y, z), n, a[:3]))
    s = torch.sin
    one = torch.ones(shape, dtype=torch.float64, device="cuda")
    rho = one + 1e-3 * (2.0 * rand(*shape) - 1.0)
    v = [0.5 * (s(z) - s(y)) * one, 0.5 * (s(x) - s(z)) * one, 0.5 * (s(y) - s(x)) * one]
    B = [0.3 * (s(2 * z) - s(y)) * one, 0.3 * (s(2 * x) - s(z)) * one, 0.3 * (s(2 * y) - s(x)) * one]
    E = 0.5 * rho * sum(q * q for q in v) + 0.6 / (GAMMA - 1.0) + 0.5 * sum(q * q for q in B)
    U = [rho] + [rho * q for q in v] + [E] + B
    if case["system"] == "glm":
        U.append(1e-2 * s(x + y) * one)
    return torch.stack(U)


def _load(ps, case, level_buf, U):
    for (lo, hi), view in zip(_boxes(case), _views(ps, 0, level_buf, U.shape[0])):
        view.copy_(U[:, lo[2]:hi[2] + 1, lo[1]:hi[1] + 1, lo[0]:hi[0] + 1])


def _dt(case):
    return (0.2 if case["system"] in ("mhd", "glm") else 0.25) * _dx(case)


RADIUS = 0.6123


def _radius(seed):
    """Radius of the reverse step's sphere integral."""
    return 0.5 + 0.25 * float(torch.rand(1, dtype=torch.float64, generator=torch.Generator().manual_seed(int(seed))))


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "amr":
        levels, N0, dx0 = synth.amr_three_levels(case["layout"])
        ps = M.Patchset(M.Hierarchy(N0, (-1, -1, -1), dx0, levels), M.System(M.MOL_CCZ4, sigma=SIGMA))
        states = ps.alloc_states()
        g = _rng(seed)
        flat = torch.tensor(synth.CCZ4_FLAT, device="cuda")
        for lv, s in enumerate(states):
            s["U"].uniform_(-1e-6, 1e-6, generator=g)
            for v in _views(ps, lv, s["U"], 25):
                v += flat[:, None, None, None]
        return dict(st, ps=ps, states=states, graph=ps.graph_create(states, 0.25 * dx0))
    if kind == "bh":
        spin = 0.1 + 0.3 * float(torch.rand(1, generator=torch.Generator().manual_seed(int(seed))))
        return dict(st, bh=bh_runs.SingleBH(nlev=case["levels"], N=case["n"], L=16.0, spin=spin))
    if kind == "channel":
        ratios = {2: (2,), 4: (4,), 22: (2, 2)}[case["ratios"]]
        width = 0.15 + 0.1 * float(torch.rand(1, generator=torch.Generator().manual_seed(int(seed))))
        return dict(st, run=fmr.ChannelRun(case["n"], ratios, width=width))
    if kind == "gradient":
        a = torch.rand(5, dtype=torch.float64, generator=torch.Generator().manual_seed(int(seed))).tolist()
        wave = case["system"] == "wave"
        prm = [1.0 if wave else 0.1, 0.25 if wave else 0.4, 0.0, 0.0, 0.0]
        prm = [p * (0.9 + 0.2 * r) + (0.1 * r if i > 1 else 0.0) for i, (p, r) in enumerate(zip(prm, a))]
        n = case["n"]
        ps = M.Patchset(M.single_patch((n, n, n), (-1, -1, -1), 2.0 / n),
                        M.System(SYSTEMS[case["system"]], sigma=SIGMA))
        return dict(st, ps=ps, prm=torch.tensor(prm, dtype=torch.float64))
    ps = _patchset(case)
    U = _initial(case, seed)
    st.update(ps=ps, dt=_dt(case))
    if kind == "step":
        states = ps.alloc_states()
        _load(ps, case, states[0]["U"], U)
        return dict(st, states=states)
    buf = ps.alloc(0)
    _load(ps, case, buf, U)
    ps.fill_ghosts(0, buf)
    if kind == "monitor":
        which = M.MOL_MON_ALL if case["system"] == "ccz4" else M.MOL_MON_KO
        return dict(st, U=buf, which=which, point=ps.alloc(0),
                    out=torch.zeros(M.MOL_MON_OUT, dtype=torch.float64, device="cuda"))
    # reverse: the four stage states of the step, kept as a program that walks back keeps them
    stages, acc = [buf] + [ps.alloc(0) for _ in range(3)], ps.alloc(0)
    for s in range(1, 4):
        ps.rk_stage(0, M.MOL_RK4, s, st["dt"], buf, stages[s - 1], acc, stages[s])
        ps.fill_ghosts(0, stages[s])
    return dict(st, radius=_radius(seed), stages=stages, lam=ps.alloc(0), w=[ps.alloc(0) for _ in range(3)], work=ps.alloc_work(0))


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "step":
        ps, s = state["ps"], state["states"]
        ps.advance(s, state["dt"], M.MOL_BATCHED | (M.MOL_ADV_SSPRK3 if case["scheme"] == "ssprk3" else 0))
        return _views(ps, 0, s[0]["U"], ps.nf)
    if kind == "amr":
        state["graph"].launch()
        return [s["U"] for s in state["states"]]  # level buffers: 200 patches are too many to name one by one
    if kind == "bh":
        bh = state["bh"]
        bh.graph.launch()
        return [_views(bh.ps, lv, s["U"], 25)[0] for lv, s in enumerate(bh.st)]
    if kind == "channel":
        r = state["run"]
        r.ps.advance(r.states, 0.25 * r.dx0, M.MOL_BATCHED | M.MOL_TIME_BOR)
        return [v for lv, s in enumerate(r.states) for v in _views(r.ps, lv, s["U"], 2)]
    if kind == "gradient":
        p = state["prm"].clone().requires_grad_(True)
        fn = adjoint.sphere_objective if case["system"] == "wave" else adjoint.ccz4_lapse_objective
        J = fn(p, state["ps"], case["steps"], 0.25 * 2.0 / case["n"], RADIUS)
        J.backward()
        return J.detach(), p.grad
    ps = state["ps"]
    if kind == "monitor":
        ps.monitor(0, state["U"], state["which"], state["out"], pointwise=state["point"])
        return state["out"], _views(ps, 0, state["point"], 6 if case["system"] == "ccz4" else 1)
    # reverse: the gradient of the objective's sphere integral through one RK4 step
    ps.sphere_adjoint(0, 18 if case["system"] == "ccz4" else 0, state["radius"], 1.0, state["lam"])
    ps.rk4_adjoint_step_stages(0, state["dt"], state["lam"], state["w"],
                               stages=state["stages"] if case["system"] == "ccz4" else None, work=state["work"])
    return _views(ps, 0, state["lam"], ps.nf)


# ---------------------------------------------------------------- the work

NF = {"wave": 2, "mhd": 8, "glm": 9, "ccz4": 25}


def _stage_flops(case):
    """Operations of one right-hand side and stage update per point."""
    s = case.get("system", "ccz4")
    if s == "wave":
        return 100.0
    if s == "ccz4":
        return 5000.0
    return {"weno5z": 4500.0, "weno5js": 4200.0, "weno3": 2200.0}[case["recon"]] * NF[s] / 8.0


def work(case):
    kind = case["kind"]
    if kind == "amr":
        levels, _, _ = synth.amr_three_levels(case["layout"])
        pts = [sum(math.prod(h - l + 1 for l, h in zip(lo, hi)) for lo, hi in b) for _, b in levels]
        return {"bytes": 400.0 * (pts[0] + 2 * pts[1] + 6 * pts[2]), "flops": 2e4 * (pts[0] + 2 * pts[1] + 6 * pts[2])}
    if kind == "bh":
        steps = case["n"] ** 3 * (2 ** case["levels"] - 1)
        return {"bytes": 400.0 * steps, "flops": 2e4 * steps}
    if kind == "channel":
        steps, f, levels = 0, 1, fmr.channel_levels(case["n"], {2: (2,), 4: (4,), 22: (2, 2)}[case["ratios"]])[0]
        for R, boxes in levels:
            f *= R
            steps += f * sum(math.prod(h - l + 1 for l, h in zip(lo, hi)) for lo, hi in boxes)
        return {"bytes": 32.0 * steps, "flops": 400.0 * steps}
    if kind == "gradient":
        nf, pts = NF[case["system"]], case["n"] ** 3 * case["steps"]
        # forward step, and the reverse step reading the step's state
        return {"bytes": 48.0 * nf * pts, "flops": 4.0 * (3.0 if nf == 25 else 2.0) * _stage_flops(case) * pts}
    pts, nf = math.prod(_dims(case)), NF[case["system"]]
    if kind == "step":
        return {"bytes": 16.0 * nf * pts, "flops": (4 if case["scheme"] == "rk4" else 3) * _stage_flops(case) * pts}
    if kind == "monitor":
        return {"bytes": 8.0 * (nf + (6 if nf == 25 else 1)) * pts, "flops": (2500.0 if nf == 25 else 60.0) * pts}
    # reverse: lam is written, and for CCZ4 the four stage states are read
    return {"bytes": 8.0 * (nf * (5 if nf == 25 else 1)) * pts, "flops": 4.0 * (2.0 if nf == 25 else 1.0) * _stage_flops(case) * pts}


# ------------------------------------------- the same outputs in plain torch

def _at(u, axis, m):
    """u at the point m further along axis (0: x), periodic."""
    return torch.roll(u, -m, dims=u.dim() - 1 - axis)


def _d1(u, k, h):
    return (8.0 * (_at(u, k, 1) - _at(u, k, -1)) - (_at(u, k, 2) - _at(u, k, -2))) / (12.0 * h)


def _d2(u, k, l, h):
    if k != l:
        return _d1(_d1(u, k, h), l, h)
    return (16.0 * (_at(u, k, 1) + _at(u, k, -1)) - (_at(u, k, 2) + _at(u, k, -2)) - 30.0 * u) / (12.0 * h * h)


def _ko(u, h):
    r = 0.0
    for k in range(3):
        r = r + (_at(u, k, 3) + _at(u, k, -3)) - 6.0 * (_at(u, k, 2) + _at(u, k, -2)) + 15.0 * (
            _at(u, k, 1) + _at(u, k, -1)) - 20.0 * u
    return SIGMA / (64.0 * h) * r


def _lop(u, k, b, h):
    up = _at(u, k, 3) - 6.0 * _at(u, k, 2) + 18.0 * _at(u, k, 1) - 10.0 * u - 3.0 * _at(u, k, -1)
    dn = _at(u, k, -3) - 6.0 * _at(u, k, -2) + 18.0 * _at(u, k, -1) - 10.0 * u - 3.0 * _at(u, k, 1)
    return torch.where(b >= 0, up, -dn) / (12.0 * h)


def _wave_rhs(U, h):
    phi, pi = U[0], U[1]
    return torch.stack([-pi + _ko(phi, h), -sum(_d2(phi, k, k, h) for k in range(3)) + _ko(pi, h)])


SYM = [(0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2)]
R3 = range(3)


def _sym(T):
    """Six packed components as a 3 x 3 list."""
    q = {}
    for m, (i, j) in enumerate(SYM):
        q[i, j] = q[j, i] = T[m]
    return [[q[i, j] for j in R3] for i in R3]


def _geometry(U, h):
    """What the CCZ4 right-hand side and the monitors share."""
    chi, g, K, A, Gh, Th = U[0], _sym(U[1:7]), U[7], _sym(U[8:14]), U[14:17], U[17]
    det = (g[0][0] * (g[1][1] * g[2][2] - g[1][2] ** 2) - g[0][1] * (g[0][1] * g[2][2] - g[1][2] * g[0][2])
           + g[0][2] * (g[0][1] * g[1][2] - g[1][1] * g[0][2]))
    c = lambda i, j, k, l: g[i][j] * g[k][l] - g[i][l] * g[k][j]  # noqa: E731
    gu = _sym([c(1, 1, 2, 2) / det, -c(0, 1, 2, 2) / det, c(0, 1, 1, 2) / det, c(0, 0, 2, 2) / det,
               -c(0, 0, 1, 2) / det, c(0, 0, 1, 1) / det])
    dg = [_sym([_d1(U[1 + m], k, h) for m in range(6)]) for k in R3]
    Gl = [[[0.5 * (dg[j][i][k] + dg[k][i][j] - dg[i][j][k]) for k in R3] for j in R3] for i in R3]
    Gu = [[[sum(gu[i][l] * Gl[l][j][k] for l in R3) for k in R3] for j in R3] for i in R3]
    Z = [0.5 * chi * (Gh[i] - sum(gu[j][k] * Gu[i][j][k] for j in R3 for k in R3)) for i in R3]
    dchi = [_d1(chi, k, h) for k in R3]
    ddchi = _sym([_d2(chi, k, l, h) for k, l in SYM])
    dG = [[_d1(Gh[k], j, h) for k in R3] for j in R3]  # [j][k]
    H = [[[sum(gu[m][n] * Gu[k][m][i] for m in R3) for n in R3] for k in R3] for i in R3]
    tr = sum(gu[k][m] * (ddchi[k][m] - 1.5 * dchi[k] * dchi[m] / chi) for k in R3 for m in R3)
    tr = tr - sum(Gh[k] * dchi[k] for k in R3)
    R = []
    for i, j in SYM:
        r = 0.5 / chi * ddchi[i][j] - 0.25 / chi ** 2 * dchi[i] * dchi[j] + 0.5 / chi * g[i][j] * tr
        for m in R3:
            for n in R3:
                r = r - 0.5 * gu[m][n] * _d2(U[1 + SYM.index((min(i, j), max(i, j)))], m, n, h)
        for k in R3:
            r = r + 0.5 * (g[k][i] * dG[j][k] + g[k][j] * dG[i][k])
            r = r + 0.5 * Gh[k] * (Gl[i][j][k] + Gl[j][i][k]) - 0.5 / chi * Gu[k][i][j] * dchi[k]
            r = r + Z[k] * (g[k][i] * dchi[j] + g[k][j] * dchi[i]) / chi ** 2
            for n in R3:
                r = r + H[i][k][n] * (Gl[j][k][n] + Gl[k][n][j]) + H[j][k][n] * Gl[i][k][n]
        R.append(r)
    Am = [[sum(gu[i][k] * A[k][j] for k in R3) for j in R3] for i in R3]
    Au = [[sum(Am[i][k] * gu[k][j] for k in R3) for j in R3] for i in R3]
    AA = sum(A[i][j] * Au[i][j] for i in R3 for j in R3)
    trace = lambda T: sum(gu[i][j] * T[i][j] for i in R3 for j in R3)  # noqa: E731
    Ric = _sym(R)
    HZ = chi * trace(Ric) + 2.0 / 3.0 * K * K + 2.0 / 3.0 * Th * (K - 2.0 * Th) - AA
    return dict(chi=chi, g=g, gu=gu, K=K, A=A, Gh=Gh, Th=Th, lndet=torch.log(det), Gu=Gu, Z=Z, dchi=dchi, Ric=Ric,
                Am=Am, Au=Au, AA=AA, trA=sum(Am[i][i] for i in R3), HZ=HZ, trace=trace)


def _ccz4_rhs(U, h):
    q = _geometry(U, h)
    chi, g, gu, K, A, Gh, Th, Z, dchi = (q[k] for k in ("chi", "g", "gu", "K", "A", "Gh", "Th", "Z", "dchi"))
    a, be, Bv = U[18], U[19:22], U[22:25]
    da = [_d1(a, k, h) for k in R3]
    db = [[_d1(be[i], k, h) for i in R3] for k in R3]  # [k][i]
    div = db[0][0] + db[1][1] + db[2][2]
    cr = sum(gu[k][m] * da[k] * dchi[m] for k in R3 for m in R3)
    DDa = _sym([_d2(a, i, j, h) - sum(q["Gu"][k][i][j] * da[k] for k in R3)
                + 0.5 / chi * (da[i] * dchi[j] + da[j] * dchi[i] - g[i][j] * cr) for i, j in SYM])
    X = [[a * q["Ric"][i][j] - DDa[i][j] for j in R3] for i in R3]
    trX = q["trace"](X)
    Kt, Zda = K + 2.0 * Th, sum(Z[i] * da[i] for i in R3)
    r = [2.0 / 3.0 * chi * (a * Kt - div)]
    for i, j in SYM:
        r.append(sum(g[i][k] * db[j][k] + g[k][j] * db[i][k] for k in R3) - 2.0 / 3.0 * g[i][j] * div
                 - 2.0 * a * (A[i][j] - g[i][j] * q["trA"] / 3.0) - KC / 3.0 * a * g[i][j] * q["lndet"])
    r.append(-chi * q["trace"](DDa) + a * (Kt * Kt / 3.0 + q["AA"] + KZ * Th) + 2.0 * Zda)
    for i, j in SYM:
        r.append(sum(A[i][k] * db[j][k] + A[k][j] * db[i][k] for k in R3) - 2.0 / 3.0 * A[i][j] * div
                 - KC / 3.0 * a * g[i][j] * q["trA"] + chi * (X[i][j] - g[i][j] * trX / 3.0)
                 + a * (K * A[i][j] - 2.0 * sum(A[i][k] * q["Am"][k][j] for k in R3)))
    dK, dT = [_d1(K, k, h) for k in R3], [_d1(Th, k, h) for k in R3]
    gdiv = [sum(_d2(be[k], k, j, h) for k in R3) for j in R3]
    GG = []
    for i in R3:
        s = 2.0 / 3.0 * Gh[i] * div + sum(gu[k][l] * _d2(be[i], k, l, h) for k in R3 for l in R3)
        b = sum(q["Gu"][i][j][k] * q["Au"][j][k] for j in R3 for k in R3) - Z[i] / chi * (KZ + 2.0 / 3.0 * Kt)
        for j in R3:
            s = s - Gh[j] * db[j][i] + gu[i][j] * gdiv[j] / 3.0 - 2.0 * q["Au"][i][j] * da[j]
            b = b - 1.5 / chi * q["Au"][i][j] * dchi[j] - gu[i][j] * (
                2.0 / 3.0 * dK[j] + dT[j] / 3.0 + Th / a * da[j])
        GG.append(s + 2.0 * a * b)
    r += GG
    r.append(0.5 * a * q["HZ"] - Zda - 2.0 * KZ * a * Th)
    r.append(-2.0 * a * K)
    r += [GD_G * Bv[i] for i in R3]
    r += [GG[i] - GD_ETA * Bv[i] for i in R3]
    r = torch.stack(r)
    for k in R3:
        r = r + be[k] * _lop(U, k, be[k], h)
    return r + _ko(U, h)


def _monitors(U, h):
    q = _geometry(U, h)
    Z = torch.sqrt(sum(q["g"][i][j] * q["Z"][i] * q["Z"][j] for i in R3 for j in R3) / q["chi"])
    return [q["Th"], Z, q["HZ"], q["lndet"], q["trA"]]


def _mhd_flux(U, d):
    rho, S, E, B = U[0], U[1:4], U[4], U[5:8]
    v = [S[i] / rho for i in R3]
    B2 = sum(b * b for b in B)
    p = (GAMMA - 1.0) * (E - 0.5 * sum(S[i] * v[i] for i in R3) - 0.5 * B2)
    pt, vB = p + 0.5 * B2, sum(v[i] * B[i] for i in R3)
    F = [S[d]] + [S[i] * v[d] - B[d] * B[i] + (pt if i == d else 0.0) for i in R3]
    F += [(E + pt) * v[d] - vB * B[d]] + [v[d] * B[i] - v[i] * B[d] for i in R3]
    a2, b2, t2 = GAMMA * p / rho, B2 / rho, sum(B[i] * B[i] for i in R3 if i != d) / rho
    cf = torch.sqrt(0.5 * (a2 + b2 + torch.sqrt((a2 - b2) ** 2 + 4.0 * a2 * t2)))
    if U.shape[0] == 9:
        F[5 + d] = F[5 + d] + U[8]
        F.append(CH * CH * B[d])
    return torch.stack(F), v[d], cf


def _weno(c, recon, eps):
    """Value at the right interface of the middle of the five cells."""
    v0, v1, v2, v3, v4 = c
    if recon == "weno3":
        w0, w1 = 2.0 / 3.0 / (eps + (v3 - v2) ** 2) ** 2, 1.0 / 3.0 / (eps + (v2 - v1) ** 2) ** 2
        return (w0 * 0.5 * (v2 + v3) + w1 * (1.5 * v2 - 0.5 * v1)) / (w0 + w1)
    b0 = 13.0 / 12.0 * (v2 - 2 * v3 + v4) ** 2 + 0.25 * (3 * v2 - 4 * v3 + v4) ** 2
    b1 = 13.0 / 12.0 * (v1 - 2 * v2 + v3) ** 2 + 0.25 * (v1 - v3) ** 2
    b2 = 13.0 / 12.0 * (v0 - 2 * v1 + v2) ** 2 + 0.25 * (v0 - 4 * v1 + 3 * v2) ** 2
    f = (lambda b: 1.0 / (eps + b) ** 2) if recon == "weno5js" else (
        lambda b: 1.0 + ((b0 - b2).abs() / (eps + b)) ** 2)
    w0, w1, w2 = 0.3 * f(b0), 0.6 * f(b1), 0.1 * f(b2)
    return (w0 * (2 * v2 + 5 * v3 - v4) + w1 * (-v1 + 5 * v2 + 2 * v3) + w2 * (2 * v0 - 7 * v1 + 11 * v2)) / (
        6.0 * (w0 + w1 + w2))


def _mhd_rhs(U, h, case):
    glm, rec, eps = U.shape[0] == 9, case["recon"], h ** (2 if case["recon"] == "weno3" else 4)
    r = torch.zeros_like(U)
    for d in R3:
        if case["flux"] == "split":
            F, v, c = _mhd_flux(U, d)
            s = v.abs() + c
            if glm:
                s = torch.clamp(s, min=CH)
            al = torch.stack([_at(s, d, m) for m in range(-2, 4)]).amax(0)
            at = [(_at(F, d, m), al * _at(U, d, m)) for m in range(-2, 4)]
            P, Q = [0.5 * (f + u) for f, u in at], [0.5 * (f - u) for f, u in at]
            H = _weno(P[:5], rec, eps) + _weno(Q[:0:-1], rec, eps)
        else:
            cells = [_at(U, d, m) for m in range(-2, 4)]
            UL, UR = _weno(cells[:5], rec, eps), _weno(cells[:0:-1], rec, eps)
            (FL, vL, cL), (FR, vR, cR) = _mhd_flux(UL, d), _mhd_flux(UR, d)
            if case["flux"] == "hll":
                SL, SR = torch.minimum(vL - cL, vR - cR), torch.maximum(vL + cL, vR + cR)
                SL, SR = (torch.clamp(SL, max=-CH), torch.clamp(SR, min=CH)) if glm else (SL, SR)
                SL, SR = torch.clamp(SL, max=0.0), torch.clamp(SR, min=0.0)
                H = (SR * FL - SL * FR + SR * SL * (UR - UL)) / (SR - SL)
            else:
                S = torch.maximum(vL.abs() + cL, vR.abs() + cR)
                S = torch.clamp(S, min=CH) if glm else S
                H = 0.5 * (FL + FR - S * (UR - UL))
        r -= (H - _at(H, d, -1)) / h
    if glm:
        r[8] -= KPSI * U[8]
    return r


def _rhs(case):
    h = _dx(case)
    return {"wave": lambda U: _wave_rhs(U, h), "ccz4": lambda U: _ccz4_rhs(U, h)}.get(
        case["system"], lambda U: _mhd_rhs(U, h, case))


def _rk(f, U, dt, scheme):
    if scheme == "ssprk3":
        V = U + dt * f(U)
        V = 0.75 * U + 0.25 * (V + dt * f(V))
        return U / 3.0 + 2.0 / 3.0 * (V + dt * f(V))
    k1 = dt * f(U)
    k2 = dt * f(U + 0.5 * k1)
    k3 = dt * f(U + 0.5 * k2)
    return U + (k1 + 2.0 * k2 + 2.0 * k3 + dt * f(U + k3)) / 6.0


def _parts(case, U):
    return [U[:, lo[2]:hi[2] + 1, lo[1]:hi[1] + 1, lo[0]:hi[0] + 1] for lo, hi in _boxes(case)]


def exact(case, seed):
    # whole hierarchies and objectives are chains of the same steps with the data movement
    # between levels: too long to restate here
    if case["kind"] not in ("step", "reverse", "monitor"):
        return None
    U, f = _initial(case, seed), _rhs(case)
    if case["kind"] == "step":
        return _parts(case, _rk(f, U, _dt(case), case["scheme"]))
    if case["kind"] == "monitor":
        h = _dx(case)
        mon = (_monitors(U, h) if case["system"] == "ccz4" else []) + [torch.sqrt((_ko(U, h) ** 2).sum(0))]
        out = torch.zeros(M.MOL_MON_OUT, dtype=torch.float64, device="cuda")
        for q, v in enumerate(mon):
            at = 3 * (q if case["system"] == "ccz4" else 5)
            out[at], out[at + 1], out[at + 2] = v.abs().sum() * h ** 3, (v * v).sum() * h ** 3, v.abs().max()
        return out, _parts(case, torch.stack(mon))
    # reverse: the vector-Jacobian product of one step; each stage is differentiated by itself
    x, y, z = _grid(case)
    lam = torch.zeros_like(U)
    lam[18 if case["system"] == "ccz4" else 0] = (x * x + y * y + z * z < _radius(seed) ** 2).double() * _dx(case) ** 3
    dt, stages = _dt(case), [U]
    for b in (0.5, 0.5, 1.0):
        stages.append(U + b * dt * f(stages[-1]))
    total, m = lam.clone(), torch.zeros_like(lam)
    for c, b, V in ((1 / 6, 0.0, stages[3]), (2 / 6, 1.0, stages[2]), (2 / 6, 0.5, stages[1]), (1 / 6, 0.5, stages[0])):
        V = V.detach().requires_grad_(True)
        m, = torch.autograd.grad(f(V), V, dt * (c * lam + b * m))
        total += m
    return _parts(case, total)
