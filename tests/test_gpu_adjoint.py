"""GPU parity of the wave adjoint (right-hand-side transpose, ghost-fill
transpose, reverse RK4 sweep) against the oracle, and of the autograd
gradient against central differences of the GPU forward."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1806_04182_amd import molamr as M
from paper_1806_04182_amd import synth
from tests.util import parity_err

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    return torch


def test_rhs_and_fill_adjoint_match_oracle():
    torch = _torch()
    rng = np.random.default_rng(3)
    n = (19, 11, 8)
    h = 0.1
    lam = synth.embed(rng.standard_normal((2, n[2], n[1], n[0])))
    ps = M.Patchset(M.single_patch(n, (0, 0, 0), h), M.System(M.MOL_WAVE, sigma=0.1))
    # garbage in lam's ghosts must be ignored
    lam_dev_h = lam.copy()
    lam_dev_h[:, :3] = 1e30
    L = torch.from_numpy(ps.pack(0, [lam_dev_h])).cuda()
    out = ps.alloc(0)
    ps.rhs_adjoint(0, None, L, out)
    torch.cuda.synchronize()
    raw = ps.unpack(0, out)[0]
    ref = O.wave_rhs_adjoint(lam, h, O.params(sigma=0.1))
    sc = max(1.0, np.max(np.abs(ref)))
    assert np.max(np.abs(raw - ref)) < 1e-12 * sc
    ps.fill_ghosts_adjoint(0, out)
    torch.cuda.synchronize()
    got = ps.unpack(0, out)[0]
    O.fill_periodic_adjoint(ref)
    assert np.max(np.abs(got - ref)) < 1e-12 * sc


def test_rk4_adjoint_sweep_matches_oracle():
    torch = _torch()
    n = (20, 16, 12)
    dx = 2.0 / 20
    xlo = (-1.0, -1.0, -1.0)
    ps = M.Patchset(M.single_patch(n, xlo, dx), M.System(M.MOL_WAVE, sigma=0.1))
    lam = ps.alloc(0)
    w = [ps.alloc(0) for _ in range(3)]
    ps.sphere_adjoint(0, 0, 0.6, 1.0, lam)
    nsteps, dt = 9, 0.25 * dx
    for _ in range(nsteps):
        ps.rk4_adjoint_step(0, dt, lam, w)
    torch.cuda.synchronize()
    got = ps.unpack(0, lam)[0]
    ref = O.wave_adjoint_run(n, (dx, dx, dx), xlo, dt, nsteps, 0.6, O.params(sigma=0.1))
    e = parity_err(synth.interior(got), synth.interior(ref))
    assert np.all(e < 1e-12), e


def test_autograd_gradient_matches_central_differences():
    torch = _torch()
    from paper_1806_04182_amd.adjoint import sphere_objective
    n = (32, 32, 32)
    dx = 2.0 / 32
    ps = M.Patchset(M.single_patch(n, (-1, -1, -1), dx), M.System(M.MOL_WAVE, sigma=0.1))
    nsteps, dt, rad = 40, 0.25 * dx, 0.6
    p0 = torch.tensor([1.0, 0.2, 0.03, -0.05, 0.02], dtype=torch.float64, requires_grad=True)
    J = sphere_objective(p0, ps, nsteps, dt, rad, every=10)
    J.backward()
    g = p0.grad.numpy()
    Jv = float(J.detach())
    assert abs(g[0] - Jv) < 1e-12 * abs(Jv)  # dJ/dA = J/A with A = 1
    base = p0.detach().numpy()
    for i in range(5):
        e = np.zeros(5)
        e[i] = 1e-6
        Jp = float(sphere_objective(torch.tensor(base + e), ps, nsteps, dt, rad))
        Jm = float(sphere_objective(torch.tensor(base - e), ps, nsteps, dt, rad))
        fd = (Jp - Jm) / 2e-6
        assert abs(fd - g[i]) <= 1e-6 * max(abs(g[i]), 1e-3 * abs(Jv)), (i, fd, g[i])


def test_gaussian_initial_data_matches_synth():
    torch = _torch()
    n = (14, 10, 9)
    dx = 2.0 / 14
    xlo = (-1.0, -1.0, -1.0)
    ps = M.Patchset(M.single_patch(n, xlo, dx), M.System(M.MOL_WAVE))
    U = ps.alloc(0)
    prm = [0.7, 0.3, 0.9, -0.1, 0.2]
    ps.wave_gaussian(0, prm, U)
    torch.cuda.synchronize()
    got = synth.interior(ps.unpack(0, U)[0])
    ref = synth.wave_gaussian(n, xlo, dx, amp=prm[0], width=prm[1], centre=prm[2:],
                              period=(n[0] * dx, n[1] * dx, n[2] * dx))
    assert np.max(np.abs(got - ref)) < 1e-14


@pytest.mark.parametrize("n,boxes", [((64, 64, 64), None),   # marching stage kernel by default
                                     ((70, 64, 61), None),   # ragged columns, marching set below
                                     ((20, 12, 9), None), ((12, 9, 1), None), ((3, 5, 4), None),
                                     ((24, 13, 10), [((0, 0, 0), (10, 12, 9)), ((11, 0, 0), (23, 5, 9)),
                                                     ((11, 6, 0), (23, 12, 9))])])
def test_wave_reverse_step_is_the_transposed_step(n, boxes):
    """The reverse RK4 step of the wave (run as forward stages of the system
    with its fields exchanged) equals sum_s m_s + lam with m_s from the
    right-hand side's and the ghost fill's transposes, on one periodic patch
    (with and without the marching kernel), thin patches and several patches;
    the ghost entries of lam keep their values.  Tolerance: the two evaluate
    the same polynomial of degree 4 in other orders, a few dozen roundings of
    values of the size of lam: 1e-13 of its maximum."""
    torch = _torch()
    print("wave reverse", n, boxes, flush=True)
    dx = 2.0 / max(n)
    dt = 0.25 * dx
    levels = [(1, boxes or [((0, 0, 0), tuple(v - 1 for v in n))])]
    ps = M.Patchset(M.Hierarchy(n, (-1, -1, -1), dx, levels), M.System(M.MOL_WAVE, sigma=0.1))
    g = torch.Generator(device="cuda").manual_seed(3)
    lam0 = torch.rand(ps.layouts[0]["nelems"], dtype=torch.float64, device="cuda", generator=g) - 0.5
    inner = torch.zeros(ps.layouts[0]["nelems"], dtype=torch.bool)
    for p, (nx, ny, nz) in enumerate(ps.layouts[0]["dims"]):
        ps._view(0, inner, p, 2)[:, 3:-3, 3:-3, 3:-3] = True
    inner = inner.cuda()
    total, m = torch.where(inner, lam0, 0.0), torch.zeros_like(lam0)
    start = total.clone()
    for c, b in ((1 / 6, 0.0), (1 / 3, 1.0), (1 / 3, 0.5), (1 / 6, 0.5)):
        k = dt * (c * start + b * m)
        m = ps.alloc(0)
        ps.rhs_adjoint(0, None, k, m)
        ps.fill_ghosts_adjoint(0, m)
        m = torch.where(inner, m, 0.0)
        total = total + m
    for tiling in (None, (64, 8, 3), (32, 4, 2)):
        if tiling is not None:
            ps.set_tiling(0, tiling)
        lam = lam0.clone()
        ps.rk4_adjoint_step_stages(0, dt, lam, [ps.alloc(0) for _ in range(3)])
        torch.cuda.synchronize()
        assert torch.equal(lam[~inner], lam0[~inner])
        assert float((lam - total)[inner].abs().max()) < 1e-13

