"""GPU parity of the fractional step of Section 10 (vfs_advect + vfs_step)
against the oracle (oracle/advect.py): one advection of a given velocity
and level set to 1e-12, several full steps (advection, body force, Stokes
solve) to the FP64 bar, and warm-started mixed solves across steps."""
import numpy as np
import pytest

import cases
from gpu_util import flat_faces, gpu_run, velocity_rel_linf
from oracle import advect, system
from oracle.grid import Grid

pytestmark = pytest.mark.gpu


def _banner(msg):
    print(f"[advect] {msg}", flush=True)


def _swirl(case, amp=0.8):
    """A smooth rotating velocity (so departure points are off the grid)."""
    out = dict(case)
    n, h, d = case["n"], case["h"], case["dim"]
    u = []
    for a in range(d):
        F = cases.face_coords(n, h, (0.0,) * d, a)
        r = [F[q] - 0.5 for q in range(d)]
        rot = [-r[1], r[0], 0.3 * r[0]][a] if d == 3 else [-r[1], r[0]][a]
        u.append(amp * rot + 0.1 * np.sin(3 * F[0] + 2 * F[1]))
    out["u"] = u
    return out


CASES = {
    "drop2d_33": lambda: _swirl(cases.drop2d(33, 3, dt=0.01)),
    "pool3d_12": lambda: _swirl(cases.pool3d(12, seed=9, dt=0.01)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_one_advection_matches_oracle(name):
    case = CASES[name]()
    grid = Grid(case["n"], case["h"])
    dt = 0.02
    ctx = gpu_run(case, step=False)
    ctx.vfs_advect(dt)
    u_g = flat_faces(grid, ctx.vfs_get_velocity())
    phi_g = ctx.vfs_get_level_set()
    u = [np.asarray(q, np.float64) for q in case["u"]]
    u_o = advect.advect_velocity(grid, u, dt)
    phi_o = advect.advect_level_set(grid, case["phi_l"], u, dt)
    du = np.abs(u_g - flat_faces(grid, u_o)).max() / np.abs(flat_faces(grid, u_o)).max()
    dp = np.abs(phi_g - phi_o).max() / np.abs(phi_o).max()
    _banner(f"{name}: velocity {du:.2e}, level set {dp:.2e}")
    assert du <= 1e-12 and dp <= 1e-12
    ctx.close()


@pytest.mark.parametrize("name", list(CASES))
def test_fractional_steps_match_oracle(name):
    """Three steps: the second and third extend the previous Stokes step's
    velocity into the air before advecting (the faces it defined), so the
    GPU's bookkeeping of known faces is checked too."""
    from paper_1010_2832_amd import vfstokes as V
    case = CASES[name]()
    dt = 0.01
    ctx = gpu_run(case, precision=V.VFS_FP64, tol=1e-12, step=False)
    c = case
    prev = None
    for step in range(3):
        c, (asm, x, u_o) = advect.ns_step(c, dt, prev)
        prev = asm
        ctx.vfs_advect(dt)
        phi_g = ctx.vfs_get_level_set()
        ctx.vfs_step(dt)
        u_g = flat_faces(asm.grid, ctx.vfs_get_velocity())
        err = velocity_rel_linf(asm, u_g, u_o)
        dphi = np.abs(phi_g - c["phi_l"]).max() / np.abs(c["phi_l"]).max()
        _banner(f"{name} step {step}: velocity rel Linf {err:.2e}, level set {dphi:.2e}, "
                f"iterations {ctx.vfs_get_stats()['iterations']}")
        assert np.array_equal(ctx.vfs_get_active(), asm.active)
        assert err <= 1e-6 and dphi <= 1e-9
    ctx.close()


def test_warm_start_across_steps():
    """Mixed solves started from the previous step's solution (masked to the
    new active set) start from the residual b - A x_prev that the oracle
    predicts from its own steps, and converge to the oracle's velocities;
    cold starts start from |b|.  The iteration counts are reported: on this
    problem the previous solution is no closer than 0 (its residual is 15-30
    times |b|, the stresses change a lot from step to step), so warm starts
    gain nothing here."""
    from paper_1010_2832_amd import vfstokes as V
    case = cases.pool2d(96, 7)
    dt = case["dt"]
    steps = 4
    want_start, want_u, asms = [1.0], [], []
    c, prev, xprev = case, None, None
    for k in range(steps):
        c, (asm, x, u) = advect.ns_step(c, dt, prev)
        if xprev is not None:
            r = asm.b_full - system.apply(asm, xprev * asm.active)
            want_start.append(np.linalg.norm(r[asm.active]) / np.linalg.norm(asm.b_full))
        want_u.append(u)
        asms.append(asm)
        prev, xprev = asm, x
    res = {}
    for warm in (False, True):
        ctx = gpu_run(case, precision=V.VFS_MIXED, tol=1e-8, step=False)
        ctx.vfs_set_warm_start(warm)
        its, start = [], []
        for k in range(steps):
            ctx.vfs_advect(dt)
            ctx.vfs_step(dt)
            st = ctx.vfs_get_stats()
            assert st["rel_residual"] <= 1e-8
            its.append(st["iterations"])
            start.append(st["rel_residual_start"])
            err = velocity_rel_linf(asms[k], flat_faces(asms[k].grid, ctx.vfs_get_velocity()),
                                    want_u[k])
            assert err <= 1e-4, (warm, k, err)
        res[warm] = (its, start)
        ctx.close()
    _banner(f"iterations cold {res[False][0]}, warm {res[True][0]}; starting residual warm "
            f"{np.round(res[True][1], 5)}, oracle {np.round(want_start, 5)}")
    assert res[False][1] == [1.0] * steps
    for got, want in zip(res[True][1], want_start):
        assert abs(got - want) <= 1e-4 * want, (got, want)


# grids of one cell (no second sample along an axis), thin ones, and the edges of
# the 64 x 4 and 64 x 2 x 2 blocks
@pytest.mark.parametrize("n", [(1, 1), (1, 6), (63, 4), (64, 5), (1, 1, 1), (5, 1, 3), (63, 2, 3), (64, 3, 2)])
def test_one_advection_at_small_extents(n):
    from paper_1010_2832_amd import vfstokes as V
    rng = np.random.default_rng(5)
    d, h, dt = len(n), 1.0 / max(n), 0.3 / max(n)
    grid = Grid(n, h)
    phi = rng.standard_normal([q + 1 for q in n])
    u = [rng.standard_normal([n[b] + (1 if b == a else 0) for b in range(d)]) for a in range(d)]
    ctx = V.Context(d, n, h)
    ctx.vfs_set_level_sets(phi)
    ctx.vfs_set_density(np.ones(n))
    ctx.vfs_set_viscosity(np.ones(n))
    ctx.vfs_set_velocity(u)
    ctx.vfs_advect(dt)
    du = np.abs(flat_faces(grid, ctx.vfs_get_velocity()) - flat_faces(grid, advect.advect_velocity(grid, u, dt))).max()
    dp = np.abs(ctx.vfs_get_level_set() - advect.advect_level_set(grid, phi, u, dt)).max()
    _banner(f"{n}: velocity {du:.2e}, level set {dp:.2e}")
    # values of size 1, weights off by the rounding of positions up to 64
    assert du <= 1e-12 and dp <= 1e-12
