"""GPU parity of the brick-local preconditioners (VFS_PRECOND_IC: block
symmetric Gauss-Seidel; VFS_PRECOND_SCHWARZ: overlapping additive Schwarz)
against the oracle (oracle/schwarz.py, the same bricks of 16^2 / 4^3 anchors):
one application to 1e-12, and FP64 PCG steps to the FP64 velocity bar with
the oracle's PCG iteration counts."""
import numpy as np
import pytest

import cases
from gpu_util import flat_faces, gpu_run, velocity_rel_linf
from oracle import schwarz, system

pytestmark = pytest.mark.gpu

BRICK = {2: 16, 3: 4}


def _banner(msg):
    print(f"[schwarz] {msg}", flush=True)


CASES = {
    "drop2d_45": lambda: cases.drop2d(45, 3),
    "pool2d_70": lambda: cases.pool2d(70, 5),
    "pool3d_14": lambda: cases.pool3d(14, seed=6),
    "column3d_19": lambda: cases.column3d(19, seed=2),
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("overlap", [0, 1])
def test_preconditioner_application_matches_oracle(name, overlap):
    from paper_1010_2832_amd import vfstokes as V
    case = CASES[name]()
    asm = system.assemble(case)
    ctx = gpu_run(case, step=False)
    pc = V.VFS_PRECOND_SCHWARZ if overlap else V.VFS_PRECOND_IC
    ctx.vfs_set_solver(pc, V.VFS_FP64, 1e-10, 100000)
    rng = np.random.default_rng(3)
    r = np.where(asm.active, rng.normal(size=asm.grid.n_samples()), 0.0)
    z = ctx.vfs_precond_apply(r)
    z_o = schwarz.preconditioner(asm, BRICK[case["dim"]], overlap)(r)
    err = np.abs(z - z_o).max() / np.abs(z_o).max()
    _banner(f"{name} overlap {overlap}: application rel err {err:.2e}")
    assert err <= 1e-12
    assert not z[~asm.active].any()
    ctx.close()


@pytest.mark.parametrize("name", list(CASES))
def test_pcg_steps_match_oracle(name):
    from paper_1010_2832_amd import vfstokes as V
    case = CASES[name]()
    asm, x, u = system.step(case)
    its_j = None
    for pc, overlap in ((V.VFS_PRECOND_JACOBI, None), (V.VFS_PRECOND_IC, 0), (V.VFS_PRECOND_SCHWARZ, 1)):
        ctx = gpu_run(case, step=False)
        ctx.vfs_set_solver(pc, V.VFS_FP64, 1e-10, 100000)
        ctx.vfs_step(case["dt"])
        st = ctx.vfs_get_stats()
        err = velocity_rel_linf(asm, flat_faces(asm.grid, ctx.vfs_get_velocity()), u)
        msg = f"{name} precond {pc}: {st['iterations']} iterations, rel {st['rel_residual']:.1e}, velocity {err:.2e}"
        if overlap is not None:
            _, its_o = schwarz.pcg(asm, schwarz.preconditioner(asm, BRICK[case["dim"]], overlap), tol=1e-10)
            msg += f" (oracle PCG {its_o} iterations)"
            assert abs(st["iterations"] - its_o) <= 2 + 0.02 * its_o
            assert st["iterations"] < its_j
        else:
            its_j = st["iterations"]
        _banner(msg)
        assert st["rel_residual"] <= 1e-10
        assert err <= 1e-6
        ctx.close()


def test_brick_preconditioners_need_fp64():
    from paper_1010_2832_amd import vfstokes as V
    ctx = gpu_run(cases.drop32(), step=False)
    for pc in (V.VFS_PRECOND_IC, V.VFS_PRECOND_SCHWARZ):
        with pytest.raises(V.VfsError) as ei:
            ctx.vfs_set_solver(pc, V.VFS_MIXED, 1e-6, 1000)
        assert ei.value.code == V.VFS_EINVAL
    ctx.close()


# bricks of 16^2 or 4^3 anchors (cells + 1), taken in rows of four: one brick, a
# full one, one anchor more, and rows that do not fill a group
@pytest.mark.parametrize("n", [(9, 14), (15, 15), (16, 31), (40, 17), (3, 3, 3), (4, 3, 7), (7, 8, 4), (9, 19, 5)])
def test_overlapping_bricks_at_grid_edges(n):
    from paper_1010_2832_amd import vfstokes as V
    pool = cases.pool2d(max(n), 5) if len(n) == 2 else cases.pool3d(max(n), seed=6)
    case = cases.crop(pool, (0,) * len(n), n)
    asm = system.assemble(case)
    ctx = gpu_run(case, step=False)
    ctx.vfs_set_solver(V.VFS_PRECOND_SCHWARZ, V.VFS_FP64, 1e-10, 100000)
    rng = np.random.default_rng(3)
    z_of = schwarz.preconditioner(asm, BRICK[len(n)], 1)
    for _ in range(2):   # the second application meets the first one's buffer
        r = np.where(asm.active, rng.normal(size=asm.grid.n_samples()), 0.0)
        z, z_o = ctx.vfs_precond_apply(r), z_of(r)
        err = np.abs(z - z_o).max() / np.abs(z_o).max()
        _banner(f"{n}: application rel err {err:.2e}")
        assert err <= 1e-12
        assert not z[~asm.active].any()
    ctx.close()
