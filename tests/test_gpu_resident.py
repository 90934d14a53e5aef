"""The resident CG solves (a whole solve in one launch): tile edges, every
tile shape, and the largest of them, checked on the FP64 residual of the
solution under the library's own operator and, where the oracle can solve the
case, on the velocity."""
import numpy as np
import pytest

import cases
from tests.gpu_util import flat_faces, gpu_run, oracle, velocity_rel_linf

pytestmark = pytest.mark.gpu


def _pool2d(nx, ny, seed=7):
    """A pool case cut to nx x ny cells."""
    return cases.crop(cases.pool2d(max(nx, ny), seed), (0, 0), (nx, ny))


def _residual(ctx):
    x, b = ctx.vfs_get_solution(), ctx.vfs_get_rhs()
    return np.linalg.norm(b - ctx.vfs_apply(x)) / np.linalg.norm(b)


# one tile is 62 x 8 anchors (cells + 1): one tile, a full one, one anchor more
# in x and y, several tiles
@pytest.mark.parametrize("nx,ny", [(20, 6), (61, 7), (62, 8), (63, 17), (124, 40), (125, 33), (9, 130)])
@pytest.mark.parametrize("precision,tol,bar", [(0, 1e-11, 1e-6), (1, 1e-9, 1e-4)])
def test_resident2d_tile_edges(nx, ny, precision, tol, bar):
    case = _pool2d(nx, ny)
    print(f"resident 2D {nx}x{ny} precision {precision}", flush=True)
    asm, x, u = oracle(case)
    ctx = gpu_run(case, precision=precision, tol=tol)
    assert ctx.vfs_get_stats()["rel_residual"] <= tol
    assert velocity_rel_linf(asm, flat_faces(asm.grid, ctx.vfs_get_velocity()), u) <= bar


# 62 x 8 anchors for up to 256 tiles, then 62 x 16, 62 x 32, 62 x 64 (FP32), and
# a grid whose active tiles are too many (the launched iteration)
@pytest.mark.parametrize("n,precision", [(300, 0), (300, 1), (640, 0), (640, 1), (1000, 0), (1000, 1),
                                         (1300, 1), (1400, 0)])
def test_resident2d_shapes(n, precision):
    tol = 1e-8
    print(f"resident 2D drop {n} precision {precision}", flush=True)
    ctx = gpu_run(cases.drop2d(n, 11), precision=precision, tol=tol)
    # the same operator in another order of additions: a few roundings of the
    # terms, far below the tolerance
    assert _residual(ctx) <= 1.01 * tol


def test_resident2d_repeats_and_cap():
    """The same solve twice gives the same bits (the stamps move on), a capped
    solve reports its cap, and the next solve is not disturbed by it."""
    case = _pool2d(130, 97)
    ctx = gpu_run(case, tol=1e-10, step=False)
    b = ctx.vfs_get_rhs()
    x0 = ctx.vfs_solve(b)
    its = ctx.vfs_get_stats()["iterations"]
    ctx.vfs_set_solver(1, 0, 1e-10, 37, 1e-3)
    ctx.vfs_solve(b, allow_unconverged=True)
    st = ctx.vfs_get_stats()
    assert st["iterations"] == 37 and st["status"] == -4
    ctx.vfs_set_solver(1, 0, 1e-10, 200000, 1e-3)
    x1 = ctx.vfs_solve(b)
    assert ctx.vfs_get_stats()["iterations"] == its
    assert np.array_equal(x0, x1)
