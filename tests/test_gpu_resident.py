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


def test_resident_batch_keeps_the_iterates_of_the_persistent_kernel():
    """A batch that fits on the chip is solved resident; with one problem too
    large for it (more tiles than compute units) the persistent kernel runs.
    Both take the same steps for the problems they share: equal iteration
    counts, equal solutions."""
    from paper_1010_2832_amd import vfstokes as V
    sizes = [24, 61, 62, 63, 130, 257, 33]
    probs = [cases.drop2d(n, 300 + q) for q, n in enumerate(sizes)]
    big = cases.drop2d(1700, 5)
    out = []
    for extra in ([], [big]):
        b = V.batch_from_cases(probs + extra, tol=1e-9)
        b.vfs_batch_step(probs[0]["dt"])
        out.append([(b.vfs_batch_get_problem(i)["iterations"], b.vfs_batch_get_solution(i))
                    for i in range(len(sizes))])
        b.close()
    for n, (i0, x0), (i1, x1) in zip(sizes, *out):
        print(f"n={n}: {i0} and {i1} iterations", flush=True)
        assert i0 == i1
        # the sums differ in order only; their rounding to FP32 may flip once in
        # millions of iterations, so equality is asked for, not a tolerance
        assert np.array_equal(x0, x1)


# one brick is 8 x 8 x 8 anchors (cells + 1), 16 x 8 x 8 in FP32 when those are
# more than the compute units: one brick, a full one, one anchor more, several,
# the folded column of the launched iteration (64), the wide bricks (48 cells a
# side), FP64 two to a unit (56 and 60) and more bricks than fit
@pytest.mark.parametrize("n", [(6, 5, 6), (7, 7, 7), (8, 8, 8), (15, 16, 17), (64, 9, 12), (9, 40, 11)])
@pytest.mark.parametrize("precision,tol,bar", [(0, 1e-11, 1e-6), (1, 1e-9, 1e-4)])
def test_resident3d_brick_edges(n, precision, tol, bar):
    case = cases.crop(cases.pool3d(max(n), 7), (0, 0, 0), n)
    print(f"resident 3D {n} precision {precision}", flush=True)
    asm, x, u = oracle(case)
    ctx = gpu_run(case, precision=precision, tol=tol)
    assert ctx.vfs_get_stats()["rel_residual"] <= tol
    assert velocity_rel_linf(asm, flat_faces(asm.grid, ctx.vfs_get_velocity()), u) <= bar


@pytest.mark.parametrize("n,precision", [((30, 33, 31), 0), ((48, 48, 48), 0), ((48, 48, 48), 1),
                                         ((65, 47, 63), 1), ((56, 56, 56), 0), ((60, 71, 63), 0), ((96, 80, 72), 0), ((96, 80, 72), 1)])
def test_resident3d_shapes(n, precision):
    tol = 1e-8
    print(f"resident 3D pool {n} precision {precision}", flush=True)
    case = cases.crop(cases.pool3d(max(n), 7), (0, 0, 0), n)
    ctx = gpu_run(case, precision=precision, tol=tol)
    assert _residual(ctx) <= 1.01 * tol


def test_resident3d_repeats_and_cap():
    case = cases.crop(cases.pool3d(40, 7), (0, 0, 0), (40, 33, 37))
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
