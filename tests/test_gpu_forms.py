"""The forms a solve can take (vfs_set_forms): which one ran, the launched and
the persistent form on problems that would run resident, and the ways back when
a resident run is given up or finds no memory."""
import numpy as np
import pytest

import cases
from tests.gpu_util import flat_faces, gpu_run, oracle, velocity_rel_linf
from oracle import system

pytestmark = pytest.mark.gpu

RESIDENT, GIVE_UP, NO_MEMORY = 1, 2, 4
MOST = 256      # compute units


def _banner(msg):
    print(f"[forms] {msg}", flush=True)


def _run(case, precision, tol, forms=None, max_iter=200000):
    """A stepped context, and what the step left."""
    ctx = gpu_run(case, precision=precision, tol=tol, step=False, max_iter=max_iter)
    if forms is not None:
        ctx.vfs_set_forms(forms)
    ctx.vfs_step(case["dt"])
    st = ctx.vfs_get_stats()
    _banner(f"{case['n']} precision {precision} forms {forms}: {ctx.vfs_get_forms()} {st['iterations']} iterations")
    return ctx, st["iterations"], ctx.vfs_get_solution(), flat_faces_of(ctx)


def flat_faces_of(ctx):
    return np.concatenate([q.ravel(order="F") for q in ctx.vfs_get_velocity()])


def _tiles(ctx, tile):
    """Tiles of this many anchors that hold an active sample."""
    found = set()
    for s in range(len(ctx.sample_shapes())):
        for ix in np.argwhere(ctx.vfs_get_active_mask(s)):
            found.add(tuple(int(i) // t for i, t in zip(ix, tile)))
    return len(found)


def _expected(ctx, precision):
    """Shape of the resident solve: the smallest tiles that fit the chip."""
    if ctx.dim == 2:
        for q in range(4 if precision else 3):
            if _tiles(ctx, (62, 8 << q)) <= MOST:
                return q
        return -1
    small = _tiles(ctx, (8, 8, 8))
    if small <= MOST:
        return 0
    if precision:
        return 1 if _tiles(ctx, (16, 8, 8)) <= MOST else -1
    return 2 if small <= 2 * MOST else -1


def _pool3d(n):
    return cases.crop(cases.pool3d(max(n), 7), (0, 0, 0), n)


# every tile and brick shape, both arithmetics, and sizes past the largest
CASES = {
    "2d_62x8": (lambda: cases.drop2d(300, 11), 0, 1), "2d_62x16": (lambda: cases.drop2d(640, 11), 1, 1),
    "2d_62x32": (lambda: cases.drop2d(1000, 11), 2, 1), "2d_62x64": (lambda: cases.drop2d(1300, 11), 3, 1),
    "2d_large": (lambda: cases.drop2d(1700, 11), -1, 1), "2d_fp64": (lambda: cases.drop2d(150, 11), 0, 0),
    "2d_fp64_62x32": (lambda: cases.drop2d(800, 11), 2, 0), "2d_fp64_large": (lambda: cases.drop2d(1400, 11), -1, 0),
    "3d_8": (lambda: _pool3d((24, 23, 25)), 0, 1), "3d_16x8": (lambda: _pool3d((60, 64, 52)), 1, 1),
    "3d_fold": (lambda: _pool3d((64, 9, 12)), 0, 1), "3d_large": (lambda: _pool3d((96, 80, 72)), -1, 1),
    "3d_fp64": (lambda: _pool3d((30, 33, 31)), 0, 0), "3d_fp64_two": (lambda: _pool3d((56, 56, 56)), 2, 0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_the_form_that_fits_runs(name):
    make, shape, precision = CASES[name]
    case = make()
    ctx = gpu_run(case, precision=precision, tol=1e-4)
    want = _expected(ctx, precision)
    _banner(f"{name}: {ctx.vfs_get_forms()}, expected {want}")
    assert want == shape                    # the case is what its name says
    assert ctx.vfs_get_forms() == dict(forms=RESIDENT, resident=want, give_ups=0)


@pytest.mark.parametrize("name", ["2d_62x8", "2d_62x16", "2d_62x32", "2d_62x64", "3d_8", "3d_16x8", "3d_fold"])
def test_mixed_solves_take_the_same_steps_in_both_forms(name):
    make, shape, _ = CASES[name]
    case = make()
    a, ia, xa, ua = _run(case, 1, 1e-6)
    b, ib, xb, ub = _run(case, 1, 1e-6, forms=0)
    assert a.vfs_get_forms()["resident"] == shape and b.vfs_get_forms()["resident"] == -1
    # the FP64 sums differ in order only, which the rounding of alpha and beta to
    # FP32 hides: equality is asked for, not a tolerance
    assert ia == ib and np.array_equal(xa, xb) and np.array_equal(ua, ub)


@pytest.mark.parametrize("precision,tol,bar", [(0, 1e-11, 1e-6), (1, 1e-9, 1e-4)])
@pytest.mark.parametrize("make", [lambda: cases.drop2d(33, 3), lambda: cases.drop2d(130, 3),
                                  lambda: _pool3d((9, 12, 17))])
def test_launched_solves_match_the_oracle(make, precision, tol, bar):
    case = make()
    asm, x, u = oracle(case)
    ctx, _, _, ug = _run(case, precision, tol, forms=0)
    assert ctx.vfs_get_forms()["resident"] == -1
    assert ctx.vfs_get_stats()["rel_residual"] <= tol
    assert velocity_rel_linf(asm, flat_faces(asm.grid, ctx.vfs_get_velocity()), u) <= bar


@pytest.mark.parametrize("name", ["2d_fp64", "2d_62x8", "3d_fp64", "3d_fp64_two", "3d_8", "3d_16x8"])
def test_a_run_that_is_given_up_is_launched(name):
    make, shape, precision = CASES[name]
    case = make()
    want = _run(case, precision, 1e-6, forms=0)
    got = _run(case, precision, 1e-6, forms=RESIDENT | GIVE_UP)
    assert got[0].vfs_get_forms() == dict(forms=RESIDENT | GIVE_UP, resident=-1, give_ups=1)
    assert got[1] == want[1] and np.array_equal(got[2], want[2]) and np.array_equal(got[3], want[3])


@pytest.mark.parametrize("name", ["2d_fp64", "3d_8"])
def test_memory_given_back_and_taken_again(name):
    make, shape, precision = CASES[name]
    case = make()
    ctx = gpu_run(case, precision=precision, tol=1e-8, step=False)
    b = ctx.vfs_get_rhs()
    x = ctx.vfs_solve(b)
    assert ctx.vfs_get_forms()["resident"] == shape
    ctx.vfs_set_forms(0)
    ctx.vfs_solve(b)
    assert ctx.vfs_get_forms()["resident"] == -1
    ctx.vfs_set_forms(RESIDENT)
    ctx.vfs_assemble(case["dt"])
    assert np.array_equal(ctx.vfs_solve(b), x)
    assert ctx.vfs_get_forms()["resident"] == shape
    from paper_1010_2832_amd import vfstokes as V
    with pytest.raises(V.VfsError):
        ctx.vfs_set_forms(8)


def test_without_memory_for_the_two_brick_shape():
    case = CASES["3d_fp64_two"][0]()
    want = _run(case, 0, 1e-6, forms=0)
    got = _run(case, 0, 1e-6, forms=RESIDENT | NO_MEMORY)
    assert got[0].vfs_get_forms()["resident"] == -1
    assert got[1] == want[1] and np.array_equal(got[2], want[2])


@pytest.mark.parametrize("make", [lambda: cases.drop2d(60, 3), lambda: _pool3d((18, 13, 15))])
def test_schwarz_without_memory_for_its_bricks(make):
    from paper_1010_2832_amd import vfstokes as V
    case = make()
    z = []
    for forms in (RESIDENT, RESIDENT | NO_MEMORY):
        ctx = gpu_run(case, step=False)
        ctx.vfs_set_forms(forms)
        ctx.vfs_set_solver(V.VFS_PRECOND_SCHWARZ, V.VFS_FP64, 1e-8, 20000, 1e-3)
        r = np.random.default_rng(2).standard_normal(ctx.n_samples())
        z.append(ctx.vfs_precond_apply(r))
    # at most eight weighted corrections a sample, added in the same order
    assert np.abs(z[0] - z[1]).max() <= 64 * np.finfo(float).eps * np.abs(z[0]).max()


# ---- batch ------------------------------------------------------------------
def _batch_problems():
    probs = [cases.drop2d(n, 700 + q) for q, n in enumerate([24, 37, 64, 50, 3, 33])]
    air = cases.drop2d(32, 1105)
    air["phi_l"] = np.ones_like(air["phi_l"])      # all air: no active sample
    return probs[:2] + [air] + probs[2:]


def _batch(probs, forms, variant=None):
    from paper_1010_2832_amd import vfstokes as V
    b = V.batch_from_cases(probs, tol=1e-9)
    b.vfs_batch_set_forms(forms)
    if variant is not None:
        b.vfs_batch_set_tiles(variant, 2)
    b.vfs_batch_step(probs[0]["dt"])
    _banner(f"batch forms {forms} variant {variant}: {b.vfs_batch_get_forms()}")
    return b


@pytest.mark.parametrize("variant", [0, 1, 2, 3, 4, 5])
def test_persistent_batch_matches_oracle_every_tile_variant(variant):
    probs = _batch_problems()
    b = _batch(probs, 0, variant)
    assert b.vfs_batch_get_forms()["resident"] == -1
    st = b.vfs_batch_get_stats()
    assert st["graph_used"] == 1 and st["status"] == 0
    for i, c in enumerate(probs):
        asm, x, u = system.step(c)
        ug = flat_faces(asm.grid, b.vfs_batch_get_velocity(i))
        pr = b.vfs_batch_get_problem(i)
        assert pr["n_active"] == int(asm.active.sum())
        if pr["n_active"] == 0:
            assert pr["iterations"] == 0 and np.array_equal(ug, u), i
            continue
        assert system.true_relative_residual(asm, b.vfs_batch_get_solution(i)) <= 2e-9
        assert velocity_rel_linf(asm, ug, u) <= 1e-4, i
    b.close()


def test_batch_given_up_runs_in_the_persistent_kernel():
    probs = _batch_problems()
    out = []
    for forms, resident, give_ups in ((0, -1, 0), (RESIDENT | GIVE_UP, -1, 1), (RESIDENT, 0, 0)):
        b = _batch(probs, forms)
        assert b.vfs_batch_get_forms() == dict(forms=forms, resident=resident, give_ups=give_ups)
        out.append([(b.vfs_batch_get_problem(i)["iterations"], b.vfs_batch_get_solution(i))
                    for i in range(len(probs))])
        b.close()
    for (i0, x0), (i1, x1) in zip(out[0], out[1]):
        assert i0 == i1 and np.array_equal(x0, x1)


def test_resident_solves_come_back_after_one_is_given_up():
    """Whatever held the compute units may have gone: after a pause of 4 s the
    resident form is tried again, from cleared words."""
    import time
    solves = []
    for name in ("2d_fp64", "3d_8"):
        make, shape, precision = CASES[name]
        ctx = gpu_run(make(), precision=precision, tol=1e-8, step=False)
        b = ctx.vfs_get_rhs()
        x = ctx.vfs_solve(b)
        assert ctx.vfs_get_forms()["resident"] == shape
        ctx.vfs_set_forms(RESIDENT | GIVE_UP)
        ctx.vfs_solve(b)
        ctx.vfs_set_forms(RESIDENT)
        ctx.vfs_solve(b)
        assert ctx.vfs_get_forms() == dict(forms=RESIDENT, resident=-1, give_ups=1)
        solves.append((ctx, b, x, shape))
    probs = _batch_problems()
    batch = _batch(probs, RESIDENT | GIVE_UP)
    batch.vfs_batch_set_forms(RESIDENT)
    for i, c in enumerate(probs):
        batch.vfs_batch_set_problem(i, c)
    batch.vfs_batch_step(probs[0]["dt"])
    assert batch.vfs_batch_get_forms() == dict(forms=RESIDENT, resident=-1, give_ups=1)
    want = [batch.vfs_batch_get_solution(i) for i in range(len(probs))]
    time.sleep(4.5)
    for ctx, b, x, shape in solves:
        assert np.array_equal(ctx.vfs_solve(b), x)
        assert ctx.vfs_get_forms() == dict(forms=RESIDENT, resident=shape, give_ups=1)
    for i, c in enumerate(probs):
        batch.vfs_batch_set_problem(i, c)
    batch.vfs_batch_step(probs[0]["dt"])
    assert batch.vfs_batch_get_forms() == dict(forms=RESIDENT, resident=0, give_ups=1)
    for i, x in enumerate(want):
        assert np.array_equal(batch.vfs_batch_get_solution(i), x)
    batch.close()


def test_batch_without_memory_for_its_plan():
    """A resident step needs memory of its own; where there is none the persistent
    kernel, which needs none of it, solves, and a later step tries again."""
    probs = _batch_problems()
    b = _batch(probs, RESIDENT | NO_MEMORY)
    assert b.vfs_batch_get_forms()["resident"] == -1
    want = [b.vfs_batch_get_solution(i) for i in range(len(probs))]
    b.vfs_batch_set_forms(RESIDENT)
    for i, c in enumerate(probs):
        b.vfs_batch_set_problem(i, c)
    b.vfs_batch_step(probs[0]["dt"])
    assert b.vfs_batch_get_forms()["resident"] == 0
    for i, x in enumerate(want):
        assert np.array_equal(b.vfs_batch_get_solution(i), x)
    b.close()


def _used():
    import torch
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info()
    return total - free


def test_memory_of_small_contexts_and_of_a_preconditioner_no_longer_set():
    """A small 3D context holds exchange words for the bricks it can have (it held
    38 MB for 512 of them), and the Schwarz corrections are held only while that
    preconditioner is set."""
    from paper_1010_2832_amd import vfstokes as V
    V.Context(3, (8, 8, 8), 0.1).close()     # the library's own first allocations
    before = _used()
    ctxs = [V.Context(3, (8, 8, 8), 0.1) for _ in range(20)]
    small = (_used() - before) / len(ctxs) / 1e6
    for c in ctxs:
        c.close()
    ctx = V.Context(3, (96, 96, 96), 0.01)
    before = _used()
    ctx.vfs_set_solver(V.VFS_PRECOND_SCHWARZ, V.VFS_FP64, 1e-6, 100, 1e-3)
    held = (_used() - before) / 1e6
    ctx.vfs_set_solver(V.VFS_PRECOND_JACOBI, V.VFS_FP64, 1e-6, 100, 1e-3)
    left = (_used() - before) / 1e6
    ctx.vfs_set_solver(V.VFS_PRECOND_SCHWARZ, V.VFS_FP64, 1e-6, 100, 1e-3)
    again = (_used() - before) / 1e6
    ctx.close()
    _banner(f"MB: {small:.1f} a small context, corrections {held:.0f}, {left:.0f} after, {again:.0f} again")
    assert small < 20
    assert 160 < held < 200 and left < 8 and abs(again - held) < 8
