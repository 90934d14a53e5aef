"""Solves whose workgroups wait for each other, in company: several host threads
with a context or a batch each, on streams of their own."""
import threading
import time

import numpy as np
import pytest

import cases
from tests.gpu_util import gpu_run

pytestmark = pytest.mark.gpu


def _banner(msg):
    print(f"[company] {msg}", flush=True)


def _on_stream(ctx):
    import torch
    ctx.stream = torch.cuda.Stream()
    ctx.vfs_set_stream(ctx.stream.cuda_stream)
    return ctx


def _together(*calls):
    """Runs the calls in a thread each; what they returned or raised."""
    out = [None] * len(calls)

    def one(q):
        try:
            out[q] = calls[q]()
        except Exception as e:   # reported by the caller's assert
            out[q] = e
    ts = [threading.Thread(target=one, args=(q,)) for q in range(len(calls))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    return out


def test_persistent_batch_and_resident_solve_wait_for_each_other():
    """The batch's persistent kernel and a resident solve both need their
    workgroups on the chip at once.  Each is longer than the other's deadline
    (2 s for a barrier, 1 s for an exchange)."""
    from paper_1010_2832_amd import vfstokes as V
    case = cases.pool2d(512, 2)
    ctx = _on_stream(gpu_run(case, tol=1e-6, step=False))
    b = ctx.vfs_get_rhs()
    # a residual that is not reached: one run of as many iterations as asked for
    ctx.vfs_set_solver(V.VFS_PRECOND_JACOBI, V.VFS_FP64, 1e-150, 600000, 1e-3)
    big = [cases.drop2d(1700, 5)]
    batch = V.batch_from_cases(big, tol=1e-9, max_iter=2000)
    batch.vfs_batch_set_forms(0)
    batch.vfs_batch_step(big[0]["dt"], allow_unconverged=True)   # first launch: code and graph

    def solve():
        t = time.time()
        ctx.vfs_solve(b, allow_unconverged=True)
        _banner(f"resident solve {time.time() - t:.2f} s, {ctx.vfs_get_forms()}, "
                f"{ctx.vfs_get_stats()['iterations']} iterations")
        return ctx.vfs_get_forms()["give_ups"]

    def step():
        time.sleep(0.5)   # the solve runs by now
        t = time.time()
        rc = batch.vfs_batch_step(big[0]["dt"], allow_unconverged=True)
        _banner(f"batch step {time.time() - t:.2f} s, {rc}")
        return rc

    give_ups, rc = _together(solve, step)
    assert give_ups == 0
    assert rc in (V.VFS_OK, V.VFS_ENOTCONV), rc
    # the other way round
    batch.vfs_batch_set_solver(1e-150, 40000)
    ctx.vfs_set_solver(V.VFS_PRECOND_JACOBI, V.VFS_FP64, 1e-150, 2000, 1e-3)

    def late():
        time.sleep(0.5)
        return solve()
    rc, give_ups = _together(lambda: batch.vfs_batch_step(big[0]["dt"], allow_unconverged=True), late)
    _banner(f"batch solve {batch.vfs_batch_get_stats()['t_solve_ms']:.0f} ms")
    assert batch.vfs_batch_get_stats()["t_solve_ms"] > 1600   # the wait was longer than a deadline
    assert give_ups == 0
    assert rc in (V.VFS_OK, V.VFS_ENOTCONV), rc
    batch.close()


def test_small_solves_run_side_by_side():
    """Two host threads with a small context each: the solves overlap (measured
    0.54 of the time in turn, 0.97 with one solve at a time on the device), and
    each gives the bits it gives alone.  A third thread's solve of the whole chip
    gets its turn between them."""
    ctxs = [_on_stream(gpu_run(cases.drop2d(96, 3 + q), tol=1e-10, step=False)) for q in range(2)]
    rhs = [c.vfs_get_rhs() for c in ctxs]
    want = [c.vfs_solve(b) for c, b in zip(ctxs, rhs)]
    count = 40

    def solves(q):
        return all(np.array_equal(ctxs[q].vfs_solve(rhs[q]), want[q]) for _ in range(count))
    t = time.time()
    assert solves(0) and solves(1)
    in_turn = time.time() - t
    t = time.time()
    assert _together(lambda: solves(0), lambda: solves(1)) == [True, True]
    together = time.time() - t
    _banner(f"in turn {in_turn:.3f} s, together {together:.3f} s")
    assert together < 0.8 * in_turn
    big = _on_stream(gpu_run(cases.drop2d(640, 11), tol=1e-6, step=False))
    b = big.vfs_get_rhs()
    x = big.vfs_solve(b)
    out = _together(lambda: solves(0), lambda: solves(1), lambda: np.array_equal(big.vfs_solve(b), x))
    assert out == [True, True, True]
    for c in ctxs + [big]:
        f = c.vfs_get_forms()
        assert f["resident"] >= 0 and f["give_ups"] == 0
