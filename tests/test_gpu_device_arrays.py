"""Device arrays of the caller's are read and written by kernels, host arrays
through a staging copy: both give the same state and results, and a bad value
leaves what it left before."""
import ctypes

import numpy as np
import pytest

import cases
from tests.gpu_util import gpu_run

pytestmark = pytest.mark.gpu

CASES = {"2d": lambda: cases.drop2d(33, 3), "3d": lambda: cases.crop(cases.pool3d(12, 9), (0, 0, 0), (12, 9, 11))}


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(np.asarray(a, np.float64).ravel(order="F"))).cuda()


def _state(V, ctx, case):
    """Device copies of what the library hands out, and the host ones."""
    import torch
    n = ctx.n_samples()
    dev = [torch.full((q.size,), np.nan, dtype=torch.float64, device="cuda") for q in case["u"]]
    b = torch.full((n,), np.nan, dtype=torch.float64, device="cuda")
    ptr = [ctypes.c_void_p(q.data_ptr()) for q in dev] + [None] * (3 - len(dev))
    assert V._lib.vfs_get_velocity(ctx.handle, *ptr) == 0
    assert V._lib.vfs_get_rhs(ctx.handle, ctypes.c_void_p(b.data_ptr())) == 0
    for d, h in zip(dev, ctx.vfs_get_velocity()):
        assert np.array_equal(d.cpu().numpy(), np.asarray(h).ravel(order="F"))
    assert np.array_equal(b.cpu().numpy(), ctx.vfs_get_rhs())
    return [d.cpu().numpy() for d in dev], b.cpu().numpy()


@pytest.mark.parametrize("name", list(CASES))
def test_device_and_host_arrays_agree(name):
    import torch
    from paper_1010_2832_amd import vfstokes as V
    case = CASES[name]()
    host = gpu_run(case, step=False)
    ctx = V.context_from_case(case)
    ctx.vfs_set_level_sets(_dev(case["phi_l"]), None if case["phi_s"] is None else _dev(case["phi_s"]))
    ctx.vfs_set_density(_dev(case["rho"]))
    ctx.vfs_set_viscosity(_dev(case["mu"]))
    ctx.vfs_set_velocity([_dev(q) for q in case["u"]])
    ctx.vfs_assemble(case["dt"])
    for x, y in zip(_state(V, host, case)[0], _state(V, ctx, case)[0]):
        assert np.array_equal(x, y)
    assert np.array_equal(host.vfs_get_rhs(), ctx.vfs_get_rhs())
    x = np.random.default_rng(1).standard_normal(ctx.n_samples())
    y = _dev(x)
    assert V._lib.vfs_apply(ctx.handle, ctypes.c_void_p(y.data_ptr()), ctypes.c_void_p(y.data_ptr())) == 0
    assert np.array_equal(y.cpu().numpy(), host.vfs_apply(x))
    # an odd byte offset goes through the staging copy
    raw = torch.zeros(8 * x.size + 8, dtype=torch.uint8, device="cuda")
    raw[4:4 + 8 * x.size] = _dev(x).view(torch.uint8)
    out = torch.zeros(x.size, dtype=torch.float64, device="cuda")
    assert V._lib.vfs_apply(ctx.handle, ctypes.c_void_p(raw.data_ptr() + 4), ctypes.c_void_p(out.data_ptr())) == 0
    assert np.array_equal(out.cpu().numpy(), host.vfs_apply(x))


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("put", [_dev, lambda a: np.array(a, np.float64)])
def test_a_bad_value_changes_neither_its_array_nor_a_later_one(name, put):
    from paper_1010_2832_amd import vfstokes as V
    case = CASES[name]()
    ctx = gpu_run(case, step=False)
    old = [np.asarray(q) for q in ctx.vfs_get_velocity()]
    new = [2.0 * np.asarray(q) for q in case["u"]]
    new[1].flat[-1] = np.inf
    with pytest.raises(V.VfsError, match="velocity: non-finite value"):
        ctx.vfs_set_velocity([put(q) for q in new])
    got = [np.asarray(q) for q in ctx.vfs_get_velocity()]
    assert np.array_equal(got[0], new[0])
    for a in range(1, len(old)):
        assert np.array_equal(got[a], old[a])
    rho = np.array(case["rho"])
    rho.flat[3] = 0.0
    with pytest.raises(V.VfsError, match="density: non-finite or non-positive value"):
        ctx.vfs_set_density(put(rho))
    solid = np.array(case["phi_l"])
    solid.flat[-1] = np.nan
    with pytest.raises(V.VfsError, match="phi_solid"):
        ctx.vfs_set_level_sets(put(case["phi_l"]), put(solid))
    with pytest.raises(V.VfsError, match="phi_liquid"):
        ctx.vfs_set_level_sets(put(solid), put(solid))
    # and the next calls are not disturbed: same results as in a fresh context
    x = np.random.default_rng(1).standard_normal(ctx.n_samples())
    bad = x.copy()
    bad[-1] = np.nan
    fresh = gpu_run(case, step=False)
    for c in (ctx, fresh):
        c.vfs_set_level_sets(put(case["phi_l"]), None if case["phi_s"] is None else put(case["phi_s"]))
        c.vfs_set_velocity([put(q) for q in case["u"]])
        c.vfs_assemble(case["dt"])
    z = put(bad)
    p = z.data_ptr() if hasattr(z, "data_ptr") else z.ctypes.data
    assert V._lib.vfs_apply(ctx.handle, ctypes.c_void_p(p), ctypes.c_void_p(p)) == V.VFS_EINVAL
    assert np.array_equal(ctx.vfs_apply(x), fresh.vfs_apply(x))
    ctx.vfs_step(case["dt"])
    fresh.vfs_step(case["dt"])
    for q, r in zip(ctx.vfs_get_velocity(), fresh.vfs_get_velocity()):
        assert np.array_equal(q, r)


def test_device_arrays_that_end_early_are_refused():
    """An array that ends before its last value is refused, as the copies that took
    it did, and not read or written past its end.  (The values missing here lie in
    the same page of memory.)"""
    from paper_1010_2832_amd import vfstokes as V
    case = cases.drop2d(16, 3)
    ctx = gpu_run(case, step=False)
    hip = V._lib   # its HIP runtime
    short = ctypes.c_void_p()
    assert hip.hipMalloc(ctypes.byref(short), ctypes.c_size_t(1024)) == 0
    try:
        zero = np.zeros(128)
        assert hip.hipMemcpy(short, ctypes.c_void_p(zero.ctypes.data), ctypes.c_size_t(1024), 1) == 0
        old = ctx.vfs_get_pressure(), ctx.vfs_get_velocity()
        assert V._lib.vfs_set_density(ctx.handle, short) == V.VFS_EHIP
        assert V._lib.vfs_set_velocity(ctx.handle, short, short, None) == V.VFS_EHIP
        assert V._lib.vfs_set_level_sets(ctx.handle, short, None) == V.VFS_EHIP
        assert V._lib.vfs_get_pressure(ctx.handle, short) == V.VFS_EHIP
        assert V._lib.vfs_get_rhs(ctx.handle, short) == V.VFS_EHIP
        assert V._lib.vfs_apply(ctx.handle, short, short) == V.VFS_EHIP
        for a, b in zip(old[1], ctx.vfs_get_velocity()):
            assert np.array_equal(a, b)
    finally:
        assert hip.hipFree(short) == 0


def test_outputs_that_share_memory_hold_the_last_one():
    """One device array given for several components of the velocity holds the last
    component's values, as with host arrays; so do parts that overlap."""
    import torch
    from paper_1010_2832_amd import vfstokes as V
    case = cases.crop(cases.pool3d(40, 9), (0, 0, 0), (40, 31, 37))
    ctx = gpu_run(case, step=False)
    u = [q.ravel(order="F") for q in ctx.vfs_get_velocity()]
    for shift in (0, 1000):
        host = np.full(max(q.size for q in u) + 2 * shift, np.nan)
        dev = _dev(host)
        for buf, p in ((host, host.ctypes.data), (dev, dev.data_ptr())):
            ptr = [ctypes.c_void_p(p + 8 * shift * a) for a in range(3)]
            assert V._lib.vfs_get_velocity(ctx.handle, *ptr) == 0
        want = np.full_like(host, np.nan)
        for a in range(3):
            want[shift * a:shift * a + u[a].size] = u[a]
        assert np.array_equal(host, want, equal_nan=True)
        assert np.array_equal(dev.cpu().numpy(), want, equal_nan=True)
