"""Volume fractions straight from the level sets: every set of both materials,
and the one-set call, bit for bit against the oracle at the edges of the kernels'
tiles (32 x 8 and 32 x 4 x 4 anchors, one more than the cells) and on level sets
that are all of one sign, of mixed signs in every cell, and both in one tile."""
import numpy as np
import pytest

from oracle import fractions
from oracle.grid import Grid

pytestmark = pytest.mark.gpu


def _field(n, kind, seed):
    rng = np.random.default_rng(seed)
    shape = tuple(q + 1 for q in n)
    phi = rng.standard_normal(shape)
    phi[rng.random(shape) < 0.1] = 0.0            # nodes on the surface
    if kind == "in":
        return -np.abs(phi) - 1e-3
    if kind == "out":
        return np.abs(phi)
    if kind == "split":                           # one sign on either side, x < n/2
        x = np.arange(shape[0]).reshape((-1,) + (1,) * (len(n) - 1))
        return np.where(x < n[0] / 2, -np.abs(phi) - 1e-3, np.abs(phi))
    return phi


@pytest.mark.parametrize("n", [(1, 1), (31, 7), (32, 8), (33, 17), (70, 9),
                               (1, 1, 1), (31, 3, 3), (32, 4, 4), (33, 5, 9), (6, 13, 8)])
@pytest.mark.parametrize("liquid,solid", [("mixed", "mixed"), ("split", "out"), ("in", "split"),
                                          ("out", "in"), ("in", None)])
def test_weights_bitexact_at_tile_edges(n, liquid, solid):
    import torch
    from paper_1010_2832_amd import vfstokes as V
    d = len(n)
    phi_l = _field(n, liquid, 3)
    phi_s = None if solid is None else _field(n, solid, 4)
    print(f"weights {n} {liquid} {solid}", flush=True)
    ctx = V.Context(d, n, 1.0 / max(n))
    cell = np.ones(n)
    ctx.vfs_set_level_sets(phi_l, phi_s)
    ctx.vfs_set_density(cell)
    ctx.vfs_set_viscosity(cell)
    ctx.vfs_set_velocity([np.zeros([n[b] + (1 if b == a else 0) for b in range(d)]) for a in range(d)])
    ctx.vfs_assemble(1e-2)
    grid = Grid(n, 1.0 / max(n))
    W = fractions.sample_weights(grid, phi_l, phi_s)
    if d == 2:
        sets = [(V.VFS_SET_CELL, (1, 1)), (V.VFS_SET_FACE_X, (0, 1)), (V.VFS_SET_FACE_Y, (1, 0)),
                (V.VFS_SET_NODE, (0, 0))]
    else:
        sets = [(V.VFS_SET_CELL, (1, 1, 1)), (V.VFS_SET_FACE_X, (0, 1, 1)), (V.VFS_SET_FACE_Y, (1, 0, 1)),
                (V.VFS_SET_FACE_Z, (1, 1, 0)), (V.VFS_SET_EDGE_Z, (0, 0, 1)), (V.VFS_SET_EDGE_Y, (0, 1, 0)),
                (V.VFS_SET_EDGE_X, (1, 0, 0))]
    dev = torch.from_numpy(np.ascontiguousarray(phi_l.ravel(order="F"))).cuda()
    for sid, st in sets:
        assert np.array_equal(ctx.vfs_get_weights(sid, V.VFS_WEIGHT_LIQUID), W[st][0]), (sid, "liquid")
        fluid = ctx.vfs_get_weights(sid, V.VFS_WEIGHT_FLUID)
        # assembly zeroes the faces next to a sample without fluid
        want = np.where(fluid == 0.0, 0.0, W[st][1]) if st in grid.faces else W[st][1]
        assert np.array_equal(fluid, want), (sid, "fluid")
        out = torch.full((W[st][0].size,), np.nan, dtype=torch.float64, device="cuda")
        V.vfs_liquid_weights_noalloc(d, n, 1e-3, dev, sid, out)
        assert np.array_equal(out.cpu().numpy(), W[st][0].ravel(order="F")), (sid, "one set")
