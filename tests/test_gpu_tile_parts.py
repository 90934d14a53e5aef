"""Launched 3D mixed iterations on short tile lists, whose 8-plane work tiles are
split in z: parts of the last tiles that lie past the grid have nothing to do."""
import numpy as np
import pytest

import cases
from tests.gpu_util import gpu_run

pytestmark = pytest.mark.gpu


def _slab(n, seed=3):
    """Liquid to nine tenths of the height (y), too many bricks to run resident."""
    rng = np.random.default_rng(seed)
    h = 1.0 / max(n)
    X = cases.node_coords(n, h, (0.0, 0.0, 0.0))
    return dict(dim=3, n=n, h=h, origin=(0.0, 0.0, 0.0), dt=1e-3, phi_l=X[1] - 0.9 * n[1] * h, phi_s=None,
                rho=rng.uniform(0.5, 2.0, size=n), mu=rng.uniform(0.5, 5.0, size=n),
                u=[rng.normal(0, 0.2, size=s) for s in cases.face_shapes(n)], u_bc=None,
                g=(0.0, -9.8, 0.0), name="slab")


# planes 0..n[2] in tiles of 8, split into two parts of 4: one plane in the last
# tile (its second part starts three past the end), four (starts at the end), five
@pytest.mark.parametrize("n", [(127, 71, 32), (127, 71, 35), (127, 71, 36), (128, 71, 32)])
def test_parts_past_the_grid(n):
    print(f"tile parts {n}", flush=True)
    ctx = gpu_run(_slab(n), precision=1, tol=1e-6)
    st = ctx.vfs_get_stats()
    tiles = st["n_tile_samples"] // (64 * 4 * 8 * 6)
    print(f"  {tiles} tiles, {st['iterations']} iterations", flush=True)
    assert 128 < tiles <= 256          # split in two, and over 256 bricks of 16 x 8 x 8
    assert st["rel_residual"] <= 1e-6
    x, b = ctx.vfs_get_solution(), ctx.vfs_get_rhs()
    assert np.linalg.norm(b - ctx.vfs_apply(x)) <= 1.01e-6 * np.linalg.norm(b)
