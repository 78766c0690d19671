"""The tiled sweeps where rows, columns and planes run out: extents around a
wave's 64 lanes of 1, 2 and 4 columns, single rows and planes, every boundary
rule, against numpy in FP64.  Nine operations per point on values of order 1:
16 roundings of the storage type."""
import numpy as np
import pytest

import paper_1207_1746_amd as G

pytestmark = pytest.mark.gpu


def _shift(u, axis, d, rule):
    if rule == G.PERIODIC:
        return np.roll(u, -d, axis)
    n = u.shape[axis]
    i = np.arange(n) + d
    v = np.take(u, np.clip(i, 0, n - 1), axis)
    if rule == G.DIRICHLET:
        s = [1, 1, 1]
        s[axis] = n
        v = np.where(((i >= 0) & (i < n)).reshape(s), v, 0.25)
    return v


@pytest.mark.parametrize("nx", [1, 2, 3, 5, 63, 64, 65, 127, 128, 129, 130, 255, 256, 257, 259])
@pytest.mark.parametrize("rule", [G.DIRICHLET, G.PERIODIC, G.CLAMP])
def test_tiled_jacobi_edges(ctx, nx, rule):
    rng = np.random.default_rng(nx)
    for ny, nz in ((1, 1), (2, 5), (5, 2), (9, 3)):
        u = rng.uniform(-1, 1, (nz, ny, nx)).astype(np.float32).astype(np.float64)
        f = rng.uniform(-1, 1, (nz, ny, nx)).astype(np.float32).astype(np.float64)
        s = sum(_shift(u, ax, d, rule) for ax in (2, 1, 0) for d in (1, -1))
        ex = 0.25 * u + 0.75 * (s - 0.5 * f) / 6
        for dt, vs, eps in ((G.F64, (1, 2), 2.0 ** -53), (G.F32, (1, 2, 4), 2.0 ** -24)):
            gu = ctx.grid(u.shape, dt, halo=1, bc=rule, bc_value=0.25 if rule == G.DIRICHLET else 0.0, data=u)
            gf = ctx.grid(u.shape, dt, halo=0, data=f)
            go = ctx.grid(u.shape, dt, halo=0)
            for v in vs:
                for cz in (1, 2):
                    ctx.tile_set(G.K_WJACOBI, gu, (v, 4, cz))
                    go.fill(7.0)
                    ctx.do_all(G.K_WJACOBI, [gu, gf], [go], p=(0.75, 0.5))
                    assert np.abs(go.numpy().astype(np.float64) - ex).max() <= 16 * eps, (ny, nz, dt, v, cz)
    ctx.tile_clear()
