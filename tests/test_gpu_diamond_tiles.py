"""The diamond kernels on enough layers to take the 64 x 32 tiles (whole and
partial tiles in both directions, the smallest grid), against the oracle: the
same operations per cell, so FP64 is bit for bit; FP32 to 256 roundings."""
import numpy as np
import pytest

import oracle
import paper_1207_1746_amd as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(512, 1, 1), (512, 31, 65), (256, 33, 70), (256, 64, 128)])
@pytest.mark.parametrize("dt", [G.F64, G.F32])
@pytest.mark.parametrize("kind", ["recur", "gs2d"])
def test_short_tiles_match_oracle(ctx, shape, dt, kind):
    g = np.random.default_rng(72)
    x = [g.uniform(-0.45, 0.45, shape), g.uniform(-0.45, 0.45, shape), g.standard_normal(shape)]
    if dt == G.F32:
        x = [v.astype(np.float32).astype(np.float64) for v in x]
    if kind == "recur":
        gi = [ctx.grid(shape, dt, halo=0, ndim=2, data=v) for v in x]
        go = ctx.grid(shape, dt, halo=0, ndim=2)
        ctx.do_diamond(G.K_DIAMOND_RECUR, gi, [go], p=(0.75,))
        ex = oracle.diamond_recur(*x, seed=0.75)
    else:
        go = ctx.grid(shape, dt, halo=1, ndim=2, bc_value=0.5, data=x[2])
        gf = ctx.grid(shape, dt, halo=0, ndim=2, data=x[0])
        ctx.do_diamond(G.K_GS2D, [go, gf], [go], p=(1.3, 0.05))
        ex = oracle.gs2d_sweep(x[2], x[0], 1.3, 0.05, 0.5)
    got = go.numpy().astype(np.float64)
    if dt == G.F64:
        assert np.array_equal(got, ex)
    else:
        assert np.abs(got - ex).max() <= 256 * 2.0 ** -24 * (np.abs(ex).max() + 1)
