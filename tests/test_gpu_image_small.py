"""Images around the size up to which a thread filters a pixel: extents on both
sides of the line, and the same result with rows per wave set, bit for bit."""
import numpy as np
import pytest

import oracle
import paper_1207_1746_amd as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lap_kind", [4, 8])
@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 2, 65), (6144, 1, 3), (3, 5, 64), (1, 640, 1024), (1, 640, 1025),
                                   (1, 641, 1024), (2, 1024, 320), (2, 1025, 319)])
def test_image_by_pixel_or_by_row(ctx, shape, lap_kind):
    img = np.random.default_rng(sum(shape)).integers(0, 256, size=shape, dtype=np.uint8)
    gi = ctx.grid(shape, G.U8, halo=2, bc=G.CLAMP, ndim=2, data=img)
    gb, gl = ctx.grid(shape, G.U8, halo=0, ndim=2).fill(1), ctx.grid(shape, G.I16, halo=0, ndim=2).fill(1)
    box, lap = (a.reshape(shape) for a in oracle.img(img, lap_kind))
    for cy in (0, 2):
        if cy:
            ctx.tile_set(G.K_IMG_BOX5_LAP, gi, (4, 4, cy))
        ctx.do_all(G.K_IMG_BOX5_LAP, [gi], [gb, gl], p=(lap_kind,))
        ctx.tile_clear()
        assert np.array_equal(gb.numpy(), box) and np.array_equal(gl.numpy(), lap), cy
