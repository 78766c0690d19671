"""A narrow, tall stack of images: 2^28 rows of 16 pixels, several rows to a
wave, more chunks of rows than fit one launch dimension if each had a wave.
Every layer is the same image, so every layer's filters equal the oracle's."""
import numpy as np
import pytest

import oracle
import paper_1207_1746_amd as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lap_kind", [4, 8])
def test_image_more_chunks_than_a_launch_dimension(ctx, lap_kind):
    import torch
    img = np.random.default_rng(3).integers(0, 256, size=(1, 16384, 16), dtype=np.uint8)
    shape = (16384, 16384, 16)
    gi = ctx.grid(shape, G.U8, halo=2, bc=G.CLAMP, ndim=2)
    gi.view.copy_(torch.as_tensor(img, device="cuda").expand(shape))
    gb, gl = ctx.grid(shape, G.U8, halo=0, ndim=2), ctx.grid(shape, G.I16, halo=0, ndim=2)
    ctx.do_all(G.K_IMG_BOX5_LAP, [gi], [gb, gl], p=(lap_kind,))
    for g, want in zip((gb, gl), oracle.img(img, lap_kind)):
        assert np.array_equal(g.view[0].cpu().numpy(), want.reshape(16384, 16))
        assert all(bool((g.view[z:z + 1024] == g.view[0]).all()) for z in range(0, 16384, 1024))
    del gi, gb, gl
    torch.cuda.empty_cache()
