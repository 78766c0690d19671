"""GPU parity of the image filters at every way a row can end: widths around
whole 16-pixel lanes and 1024-pixel waves, heights around the rows of a wave's
march, both Laplacians, bit for bit; the bytes of the row padding stay as the
caller left them."""
import numpy as np
import pytest

import oracle
import paper_1207_1746_amd as G

pytestmark = pytest.mark.gpu

WIDTHS = [1, 2, 3, 4, 5, 7, 12, 15, 16, 17, 19, 31, 33, 1007, 1008, 1019, 1020, 1021, 1023, 1024, 1025, 1027, 1028, 1039,
          1040, 2047, 2052]


@pytest.mark.parametrize("lap_kind", [4, 8])
@pytest.mark.parametrize("cy", [0, 1, 2, 3, 4, 8])
def test_image_every_row_end(ctx, lap_kind, cy):
    import torch
    g = np.random.default_rng(100 + cy)
    for nx in WIDTHS:
        for nz, ny in ((2, 7), (1, 1), (1, 9)):
            img = g.integers(0, 256, size=(nz, ny, nx), dtype=np.uint8)
            if nx > 8:
                img[:, :, nx // 2:] = g.choice([0, 255], size=img[:, :, nx // 2:].shape)
            gi = ctx.grid(img.shape, G.U8, halo=2, bc=G.CLAMP, ndim=2, data=img)
            gb = ctx.grid(img.shape, G.U8, halo=0, ndim=2)
            gl = ctx.grid(img.shape, G.I16, halo=0, ndim=2)
            gb.storage.fill_(0xA5)
            gl.storage.fill_(0x5A5A)
            if cy:
                ctx.tile_set(G.K_IMG_BOX5_LAP, gi, (4, 4, cy))
            ctx.do_all(G.K_IMG_BOX5_LAP, [gi], [gb, gl], p=(lap_kind,))
            ctx.tile_clear()
            box, lap = oracle.img(img, lap_kind)
            assert np.array_equal(gb.numpy(), box.reshape(img.shape)), (nx, ny)
            assert np.array_equal(gl.numpy(), lap.reshape(img.shape)), (nx, ny)
            pitch = gb.desc.pitch[0]
            if pitch > nx:
                pad_b = gb.storage[:nz * ny * pitch].view(nz, ny, pitch)[:, :, nx:]
                pad_l = gl.storage[:nz * ny * pitch].view(nz, ny, pitch)[:, :, nx:]
                assert bool((pad_b == 0xA5).all()) and bool((pad_l == 0x5A5A).all()), (nx, ny)


@pytest.mark.parametrize("nx", [127, 128, 129, 255, 256, 257, 511, 512, 513])
def test_image_rows_sharing_a_wave(ctx, nx):
    """Widths around the rows that share a wave (8, 16 and 32 lanes each), with
    chunk counts that leave lanes of the last wave without a chunk."""
    g = np.random.default_rng(nx)
    for nz, ny in ((1, 1), (3, 11), (1, 17)):
        img = g.integers(0, 256, size=(nz, ny, nx), dtype=np.uint8)
        gi = ctx.grid(img.shape, G.U8, halo=2, bc=G.CLAMP, ndim=2, data=img)
        gb = ctx.grid(img.shape, G.U8, halo=0, ndim=2)
        gl = ctx.grid(img.shape, G.I16, halo=0, ndim=2)
        for lap_kind in (4, 8):
            for cy in (1, 2, 4):
                ctx.tile_set(G.K_IMG_BOX5_LAP, gi, (4, 4, cy))
                ctx.do_all(G.K_IMG_BOX5_LAP, [gi], [gb, gl], p=(lap_kind,))
                box, lap = oracle.img(img, lap_kind)
                assert np.array_equal(gb.numpy(), box.reshape(img.shape)), (ny, lap_kind, cy)
                assert np.array_equal(gl.numpy(), lap.reshape(img.shape)), (ny, lap_kind, cy)
    ctx.tile_clear()
