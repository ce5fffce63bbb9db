"""The persistent batch form's claims: a wave's first claim is its own number and later ones come
from the counter, so every tile is rendered once whether the launch has fewer tiles than waves,
about as many, or many per wave; twice in a row, as the counter starts again at each call.  Each
image is the per-tile form's, bit for bit."""
import numpy as np
import pytest

from paper_2010_08735_amd import bh, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[(8, 8)], [(33, 17), (5, 70)], [(700, 500), (801, 603)],
                                   [(1920, 1080), (64, 64), (1283, 999)]])
def test_every_tile_is_rendered_once(gpu_ctx, gpu_tables, small_scene, sizes):
    import torch
    field, n0, sh, cube = small_scene
    views = []
    for w, h in sizes:
        v = scenes.small_static_view()
        v.width, v.height = w, h
        views.append(bh.make_view(v, sh))
    images = []
    try:
        for form in (0, 1, 1):
            bh.bh_set_batch_form(gpu_ctx, form)
            outs = [torch.full((h, w, 4), float("nan"), dtype=torch.float32, device="cuda")
                    for w, h in sizes]
            bh.bh_render_batch(gpu_ctx, gpu_tables, views, [o.data_ptr() for o in outs],
                               bh.current_stream())
            torch.cuda.synchronize()
            images.append([o.cpu().numpy() for o in outs])
    finally:
        bh.bh_set_batch_form(gpu_ctx, 0)
    for tiles, first, second in zip(*images):
        assert np.isfinite(tiles).all()
        assert np.array_equal(tiles, first) and np.array_equal(tiles, second)
