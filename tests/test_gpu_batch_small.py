"""The persistent batch form at both ends: with a few tiles a wave every wave has its share, so
the form stays close to one workgroup per tile (dealt in claims of 16 tiles it took 4 to 5 times as
long on a 512 x 512 frame, since most waves got none)."""
import pytest

from paper_2010_08735_amd import bh, scenes

from test_gpu_area import gpu_area

pytestmark = pytest.mark.gpu


def _us(run, n=60):
    import torch
    best = float("inf")
    for _ in range(5):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(n):
            run()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / n)
    return best


def test_small_persistent_launches_use_every_wave(gpu_ctx, gpu_tables, small_scene):
    import torch
    field, n0, sh, cube = small_scene
    v = scenes.small_static_view()
    v.width = v.height = 512
    v.disc_opacity, v.k_area = 0.0, 0.5
    area = gpu_area(gpu_ctx, scenes.area_map(512, 21))
    view = bh.make_view(v, sh, None, area)
    out = torch.zeros((512, 512, 4), device="cuda")
    us = []
    try:
        for form in (0, 1):
            bh.bh_set_batch_form(gpu_ctx, form)
            us.append(_us(lambda: bh.bh_render_batch(gpu_ctx, gpu_tables, [view],
                                                     [out.data_ptr()], bh.current_stream())))
    finally:
        bh.bh_set_batch_form(gpu_ctx, 0)
        bh.bh_release_area(area)
    print("per tile %.1f us, persistent %.1f us" % tuple(us))
    assert us[1] < 2 * us[0], us


@pytest.mark.parametrize("cfg,sizes", [
    (3, [(3840, 2160)] * 3 + [(2049, 2047), (8, 8)]),  # 70 blocks a wave: half dealt, half claimed
    (6, [(1283, 999), (33, 65)]), (6, [(31, 31)]), (7, [(1920, 1080), (700, 501)])])  # 16 blocks
def test_dealt_and_claimed_tiles_are_rendered_once(gpu_ctx, gpu_tables, small_scene, cfg, sizes):
    """Twice in the persistent form, as the counter starts again at each call; each image is the
    per-tile form's, bit for bit."""
    import torch
    field, n0, sh, cube = small_scene
    views = []
    for w, h in sizes:
        v = scenes.small_static_view()
        v.width, v.height = w, h
        views.append(bh.make_view(v, sh))
    images = []
    try:
        bh.bh_set_tile_config(gpu_ctx, cfg)
        for form in (0, 1, 1):
            bh.bh_set_batch_form(gpu_ctx, form)
            outs = [torch.full((h, w, 4), float("nan"), device="cuda") for w, h in sizes]
            bh.bh_render_batch(gpu_ctx, gpu_tables, views, [o.data_ptr() for o in outs],
                               bh.current_stream())
            torch.cuda.synchronize()
            images.append(outs)
    finally:
        bh.bh_set_batch_form(gpu_ctx, 0)
        bh.bh_set_tile_config(gpu_ctx, -1)
    for tiles, one, two in zip(*images):
        assert torch.isfinite(tiles).all()
        assert torch.equal(tiles, one) and torch.equal(tiles, two)
