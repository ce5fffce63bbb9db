"""The area-source filter's probe paths at the map sizes where they part: one texel a face (the
level that is a single texel is level 0), two, the sizes whose footprints take one probe and
level 0 alone, and one whose footprints take many probes on two levels.

Tolerances: as for the 64 x 64 map of the same patches (test_gpu_area.py), a pixel's filtered
radiance moves with the escape direction's error times the patches' slope, which does not depend
on the map's size: 2e-5 at the 99th percentile.  Pixels whose probes lie within that error of a
cube edge read another face, where a map of few texels steps, and probe counts and levels are
discrete choices that may flip: 1 pixel in 100 is left to those."""
import numpy as np
import pytest

from paper_2010_08735_amd import bh, scenes

import parity
from test_gpu_area import _frame_stats, gpu_area

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n0", [1, 2, 16, 512])
def test_area_sizes_match_oracle(gpu_ctx, gpu_tables, orc, orc_tables, n0):
    it = scenes.area_map(n0, 21)
    h = gpu_area(gpu_ctx, it)
    try:
        v = scenes.small_static_view()
        v.disc_opacity = 0.0
        v.k_area = 3.0
        rgb, aov = parity.render_gpu(gpu_ctx, gpu_tables, v, None, area=h)
        pt = orc.render_quads(v, scenes.all_quads(v.width, v.height), tables=orc_tables,
                              area=orc.area_levels(it), area_n0=n0)
        g = parity.gpu_at(rgb, aov, pt)
        m = parity.mask_of(pt, g)
        lit = ~m & (pt["star_zeroed"] == 0) & (pt["area_A"] > 0)
        r = _frame_stats(pt, g, lit)
        print(n0, "p50 %.2g p99 %.2g max %.2g" % (np.median(r), np.percentile(r, 99), r.max()))
        assert lit.sum() > 10000
        assert np.percentile(r, 99) < 2e-5
    finally:
        bh.bh_release_area(h)


@pytest.mark.parametrize("opacity", [0.0, 0.6, 1.0])
def test_image_is_the_same_with_and_without_the_pixel_record(gpu_ctx, gpu_tables, small_scene,
                                                             opacity):
    """Waves of hidden pixels end early, and a crossing behind an opaque one is not looked for,
    only when no per-pixel record is written: the images are equal bit for bit."""
    field, sn0, sh, cube = small_scene
    h = gpu_area(gpu_ctx, scenes.area_map(64, 21))
    try:
        for area in (None, h):
            v = scenes.small_static_view()
            v.disc_opacity = opacity
            v.k_area = 0.5
            with_record, _ = parity.render_gpu(gpu_ctx, gpu_tables, v, sh, area=area)
            without, _ = parity.render_gpu(gpu_ctx, gpu_tables, v, sh, aov=False, area=area)
            assert np.array_equal(with_record, without)
    finally:
        bh.bh_release_area(h)


@pytest.mark.parametrize("bands", [False, True])
def test_largest_map_reads_its_own_texels(gpu_ctx, gpu_tables, bands):
    """The largest area map (2 GiB with band colours, byte offsets to the end of 32 bits).  Bilinear
    reads and box-filtered levels reproduce a field that is linear on each face, so its frame is
    the 256 x 256 map's of the same field: to 2^-24 of the texel count in the position, times the
    field's slope of a texel, and the roundings of some ten products (1e-6), except where a
    footprint reaches the outermost half texels of a face of either map (1 pixel in 30)."""
    import torch

    def build(n0):
        c = (torch.arange(n0, device="cuda", dtype=torch.float64) + 0.5) * (2.0 / n0) - 1.0
        f = torch.arange(6, device="cuda", dtype=torch.float64)
        I = (2.0 + 0.3 * f[:, None, None] + 0.5 * c[None, None, :] + 0.25 * c[None, :, None])
        I = I.float()
        if bands:
            tex = torch.stack([I, 0.5 * I, 0.25 * I, torch.zeros_like(I)], -1).contiguous()
        else:
            tex = torch.stack([I, torch.full_like(I, 6000.0)], -1).contiguous()
        del I
        make = bh.bh_build_area_bands if bands else bh.bh_build_area
        h = make(gpu_ctx, tex.data_ptr(), n0, bh.current_stream())
        torch.cuda.synchronize()
        return h

    small, large = build(256), build(4096)
    try:
        for aim in ((0.4, 0.7), (1.6, 2.4), (2.7, 4.5)):
            v = scenes.small_static_view()
            v.width, v.height, v.fov_y, v.disc_opacity, v.k_area = 201, 163, 2.0, 0.0, 1.0
            v.cam_rot = scenes.look_rotation(scenes.spherical_position(1.0, *aim))
            a, b = (parity.render_gpu(gpu_ctx, gpu_tables, v, None, aov=False, area=h)[0]
                    for h in (small, large))
            r = np.abs(a - b)[..., :3].max(-1) / np.maximum(a[..., :3].max(-1), 1e-3)
            assert (a[..., :3].max(-1) > 0).mean() > 0.5
            assert np.percentile(r, 97) < 1e-5, float(np.percentile(r, 97))
    finally:
        bh.bh_release_area(small)
        bh.bh_release_area(large)
        bh.bh_trim(gpu_ctx)
