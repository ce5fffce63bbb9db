"""Star maps at the edges of the build's tiling, against the same merge in numpy: faces smaller
than a tile, one tile a face and many, occupancy words shared by tiles, tiles with more stars
than fit in LDS, many stars in one texel, unlit stars, and an empty field."""
import numpy as np
import pytest

from paper_2010_08735_amd import bh, scenes

pytestmark = pytest.mark.gpu


def _place(dirs, n0):
    """Level-0 texel and position of each direction, in float32 as the map's definition."""
    a = np.abs(dirs)
    k = np.where(a[:, 1] > a[:, 0], 1, 0)
    k = np.where(a[:, 2] > np.maximum(a[:, 0], a[:, 1]), 2, k)
    i = np.arange(len(dirs))
    m = a[i, k]
    face = 2 * k + (dirs[i, k] < 0)
    g = [np.float32(0.5) * (dirs[i, (k + j) % 3] / m + np.float32(1)) * np.float32(n0)
         for j in (1, 2)]
    c = [np.clip(np.floor(x).astype(np.int64), 0, n0 - 1) for x in g]
    return (face * n0 + c[1]) * n0 + c[0], g[0] - c[0].astype(np.float32), \
        g[1] - c[1].astype(np.float32)


def _levels(dirs, channels, weight, n0):
    """(texels, channels + 2) sums per level: channels, weight u, weight v."""
    key, pu, pv = _place(dirs, n0)
    lev = np.zeros((6 * n0 * n0, channels.shape[1] + 2))
    np.add.at(lev, key, np.concatenate([channels, (weight * pu)[:, None],
                                        (weight * pv)[:, None]], 1))
    return lev


def _field(n, n0, kind, seed):
    rng = np.random.default_rng(seed)
    f = scenes.star_field(max(n, 1), seed)
    d, inten, temp = f.dirs[:n].copy(), f.intensity[:n].copy(), f.temperature[:n].copy()
    if kind == "clustered" and n:
        d[: n // 2] = d[0] + rng.normal(0, 0.02, (n // 2, 3)).astype(np.float32)
        d[: n // 40] = d[1]  # many stars in one texel
        inten[::17] = 0.0    # unlit
        d[3] = 0.0           # no direction
    return d, inten, temp


CASES = [(1, 50, "plain"), (2, 50, "plain"), (4, 300, "plain"), (16, 3000, "plain"),
         (32, 3000, "clustered"), (64, 30000, "clustered"), (64, 60000, "clustered"), (512, 20000, "clustered"),
         (1024, 40000, "clustered"), (2048, 5000, "plain"), (64, 0, "plain")]


@pytest.mark.parametrize("n0,n,kind", CASES)
@pytest.mark.parametrize("bands", [False, True])
def test_star_map_levels_match_numpy(gpu_ctx, n0, n, kind, bands):
    import torch
    d, inten, temp = _field(n, n0, kind, 5)
    one = np.zeros((1, 3), np.float32)
    dd = torch.from_numpy(d if n else one).cuda()
    if bands:
        col = np.random.default_rng(3).uniform(0.1, 1.0, (n, 3)).astype(np.float32)
        rgb = (inten[:, None] * col).astype(np.float32)
        tt = torch.from_numpy(rgb if n else one).cuda()
        h = bh.bh_build_star_bands(gpu_ctx, dd.data_ptr(), tt.data_ptr(), n, n0,
                                   bh.BH_TEXEL_FP32, bh.current_stream())
        ch, w = rgb.astype(np.float64), rgb.astype(np.float64).sum(1)
    else:
        ii, tt = (torch.from_numpy(x if n else one[0]).cuda() for x in (inten, temp))
        h = bh.bh_build_stars(gpu_ctx, dd.data_ptr(), ii.data_ptr(), tt.data_ptr(), n, n0,
                              bh.BH_TEXEL_FP32, bh.current_stream())
        w = inten.astype(np.float64)
        ch = np.stack([w, w * temp], 1)
    ok = (w > 0) & (np.abs(d).max(1, initial=0) > 0)
    lev = _levels(d[ok], ch[ok], w[ok], n0)
    nl, level, per = n0, 0, 8 if bands else 4
    while True:
        got = np.full((6 * nl * nl, per), np.nan, np.float32)
        bh.bh_stars_download(h, level, got.ctypes.data)
        S = lev[:, :3].sum(1) if bands else lev[:, 0]
        lit, s = S > 0, np.where(S > 0, S, 1.0)
        want = np.concatenate([lev[:, :3] if bands else np.stack([S, lev[:, 1] / s], 1),
                               lev[:, -2:] / s[:, None]], 1)
        assert not got[~lit].any() and not got[:, want.shape[1]:].any()
        # each level rounds its texels to FP32 (2^-24 relative) from the level below's
        np.testing.assert_allclose(got[:, :want.shape[1]][lit], want[lit],
                                   rtol=2.0 ** -23 * (level + 1), atol=2.0 ** -23 * (level + 1))
        if nl == 1:
            break
        q = lev.reshape(6, nl // 2, 2, nl // 2, 2, -1)
        up = 0.0
        for y in (0, 1):
            for x in (0, 1):
                c = q[:, :, y, :, x].copy()
                cs = c[..., :3].sum(-1) if bands else c[..., 0]
                c[..., -2] = 0.5 * (x * cs + c[..., -2])
                c[..., -1] = 0.5 * (y * cs + c[..., -1])
                up = up + c
        nl, level = nl // 2, level + 1
        lev = up.reshape(6 * nl * nl, -1)
    bh.bh_release_stars(h)


@pytest.mark.parametrize("n0,n,kind", [
    (1, 700, "plain"), (2, 3000, "plain"),  # one sorted texel a tile; tiles of one texel
    (16, 20000, "clustered"),               # texels found again from the stars
    (32, 60000, "plain"), (64, 20000, "plain"), (64, 300000, "clustered"),
    (1024, 1000000, "plain"),               # sorted tiles of few stars a texel
    (2048, 300000, "clustered")])           # bins of several tiles, some sorted
@pytest.mark.parametrize("bands", [False, True])
def test_dense_tiles_match_numpy(gpu_ctx, n0, n, kind, bands):
    """Tiles whose stars are sorted by texel and index before they are merged, among tiles whose
    stars are listed."""
    test_star_map_levels_match_numpy(gpu_ctx, n0, n, kind, bands)


@pytest.mark.parametrize("n0", [2, 16, 32, 64, 256])
@pytest.mark.parametrize("fmt", [bh.BH_TEXEL_FP16, bh.BH_TEXEL_FP32])
def test_every_star_is_found_by_a_frame(gpu_ctx, gpu_tables, orc, orc_tables, n0, fmt):
    """The occupancy bits (words that tiles share, guard words, paired rows): a frame of the
    whole map's stars against the oracle."""
    import torch
    field = scenes.star_field(6 * n0 * n0 // 3 + 4, 11)
    d, i, t = (torch.from_numpy(a).cuda() for a in (field.dirs, field.intensity,
                                                    field.temperature))
    h = bh.bh_build_stars(gpu_ctx, d.data_ptr(), i.data_ptr(), t.data_ptr(), len(field), n0,
                          fmt, bh.current_stream())
    cube = orc.cubemap(field, n0)
    for aim in ((0.3, 1.0), (2.6, 4.1)):
        v = scenes.small_static_view()
        v.width, v.height, v.fov_y = 61, 47, 1.9
        v.cam_rot = scenes.look_rotation(scenes.spherical_position(1.0, *aim))
        out = torch.full((47, 61, 4), -1.0, device="cuda")
        bh.bh_render(gpu_ctx, gpu_tables, bh.make_view(v, h), out.data_ptr(), None,
                     bh.current_stream())
        px = orc.render_quads(v, scenes.all_quads(61, 47), cube=cube, n0=n0, tables=orc_tables)
        px = px[(px["x"] < 61) & (px["y"] < 47) & (px["n_cross"] == 0) & (px["star_zeroed"] == 0)]
        g, o = out.cpu().numpy()[px["y"], px["x"], :3], px["rgb"]
        # the escape angle is FP32 (~2e-6 rad, pixels are 4e-2 rad) and FP16 positions are
        # within 2^-12 texel: tent weights move by less than 1e-3 of the brightest neighbour
        err = np.abs(g - o).max(1) / np.maximum(o.max(1), 1e-2 * o.max())
        assert np.percentile(err, 98) < 5e-3, float(np.percentile(err, 98))
    bh.bh_release_stars(h)


def _level0(h, n0):
    g = np.empty((6 * n0 * n0, 4), np.float32)
    bh.bh_stars_download(h, 0, g.ctypes.data)
    return g


@pytest.mark.parametrize("budget", [0, 4 << 30])
def test_maps_built_in_released_blocks(budget):
    """Maps built and released in turn by two threads on streams of their own, in blocks that
    earlier maps of other contents held, against maps of a fresh context; nothing stays counted."""
    import threading
    import torch
    n0, fields = 512, [scenes.star_field(n, 30 + n % 7) for n in (40000, 41000, 300, 39500)]
    dev = [[torch.from_numpy(a).cuda() for a in (f.dirs, f.intensity, f.temperature)]
           for f in fields]
    torch.cuda.synchronize()

    def build(ctx, k, stream):
        d, i, t = dev[k]
        return bh.bh_build_stars(ctx, d.data_ptr(), i.data_ptr(), t.data_ptr(), len(d), n0,
                                 bh.BH_TEXEL_FP16, stream.cuda_stream)
    ref = []
    for k in range(len(fields)):
        ctx = bh.bh_create(0, 0)
        ref.append(_level0(build(ctx, k, torch.cuda.Stream()), n0))
        bh.bh_destroy(ctx)
    ctx = bh.bh_create(0, budget)
    base, bad = bh.bh_bytes_in_use(ctx), []

    def work(first):
        s = torch.cuda.Stream()
        for r in range(12):
            k = (first + r) % len(fields)
            h = build(ctx, k, s)
            if not np.array_equal(_level0(h, n0), ref[k]):
                bad.append((first, r, k))
            bh.bh_release_stars(h)
    threads = [threading.Thread(target=work, args=(q,)) for q in (0, 2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    assert bh.bh_bytes_in_use(ctx) == base
    bh.bh_destroy(ctx)


def test_a_resident_map_is_found_without_scratch():
    """While a thread asks again and again for a map that is resident, another's allocations still
    find the budget's rest, which the scratch of a build would take."""
    import threading
    import torch
    n, n0 = 2_000_000, 64  # scratch of a build: 12 bytes a star and more
    f = scenes.star_field(n, 2)
    d, i, t = (torch.from_numpy(a).cuda() for a in (f.dirs, f.intensity, f.temperature))
    torch.cuda.synchronize()

    def build(ctx, stream=None):
        return bh.bh_build_stars(ctx, d.data_ptr(), i.data_ptr(), t.data_ptr(), n, n0,
                                 bh.BH_TEXEL_FP16, stream)
    probe = bh.bh_create(0, 0)
    build(probe)
    used = bh.bh_bytes_in_use(probe)
    bh.bh_destroy(probe)
    ctx = bh.bh_create(0, used + 40 * n)
    h, stop, failed = build(ctx), threading.Event(), []

    def ask():
        s = torch.cuda.Stream()
        while not stop.is_set():
            assert build(ctx, s.cuda_stream) == h
            bh.bh_release_stars(h)
    asking = threading.Thread(target=ask)
    asking.start()
    try:
        for _ in range(200):
            try:  # 2 x 32 MB of the 80
                bh.bh_release(bh.bh_bloom_create(ctx, 2 * 1600, 2 * 1250, 1))
            except bh.BhError as e:
                failed.append(e)
    finally:
        stop.set()
        asking.join()
        bh.bh_destroy(ctx)
    assert not failed, failed[0]


def test_trim_gives_kept_blocks_back():
    """A released pyramid's blocks stay with the context, and bh_trim gives them back."""
    import torch
    ctx = bh.bh_create(0, 0)
    try:
        start = torch.cuda.mem_get_info()[0]
        bh.bh_release(bh.bh_bloom_create(ctx, 8192, 4096, 1))  # 2 x 128 MiB
        kept = start - torch.cuda.mem_get_info()[0]
        bh.bh_trim(ctx)
        left = start - torch.cuda.mem_get_info()[0]
        assert kept >= 2 << 27 and left < 1 << 24, (kept, left)
    finally:
        bh.bh_destroy(ctx)


@pytest.mark.parametrize("fmt", [bh.BH_TEXEL_FP16, bh.BH_TEXEL_FP32])
def test_infinite_temperatures_stay_infinite(gpu_ctx, fmt):
    """A texel's temperature is the weighted mean of its stars', in every level: infinite when one
    of them is (a NaN would reach the image), and the others' texels are not touched."""
    import torch
    n0 = 4
    d = np.array([[1, 0.1, 0.1], [1, 0.1, 0.1], [1, -0.9, -0.9], [-1, 0.2, 0.3]], np.float32)
    inten = np.array([2.0, 1.0, 1.0, 3.0], np.float32)
    temp = np.array([np.inf, 5000.0, 4000.0, 6000.0], np.float32)
    dd, ii, tt = (torch.from_numpy(x).cuda() for x in (d, inten, temp))
    h = bh.bh_build_stars(gpu_ctx, dd.data_ptr(), ii.data_ptr(), tt.data_ptr(), len(d), n0, fmt,
                          bh.current_stream())
    for level in range(3):
        nl = n0 >> level
        got = np.empty((6, nl, nl, 4), np.float32)
        bh.bh_stars_download(h, level, got.ctypes.data)
        assert not np.isnan(got).any(), level
        assert np.isinf(got[0, ..., 1]).sum() == 1 and np.isfinite(got[1:]).all(), level
        assert got[1, ..., 1].max() == pytest.approx(6000.0, rel=2.0 ** -11)
        if level < 2:  # the finite star's own texel
            assert got[0, 0, 0, 1] == pytest.approx(4000.0, rel=2.0 ** -11)
    bh.bh_release_stars(h)


@pytest.mark.parametrize("n0,n", [(64, 3000), (64, 60000)])
def test_level0_quotients_are_the_rounded_division(gpu_ctx, n0, n):
    """FP32 texels are FP64 sums in star order and one FP64 division each: the same bits as numpy's
    (every product of two FP32 values is exact in FP64)."""
    import torch
    d, inten, temp = _field(n, n0, "clustered", 9)
    dd, ii, tt = (torch.from_numpy(x).cuda() for x in (d, inten, temp))
    h = bh.bh_build_stars(gpu_ctx, dd.data_ptr(), ii.data_ptr(), tt.data_ptr(), n, n0,
                          bh.BH_TEXEL_FP32, bh.current_stream())
    w = inten.astype(np.float64)
    ok = (w > 0) & (np.abs(d).max(1) > 0)
    lev = _levels(d[ok], np.stack([w, w * temp], 1)[ok], w[ok], n0)
    lit = lev[:, 0] > 0
    want = np.concatenate([lev[lit, :1], lev[lit, 1:] / lev[lit, :1]], 1).astype(np.float32)
    assert np.array_equal(_level0(h, n0)[lit], want)
    bh.bh_release_stars(h)
