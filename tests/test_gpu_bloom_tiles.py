"""The glare pass in each of its output tile shapes, at sizes around the lines between them: the
linear result against the oracle where that is quick, and the fused display encoding equal, code
for code, to the encoding of the linear result (the same arithmetic in other tiles)."""
import numpy as np
import pytest

from paper_2010_08735_amd import bh, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,levels", [
    (33, 31, 7), (31, 65, 1), (97, 95, 2), (959, 513, 7), (1025, 513, 9), (1023, 512, 6),
    (2049, 63, 3), (65, 2111, 16), (4161, 4159, 7), (8191, 2049, 8)])
def test_fused_display_equals_encoded_linear(gpu_ctx, orc, w, h, levels):
    import torch
    g = torch.Generator(device="cuda").manual_seed(w + 3 * h)
    img = torch.rand((h, w, 4), generator=g, device="cuda") ** 6 * 4.0
    lin, wt = torch.full_like(img, float("nan")), scenes.bloom_weights(levels)
    one, two = (torch.zeros((h, w), dtype=torch.int32, device="cuda") for _ in "ab")
    b, st = bh.bh_bloom_create(gpu_ctx, w, h, levels), bh.current_stream()
    bh.bh_bloom_apply_display(b, wt, 0.8, img.data_ptr(), one.data_ptr(), st)
    bh.bh_bloom_apply(b, wt, img.data_ptr(), lin.data_ptr(), st)
    bh.bh_tonemap(gpu_ctx, lin.data_ptr(), two.data_ptr(), w, h, 0.8, st)
    bh.bh_bloom_apply(b, wt, img.data_ptr(), img.data_ptr(), st)  # in place: the same bits
    torch.cuda.synchronize()
    assert torch.equal(one, two) and torch.equal(img, lin)
    bh.bh_bloom_release(b)
    if w * h < 1 << 21:
        g.manual_seed(w + 3 * h)
        src = (torch.rand((h, w, 4), generator=g, device="cuda") ** 6 * 4.0).cpu().numpy()
        ref = orc.bloom(src.astype(np.float64), levels,
                        np.asarray(wt, np.float32).astype(np.float64))
        # ~4 roundings of 2^-24 a level on sums of non-negative terms
        assert np.abs(lin.cpu().numpy() - ref).max() <= 4 * (levels + 1) * 2.0 ** -23 * ref.max()


@pytest.mark.parametrize("w,h,levels", [(2047, 1024, 7), (2049, 1024, 7), (1937, 1087, 8)])
def test_around_one_round_of_workgroups(gpu_ctx, orc, w, h, levels):
    """512 and 528 tiles of 64 x 64: the line between the display shapes."""
    test_fused_display_equals_encoded_linear(gpu_ctx, orc, w, h, levels)
