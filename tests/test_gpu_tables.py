"""Table precompute at the edges of its work split: the smallest tables, columns and rows that
do not fill a wave, more rows than steps in a chunk, step counts that end inside, at and past a
block of steps, narrow and wide FP64 bands, against quadrature at the texel centres."""
import numpy as np
import pytest

from paper_2010_08735_amd import bh

pytestmark = pytest.mark.gpu

B, S, A = bh.BH_TAB_FP64_BAND, bh.BH_TAB_FP32, bh.BH_TAB_FP64_ALL


@pytest.mark.parametrize("d_n,u_ne,u_nphi,prec,band,step", [
    (8, 4, 4, B, 0.05, 0.0), (10, 5, 7, A, 0.0, 2e-3), (130, 65, 33, B, 0.05, 1.7e-3),
    (66, 67, 257, B, 0.3, 2e-3), (1026, 16, 300, B, 0.05, 2e-3), (64, 64, 32, A, 0.0, 5e-4),
    (64, 64, 32, S, 0.0, 2e-3), (64, 31, 65, B, 0.0, 2e-3), (64, 31, 65, B, 1e-4, 2e-3)])
def test_tables_at_the_edges_of_their_split(gpu_ctx, orc, d_n, u_ne, u_nphi, prec, band, step):
    ref = orc.Tables(d_n, u_ne, u_nphi, time=True)
    t = bh.bh_precompute_tables(gpu_ctx, d_n, u_ne, u_nphi, prec, band, step)
    D, Dt = np.full((2, d_n, d_n), np.nan, np.float32)
    U, Ut = np.full((2, u_nphi, u_ne), np.nan, np.float32)
    bh.bh_tables_download(t, D.ctypes.data, U.ctypes.data)
    bh.bh_tables_download_time(t, Dt.ctypes.data, Ut.ctypes.data)
    bh.bh_release_tables(t)
    # FP64 near the photon sphere: the bound of the 512 x 512 tables.  Without it, the FP32
    # rounding of e^2 near mu (mu 2^-24 ~ 9e-9) over the distance of the outermost columns from
    # mu (mu exp(-12.5) ~ 5.5e-7) moves the deflection by 1.6e-2 rad.
    tol = 1e-6 if band >= 0.05 or prec == A else 2e-2
    for name, got, want in (("D", D, ref.D), ("Dt", Dt, ref.Dt), ("U", U, ref.U),
                            ("Ut", Ut, ref.Ut)):
        want = np.asarray(want).reshape(got.shape)
        assert np.isfinite(got).all(), name
        err = np.abs(got - want) / np.maximum(1.0, np.abs(want))
        assert err.max() < tol, (name, float(err.max()),
                                 [int(v) for v in np.unravel_index(err.argmax(), err.shape)])


def test_every_row_is_written_at_small_steps(gpu_ctx, orc):
    """Steps below 5e-6 take the longest columns past 4e6 steps: their last rows were left as the
    memory was.  Tolerance: the default step's 1e-6, and 14.7 rad at the FP32 step's rounding."""
    ref = orc.Tables(64, 8, 8, time=True)
    t = bh.bh_precompute_tables(gpu_ctx, 64, 8, 8, B, 0.05, 3e-6)
    D, Dt = np.full((2, 64, 64), np.nan, np.float32)
    U, Ut = np.full((2, 8, 8), np.nan, np.float32)
    bh.bh_tables_download(t, D.ctypes.data, U.ctypes.data)
    bh.bh_tables_download_time(t, Dt.ctypes.data, Ut.ctypes.data)
    bh.bh_release_tables(t)
    for name, got, want in (("D", D, ref.D), ("Dt", Dt, ref.Dt), ("U", U, ref.U),
                            ("Ut", Ut, ref.Ut)):
        want = np.asarray(want).reshape(got.shape)
        err = np.abs(got - want) / np.maximum(1.0, np.abs(want))
        assert err.max() < 1e-6 + 14.7 * 2.0 ** -24, (name, float(err.max()))
