"""Host planner of the wave-tile passes: strips and segments cover every pixel of a
plane once, segments are whole 32-row steps, and what a work-group needs fits its LDS.
The kernels index with these numbers alone."""
import ctypes

import pytest

from paper_1503_07998_amd import _native as N
from paper_1503_07998_amd import api

SIZES = [(1, 1, 1), (1, 32, 32), (3, 33, 31), (61, 203, 331), (512, 512, 512), (16, 2048, 2048), (1, 4095, 257),
         (7, 31, 4096), (1953, 128, 128), (1, 97, 260), (2, 513, 272)]


def _plan(ctx, planes, k, views, fused):
    f = N.lib().mvd_internal_march_plan
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_void_p] + [ctypes.c_int] * 4 + [ctypes.POINTER(ctypes.c_long)]
    out = (ctypes.c_long * 7)()
    return f(ctx, planes, k, views, fused, out), list(out)


@pytest.mark.parametrize("planes,z,x", SIZES)
@pytest.mark.parametrize("k,views,fused", [(9, 1, 0), (31, 2, 0), (41, 1, 0), (63, 1, 0), (15, 2, 1), (31, 2, 1)])
def test_tiles_cover_every_pixel_once(planes, z, x, k, views, fused):
    ctx = api.mvd_create(2, z, x, N.MVD_DEVICE_NONE)
    try:
        st, (kb, zseg, nseg, nstrip, pairs, ntiles, lds) = _plan(ctx, planes, k, views, fused)
    finally:
        api.mvd_destroy(ctx)
    assert st == 0 and kb >= k
    assert zseg >= 32 and zseg % 32 == 0
    rows = [(s * zseg, min((s + 1) * zseg, z)) for s in range(nseg)]
    assert rows[0][0] == 0 and rows[-1][1] == z and all(a < b for a, b in rows)
    w = 32 * pairs
    assert 1 <= pairs <= 8 and nstrip * w >= x and (nstrip - 1) * w < x
    assert ntiles == planes * nseg * nstrip
    assert 0 < lds <= 160 * 1024


@pytest.mark.parametrize("k,views,fused", [(41, 2, 0), (41, 2, 1), (65, 1, 0)])
def test_forms_that_do_not_exist_are_refused(k, views, fused):
    ctx = api.mvd_create(2, 64, 64, N.MVD_DEVICE_NONE)
    st, _ = _plan(ctx, 1, k, views, fused)
    api.mvd_destroy(ctx)
    assert st == N.MVD_ERR_UNSUPPORTED


SIM, SEQ = 0, 1


@pytest.mark.parametrize("update,k,z,x,tiles", [
    # few planes of these take up to three times as long on the float32 units, many
    # of them at most a quarter less: wave tiles whatever the plane's size
    (SIM, 9, 512, 384, True), (SIM, 15, 104, 640, True), (SIM, 15, 512, 512, True), (SIM, 11, 512, 1024, True),
    (SEQ, 15, 104, 640, True), (SEQ, 11, 512, 384, True), (SEQ, 41, 512, 512, True), (SEQ, 41, 128, 480, True),
    # one input per launch on rows that fill a power-of-two work-group
    (SEQ, 11, 512, 512, False), (SEQ, 21, 128, 480, False), (SEQ, 41, 256, 256, False),
    (SEQ, 31, 512, 512, True), (SIM, 31, 512, 512, True), (SIM, 41, 512, 512, False)])
def test_units_do_not_depend_on_the_plane_s_size(update, k, z, x, tiles):
    import numpy as np

    f = N.lib().mvd_internal_wave_tiles
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int]
    for rows in (z, 2 * z, 64):
        d = api.Deconvolver(2, rows, x, N.MVD_DEVICE_NONE)
        for v in range(2):
            d.set_psf(v, np.full((k, k), 1.0 / (k * k), np.float32))
        got = f(d.ctx, N.BOUNDARY["zero"], update)
        d.close()
        assert got == int(tiles)
