"""Values of very different size beside each other on the 16-bit matrix units.

Where one view sees nothing over a region (a crop, a shadow, the padding after a
registration) and the other does, ψ falls towards zero there, b passes through
the guard and ratios of 1e8 stand beside ratios near 1.  A pixel's result must not
depend on how large its neighbours' values are.

Tolerance.  Every term of a convolution is ≥ 0, so rounding errors are relative to
the pixel itself: a 1D convolution of split operands is off by the products left
out (3·2⁻²⁴) and at most a dozen roundings of 2⁻²⁴, less than 1e-6; four of them, a
quotient and an update per view and iteration are less than 5e-6, and T iterations
of V views add up to 5e-6 · T · V of the pixel's own value (ψ > 1).
"""
import numpy as np
import pytest

import oracle
from synthetic import gaussian_psf

pytestmark = pytest.mark.gpu

SIM, SEQ = "simultaneous", "sequential"
RANGE = [
    # (Z, X, K, σx, σz, views, cropped, update, rank)
    (128, 128, 15, 1.2, 3.0, 2, "one", SIM, 1),
    (128, 128, 21, 1.5, 4.0, 2, "one", SIM, 1),
    (128, 128, 31, 1.5, 6.0, 2, "one", SIM, 1),
    (120, 131, 31, 1.5, 6.0, 2, "both", SIM, 1),
    (100, 134, 25, 1.5, 5.0, 2, "one", SEQ, 1),
    (100, 130, 41, 2.0, 7.0, 2, "both", SEQ, 1),
    (110, 128, 21, 1.5, 4.0, 2, "both", SIM, 2),
]


def _problem(Z, X, k, sx, sz, V, cropped, rank, full=False):
    rng = np.random.default_rng(Z * 1009 + X + k)
    zz, xx = np.mgrid[:Z, :X]
    truth = np.full((2, Z, X), 150.0)
    for y in range(2):
        for _ in range(25):
            c, s, a = rng.uniform(0, [Z, X]), rng.uniform(2.0, 4.0), rng.uniform(200.0, 1000.0)
            truth[y] += a * np.exp(-((zz - c[0]) ** 2 + (xx - c[1]) ** 2) / (2 * s * s))
    psfs, obs = [], []
    for v in range(V):
        p = gaussian_psf(k, *((sx, sz) if v % 2 == 0 else (sz, sx)))
        for _ in range(rank - 1):
            p = p + 0.3 * np.roll(gaussian_psf(k, 2.0 * sx, 0.5 * sz), (2, -1), (0, 1))
        if full:
            p = p * (1.0 + 0.2 * rng.uniform(-1.0, 1.0, p.shape))
        p = (p / p.sum()).astype(np.float32)
        o = rng.poisson(np.maximum(np.stack([oracle.conv2d(t, p.astype(np.float64)) for t in truth]), 100.0))
        if v == 0:
            o[:, :, :60] = 0
        elif cropped == "both":
            o[:, :37] = 0
        psfs.append(p)
        obs.append(o.astype(np.float32))
    return psfs, obs


def _errors(psfs, obs, T, update):
    """Largest relative error where ψ > 1 on the 16-bit and on the float32 units."""
    import torch

    from paper_1503_07998_amd import Deconvolver, api

    _, Z, X = obs[0].shape
    d = Deconvolver(len(obs), Z, X, 0)
    for v, p in enumerate(psfs):
        d.set_psf(v, p)
    dev = [torch.from_numpy(o).to("cuda:0") for o in obs]
    kw = dict(iters=T, update=update, layout="planes_yzx")
    split = d.run(dev, **kw).cpu().numpy().astype(np.float64)
    api.mvd_set_float32_units(d.ctx)
    plain = d.run(dev, **kw).cpu().numpy().astype(np.float64)
    info = [api.mvd_psf_info(d.ctx, v) for v in range(len(obs))]
    d.close()
    assert not np.array_equal(split, plain), "both runs took the same units"
    ref = oracle.deconvolve(obs, [p.astype(np.float64) for p in psfs], T, update=update, layout="planes_yzx")
    at = ref > 1.0
    assert at.sum() > ref.size // 3
    err = [float((np.abs(x - ref)[at] / ref[at]).max()) for x in (split, plain)]
    print(f"[result] relative error 16-bit units {err[0]:.2e}, float32 units {err[1]:.2e}", flush=True)
    return err, info


@pytest.mark.parametrize("case", RANGE, ids=[f"r{i}" for i in range(len(RANGE))])
def test_cropped_views_keep_every_pixel(case):
    Z, X, k, sx, sz, V, cropped, update, rank = case
    print(f"[case] range Z={Z} X={X} K={k} V={V} cropped={cropped} {update} rank={rank}", flush=True)
    T = 10
    psfs, obs = _problem(Z, X, k, sx, sz, V, cropped, rank)
    err, _ = _errors(psfs, obs, T, update)
    assert err[0] <= 5e-6 * T * V, err
