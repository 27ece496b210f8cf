"""Strips whose width is no multiple of 4, on the float32 units.

The row pass of a strip with halo columns forms 4 outputs at a time; past the last
input column of a ragged strip it meets up to 3 LDS columns with zero taps.  What an
earlier work-group left there must not reach the outputs.  A run on infinite
observations first leaves infinities (zero times which is NaN) in the LDS of every
compute unit: its ratios are infinite, and so are its back-projections.

Tolerance.  Every term is ≥ 0, so rounding errors are relative to the pixel itself.
A 1D convolution of K float32 taps is off by at most (K + 1) · 2⁻²⁴; four of them, a
quotient and an update with a few roundings each are (4 K + 16) · 2⁻²⁴ per view and
iteration, and the two errors of a sequential or simultaneous chain add up over T
iterations of V views.  Sums of rank-one terms have terms of either sign, which
cancel: their largest term may exceed the sum, so twice that.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SIM, SEQ = "simultaneous", "sequential"
CASES = [
    # (Z, X, K, views, update, boundary, rank)
    (5, 17, 31, 2, SEQ, "periodic", 2),
    (21, 57, 31, 4, SEQ, "periodic", 1),
    (33, 30, 9, 2, SIM, "periodic", 1),
    (20, 35, 41, 1, SIM, "periodic", 1),
    (12, 99, 63, 2, SIM, "periodic", 1),
    (40, 530, 63, 2, SEQ, "zero", 1),     # last strip 258 columns
    (24, 1030, 15, 2, SIM, "zero", 1),    # last strip 510 columns
]


@pytest.mark.parametrize("case", CASES, ids=[f"s{i}" for i in range(len(CASES))])
def test_earlier_values_stay_out(case):
    import torch

    from paper_1503_07998_amd import Deconvolver, api

    print(f"[case] strip tails {case}", flush=True)
    Z, X, k, V, update, boundary, rank = case
    Y, T = 2, 1
    rng = np.random.default_rng(Z * 1009 + X + k)
    psfs = []
    for _ in range(V):
        p = sum(np.outer(rng.uniform(0.05, 1.0, k), rng.uniform(0.05, 1.0, k)) for _ in range(rank))
        psfs.append((p / p.sum()).astype(np.float32))
    obs = [rng.uniform(50.0, 900.0, (Y, Z, X)).astype(np.float32) for _ in range(V)]

    d = Deconvolver(V, Z, X, 0)
    for v, p in enumerate(psfs):
        d.set_psf(v, p)
    api.mvd_set_float32_units(d.ctx, True)
    dev = [torch.from_numpy(o).to("cuda:0") for o in obs]

    # whole rows of 1000 columns: about 70 KB of LDS per work-group and pass
    dirty = Deconvolver(1, 64, 1000, 0)
    dirty.set_psf(0, np.full((31, 31), 1.0 / 961.0, np.float32))
    api.mvd_set_float32_units(dirty.ctx, True)
    inf = torch.full((256, 64, 1000), float("inf"), device="cuda:0")
    one = torch.ones((256, 64, 1000), device="cuda:0")
    dirty.run([inf], iters=1, init="given", est=one, layout="planes_yzx")
    got = d.run(dev, iters=T, update=update, boundary=boundary, layout="planes_yzx").cpu().numpy()
    dirty.close()
    d.close()

    ref = oracle.deconvolve(obs, [p.astype(np.float64) for p in psfs], T, update=update, boundary=boundary,
                            layout="planes_yzx")
    assert np.isfinite(got).all(), f"{(~np.isfinite(got)).sum()} values are not finite"
    rtol = (4 * k + 16) * 2.0 ** -24 * T * V * (2 if rank > 1 else 1)
    np.testing.assert_allclose(got, ref, rtol=rtol)
