"""One infinity, NaN or huge value in an input of the 16-bit matrix units.

Pixels out of its reach keep the values that they have without it.  One update
moves an input value by two kernel radii at most; beyond that the result is
compared with the float32 units' on the same input without the value.  Both are
within 5e-6 · T · V of the exact value (the derivation stands in
test_gpu_range.py), so within twice that of each other.  Within reach the oracle
says what comes out: a blurred estimate that is NaN counts as below the guard
(ratio 1).  (An infinite one does not: φ / ∞ is NaN here and 0 there, so infinities
are compared out of reach only, and so is 1e30 with kernels that are sums of
rank-one terms, which cancel.)
"""
import numpy as np
import pytest

import oracle
from synthetic import gaussian_psf

pytestmark = pytest.mark.gpu

SIM, SEQ = "simultaneous", "sequential"
CASES = [
    # (Z, X, K, views, update, rank, normalize)
    (96, 128, 31, 2, SIM, 1, False),
    (100, 131, 9, 2, SIM, 1, False),
    (90, 150, 21, 1, SIM, 1, False),
    (97, 165, 21, 3, SEQ, 1, False),
    (120, 230, 41, 2, SEQ, 1, False),
    (96, 132, 21, 2, SIM, 1, True),
    (96, 130, 15, 1, SIM, 1, True),
    (100, 132, 21, 2, SIM, 2, False),
    (100, 131, 41, 1, SEQ, 2, False),
]


def _check(case, value, where, full=False):
    import torch

    from paper_1503_07998_amd import Deconvolver, api

    print(f"[case] nonfinite {value} in {where}: {case} full={full}", flush=True)
    Z, X, k, V, update, rank, normalize = case
    rng = np.random.default_rng(Z * 1009 + X + k)
    psfs = []
    for _ in range(V):
        p = gaussian_psf(k, 0.1 * k, 0.2 * k)
        for _ in range(rank - 1):
            p = p + 0.3 * np.roll(gaussian_psf(k, 0.2 * k, 0.1 * k), (2, -1), (0, 1))
        if full:
            p = p * (1.0 + 0.2 * rng.uniform(-1.0, 1.0, p.shape))
        psfs.append((p / p.sum()).astype(np.float32))
    obs = [rng.uniform(50.0, 900.0, (1, Z, X)).astype(np.float32) for _ in range(V)]
    est = rng.uniform(50.0, 900.0, (1, Z, X)).astype(np.float32)
    kw = dict(update=update, layout="planes_yzx", normalize=normalize)
    d = Deconvolver(V, Z, X, 0)
    for v, p in enumerate(psfs):
        d.set_psf(v, p)

    def run(float32):
        api.mvd_set_float32_units(d.ctx, float32)
        out = d.run([torch.from_numpy(o).to("cuda:0") for o in obs], iters=1, init="given",
                    est=torch.from_numpy(est).to("cuda:0"), **kw)
        return out.cpu().numpy()[0].astype(np.float64)

    clean, clean16 = run(True), run(False)
    assert not np.array_equal(clean, clean16), "both runs took the same units"
    at = (Z // 2 + 3, X // 2 - 5)
    (est if where == "psi" else obs[0])[0][at] = value
    got = run(False)
    d.close()
    zz, xx = np.mgrid[:Z, :X]
    away = np.maximum(abs(zz - at[0]), abs(xx - at[1]))
    far = away > 2 * (k // 2) * (V if update == SEQ else 1)
    rtol = 2 * 5e-6 * V
    np.testing.assert_allclose(got[far], clean[far], rtol=rtol)
    assert far.any() or value != value
    if value != value or (value == 1e30 and rank == 1 and not full):
        ref = oracle.deconvolve(obs, [p.astype(np.float64) for p in psfs], 1, init="given", init_given=est, **kw)[0]
        assert np.array_equal(np.isnan(got), np.isnan(ref)), np.isnan(got).sum()
        np.testing.assert_allclose(got, ref, rtol=rtol)


@pytest.mark.parametrize("value", [np.inf, np.nan, 1e30])
@pytest.mark.parametrize("case", CASES, ids=[f"n{i}" for i in range(len(CASES))])
def test_one_value_stays_in_its_reach(case, value):
    _check(case, value, "psi")


@pytest.mark.parametrize("case", [CASES[1], CASES[2]], ids=["n1", "n2"])
def test_an_infinite_observation_stays_in_its_reach(case):
    _check(case, np.inf, "obs")
