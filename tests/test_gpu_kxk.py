"""The K×K passes on the 16-bit matrix units (kernels of up to 33 columns that are no
short sum of rank-one terms): the edges of their 64×64 tiles and of planes smaller
than one, very different values beside each other, and values that are not finite.
Every case checks that its kernels do run as K×K passes.

Tolerance.  A convolution's products are off by at most 3·2⁻²⁴ (parts left out), and
its sum is rounded three times per tap row at most: with a quotient and the update
less than 2e-6 + 2.4e-7 · kz per view and iteration, of the largest value, or of the
pixel's own where every term is ≥ 0.
"""
import numpy as np
import pytest

import oracle
from test_gpu_nonfinite import _check
from test_gpu_range import _errors, _problem

pytestmark = pytest.mark.gpu

Z0, PER, SIM, SEQ = "zero", "periodic", "simultaneous", "sequential"


def _bound(kz, T, V):
    return (2e-6 + 2.4e-7 * kz) * T * V


EDGES = [
    # (Y, Z, X, kernel shape, boundary, update, T)
    (2, 1, 130, (63, 9), Z0, SIM, 2),
    (2, 1, 1, (9, 9), Z0, SEQ, 3),
    (1, 130, 1, (7, 31), Z0, SIM, 2),
    (2, 70, 61, (23, 23), Z0, SIM, 2),
    (1, 66, 129, (63, 33), Z0, SEQ, 1),
    (1, 383, 449, (7, 7), Z0, SIM, 2),     # 48 tiles
    (1, 383, 448, (7, 7), Z0, SIM, 2),     # 42 tiles: the float32 form
    (2, 64, 64, (31, 31), PER, SIM, 2),
    (1, 20, 33, (29, 33), PER, SEQ, 1),
]


@pytest.mark.parametrize("case", EDGES, ids=[f"e{i}" for i in range(len(EDGES))])
def test_edges_match_oracle(case):
    import torch

    from paper_1503_07998_amd import Deconvolver, api

    Y, Z, X, (kz, kx), boundary, update, T = case
    print(f"[case] K×K edges {case}", flush=True)
    rng = np.random.default_rng(Z * 1009 + X)
    V = 2
    psfs = []
    for _ in range(V):
        p = rng.uniform(0.05, 1.0, (kz, kx))
        psfs.append((p / p.sum()).astype(np.float32))
    obs = [rng.uniform(20.0, 2000.0, (Y, Z, X)).astype(np.float32) for _ in range(V)]
    d = Deconvolver(V, Z, X, 0)
    for v in range(V):
        d.set_psf(v, psfs[v])
    assert [api.mvd_psf_info(d.ctx, v) for v in range(V)] == [(0, 0)] * V
    kw = dict(update=update, boundary=boundary, layout="planes_yzx")
    got = d.run([torch.from_numpy(o).to("cuda:0") for o in obs], iters=T, **kw).cpu().numpy().astype(np.float64)
    d.close()
    ref = oracle.deconvolve(obs, [p.astype(np.float64) for p in psfs], T, **kw)
    assert np.all(np.isfinite(got))
    err = np.abs(got - ref).max() / np.abs(ref).max()
    assert err <= _bound(kz, T, V), err


RANGE = [
    # (Z, X, K, σx, σz, cropped, update)
    (128, 128, 15, 1.2, 3.0, "one", SIM),
    (128, 128, 21, 1.5, 4.0, "one", SIM),
    (120, 131, 31, 1.5, 6.0, "both", SIM),
    (100, 134, 21, 1.5, 4.0, "both", SEQ),
]


@pytest.mark.parametrize("case", RANGE, ids=[f"r{i}" for i in range(len(RANGE))])
def test_cropped_views_keep_every_pixel(case):
    Z, X, k, sx, sz, cropped, update = case
    print(f"[case] K×K range {case}", flush=True)
    T, V = 10, 2
    psfs, obs = _problem(Z, X, k, sx, sz, V, cropped, 1, full=True)
    err, info = _errors(psfs, obs, T, update)
    assert info == [(0, 0)] * V
    assert err[0] <= _bound(k, T, V), err


@pytest.mark.parametrize("value", [np.inf, np.nan, 1e30])
@pytest.mark.parametrize("case", [(96, 128, 21, 2, SIM, 1, False), (100, 131, 9, 2, SEQ, 1, False)], ids=["v", "e"])
def test_one_value_stays_in_its_reach(case, value):
    _check(case, value, "psi", full=True)
