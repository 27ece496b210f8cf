"""The fused iteration where it is chosen by itself, in batches of planes copied from
the host, and on the float32 units at every kernel size that it is compiled for.
It must equal the two-launch form bitwise; the launch timings say which one ran.
"""
import ctypes

import numpy as np
import pytest

from synthetic import gaussian_psf

pytestmark = pytest.mark.gpu


def _tune(spec):
    from paper_1503_07998_amd import _native as N

    lib = N.lib()
    lib.mvd_internal_set_tune.restype = ctypes.c_int
    lib.mvd_internal_set_tune.argtypes = [ctypes.c_char_p]
    lib.mvd_internal_set_tune(spec.encode() if spec is not None else None)


def _context(Z, X, k, float32=False):
    from paper_1503_07998_amd import Deconvolver, api

    d = Deconvolver(2, Z, X, 0)
    for v, s in enumerate([(1.3, 0.4 + 0.15 * k), (0.4 + 0.15 * k, 0.9)]):
        d.set_psf(v, gaussian_psf(k, *s).astype(np.float32))
    if float32:
        api.mvd_set_float32_units(d.ctx)
    return d


def _run(d, obs, iters, dtype, est=None, spec=None):
    """(ψ^T, fused launches, forward launches) of stacks [Z][Y][X] on the device."""
    import torch

    from paper_1503_07998_amd import api

    Z, Y, X = obs[0].shape
    given = est is not None
    est = torch.empty((Y, Z, X), device="cuda:0") if est is None else est.clone()
    _tune(spec)
    try:
        run = api.make_run(Y, iters, obs_dtype=dtype, timing=True, init="given" if given else "mean")
        nb = api.mvd_workspace_bytes(d.ctx, run)
        ws = torch.empty(nb + 256, dtype=torch.uint8, device="cuda:0")
        run.workspace = (ws.data_ptr() + 255) // 256 * 256
        run.workspace_bytes = nb
        api.mvd_get_timing(d.ctx, reset=True)
        api.mvd_deconvolve_planes(d.ctx, obs, est, run)
        torch.cuda.synchronize()
        tim = api.mvd_get_timing(d.ctx, reset=True)
    finally:
        _tune(None)
    return est, tim["fused"][0], tim["forward"][0]


def _stacks(Z, Y, X, dtype, seed):
    import torch

    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    out = [torch.rand((Z, Y, X), generator=g, device="cuda:0") * 3000 + 50 for _ in range(2)]
    return [o.to(torch.int32).to(torch.uint16) for o in out] if dtype == "u16" else out


@pytest.mark.parametrize("k,Z,Y,X", [(11, 33, 3, 264), (15, 64, 2, 136), (21, 50, 2, 512), (31, 70, 2, 520)])
def test_fused_on_the_float32_units(k, Z, Y, X):
    import torch

    print(f"[case] fused, float32 units K={k} Z={Z} Y={Y} X={X}", flush=True)
    d = _context(Z, X, k, float32=True)
    obs = _stacks(Z, Y, X, "u16", k)
    a, nf, _ = _run(d, obs, 3, "u16", spec="fused=1")
    b, n0, fw = _run(d, obs, 3, "u16", spec="fused=0")
    d.close()
    assert nf == 3 and n0 == 0 and fw == 3
    assert torch.equal(a, b)


def test_large_volumes_choose_the_fused_form():
    """32 Mvoxel of uint16 in two views; with ψ^0 given or float32 observations, which
    may hold infinities or NaN, two launches; in batches from the host as in one run."""
    import torch

    from paper_1503_07998_amd import api

    Z, Y, X, T = 512, 128, 512, 3
    print(f"[case] fused by size Z={Z} Y={Y} X={X}", flush=True)
    d = _context(Z, X, 21)
    obs = _stacks(Z, Y, X, "u16", 5)
    a, nf, fw = _run(d, obs, T, "u16")
    assert nf == T and fw == 0
    b, n0, _ = _run(d, obs, T, "u16", spec="fused=0")
    assert n0 == 0 and torch.equal(a, b)
    _, nf, fw = _run(d, obs, 1, "u16", est=a)
    assert nf == 0 and fw == 1
    host = [torch.empty(o.shape, dtype=torch.uint16, pin_memory=True) for o in obs]
    for h, o in zip(host, obs):
        h.copy_(o)
    run = api.make_run(Y, T, obs_dtype="u16")
    batch = 120   # the first batch is large enough, the second of 8 planes is not
    nb = api.mvd_stream_workspace_bytes(d.ctx, run, batch, False)
    ws = torch.empty(nb + 256, dtype=torch.uint8, device="cuda:0")
    run.workspace = (ws.data_ptr() + 255) // 256 * 256
    run.workspace_bytes = nb
    b.zero_()
    api.mvd_deconvolve_stream(d.ctx, host, b, run, batch)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    del host, ws, b
    obs = [o.to(torch.int32).float() for o in obs]
    c, nf, fw = _run(d, obs, T, "f32")
    d.close()
    assert nf == 0 and fw == T and torch.equal(a, c)
