"""The form an untuned batch takes, and the queue's float32 tiles.

The queue runs wave tiles or, where the plain runs do (short kernels, the periodic
boundary, contexts on the float32 units, rows that suit them), the float32 passes in
tiles of half a work-group's threads; rows wider than that are strips with halo
columns.  Every volume must equal its plain run bitwise.
"""
import numpy as np
import pytest

from synthetic import gaussian_psf

pytestmark = pytest.mark.gpu

SIM, SEQ = "simultaneous", "sequential"


def _item(nz, nx, ny, views, k, iters, update, seed, boundary="zero", float32=False, dtype="f32"):
    import torch

    from paper_1503_07998_amd import Deconvolver, api

    rng = np.random.default_rng(seed)
    d = Deconvolver(views, nz, nx, 0)
    for v in range(views):
        d.set_psf(v, gaussian_psf(k, 0.5 + 0.08 * k, 0.5 + 0.15 * k).astype(np.float32))
    if float32:
        api.mvd_set_float32_units(d.ctx)
    obs = [torch.from_numpy(rng.uniform(50.0, 3000.0, (ny, nz, nx)).astype(np.uint16 if dtype == "u16" else np.float32))
           .to("cuda:0") for _ in range(views)]
    run = api.make_run(ny, iters, update=update, boundary=boundary, obs_dtype=dtype, layout="planes_yzx")
    nb = api.mvd_workspace_bytes(d.ctx, run)
    ws = torch.empty(nb + 256, dtype=torch.uint8, device="cuda:0")
    run.workspace = (ws.data_ptr() + 255) // 256 * 256
    run.workspace_bytes = nb
    est = torch.empty((ny, nz, nx), device="cuda:0")
    api.mvd_deconvolve_planes(d.ctx, obs, est, run)
    torch.cuda.synchronize()
    want = est.cpu().numpy()
    est.zero_()
    return dict(ctx=d, obs=obs, est=est, run=run, ws=ws, want=want)


def _check(items, persistent):
    import torch

    from paper_1503_07998_amd import api

    b = api.Batch([(i["ctx"].ctx, i["obs"], i["est"], i["run"]) for i in items])
    assert b.info()["persistent"] == persistent, b.info()
    for _ in range(2):
        b.launch()
        b.wait()
        torch.cuda.synchronize()
        for n, i in enumerate(items):
            assert np.array_equal(i["est"].cpu().numpy(), i["want"]), f"item {n}"
            i["est"].zero_()
    b.close()
    for i in items:
        i["ctx"].close()


FLOAT32 = [
    # (nz, nx, ny, views, k, iters, update, boundary, dtype)
    [(40, 264, 2, 2, 11, 3, SEQ, "zero", "f32"), (33, 512, 2, 1, 15, 2, SIM, "zero", "u16")],
    [(20, 1000, 1, 2, 21, 2, SIM, "zero", "f32"), (70, 256, 2, 3, 31, 2, SEQ, "zero", "f32")],
    [(50, 520, 1, 2, 41, 2, SEQ, "zero", "u16"), (45, 48, 3, 2, 21, 2, SIM, "periodic", "f32")],
]


@pytest.mark.parametrize("case", FLOAT32, ids=["a", "b", "c"])
def test_queue_on_float32_tiles(case):
    print(f"[case] queue, float32 tiles {case}", flush=True)
    _check([_item(*c[:7], seed=n, boundary=c[7], dtype=c[8], float32=True) for n, c in enumerate(case)], True)


def test_queue_on_float32_tiles_by_the_rule():
    """Sequential 11 taps on whole rows of 512 columns: float32 passes without being asked."""
    print("[case] queue, float32 tiles chosen by size", flush=True)
    _check([_item(64, 512, 2, 2, 11, 2, SEQ, seed=3), _item(24, 64, 2, 2, 31, 2, SIM, seed=4)], True)


@pytest.mark.parametrize("float32", [False, True])
def test_few_large_volumes_run_as_a_graph(float32):
    print(f"[case] batch of three volumes of 0.5 Mvoxel, float32={float32}", flush=True)
    _check([_item(128, 256, 16, 2, 21, 2, SEQ, seed=n, float32=float32) for n in range(3)], False)


def test_many_small_volumes_stay_in_the_queue():
    print("[case] batch of 20 volumes, 1.3 Mvoxel", flush=True)
    _check([_item(64, 128, 8, 2, 15, 2, SIM, seed=n) for n in range(20)], True)
