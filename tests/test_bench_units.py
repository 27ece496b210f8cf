"""The bench's roofline entry names the kernel family that ran: a traffic record of
one family is never used for another, and the wave tiles' ceiling is that of the
16-bit matrix units."""
import json
import os

import numpy as np
import pytest

import bench
from paper_1503_07998_amd import Deconvolver, api
from paper_1503_07998_amd import _native as N
from synthetic import CONFIGS, gaussian_psf

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_kernel_families():
    assert bench.kernel_family("void mvd::march::fused_kernel<1>(mvd::MarchFusedArgs)") == "tiles"
    assert bench.kernel_family("void mvd::sepk::fused_kernel<31, 1>(mvd::FusedArgs)") == "fused"
    assert bench.kernel_family("void mvd::sepk::sep_forward_kernel<31, 1, 2, 4, 5, 1>(mvd::SepPassArgs)") == "sep"
    assert bench.kernel_family("mvd::(anonymous namespace)::copy_kernel(float const*, float*, unsigned long)") is None


@pytest.mark.parametrize("kind", ["forward", "backward", "fused"])
@pytest.mark.parametrize("tiles", [False, True])
def test_traffic_comes_from_the_family_that_ran(kind, tiles):
    rec = json.load(open(os.path.join(ROOT, "profiles", "sep_passes_vol512_traffic.json")))
    family = bench.pass_family(kind, tiles)
    got = bench.measured_traffic("vol512", kind, tiles)
    if rec["code_sha256"].get(family) != bench.pass_code_hash(family):
        assert got is None
    elif got is not None:
        assert bench.kernel_family(got["instance"]) == family
    # whatever the record holds, the default run's dominant kernel is not another family's
    spec = CONFIGS["vol512"]
    b, f, _, fm = bench.step_work_split(spec, kind, spec.n_planes * spec.n_z * spec.n_x, 1)
    r = bench.roofline(spec, {kind: dict(launches=10, avg_ms=1.0, bytes=b, flops=f, flops_valu=0.0, flops_mfma=fm)},
                       tiles=tiles)
    assert ("march::" in r["kernel"]) == tiles
    assert r["floor_ms"]["mfma"] == pytest.approx(1e3 * (6 * fm / 2.5e15 if tiles else fm / 157.3e12))


def test_the_library_says_which_units_run():
    d = Deconvolver(2, 512, 512, N.MVD_DEVICE_NONE)   # planning only
    for v in range(2):
        d.set_psf(v, gaussian_psf(31, 1.5, 6.0).astype(np.float32))
    assert bench.wave_tiles(d.ctx, CONFIGS["vol512"])
    api.mvd_set_float32_units(d.ctx)
    assert not bench.wave_tiles(d.ctx, CONFIGS["vol512"])
    d.close()
