"""The visibility route in passes over time (staged samples beyond the workspace, the
visibilities summed in float64 between), for 4+4-bit samples and for several table
types, against float64 sums (tolerance of test_gpu_fx.py).  Two antennas: the image
holds e_0 conj(e_1) only, so one sample with the mean product has the same image."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import TOL, moff, to_dev, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


# eight channels of one 64-antenna block of 2 GiB: passes of at most 2.1 million
# 4+4-bit and 350 thousand complex64 samples; the last pass ragged
@pytest.mark.parametrize("fmt,T", [(synth.IN_CI4, 2_100_007), (synth.IN_C64, 360_011)])
@pytest.mark.parametrize("types", [1, 2])
def test_passes(torch, moff, fmt, T, types):
    C, rng = 8, np.random.default_rng(types)
    tabs = [synth.random_kernel(rng, 2), synth.random_kernel(rng, 3)][:types]
    w = synth.random_case(1, 2, 16, C, 1, tabs, fmt=fmt, extent_m=3.0, cell_m=1.0)
    w.geom.ant_ktype = np.array([0, types - 1], np.int32)
    if fmt == synth.IN_CI4:
        n = rng.integers(-8, 8, (2, T, C, 2), np.int8)
        n[:, :, :, 1] = np.clip(n[:, :, :, 0] + n[:, :, :, 1] // 4, -8, 7)
        raw = (((n[0] & 15) << 4) | (n[1] & 15)).astype(np.uint8)
    else:
        raw = rng.standard_normal((T, C, 4), np.float32).view(np.complex64)
        raw[:, :, 1] += raw[:, :, 0]
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        got = p.image_fx(to_dev(torch, raw), to_dev(torch, w.gains)).cpu().numpy().astype(np.float64)
    for c in range(C):
        if fmt == synth.IN_CI4:
            e = n[0, :, c].astype(np.float64) + 1j * n[1, :, c]
        else:
            e = raw[:, c].astype(np.complex128)
        e = e * w.gains[c].astype(np.complex128)
        v = np.mean(e[:, 0] * np.conj(e[:, 1]))
        one = synth.random_case(1, 2, 16, 1, 1, tabs, extent_m=3.0, cell_m=1.0).geom
        one.ant_xy, one.ant_ktype = w.geom.ant_xy, w.geom.ant_ktype
        ref, parts = oracle.moff_channel(one, np.array([[[v, 1.0]]]), None, 0, keep=True)
        scale = np.mean(np.abs(e) ** 2) / np.mean([abs(v) ** 2, 1.0]) * np.abs(parts["S"]).max()
        assert np.abs(got[c] - ref).max() <= TOL * scale, f"channel {c}"
