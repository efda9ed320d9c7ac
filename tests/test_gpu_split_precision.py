"""The matrix-core float32 frame transform (grids of 64 and 128) loses nothing
against the float32 FFT: its distance from the FP64 oracle, in the 2-norm of a
channel's image, is at most that of the FFT shape on the same input, and below the
tolerance of test_gpu_split.py where one antenna is far louder than the others.
"""
import numpy as np
import pytest

import oracle
import synth
from oracle import uv_autocorr
from test_gpu_parity import moff, to_dev, torch  # noqa: F401 (fixtures)
from test_gpu_split import _check, _tables

pytestmark = pytest.mark.gpu


# dense complex tables; the uv-plane rule takes out an error proportional to the
# image, most of the FFT's, and leaves what the phase factors' rounding leaves
@pytest.mark.parametrize("N", [64, 128])
@pytest.mark.parametrize("flags", [0, synth.AUTOCORR_UV])
def test_no_further_from_64_bits_than_the_fft(torch, moff, N, flags):
    w = synth.random_case(N, 203, N, 2, 120, _tables(False, (3, 5)), extent_m=0.8 * N / 2, cell_m=1.0)
    w.geom.flags |= flags
    P = oracle.plan(w.geom)
    one = uv_autocorr.uv_channel if flags else oracle.moff_channel
    ref = [one(w.geom, w.E, w.gains, c, P) for c in range(2)]
    err = []
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        for v in (0, p.config(120)["n_variants"] - 1):
            p.set_config(v, 30)
            got = p.image(to_dev(torch, w.E), to_dev(torch, w.gains)).cpu().numpy()
            err.append([np.linalg.norm(got[c] - ref[c]) / np.linalg.norm(ref[c]) for c in range(2)])
    assert max(err[1]) <= max(err[0]), f"FFT {err[0]}, matrix cores {err[1]}"


@pytest.mark.parametrize("N", [64, 128])
@pytest.mark.parametrize("slices", [1, 7])
def test_one_loud_antenna(torch, moff, N, slices):
    w = synth.random_case(N + 1, 203, N, 2, 7, _tables(False, (3, 5)), extent_m=0.8 * N / 2, cell_m=1.0)
    w.E[:, :, 67] *= np.float32(1e4)
    _check(torch, moff, w, slices, f"N={N} one loud antenna, {slices} slices")
