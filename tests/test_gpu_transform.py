"""GPU parity of the float32 FFT frame transform against the FP64 oracle, every
grid and shape variant: the twiddles taken as twists of the radix passes.

Tolerance: that of the float32 path (1e-5 of max |Pbar|) and, in the 2-norm, one
derived from its roundings.  A frame passes 2 log2 N butterfly levels of at most
three roundings and some eight in calibration and gridding, each of relative size
below 2^-24 and independent, so a field sample carries at most
sqrt(6 log2 N + 8) 2^-24 and its power twice that.  The power of a channel's
frames is its image plus the antennas' mean power times Pbar.
"""
import math

import numpy as np
import pytest

import synth
from oracle.moff import decode_ci4
from test_gpu_parity import assert_image_close, moff, oracle_channels, to_dev, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


# every column class and twist (random footprints fill the whole aperture), more
# antennas than a lane ingests, ragged slices, and a frame of two antennas
@pytest.mark.parametrize("N,variant", [(8, 0), (16, 0), (32, 0), (64, 0), (128, 0), (128, 1), (256, 0), (256, 1)])
@pytest.mark.parametrize("ant,chan,time,slices", [(2, 1, 1, 1), (300, 3, 5, 2)])
@pytest.mark.parametrize("fmt", [synth.IN_C64, synth.IN_CI4])
def test_transform_parity(torch, moff, N, variant, ant, chan, time, slices, fmt):
    rng = np.random.default_rng(N)
    w = synth.random_case(ant + N, ant, N, chan, time, [synth.random_kernel(rng, 3)], fmt=fmt,
                          extent_m=min(0.7 * N / 2, N / 2 - 3), cell_m=1.0)   # (footprints of three cells fit)
    ref, pbar = oracle_channels(w, range(chan))
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        p.set_config(variant, slices)
        got = p.image(to_dev(torch, w.E), to_dev(torch, w.gains) if w.gains is not None else None)
        torch.cuda.synchronize()
        got = got.cpu().numpy()
    assert_image_close(got, ref, pbar, label=f"N={N} variant {variant}")
    tol = 2 * math.sqrt(6 * math.log2(N) + 8) * 2.0 ** -24
    for c in range(chan):
        E = w.E[:, c] if fmt == synth.IN_C64 else decode_ci4(w.E[:, c])
        power = np.linalg.norm(ref[c]) + np.mean(np.abs(E * w.gains[c]) ** 2) * np.linalg.norm(pbar[c])
        assert np.linalg.norm(got[c] - ref[c]) <= tol * power, f"N={N} variant {variant} channel {c}"
