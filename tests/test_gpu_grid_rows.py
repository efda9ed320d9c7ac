"""Gridding where cells have few, many and unequal numbers of entries, against the
FP64 oracle: a thread takes four entries of a cell at a time, and beyond 1024 cells
two cells ahead and several workgroups to a frame of few.

Tolerance: every entry adds two roundings of a running sum that stays below the sum
of the magnitudes, 2^-24 of it each, and the calibration three of its own."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import moff, to_dev, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


# antennas stacked 1 .. 13 deep at a cell, with the same footprint; frames that keep
# several workgroups to a frame and that do not (1024 is the border)
@pytest.mark.parametrize("N,frames", [(8, 5), (16, 3), (32, 2), (64, 3), (128, 3), (128, 1025), (256, 2)])
@pytest.mark.parametrize("fmt", [synth.IN_C64, synth.IN_CI4])
def test_stacked_antennas(torch, moff, N, frames, fmt):
    L = N // 2
    rng = np.random.default_rng(N)
    k = 2 if N > 8 else 1
    spots = rng.integers(0, L - k + 1, (13, 2))
    xy = np.concatenate([np.repeat(spots[i:i + 1], i + 1, axis=0) for i in range(13)]).astype(float) + 0.3
    xy[0], xy[-1] = 0.0, L - k      # (the aperture's corners)
    w = synth.random_case(N, len(xy), N, 1, frames, [synth.random_kernel(rng, k)], fmt=fmt, cell_m=1.0, extent_m=1.0)
    w.geom.ant_xy = xy
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        got = p.grid(to_dev(torch, w.E), to_dev(torch, w.gains)).cpu().numpy()
    P = oracle.plan(w.geom)
    for t in (0, frames - 1):
        e = oracle.calibrated_field(w.E[t:t + 1], w.gains, w.geom.flags, 0)
        ref = oracle.grid_field(e, P)[0]
        mag = np.abs(e).sum() * np.abs(w.geom.ktype_vals[0]).max()
        assert np.abs(got[t, 0] - ref).max() <= (2 * len(xy) + 3) * 2.0 ** -24 * mag
        assert np.all(got[t, 0][ref == 0] == 0)


def test_crowded_centre(torch, moff):
    """400 antennas of 9 x 9 tables within a few cells: rows of hundreds of entries."""
    rng = np.random.default_rng(1)
    w = synth.random_case(1, 400, 128, 2, 2, [synth.random_kernel(rng, 9)], cell_m=1.0, extent_m=5.0)
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        got = p.grid(to_dev(torch, w.E), to_dev(torch, w.gains)).cpu().numpy()
    P = oracle.plan(w.geom)
    for c in range(2):
        e = oracle.calibrated_field(w.E, w.gains, w.geom.flags, c)
        ref = oracle.grid_field(e, P)
        mag = np.abs(e).sum() * np.abs(w.geom.ktype_vals[0]).max()
        assert np.abs(got[:, c] - ref).max() <= (2 * 400 + 3) * 2.0 ** -24 * mag
