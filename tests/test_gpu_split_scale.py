"""The scale of the matrix-core float32 frame transform (grids of 64 and 128),
against the FP64 oracle: it follows the calibrated samples, not the gains.

Tolerance: that of test_gpu_split.py, which holds whatever the scale.
"""
import numpy as np
import pytest

import synth
from test_gpu_parity import moff, torch  # noqa: F401 (fixtures)
from test_gpu_split import _check, _tables

pytestmark = pytest.mark.gpu


# antennas one per lane, and more than the samples that are loaded a frame ahead
@pytest.mark.parametrize("N", [64, 128])
@pytest.mark.parametrize("ant", [61, 530])
@pytest.mark.parametrize("gain", [1e4, 1e6, 1e8])
def test_dead_antenna_with_a_runaway_gain(torch, moff, N, ant, gain):
    """4+4-bit samples of one antenna are all zero and its gain is far from the
    others': it adds nothing to the image and takes nothing from the others."""
    w = synth.random_case(ant + N, ant, N, 2, 6, _tables(False, (3,)), fmt=synth.IN_CI4, extent_m=0.7 * N / 2,
                          cell_m=1.0)
    for dead in (0, ant - 1):
        w.E[:, :, dead] = 0
        w.gains[:, dead] = gain
    _check(torch, moff, w, 2, f"N={N} ant={ant} gain={gain}")


@pytest.mark.parametrize("N", [64, 128])
@pytest.mark.parametrize("gain", [1e2, 1e5])
def test_antenna_that_wakes_up(torch, moff, N, gain):
    """A 4+4-bit antenna with the largest gain whose samples are zero at first: the
    sums so far are rescaled when it starts."""
    w = synth.random_case(N, 40, N, 2, 9, _tables(True, (3,)), fmt=synth.IN_CI4, extent_m=0.7 * N / 2, cell_m=1.0)
    w.E[:4, :, 7] = 0
    w.gains[:, 7] = gain
    _check(torch, moff, w, 1, f"N={N} gain={gain}")


@pytest.mark.parametrize("N", [64, 128])
def test_no_samples_at_all(torch, moff, N):
    """Frames of zeros, at the start and throughout."""
    w = synth.random_case(N, 20, N, 2, 5, _tables(True, (2,)), fmt=synth.IN_CI4, extent_m=0.7 * N / 2, cell_m=1.0)
    w.E[:3] = 0
    w.E[:, 1] = 0
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        p.set_config(p.config(5)["n_variants"] - 1, 1)
        got = p.image(torch.from_numpy(w.E).to("cuda:0"), torch.from_numpy(w.gains).to("cuda:0")).cpu().numpy()
    assert np.all(got[1] == 0) and np.any(got[0] != 0)
