"""The launch of a plan that is neither tuned nor set: variant and slices of least
modelled time.  What the model has to see: programs and antennas that outweigh the
transform (a short call is cut into slices), many workgroups of a single frame (the
matrix cores' tables do not pay), and that a set choice ends the rule."""
import numpy as np
import pytest

import synth
from test_gpu_parity import assert_image_close, moff, oracle_channels, to_dev, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


def _line(N, ant, chan, time, k, fmt=synth.IN_CI4):
    w = synth.random_case(ant, ant, N, chan, time, [synth.random_kernel(np.random.default_rng(k), k).real.astype(np.complex64)],
                          fmt=fmt, extent_m=1.0, cell_m=1.0)
    x = np.random.default_rng(ant).uniform(0, N / 2 - k - 2, ant)
    w.geom.ant_xy = np.stack([x, np.full(ant, 5.0)], axis=1)
    return w


def test_gather_counts(torch, moff):
    """849 antennas of 9 x 9 tables in a line, 72 channels x 4 samples: a frame is
    mostly gathering, and one slice leaves most of the card idle."""
    w = _line(128, 849, 72, 4, 9)
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        assert p.config(4)["slices"] == 4
        assert p.config(4) == p.config(4)
        got = p.image(to_dev(torch, w.E), to_dev(torch, w.gains)).cpu().numpy()
        p.set_config(0, 1)
        assert p.config(4)["slices"] == 1 and p.config(4)["variant"] == 0
    ref, pbar = oracle_channels(w, (0, 71))
    assert_image_close(got[[0, 71]], ref, pbar)


@pytest.mark.parametrize("N,ant,chan,time,variant", [
    (128, 256, 128, 1000, 2),   # a long integration: the matrix cores
    (64, 203, 33, 257, 1),
    (128, 88, 1700, 1, 0),      # single frames of many channels: the FFT
    (128, 16, 1, 8, 0),         # a call too small to fill the card
    (256, 350, 64, 64, 1)])
def test_variant_by_size(torch, moff, N, ant, chan, time, variant):
    w = synth.random_case(1, ant, N, chan, 1, [synth.random_kernel(np.random.default_rng(1), 3).real.astype(np.complex64)],
                          extent_m=0.7 * N / 2, cell_m=1.0)
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        assert p.config(time)["variant"] == variant
