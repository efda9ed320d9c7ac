"""Pair sums of long lag rows (antennas in a line, 256 pairs or more to a lag cell): the
image against the FP64 oracle's FX route and bit for bit from one call to the next."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import assert_image_close, moff, oracle_channels, to_dev, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


# just past 256 pairs to a cell; few workgroups and more than 512
@pytest.mark.parametrize("N, n_ant, n_chan", [(32, 130, 1), (32, 130, 520), (64, 182, 3), (64, 182, 520),
                                              (128, 256, 1), (128, 257, 520), (256, 364, 2), (256, 380, 520)])
def test_lines(torch, moff, N, n_ant, n_chan):
    rng = np.random.default_rng(N)
    w = synth.random_case(N, n_ant, N, n_chan, 2, [synth.random_kernel(rng, 2)], fmt=synth.IN_CI4, cell_m=1.0)
    w.geom.ant_xy = np.stack([rng.uniform(0, N / 2 - 3, n_ant), np.full(n_ant, N / 4)], axis=1)
    E, g = to_dev(torch, w.E), to_dev(torch, w.gains)
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        got = p.image_fx(E, g).cpu()
        for _ in range(3):
            assert torch.equal(p.image_fx(E, g).cpu(), got)
    chans = sorted({0, n_chan - 1})
    _, pbar = oracle_channels(w, chans)
    ref = np.stack([oracle.fx_discrete_image(w.geom, w.E, w.gains, c) for c in chans])
    assert_image_close(got.numpy()[chans], ref, pbar, label=f"N={N} {n_ant} {n_chan}")
