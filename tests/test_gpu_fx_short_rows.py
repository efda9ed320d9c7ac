"""Pair sums of short lag rows, four to a workgroup: the image against the FP64 oracle's FX
route at both sides of the rule's line and with row counts that leave waves without a row."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import assert_image_close, moff, oracle_channels, to_dev, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


def _check(torch, moff, w, label):
    E, g = to_dev(torch, w.E), to_dev(torch, w.gains)
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        got = p.image_fx(E, g).cpu()
        assert torch.equal(p.image_fx(E, g).cpu(), got)
    chans = range(w.geom.n_chan)
    _, pbar = oracle_channels(w, chans)
    ref = np.stack([oracle.fx_discrete_image(w.geom, w.E, w.gains, c) for c in chans])
    assert_image_close(got.numpy(), ref, pbar, label=label)


def _case(N, xy, n_types, fmt, flags=0, n_chan=2):
    rng = np.random.default_rng(N + len(xy))
    w = synth.random_case(N, len(xy), N, n_chan, 5,
                          [synth.random_kernel(rng, 1 if N == 8 else 2) for _ in range(n_types)],
                          fmt=fmt, cell_m=1.0)
    w.geom.flags |= flags
    w.geom.ant_xy = np.asarray(xy, np.float64)
    return w


# all antennas in one cell: one row, of up to 1035 pairs with 45 and to 1081 with 46
@pytest.mark.parametrize("n_ant", [2, 44, 45, 46, 47])
@pytest.mark.parametrize("flags", [0, synth.AUTOCORR_NONE])
def test_one_row(torch, moff, n_ant, flags):
    _check(torch, moff, _case(32, [[3, 4]] * n_ant, 1, synth.IN_C64, flags), f"{n_ant} {flags}")


# a column of k + 1 cells has k + 1 rows per type pair or, of one type, as many as its
# kernels reach; up to three waves of the last workgroup have no row
@pytest.mark.parametrize("N", [8, 32, 128, 256])
@pytest.mark.parametrize("n_types", [1, 2, 3])
@pytest.mark.parametrize("rows", [1, 2, 3])
def test_rows(torch, moff, N, n_types, rows):
    for fmt in (synth.IN_C64, synth.IN_CI4):
        xy = [[i % 3, i % rows] for i in range(9)]
        _check(torch, moff, _case(N, xy, n_types, fmt), f"N={N} {n_types} {rows}")


# more channels than a launch's workgroups are dealt out to at a time
@pytest.mark.parametrize("n_chan", [1, 7, 9, 17])
def test_channels(torch, moff, n_chan):
    rng = np.random.default_rng(n_chan)
    xy = rng.uniform(0, 25, (12, 2))
    _check(torch, moff, _case(64, xy, 2, synth.IN_CI4, n_chan=n_chan), f"{n_chan}")
