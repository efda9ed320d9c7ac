"""Pair sums where many pairs share a lag cell (regular arrays, arrays in a line): the
image against the FP64 oracle's FX route, and bit for bit from one call to the next."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import assert_image_close, moff, oracle_channels, to_dev, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


# every number of copies of a row's sums; a wave whose lanes all meet in one cell (all
# antennas of a column) and in a few
@pytest.mark.parametrize("N", [8, 16, 32, 64, 128, 256])
@pytest.mark.parametrize("shape", ["square", "line", "column"])
@pytest.mark.parametrize("fmt", [synth.IN_C64, synth.IN_CI4])
def test_redundant_arrays(torch, moff, N, shape, fmt):
    side = min(8, N // 2 - 1)
    j, i = np.meshgrid(np.arange(side), np.arange(side), indexing="ij")
    if shape == "square":
        xy = np.stack([i.ravel(), j.ravel()], axis=1)
    else:
        x = np.arange(70) % (N // 2 - 1)
        xy = np.stack([x, np.zeros(70)], axis=1) if shape == "line" else np.stack([np.zeros(70), x], axis=1)
    w = synth.random_case(N, len(xy), N, 2, 5, [synth.random_kernel(np.random.default_rng(N), 1 if N == 8 else 2)],
                          fmt=fmt, cell_m=1.0)
    w.geom.ant_xy = xy.astype(np.float64)
    E, g = to_dev(torch, w.E), to_dev(torch, w.gains)
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        got = p.image_fx(E, g).cpu()
        for _ in range(3):
            assert torch.equal(p.image_fx(E, g).cpu(), got)
    _, pbar = oracle_channels(w, range(2))
    ref = np.stack([oracle.fx_discrete_image(w.geom, w.E, w.gains, c) for c in range(2)])
    assert_image_close(got.numpy(), ref, pbar, label=f"N={N} {shape}")
