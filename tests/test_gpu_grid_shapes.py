"""Staged gridding at the edges of its launch shapes, against the FP64 oracle grid:
a frame's cells one at a time, eight side by side in one or several workgroups, and
in batches of one workgroup where the frames alone fill the card.

Tolerance: a cell sums at most the entries of its row, each of two float32 products
(2^-24 each) of a calibrated sample (2^-23); the largest cell bounds them all, 1e-6.
"""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import moff, to_dev, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,chan,time", [(32, 1, 3), (64, 3, 2), (128, 1, 2047), (128, 2, 1024), (256, 1, 2), (256, 1, 2048)])
@pytest.mark.parametrize("fmt", [synth.IN_C64, synth.IN_CI4])
def test_grid_shapes(torch, moff, N, chan, time, fmt):
    rng = np.random.default_rng(N + time)
    w = synth.random_case(N, 40, N, chan, time, [synth.random_kernel(rng, 3)], fmt=fmt, extent_m=0.35 * N, cell_m=1.0)
    P = oracle.plan(w.geom)
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        eg = p.grid(to_dev(torch, w.E), to_dev(torch, w.gains))
        torch.cuda.synchronize()
        pick = sorted({0, 1, time // 2, time - 1})
        got = eg[pick].cpu().numpy()
    for c in range(chan):
        ref = oracle.grid_field(oracle.calibrated_field(w.E[pick], w.gains, w.geom.flags, c), P)
        assert np.abs(got[:, c] - ref).max() <= 1e-6 * np.abs(ref).max()
