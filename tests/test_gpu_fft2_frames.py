"""The padded transform of gridded frames on both sides of its launch rule (few frames
store each output as it comes, many two adjacent pixels at a time), against 64 bits.

Tolerance: a value passes 2 log2 N butterfly levels of at most three roundings, each
below 2^-24 and independent, so a frame's relative 2-norm error stays below
sqrt(6 log2 N) 2^-24."""
import math

import numpy as np
import pytest

from oracle.moff import image_field
from test_gpu_parity import moff, to_dev, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,frames", [(64, 3), (128, 1), (128, 200), (128, 201), (256, 1), (256, 20), (256, 21)])
def test_fft2_frames(torch, moff, N, frames):
    rng = np.random.default_rng(N + frames)
    L = N // 2
    eg = (rng.standard_normal((frames, L, L)) + 1j * rng.standard_normal((frames, L, L))).astype(np.complex64)
    with moff.Plan(np.array([[0.0, 0.0], [1.0, 1.0]]), [1], [np.ones((1, 1), np.complex64)], np.zeros(2, np.int32),
                   np.full(1, 1e8), N, 1.0, 0, 0) as p:
        got = p.fft2(to_dev(torch, eg)).cpu().numpy()
    for f in sorted({0, frames // 2, frames - 1}):
        ref = image_field(eg[f:f + 1].astype(np.complex128), N)[0]
        err = np.linalg.norm(got[f] - ref) / np.linalg.norm(ref)
        assert err <= math.sqrt(6 * math.log2(N)) * 2.0 ** -24, f"frame {f}: {err:.3g}"
