"""The sums of the gain gradient (self power, power-pattern products, partials of
slices and classes) at the sizes where their split can go wrong, against the FP64
oracle gradient.

Tolerance: the gradient's own, 1e-4 of the channel's largest entry.  The sums run
in float64, so the transforms' float32 roundings are all that is left of it.
"""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_grad import TOL, gpu_grad, moff, rel_err, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


# antennas about a wave's lanes, samples fewer than its workgroup's waves and not a
# multiple of their batches of eight; with self power and without (no sums but the
# partials'), from one workgroup's partials and from those of the staged form
@pytest.mark.parametrize("ant,time", [(2, 1), (64, 7), (65, 67), (130, 9)])
@pytest.mark.parametrize("flags", [0, synth.AUTOCORR_NONE])
@pytest.mark.parametrize("fmt", [synth.IN_C64, synth.IN_CI4])
@pytest.mark.parametrize("staged", [False, True])
def test_gradient_sums(torch, moff, ant, time, flags, fmt, staged):
    rng = np.random.default_rng(ant)
    w = synth.random_case(ant, ant, 64, 3, time, [synth.random_kernel(rng, 2), synth.random_kernel(rng, 3)], fmt=fmt,
                          extent_m=26.0, cell_m=1.0)
    w.geom.flags |= flags
    R = rng.standard_normal((3, 64, 64)).astype(np.float32)
    ref = oracle.gain_gradient(w.geom, w.E, w.gains, R.astype(np.float64))
    err = rel_err(gpu_grad(torch, moff, w, R, staged), ref)
    assert err <= TOL, f"{ant} antennas, {time} samples: {err:.3g}"
