"""The gain adjoint's launch choices survive what does not concern them: forcing the
image's matrix-core variant, and an autotune that fails.  The adjoint of one shape
repeats its bits; two shapes differ in float32 rounding."""
import numpy as np
import pytest

import synth
from test_gpu_parity import moff, to_dev, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


def test_forcing_the_matrix_core_image_leaves_the_adjoint(torch, moff):
    N = 128
    w = synth.random_case(N, 90, N, 3, 11, [synth.random_kernel(np.random.default_rng(4), 3)], extent_m=40.0, cell_m=1.0)
    rng = np.random.default_rng(5)
    R = to_dev(torch, rng.standard_normal((3, N, N)).astype(np.float32))
    E, g = to_dev(torch, w.E), to_dev(torch, w.gains)
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        n = p.config(11)["n_variants"]
        default = p.gain_vjp(E, g, R).cpu()
        assert torch.equal(p.gain_vjp(E, g, R).cpu(), default)
        by_fft = []
        for v in (1, 0):
            p.set_config(v, 0)
            by_fft.append(p.gain_vjp(E, g, R).cpu())
        assert not torch.equal(*by_fft) and torch.equal(by_fft[1], default)
        p.set_config(n - 1, 0)
        assert torch.equal(p.gain_vjp(E, g, R).cpu(), default)
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        p.set_config(n - 1, 4)
        assert torch.equal(p.gain_vjp(E, g, R).cpu(), default)


def test_failed_autotune_keeps_the_choices(torch, moff):
    """An image shape whose tables do not fit a compute unit's LDS is refused; the
    adjoint's register budget stays as it was set."""
    w = synth.random_case(7, 4000, 256, 1, 2, [np.ones((2, 2), np.complex64)], extent_m=100.0, cell_m=1.0)
    E, g = to_dev(torch, w.E), to_dev(torch, w.gains)
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        p.set_config(1, 0)
        p.set_adjoint_waves(2)
        with pytest.raises(moff.MoffError, match="MOFF_ERR_UNSUPPORTED"):
            p.autotune(E, g)
        assert p.adjoint_waves()[0] == 2 and p.config(2)["variant"] == 1 and not p.config(2)["tuned"]
