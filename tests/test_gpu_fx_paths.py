"""The visibility route's kernels at the sizes where they can go wrong, against
the FP64 oracle's FX route (tolerance of test_gpu_fx.py): one table type (lists
of cells, the response applied to the image) and two (dense lag grid), real and
complex tables, few and many pairs per cell, antenna counts below and around a
4-antenna load, a 16-wide block and a 64-wide tile, samples around a chunk of 32
and a step of 64, and every grid size."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import assert_image_close, moff, oracle_channels, to_dev, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


def _check(torch, moff, w, label):
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        got = p.image_fx(to_dev(torch, w.E), to_dev(torch, w.gains) if w.gains is not None else None)
        torch.cuda.synchronize()
        got = got.cpu().numpy()
    C = w.geom.n_chan
    _, pbar = oracle_channels(w, range(C))
    ref = np.stack([oracle.fx_discrete_image(w.geom, w.E, w.gains, c) for c in range(C)])
    assert_image_close(got, ref, pbar, label=label)


def _tables(seed, real, types):
    rng = np.random.default_rng(seed)
    tabs = [synth.random_kernel(rng, 2 + i) for i in range(types)]
    return [t.real.astype(np.complex64) for t in tabs] if real else tabs


@pytest.mark.parametrize("ant,time", [(2, 1), (3, 33), (5, 64), (17, 65), (63, 32), (66, 31)])
@pytest.mark.parametrize("fmt", [synth.IN_C64, synth.IN_CI4])
@pytest.mark.parametrize("types,real", [(1, False), (2, True), (2, False)])
def test_fx_antennas_and_samples(torch, moff, ant, time, fmt, types, real):
    w = synth.random_case(ant + time, ant, 32, 2, time, _tables(ant, real, types), fmt=fmt, extent_m=11.0, cell_m=1.0)
    _check(torch, moff, w, f"{ant} antennas, {time} samples")


@pytest.mark.parametrize("N", [8, 16, 32, 64, 128, 256])
@pytest.mark.parametrize("types", [1, 2])
def test_fx_every_grid(torch, moff, N, types):
    w = synth.random_case(N, 9, N, 9, 3, _tables(N, False, types), extent_m=0.6 * (N / 2 - 4), cell_m=1.0)
    _check(torch, moff, w, f"N={N}")


def test_fx_redundant_array(torch, moff):
    """A regular array: up to 48 pairs per cell, several lanes per cell."""
    w = synth.random_case(3, 49, 32, 3, 5, _tables(3, False, 1), fmt=synth.IN_CI4, extent_m=6.0, cell_m=1.0)
    j, i = np.meshgrid(np.arange(7), np.arange(7), indexing="ij")
    w.geom.ant_xy = np.stack([i.ravel(), j.ravel()], axis=1).astype(np.float64) * 1.0
    _check(torch, moff, w, "redundant")


@pytest.mark.parametrize("scale", [1e-14, 1e14])
def test_fx_sample_scale(torch, moff, scale):
    """bfloat16 levels keep float32's range: no scale is lost."""
    w = synth.random_case(8, 20, 32, 1, 40, _tables(8, False, 1), extent_m=9.0, cell_m=1.0)
    w.E = (w.E * np.float32(scale)).astype(np.complex64)
    _check(torch, moff, w, f"scale {scale}")


def test_fx_long_integration_in_passes(torch, moff):
    """Staged samples that do not fit the workspace (about 2 GiB for eight
    channels): the integration runs in two passes over time, the second ragged,
    its visibilities summed in float64.  Two antennas give V = e_0 conj(e_1) and
    an image that is its fringe, so the reference is one float64 sum."""
    T, C = 400_003, 8
    w = synth.random_case(1, 2, 8, C, 8, [np.ones((1, 1), np.complex64)], extent_m=2.0, cell_m=1.0)
    rng = np.random.default_rng(0)
    E = (rng.standard_normal((T, C, 2)) + 1j * rng.standard_normal((T, C, 2))).astype(np.complex64)
    E[:, :, 1] += E[:, :, 0]
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        got = p.image_fx(to_dev(torch, E), to_dev(torch, w.gains))
        torch.cuda.synchronize()
        got = got.cpu().numpy().astype(np.float64)
    for c in (0, C - 1):
        e = E[:, c].astype(np.complex128) * w.gains[c]
        # one sample with the same product e_0 conj(e_1) has the same image
        v = np.mean(e[:, 0] * np.conj(e[:, 1]))
        one = np.array([[[v, 1.0]]])
        g1 = synth.random_case(1, 2, 8, 1, 1, [np.ones((1, 1), np.complex64)], extent_m=2.0, cell_m=1.0).geom
        ref = oracle.moff_channel(g1, one, None, 0)
        assert np.abs(got[c] - ref).max() <= 1e-5 * np.abs(e).max() ** 2
        assert np.abs(got[c] - ref).max() <= 1e-5 * np.mean(np.abs(e) ** 2) * 4
