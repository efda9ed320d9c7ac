"""GPU parity of the matrix-core float32 frame transform (grids of 64 and 128)
against the FP64 oracle, at the sizes where it can go wrong.

Tolerance: that of the float32 path (1e-5 of max |Pbar|), and the claim that
the split products lose nothing against the float32 FFT: each operand keeps 22
bits (relative 2^-23), three roundings along a pixel's path, so the relative
2-norm error of a frame stays below 4 x 2^-23 = 4.8e-7; sums over the few
frames here add less.
"""
import numpy as np
import pytest

import synth
from test_gpu_parity import assert_image_close, moff, oracle_channels, to_dev, torch  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu
TOL2 = 4 * 2.0 ** -23


def _tables(real, ks, seed=3):
    rng = np.random.default_rng(seed)
    tabs = [synth.random_kernel(rng, k) for k in ks]
    return [t.real.astype(np.complex64) for t in tabs] if real else tabs


def _check(torch, moff, w, slices, label):
    ref, pbar = oracle_channels(w, range(w.geom.n_chan))
    with moff.Plan.from_geometry(w.geom, device=0) as p:
        v = p.config(w.E.shape[0])["n_variants"] - 1      # the matrix-core shape follows the FFT's
        p.set_config(v, slices)
        assert p.config(w.E.shape[0])["variant"] == v
        got = p.image(to_dev(torch, w.E), to_dev(torch, w.gains) if w.gains is not None else None)
        torch.cuda.synchronize()
        got = got.cpu().numpy()
    assert_image_close(got, ref, pbar, label=label)
    for c in range(ref.shape[0]):
        assert np.linalg.norm(got[c] - ref[c]) <= TOL2 * np.linalg.norm(pbar[c]), f"{label} channel {c}"


# antennas: two, fewer than a wave's lanes, more than two per lane (N = 64: 128
# threads; N = 128: 256); channels and samples that leave ragged XCD rounds and
# slices; one slice and more slices than samples per slice divide evenly
@pytest.mark.parametrize("N", [64, 128])
@pytest.mark.parametrize("real", [True, False])
@pytest.mark.parametrize("ant,chan,time,slices", [(2, 1, 1, 1), (61, 9, 5, 2), (700, 2, 3, 3)])
@pytest.mark.parametrize("fmt", [synth.IN_C64, synth.IN_CI4])
def test_split_parity(torch, moff, N, real, ant, chan, time, slices, fmt):
    w = synth.random_case(ant + N, ant, N, chan, time, _tables(real, (3, 5)), fmt=fmt, extent_m=0.7 * N / 2, cell_m=1.0)
    _check(torch, moff, w, slices, f"N={N} real={real} ant={ant}")


@pytest.mark.parametrize("scale", [1e-16, 1.0, 1e12])
def test_split_scale_follows_the_samples(torch, moff, scale):
    """complex64 samples of any size, and frames that grow and shrink by large
    factors within a slice (each new largest frame rescales the sums)."""
    w = synth.random_case(5, 40, 64, 2, 9, _tables(False, (3,)), extent_m=20.0, cell_m=1.0)
    steps = np.array([1.0, 1e-3, 30.0, 2.0, 1e4, 0.0, 1e4, 1e-2, 3e4], np.float32) * np.float32(scale)
    w.E = (w.E * steps[:, None, None]).astype(np.complex64)
    _check(torch, moff, w, 1, f"scale {scale}")


@pytest.mark.parametrize("N", [64, 128])
def test_split_blocked_accumulation(torch, moff, N):
    """600 samples in one slice: the float32 sums go into float64 twice."""
    w = synth.random_case(N, 6, N, 1, 600, _tables(True, (2,)), extent_m=N / 6.0, cell_m=1.0)
    _check(torch, moff, w, 1, f"N={N} blocked")
