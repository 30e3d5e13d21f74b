"""Upstream gradients that are not finite at one pixel: the sums of Gaussians
that the pixel does not blend keep their values, though pixels of the same
wavefront blend them, and so do the colour sums of those that it blends where
the pixel's own colour gradients are finite.  (A NaN colour gradient reaches
that channel's sum of every Gaussian of the wavefront.)  The sums are the same
FP32 additions with and without it, so they agree to a few of their roundings:
1e-6 of the largest."""
import numpy as np
import pytest

import workloads as W
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu
SIZE, PIXEL = (16, 16), (5, 4)  # (row, column)


def _scene(wide):
    """Gaussian 0 around the pixel, 1 beside it in the same four rows, and
    `wide` more over the whole tile behind them."""
    n = 2 + wide
    sc = W.random_scene(n, seed=1)
    f = 40.0
    cam = W.camera_small().with_size(f, f, 8.0, 8.0, *SIZE)
    for i, (x, y, z) in enumerate([(4.0, 5.5, 1.5), (12.0, 5.5, 1.6)] + [(8.0, 8.0, 2.0 + 0.1 * k) for k in range(wide)]):
        sc.mean[i] = [(x - 8.0) / f * z, (y - 8.0) / f * z, z]
    sc.log_scale[:2] = -4.0
    sc.log_scale[2:] = -1.0
    sc.opacity_logit[:2] = 1.0
    sc.opacity_logit[2:] = -2.0
    return sc, cam


def _grads(gsr, wide, bad):
    sc, cam = _scene(wide)
    r = gsr.Renderer()
    r.plan(sc.n, [SIZE])
    cfg = gsr.Config()
    g, cams = H.gpu_scene(gsr, sc), gsr.pack_cameras([cam])
    r.render_forward(g, cams, cfg)
    up = list(H.flat_upstream([SIZE], seed=3))
    if bad is not None:
        which, value = bad
        up[which][PIXEL[0] * 16 + PIXEL[1]] = value  # (which 0: the red plane)
    return H.gpu_grads_numpy(r.render_backward(g, cams, cfg, *(H.to_dev(x) for x in up)))


def _same(got, want, scale):
    assert np.isfinite(want).all() and np.abs(want).max() > 0
    np.testing.assert_allclose(got, want, rtol=0, atol=1e-6 * np.abs(scale).max())


@pytest.mark.parametrize("wide", [0, 3, 14])
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf, 1e37])
@pytest.mark.parametrize("which", [0, 1, 2], ids=["red", "depth", "T"])
def test_a_bad_upstream_stays_with_its_pixel(gsr_lib, which, value, wide):
    print("CASE nonfinite", which, value, wide, flush=True)
    want, got = _grads(gsr_lib, wide, None), _grads(gsr_lib, wide, (which, value))
    if value == 1e37:
        assert np.abs(got["opacity_logit"][0]) > 1e30
    else:
        assert not np.isfinite(got["opacity_logit"][0])
    for k in ("opacity_logit", "mean", "log_scale", "quat"):
        # (a depth gradient goes to the depth sum, hence the mean, of the whole wavefront)
        if not (which == 1 and k == "mean"):
            _same(got[k][1], want[k][1], want[k])
    # Colour sums: of all Gaussians, but for the channel whose gradient is bad.
    c = 1 if which == 0 else 0
    _same(got["rgb"][:, c:], want["rgb"][:, c:], want["rgb"])
