"""The rasteriser at list lengths where its walks change their way: the
forward takes list entries four at a time, the backward eight (two halves),
sub-batches hold 64 and staged batches 192 (separate forward) or more.  Every
Gaussian covers the whole image, so that each tile's list has the length
asked for.  Images, `last`, work counts and gradients against the CPU oracle,
with the tolerances of the other parity tests."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu

LENGTHS = (1, 3, 4, 5, 7, 8, 9, 12, 63, 64, 65, 191, 192, 193, 260)


def _config(gsr, mode):
    if mode == "open":  # every entry blends in every pixel, also one of alpha 0
        return gsr.Config(alpha_min=0.0, alpha_max=1.0, T_min=0.0, flags=gsr.GSR_GAUSS_GRAD | gsr.GSR_POSE_GRAD | 1)
    if mode == "early":  # pixels stop inside the first groups
        return gsr.Config(T_min=0.6, bg=(0.3, 0.1, 0.2))
    return gsr.Config(bg=(0.3, 0.1, 0.2))


def _wide(n, seed):
    sc = W.random_scene(n, seed=seed, xy=0.1, z=(1.0, 3.0), log_scale_mu=-0.5)
    sc.opacity_logit[:] = np.random.default_rng(seed).uniform(-3.5, -2.0, n).astype(np.float32)
    sc.opacity_logit[::17] = 7.0  # clamped at alpha_max near its centre
    return sc


@pytest.mark.parametrize("mode", ["default", "open", "early"])
@pytest.mark.parametrize("n", LENGTHS)
def test_list_lengths(gsr_lib, n, mode):
    gsr = gsr_lib
    print("CASE raster", n, mode, flush=True)
    sc = _wide(n, n)
    if mode == "open":
        sc.opacity_logit[:] = np.minimum(sc.opacity_logit, -2.0)
    cam = W.camera_small().with_size(30.0, 30.0, 8.0, 4.0, 19, 21)
    size = (cam.width, cam.height)
    cfg = _config(gsr, mode)
    ocfg = H.oracle_cfg_of(cfg)
    r = gsr.Renderer()
    r.plan(n, [size])
    g, cams = H.gpu_scene(gsr, sc), gsr.pack_cameras([cam])
    out = r.render_forward(g, cams, cfg)
    rng, ids = (x.numpy() for x in r.debug_tiles())
    assert (rng[:, 1] - rng[:, 0]).max() == n
    img = H.split_images(out, r.sizes)[0]
    o = O.render(sc, cam, ocfg)
    H.assert_images_close(img, o, max_ambiguous=0.05, gpu_lists=(rng, ids, 0, 0))
    T = o["proj"]["TX"] * o["proj"]["TY"]
    work, ow = r.work_counts(g, cfg), H.oracle_work(o, cam, ocfg, H.gpu_view_lists(rng, ids, 0, T, 0))
    for k in ("fwd_evals", "blended"):
        assert abs(work[k] - ow[k]) <= ow["slack"], (k, work[k], ow[k], ow["slack"])
    up = H.flat_upstream([size], seed=n, zero_masks=[o["ambiguous_grad"]])
    got = H.gpu_grads_numpy(r.render_backward(g, cams, cfg, *(H.to_dev(x) for x in up)))
    ref = O.render_backward(sc, cam, ocfg, *H.view_slices(*up, [size])[0], fwd=o)
    H.assert_grads_close(got, ref)
    # The fused step on targets that the image misses by far more than its
    # error: the residual signs, hence the upstream gradients, are certain.
    t_rgb, t_d = (np.where(np.random.default_rng(n).random(x.shape) < 0.5, x - 1.0, x + 1.0).astype(np.float32)
                  for x in (o["rgb"], o["depth"]))
    t_d = np.where(o["ambiguous_grad"], 0.0, np.maximum(t_d, 0.0)).astype(np.float32)
    mask = ~o["ambiguous_grad"]
    loss, grads = r.render_l1_fused(g, cams, cfg, H.to_dev(t_rgb.reshape(-1)), H.to_dev(t_d.reshape(-1)),
                                    H.to_dev(mask.reshape(-1), torch.uint8), w_rgb=0.8, w_depth=0.3)
    ref_loss, gC, gD = O.l1_loss(o["rgb"], o["depth"], t_rgb, t_d, mask, 0.8, 0.3)
    assert abs(float(loss.item()) - ref_loss) <= 1e-4 * abs(ref_loss) + 1e-12
    H.assert_grads_close(H.gpu_grads_numpy(grads), O.render_backward(sc, cam, ocfg, gC, gD, None, fwd=o))


def test_a_nan_upstream_stays_with_the_wavefront_of_its_pixel(gsr_lib):
    """A Gaussian that no pixel of the four rows around a NaN upstream
    gradient blends keeps the gradient that it has without it."""
    gsr = gsr_lib
    # Two small Gaussians in one tile, around rows 2 and 13.
    cam = W.camera_small().with_size(40.0, 40.0, 8.0, 8.0, 16, 16)
    sc = W.random_scene(2, seed=1)
    sc.mean[:] = [[0.0, -6.0 / 40.0 * 2.0, 2.0], [0.0, 5.0 / 40.0 * 1.5, 1.5]]
    sc.log_scale[:] = -4.0
    sc.opacity_logit[:] = 1.0
    grads = []
    for nan in (False, True):
        r = gsr.Renderer()
        r.plan(2, [(16, 16)])
        cfg = gsr.Config()
        g, cams = H.gpu_scene(gsr, sc), gsr.pack_cameras([cam])
        r.render_forward(g, cams, cfg)
        rng, _ = r.debug_tiles()
        assert int(rng[0, 1] - rng[0, 0]) == 2
        up = H.flat_upstream([(16, 16)], seed=3)
        if nan:
            up[0][13 * 16 + 8] = np.nan
        grads.append(H.gpu_grads_numpy(r.render_backward(g, cams, cfg, *(H.to_dev(x) for x in up))))
    for k in ("mean", "log_scale", "opacity_logit", "rgb"):
        assert np.abs(grads[0][k][0]).max() > 0
        np.testing.assert_array_equal(grads[1][k][0], grads[0][k][0])
