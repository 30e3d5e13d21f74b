"""The chain to the parameters and poses at the view counts where a block's
share of the views changes: counts are read eight views at a time, and without
Gaussian gradients a block takes eight views."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_views", [1, 7, 8, 9, 17])
@pytest.mark.parametrize("n", [64, 300])
def test_chain_over_views(gsr_lib, n, n_views):
    gsr = gsr_lib
    print("CASE chain", n, n_views, flush=True)
    sc = W.random_scene(n, seed=n_views, log_scale_mu=-2.0)
    rng = np.random.default_rng(n_views)
    # Every third camera looks away: views that no lane sees between others.
    cams = [W.perturb_pose(W.camera_small().with_size(30.0, 30.0, 16.0, 12.0, 33, 25),
                           rng.uniform(-0.05, 0.05, 6) + (np.array([0, 0, -20.0, 0, 0, 0]) if v % 3 == 2 else 0.0))
            for v in range(n_views)]
    sizes = [(c.width, c.height) for c in cams]
    r = gsr.Renderer()
    r.plan(n, sizes)
    g, cams_d = H.gpu_scene(gsr, sc), gsr.pack_cameras(cams)
    both = gsr.Config()
    pose = gsr.Config(flags=gsr.GSR_POSE_GRAD)
    ocfg = H.oracle_cfg_of(both)
    fwds = [O.render(sc, c, ocfg) for c in cams]
    up = H.flat_upstream(sizes, seed=n, zero_masks=[f["ambiguous_grad"] for f in fwds])
    dev = [H.to_dev(x) for x in up]
    r.render_forward(g, cams_d, both)
    got = H.gpu_grads_numpy(r.render_backward(g, cams_d, both, *dev))
    r.render_forward(g, cams_d, pose)
    alone = r.render_backward(g, cams_d, pose, *dev)["d_pose"].cpu().numpy()
    ref = [O.render_backward(sc, c, ocfg, *u, fwd=f) for c, f, u in zip(cams, fwds, H.view_slices(*up, sizes))]
    H.assert_grads_close(got, {k: sum(b[k] for b in ref) for k in ("mean", "log_scale", "quat", "opacity_logit", "rgb")})
    for v, b in enumerate(ref):
        assert H.rel_err(got["pose"][v], b["pose"]) <= 1e-3 or np.abs(b["pose"]).max() == 0.0
        # The same FP64 sums in the same order, but for the order of the 2D
        # gradients' FP64 atomics: equal to a float32 rounding.
        np.testing.assert_allclose(alone[v], got["pose"][v], rtol=3e-7, atol=1e-7 * np.abs(got["pose"][v]).max())


@pytest.mark.parametrize("which", ["gauss", "pose", "both"])
def test_autograd_buffers_are_written(gsr_lib, which):
    """The autograd backward's buffers: written where the flags ask for the
    gradient and zero elsewhere, whatever their memory held before."""
    import torch
    gsr = gsr_lib
    flags = dict(gauss=gsr.GSR_GAUSS_GRAD, pose=gsr.GSR_POSE_GRAD, both=gsr.GSR_GAUSS_GRAD | gsr.GSR_POSE_GRAD)[which]
    n = 300
    sc, cam = W.random_scene(n, seed=3, log_scale_mu=-2.0), W.camera_small().with_size(30.0, 30.0, 16.0, 12.0, 33, 25)
    r = gsr.Renderer()
    r.plan(n, [(33, 25)])
    cams, cfg = gsr.pack_cameras([cam]), gsr.Config(flags=flags)
    g = H.gpu_scene(gsr, sc)
    leaves = [x.clone().requires_grad_() for x in (g.mean, g.log_scale, g.quat, g.opacity_logit, g.rgb)]
    xi = torch.zeros(1, 6, device="cuda", requires_grad=True)
    up = [H.to_dev(x) for x in H.flat_upstream([(33, 25)], seed=2)]
    out = gsr.render(r, *leaves, cams, cfg, pose_xi=xi)
    junk = [torch.full(s, float("nan"), device="cuda") for s in ((n, 3), (n, 3), (n, 4), (n,), (n, 3), (1, 6)) for _ in range(4)]
    del junk  # the allocator hands these out next
    got = torch.autograd.grad(out, [*leaves, xi], grad_outputs=up)
    r.render_forward(g, cams, cfg)
    ref = r.render_backward(g, cams, cfg, *up)
    for a, k in zip(got, ("d_mean", "d_log_scale", "d_quat", "d_opacity_logit", "d_rgb", "d_pose")):
        np.testing.assert_allclose(a.cpu().numpy(), ref[k].cpu().numpy(), rtol=1e-6, atol=1e-7 * float(ref[k].abs().max()))
        asked = which == "both" or (k == "d_pose") == (which == "pose")
        assert bool((a != 0).any()) == asked, k
