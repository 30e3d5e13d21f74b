"""The separate backward clears the gradient rows of the visible records and
reads no others: the same gradients whatever the workspace held before, at
record counts around the clearing kernel's blocks (256) and wavefronts (64),
over views that see different parts of the scene, with and without the
Gaussians' gradients and spherical-harmonic colour."""
import numpy as np
import pytest
import torch

import workloads as W
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sh", [False, True])
@pytest.mark.parametrize("pose_only", [False, True])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 1500])
def test_backward_in_a_workspace_of_any_contents(gsr_lib, n, pose_only, sh):
    gsr = gsr_lib
    print("CASE clear rows", n, pose_only, sh, flush=True)
    sc = W.random_scene(n, seed=n)
    if sh:
        sc.sh = np.random.default_rng(n).normal(0.3, 0.3, (n, 4, 3)).astype(np.float32)
    cam = W.camera_small()
    cams = [cam, W.perturb_pose(cam, [0.9, 0.0, 0.0, 0.0, 0.2, 0.0]), W.perturb_pose(cam, [0.0, 0.0, -9.0, 0.0, 0.0, 0.0])]
    sizes = [(c.width, c.height) for c in cams]
    cfg = gsr.Config(flags=gsr.GSR_POSE_GRAD if pose_only else gsr.GSR_POSE_GRAD | gsr.GSR_GAUSS_GRAD)
    up = H.flat_upstream(sizes, seed=5)
    grads = []
    for fill in (0, 255):
        r = gsr.Renderer()
        r.plan(n, sizes)
        r.workspace.fill_(fill)
        g, packed = H.gpu_scene(gsr, sc), gsr.pack_cameras(cams)
        r.render_forward(g, packed, cfg)
        for _ in range(2):  # the second finds the rows as the first left them
            got = H.gpu_grads_numpy(r.render_backward(g, packed, cfg, *(H.to_dev(x) for x in up)))
            grads.append(got)
        torch.cuda.synchronize()
    for got in grads[1:]:
        for k, want in grads[0].items():
            assert np.isfinite(want).all()
            # (FP64 sums over tiles in the order they finish)
            np.testing.assert_allclose(got[k], want, rtol=1e-5, atol=1e-6 * max(np.abs(want).max(), 1e-30), err_msg=k)
