"""Calls out of order: a backward whose forward state a graph replay has
overwritten, and a replay of a graph captured before the last plan.  Both are
refused on the host, before any kernel starts."""
import numpy as np
import pytest
import torch

import workloads as W
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu


def _captured(gsr):
    """A renderer with a captured step, and what its calls take."""
    cam = W.camera_small()
    sc = W.random_scene(500, seed=2)
    sizes = [(cam.width, cam.height)]
    r = gsr.Renderer()
    r.plan(sc.n, sizes)
    g, cams, cfg = H.gpu_scene(gsr, sc), gsr.pack_cameras([cam]), gsr.Config()
    t_rgb, t_d, _ = (H.to_dev(x) for x in W.random_targets(sizes, seed=3))
    grads, loss = r.new_grads(sc.n), torch.zeros(1, device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        r.render_l1_fused(g, cams, cfg, t_rgb, t_d, grads=grads, loss=loss)
        r.graph_capture(g, cams, cfg, t_rgb, t_d, grads=grads, loss=loss, stream=s)
    s.synchronize()
    up = [H.to_dev(x) for x in H.flat_upstream(sizes, seed=4)]
    return r, (g, cams, cfg), up, s, (grads, loss)


def test_backward_after_a_replay(gsr_lib):
    gsr = gsr_lib
    r, scene, up, s, _ = _captured(gsr)
    r.render_forward(*scene)
    want = H.gpu_grads_numpy(r.render_backward(*scene, *up))
    r.render_forward(*scene)
    r.graph_launch(stream=s)
    s.synchronize()
    with pytest.raises(gsr.GsrError) as e:
        r.render_backward(*scene, *up)
    assert e.value.status == gsr.GSR_E_STATE
    # The next forward is whole again.
    r.render_forward(*scene)
    got = H.gpu_grads_numpy(r.render_backward(*scene, *up))
    for k in want:
        if want[k] is not None:
            assert H.rel_err(got[k], want[k]) <= 1e-5, k


def test_replay_on_another_workspace_leaves_the_forward(gsr_lib):
    gsr = gsr_lib
    r, scene, up, s, _ = _captured(gsr)
    mine = r.workspace
    r.workspace = torch.empty_like(mine)
    r.render_forward(*scene)
    r.graph_launch(stream=s)
    s.synchronize()
    got = H.gpu_grads_numpy(r.render_backward(*scene, *up))
    assert np.abs(got["mean"]).max() > 0
    del mine


def test_replay_after_a_plan(gsr_lib):
    gsr = gsr_lib
    r, scene, up, s, (grads, loss) = _captured(gsr)
    r.graph_launch(stream=s)
    s.synchronize()
    r.plan(r.n, r.sizes, r.capacity)
    with pytest.raises(gsr.GsrError) as e:
        r.graph_launch(stream=s)
    assert e.value.status == gsr.GSR_E_STATE
