"""The projection's early test with a camera matrix that is not a rotation (a
similarity's scale, a sheared product of rotations): the projection takes it as
it is, so the pairs and lists are the oracle's, also of Gaussians that reach
the view from beside it by the matrix's scale alone."""
import dataclasses

import numpy as np
import pytest

import oracle as O
import workloads as W
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu

MATRICES = {
    "rotation": np.eye(3),
    "scale_4": 4.0 * np.eye(3),
    "scale_half": 0.5 * np.eye(3),
    "stretch_x": np.diag([5.0, 1.0, 1.0]),
    "stretch_z": np.diag([1.0, 1.0, 3.0]),
    "shear": np.array([[1.0, 2.5, 0.0], [0.0, 1.0, -1.5], [0.3, 0.0, 1.0]]),
}


@pytest.mark.parametrize("guard", [1.3, 0.0])
@pytest.mark.parametrize("name", list(MATRICES))
def test_pairs_and_lists_with_any_matrix(gsr_lib, name, guard):
    gsr = gsr_lib
    print("CASE early", name, guard, flush=True)
    sc = W.random_scene(6000, seed=9, xy=1.2, z=(1.0, 4.0), log_scale_mu=-2.2, log_scale_sd=0.5)
    cam = W.camera_small().with_size(70.0, 66.0, 47.5, 31.5, 96, 64)
    cam = W.perturb_pose(cam, [0.05, -0.03, 0.02, 0.04, 0.05, -0.03])
    cam = cam.with_pose(np.asarray(cam.R, np.float64) @ MATRICES[name], cam.t)
    r = gsr.Renderer()
    r.plan(sc.n, [(96, 64)])
    cfg = gsr.Config(fov_guard=guard)
    r.render_forward(H.gpu_scene(gsr, sc), gsr.pack_cameras([cam]), cfg)
    rng, ids = (x.numpy() for x in r.debug_tiles())
    ocfg = dataclasses.replace(H.oracle_cfg_of(cfg), fov_guard=guard)
    proj = O.project(sc, cam, ocfg.as_f32())
    assert r.pair_count() == H.rect_pairs(proj) > 0
    H.check_view_lists(rng, ids, 0, 0, proj, O.tile_lists(proj), 96, 64, ocfg)
