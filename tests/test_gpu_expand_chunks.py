"""The adding step at pixel counts around a chunk (2 048 pixels) and around the
number of chunks up to which a block adds the counts in front of it itself
(4 096), with chunks in which every pixel, none or a few are added.  Count and
order exact, new Gaussians as in test_gpu_expand."""
import numpy as np
import pytest
import torch

import gpu_helpers as H
import oracle.expand as E
import workloads as W
from test_gpu_expand import _check_new, _out_arrays, _split

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [(1, 1), (2048, 1), (2049, 1), (97, 64), (4096, 2048), (4099, 2048)])
def test_expand_add_chunks(gsr_lib, size):
    gsr = gsr_lib
    w, h = size
    P = w * h
    print("CASE expand chunks", size, flush=True)
    rng = np.random.default_rng(P)
    cam = W.perturb_pose(W.camera_small().with_size(0.8 * w + 1.0, 0.7 * w + 1.0, 0.5 * w, 0.5 * h, w, h),
                         [0.1, -0.2, 0.05, 0.02, 0.1, -0.03])
    do = rng.uniform(1.0, 3.0, P).astype(np.float32)
    dr, T = do.copy(), np.zeros(P, np.float32)
    hit = rng.choice(P, max(1, min(P, 5000) // 3), replace=False)
    dr[hit] += 1.0                            # a few in most chunks
    T[: min(P, 2048)] = 1.0                   # every pixel of the first chunk
    T[max(0, P - 5):] = 1.0                   # the last pixels
    do[rng.choice(P, P // 50, replace=False)] = 0.0
    rgb = rng.random(3 * P).astype(np.float32)
    sizes = [size]
    masks, new = E.add_gaussians([cam], _split(T, sizes), _split(dr, sizes), _split(do, sizes), _split(rgb, sizes, 3),
                                 0.5, 0.25, 1.3, -2.0)
    count = int(new["mean"].shape[0])
    r = gsr.Renderer()
    r.plan(1, sizes)
    for room in (7, -1) if count > 1 else (7,):  # all fit, the last does not
        cap = 3 + max(0, count + room)
        out = _out_arrays(cap)
        flag = torch.full((P,), 7, dtype=torch.uint8, device="cuda")
        cnt = r.expand_add(gsr.pack_cameras([cam]), H.to_dev(T), H.to_dev(dr), H.to_dev(do), H.to_dev(rgb), out, 3, cap,
                           0.5, 0.25, 1.3, -2.0, pixel_flag=flag)
        assert int(cnt.item()) == count
        np.testing.assert_array_equal(flag.cpu().numpy(), masks[0].ravel().astype(np.uint8))
        _check_new(out, 3, new, count)
