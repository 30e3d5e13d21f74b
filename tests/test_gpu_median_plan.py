"""The loss cap right behind a plan, on a stream that does not wait for the
null stream: the counters that the plan clears are clear by then."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu


def test_median_on_another_stream_behind_a_plan(gsr_lib):
    gsr = gsr_lib
    r = gsr.Renderer()
    s = torch.cuda.Stream()
    for k, views in enumerate((1, 64, 7, 128)):
        sizes = [(182, 181)] * views
        px, _ = W.loss_images(sizes, seed=k)
        dev, cap = H.to_dev(px), torch.empty(views, device="cuda")
        torch.cuda.synchronize()
        r.plan(1, sizes, workspace=False)
        r.loss_median(dev, None, 10.0, cap_out=cap, stream=s)
        s.synchronize()
        want = [O.loss_cap(p, None, 10.0) for p in px.reshape(views, -1)]
        np.testing.assert_array_equal(cap.cpu().numpy(), np.array(want, np.float32))
