"""The loss cap right behind a plan, on a stream that does not wait for the
null stream: the counters that the plan clears are clear by then; and on the
null stream while another stream is being captured."""
import ctypes

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


@pytest.mark.parametrize("mode", [1, 2])
def test_median_on_the_null_stream_beside_a_capture(gsr_lib, mode):
    """mode: hipStreamCaptureModeThreadLocal, hipStreamCaptureModeRelaxed."""
    gsr = gsr_lib
    sizes = [(640, 480)]
    r = gsr.Renderer()
    r.plan(1, sizes)
    px, _ = W.loss_images(sizes, seed=1)
    dev, cap = H.to_dev(px), torch.empty(1, device="cuda")
    want = np.array([O.loss_cap(px, None, 10.0)], np.float32)
    torch.cuda.synchronize()
    hip = ctypes.CDLL("libamdhip64.so")
    s, graph = ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipStreamCreate(ctypes.byref(s)) == 0
    assert hip.hipStreamBeginCapture(s, mode) == 0
    try:
        r.loss_median(dev, None, 10.0, cap_out=cap)
    finally:
        assert hip.hipStreamEndCapture(s, ctypes.byref(graph)) == 0
    torch.cuda.synchronize()
    np.testing.assert_array_equal(cap.cpu().numpy(), want)
    # and with the counters again
    cap.zero_()
    r.loss_median(dev, None, 10.0, cap_out=cap)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(cap.cpu().numpy(), want)
    hip.hipStreamDestroy(s)
