"""The loss cap of views that many blocks share (over 32 768 pixels): the
exact lower median against the oracle at the sizes around that line, from
several streams in turn, and captured in a graph."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu


def _want(px, mask, sizes, factor):
    out, po = [], 0
    for w, h in sizes:
        out.append(O.loss_cap(px[po:po + w * h], mask[po:po + w * h] if mask is not None else None, factor))
        po += w * h
    return np.array(out, np.float32)


@pytest.mark.parametrize("sizes", [[(256, 128)], [(10923, 3)], [(1200, 680), (1, 1), (91, 90), (640, 480)],
                                   [(8192, 5), (8193, 5), (8191, 5)]])
@pytest.mark.parametrize("masked", [False, True])
def test_median_of_large_views(gsr_lib, sizes, masked):
    gsr = gsr_lib
    print("CASE median", sizes, masked, flush=True)
    r = gsr.Renderer()
    r.plan(1, sizes)
    for seed in (3, 4):  # the second call finds the counters as the first left them
        px, mask = W.loss_images(sizes, seed=seed)
        got = r.loss_median(H.to_dev(px), H.to_dev(mask, torch.uint8) if masked else None, 10.0).cpu().numpy()
        np.testing.assert_array_equal(got, _want(px, mask if masked else None, sizes, 10.0))


def test_median_on_several_streams_and_captured(gsr_lib):
    gsr = gsr_lib
    sizes = [(640, 480), (300, 200)]
    r = gsr.Renderer()
    r.plan(1, sizes)
    px = [H.to_dev(W.loss_images(sizes, seed=s)[0]) for s in range(4)]
    want = [_want(p.cpu().numpy(), None, sizes, 2.0) for p in px]
    streams = [torch.cuda.Stream() for _ in range(3)] + [torch.cuda.current_stream()]
    outs = [[torch.zeros(2, device="cuda") for _ in px] for _ in range(8)]
    torch.cuda.synchronize()
    for rep in range(8):
        for k, (p, s) in enumerate(zip(px, streams)):
            r.loss_median(p, None, 2.0, cap_out=outs[rep][k], stream=s)
    torch.cuda.synchronize()
    for rep in range(8):
        for k in range(4):
            np.testing.assert_array_equal(outs[rep][k].cpu().numpy(), want[k])
    src, cap = px[0].clone(), torch.zeros(2, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        r.loss_median(src, None, 2.0, cap_out=cap)
    for k in (1, 2, 3, 0):
        src.copy_(px[k])
        graph.replay()
        r.loss_median(px[k], None, 2.0, cap_out=outs[0][0])
        torch.cuda.synchronize()
        np.testing.assert_array_equal(cap.cpu().numpy(), want[k])
        np.testing.assert_array_equal(outs[0][0].cpu().numpy(), want[k])
