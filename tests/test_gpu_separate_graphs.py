"""Forward and backward captured into graphs of their own, replayed in any
order and between eager calls: a replayed backward finds clear accumulators
and a clear tile-order histogram however often it ran since the last forward."""
import numpy as np
import pytest
import torch

import scenegen
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

GRADS = ("means", "log_scales", "quats", "opacity_logits", "sh", "masks")


def _capture(fn):
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        fn()
    torch.cuda.synchronize()
    return g


@pytest.mark.parametrize("away", [False, True], ids=["small-splat", "tile-wide"])
def test_backward_graph_replayed_more_often_than_its_forward(away):
    from paper_2412_20522_amd.raster import Grads, Rasterizer
    s = scenegen.small_scene(2500, 149, 91, seed=951, sh_degree=1, log_scale_mean=-2.3)
    cams = [s["cameras"][0]] + ([scenegen.orbit_camera(4.0, 0.0, 0.0, 2048, 1600)] if away else [])
    dev = U.to_device(s)
    params = {k: dev[k] for k in U.PARAM_KEYS}
    P = sum(c["width"] * c["height"] for c in cams)
    images, dl = torch.empty(3 * P, device="cuda"), torch.zeros(3 * P, device="cuda")
    dl[:3 * 149 * 91] = torch.from_numpy(np.random.default_rng(6).normal(size=3 * 149 * 91).astype(np.float32)).cuda()
    out = Grads(*(torch.empty_like(params[k]) for k in U.PARAM_KEYS), torch.empty_like(dev["masks"]))
    # (the first forward over these views has no measured batch counts, so the
    # captured backward forms a tile order of its own)
    rast = Rasterizer(0, sh_degree=1, batch_depth=64, stats=0)
    frame = rast.acquire_frame()

    def forward():
        rast.forward(frame, params, dev["masks"], cams, images=images)

    def backward():
        rast.backward(frame, params, dl, out=out)

    def check(what):
        torch.cuda.synchronize()
        for k in GRADS:
            e = U.rel_err(getattr(out, k).cpu().numpy(), ref[k])
            assert e <= 1e-5, (what, k, e)
            getattr(out, k).fill_(77.0)

    forward()
    backward()
    torch.cuda.synchronize()
    ref = {k: getattr(out, k).cpu().numpy().copy() for k in GRADS}
    rast.reserve(frame, 1.25)
    # a forward over another view in between, so that the next one over these
    # has no measured counts again
    rast.forward(frame, params, dev["masks"], [scenegen.orbit_camera(4.0, 15.0, 0.0, 149, 91)] + cams[1:],
                 images=images)
    rast.check(frame)
    forward()
    bwd = _capture(backward)
    fwd = _capture(forward)
    for rep in range(3):
        bwd.replay()
        check(("backward graph again", rep))
    fwd.replay()
    bwd.replay()
    check("both graphs")
    backward()
    check("eager backward after a replayed one")
    forward()
    bwd.replay()
    check("replay after an eager forward")
    backward()
    check("eager backward after a replay that an eager forward preceded")
    fwd.replay()
    backward()
    check("eager backward of a replayed forward")
    both = _capture(lambda: (forward(), backward(), backward(), forward(), backward()))
    for rep in range(3):
        both.replay()
        check(("steps in one graph", rep))
        _ = (images * 2.0).sum().item()
    rast.check(frame)
    del bwd, fwd, both
    rast.reserve(frame, 0)
    rast.release_frame(frame)
