"""A staged list that is too small for some batches: the backward forms these
batches again and gives the gradients of a list with room for all."""
import numpy as np
import pytest
import torch

import scenegen
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

GRADS = ("means", "log_scales", "quats", "opacity_logits", "sh", "masks")


@pytest.mark.parametrize("tile,bwd_ppt", [((16, 16), 4), ((16, 16), 1), ((8, 8), 1)])
@pytest.mark.parametrize("cull,wide", [(1, -1), (1, 8), (0, 8)])
def test_batches_that_the_staged_list_does_not_hold(tile, bwd_ppt, cull, wide):
    """The fixed workspace is sized by a frame whose tiles stay within their
    first chunks, with room for some further ones; then all splats move into
    a few tiles, whose lists need many."""
    from paper_2412_20522_amd import maskgs as M
    from paper_2412_20522_amd.raster import Rasterizer
    n, w, h = 20_000, 2048, 1600  # tile-wide kernels at any splat size
    s = scenegen.small_scene(n, w, h, seed=960, sh_degree=0, log_scale_mean=-6.5)
    rng = np.random.default_rng(7)
    spread = rng.uniform(-1.5, 1.5, (n, 3)).astype(np.float32)
    # one splat in ten over several tiles (listed per region with wide = 8)
    s["log_scales"][::10] += 2.0
    s["opacity_logits"][:] = -4.0  # no pixel stops: every entry is staged
    s["means"] = spread
    dev = U.to_device(s)
    params = {k: dev[k] for k in U.PARAM_KEYS}
    crowd = dict(params, means=torch.from_numpy((0.02 * spread).astype(np.float32)).cuda())
    cams = [scenegen.orbit_camera(4.0, 0.0, 0.0, w, h)]
    dl = torch.from_numpy(rng.normal(size=3 * w * h).astype(np.float32)).cuda()
    rast = Rasterizer(0, sh_degree=0, tile_w=tile[0], tile_h=tile[1], batch_depth=64, fwd_ppt=1, bwd_ppt=bwd_ppt,
                      tile_cull=cull, wide_tiles=wide, stats=0)
    plain, fixed = rast.acquire_frame(), M.mgs_frame_create(rast.ctx)
    img = rast.forward(plain, crowd, dev["masks"], cams)
    ref = rast.backward(plain, crowd, dl)
    r = U.u32(M.mgs_frame_export(rast.ctx, plain, "ranges")).reshape(-1, 2).astype(np.int64)
    longest = (r[:, 1] - r[:, 0])[:rast.stats(plain)["total_tiles"]]
    # counter chunks that the lists need, against the 8 beyond the first ones
    assert np.maximum(0, np.ceil((longest - 256) / 512)).sum() > 16
    rast.forward(fixed, params, dev["masks"], cams)
    rast.reserve(fixed, 1.0)
    again = rast.forward(fixed, crowd, dev["masks"], cams)
    rast.check(fixed)
    got = rast.backward(fixed, crowd, dl)
    torch.cuda.synchronize()
    assert torch.equal(img, again)
    for k in GRADS:
        e = U.rel_err(getattr(got, k).cpu().numpy(), getattr(ref, k).cpu().numpy())
        assert e <= 1e-6, (k, e)
    rast.reserve(fixed, 0)
    for f in (plain, fixed):
        rast.release_frame(f)
