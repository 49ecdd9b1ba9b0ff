"""The oracle, importance and fixed-workspace tests once more on the tile-wide
compositing kernels.  Frames of few pixels, which those tests use, take the
kernels for small splats, where pixels per thread and batch depth have no
effect; a further view that sees nothing makes the frame large enough for the
tile-wide ones without changing any result of the other views.  Also the
overflow of the batch checkpoints of a fixed workspace, on both sets."""
import numpy as np
import pytest
import torch

import scenegen
from tests import gpu_util as U
from tests import test_gpu_end_to_end as E2E
from tests import test_gpu_graph as G
from tests import test_gpu_importance as I
from tests import test_gpu_stages as S
from tests import test_gpu_variants as V

pytestmark = pytest.mark.gpu

SIZE = (1408, 1320)  # 1,858,560 pixels: beyond the small-splat kernels at any splat size


def _away():
    """A camera that looks the other way: every splat lies behind it."""
    c = scenegen.orbit_camera(4.0, 0.0, 0.0, *SIZE)
    vm = np.asarray(c["viewmat"], np.float32).copy().reshape(4, 4)
    vm[[0, 2]] *= -1.0
    return dict(c, viewmat=vm)


@pytest.fixture
def large_frames(monkeypatch):
    """scenegen's small scenes with the empty view behind their own."""
    for name in ("tiny_scene", "small_scene"):
        plain = getattr(scenegen, name)

        def scene(*args, _plain=plain, **kw):
            s = _plain(*args, **kw)
            s["cameras"] = list(s["cameras"]) + [_away()]
            return s

        monkeypatch.setattr(scenegen, name, scene)


@pytest.fixture(scope="module")
def ctx():
    return U.M().mgs_create(0)


@pytest.fixture(scope="module")
def rast():
    from paper_2412_20522_amd.raster import Rasterizer
    return Rasterizer(0)


@pytest.fixture(scope="module")
def graph_rast():
    from paper_2412_20522_amd.raster import Rasterizer
    return Rasterizer(0, sh_degree=2, bg=(0.1, 0.2, 0.3), persistent=1)


@pytest.mark.parametrize("kind", ["tiny", "ragged_sh3", "multiview"])
@pytest.mark.parametrize("shape", S.SHAPES)
@pytest.mark.parametrize("cull", [0, 1])
def test_compositing_matches_oracle(large_frames, ctx, kind, shape, cull):
    S.test_product_compositing_matches_oracle(ctx, kind, shape, cull)


@pytest.mark.parametrize("kind", ["tiny", "ragged"])
@pytest.mark.parametrize("wide", [-1, 0, 1])
@pytest.mark.parametrize("cull", [0, 1])
def test_full_path_matches_oracle(large_frames, rast, kind, wide, cull):
    E2E.test_full_path_matches_oracle(rast, kind, wide, cull)


@pytest.mark.parametrize("wide,cull", [(-1, 0), (8, 1), (1, 1)])
def test_opacity_mode_matches_oracle(large_frames, rast, wide, cull):
    V.test_opacity_mode_matches_oracle(rast, "ragged", wide, cull, True)


def test_exact_mode_matches_oracle(large_frames, rast):
    V.test_opacity_mode_exact_mode_matches_oracle(rast)


@pytest.mark.parametrize("kind", ["tiny", "ragged", "multiview"])
@pytest.mark.parametrize("wide,cull,ppt", [(-1, 0, 1), (8, 1, 4), (1, 1, 2)])
def test_importance_matches_oracle(large_frames, rast, kind, wide, cull, ppt):
    I.test_importance_matches_oracle(rast, kind, wide, cull, ppt)


def test_backward_after_importance_forward(large_frames, rast):
    I.test_backward_after_importance_forward(rast)


def test_reserved_frame_and_graph_replays_match_eager(large_frames, graph_rast):
    G.test_reserved_frame_and_graph_replays_match_eager(graph_rast)


def test_reserved_frame_reports_overflow_and_recovers(large_frames, graph_rast):
    G.test_reserved_frame_reports_overflow_and_recovers(graph_rast)


def test_graph_step_matches_oracle(large_frames, graph_rast):
    G.test_graph_step_matches_oracle(graph_rast)


def test_captured_importance_forward_matches_eager(large_frames, graph_rast):
    G.test_captured_importance_forward_matches_eager(graph_rast)


@pytest.mark.parametrize("large", [False, True], ids=["small-splat", "tile-wide"])
def test_checkpoints_beyond_a_fixed_workspace_are_reported(large):
    """Sized with batches of 256 entries, used with batches of 32: the same list
    entries need more checkpoints than reserved.  The forward and a backward
    behind it leave the frame usable."""
    from paper_2412_20522_amd import maskgs as M
    from paper_2412_20522_amd.raster import Rasterizer
    s = scenegen.small_scene(25_000, 160, 120, seed=990, sh_degree=0, log_scale_mean=-1.6)
    cams = s["cameras"] + ([_away()] if large else [])
    dev = U.to_device(s)
    params = {k: dev[k] for k in U.PARAM_KEYS}
    P = sum(c["width"] * c["height"] for c in cams)
    dl = torch.from_numpy(np.random.default_rng(4).normal(size=3 * P).astype(np.float32)).cuda()
    rast = Rasterizer(0, sh_degree=0, stats=0, wide_tiles=-1, batch_depth=256)
    frame = rast.acquire_frame()
    ref = rast.forward(frame, params, dev["masks"], cams).clone()
    g_ref = rast.backward(frame, params, dl)
    # two checkpoints for every 32 entries instead of every 256, beyond the
    # 4,096 that a reservation adds
    assert rast.stats(frame)["n_instances"] * 2 * (1 / 32 - 1 / 256) > 2 * 4096
    rast.reserve(frame, 1.0)
    rast.set(batch_depth=32)
    img = torch.full((3 * P,), -3.0, device="cuda")
    rast.forward(frame, params, dev["masks"], cams, images=img)
    rast.backward(frame, params, dl)
    with pytest.raises(M.MaskGSError) as e:
        rast.check(frame)
    assert e.value.status == 3  # MGS_ERR_CAPACITY
    assert (img == -3.0).all()  # nothing was composited
    rast.set(batch_depth=256)
    for _ in range(2):
        img = rast.forward(frame, params, dev["masks"], cams)
        g = rast.backward(frame, params, dl)
        rast.check(frame)
        assert torch.equal(img, ref)
        for k in (*U.PARAM_KEYS, "masks"):
            assert U.rel_err(getattr(g, k).cpu().numpy(), getattr(g_ref, k).cpu().numpy()) <= 1e-5, k
    rast.reserve(frame, 0)
    rast.release_frame(frame)


@pytest.mark.parametrize("width", [1352, 1400], ids=["7,392 tiles", "7,656 tiles"])
@pytest.mark.parametrize("tile,fwd_ppt", [((16, 16), 2), ((32, 8), 2)])
def test_backward_on_both_sides_of_the_line_for_sums_over_a_tile_s_waves(width, tile, fwd_ppt):
    """Two pixels per thread and batches of 256: the waves' totals meet in LDS up
    to 7,424 tiles and go to the accumulators one by one beyond; with batches of
    128 they always meet."""
    from paper_2412_20522_amd.raster import Rasterizer
    s = scenegen.small_scene(6000, width, 1392, seed=995, sh_degree=0, log_scale_mean=-2.8)
    cams = s["cameras"]
    dev = U.to_device(s)
    params = {k: dev[k] for k in U.PARAM_KEYS}
    dl = torch.from_numpy(np.random.default_rng(5).normal(size=3 * width * 1392).astype(np.float32)).cuda()
    out = []
    for batch, ppt in ((256, 2), (128, 2), (256, 1)):
        rast = Rasterizer(0, sh_degree=0, stats=0, tile_w=tile[0], tile_h=tile[1], batch_depth=batch, fwd_ppt=fwd_ppt,
                          bwd_ppt=ppt)
        frame = rast.acquire_frame()
        img = rast.forward(frame, params, dev["masks"], cams)
        g = rast.backward(frame, params, dl)
        torch.cuda.synchronize()
        out.append((img.cpu().numpy(), {k: getattr(g, k).cpu().numpy() for k in (*U.PARAM_KEYS, "masks")}))
        rast.release_frame(frame)
    for img, g in out[1:]:
        assert np.array_equal(img, out[0][0])
        for k, v in g.items():
            assert U.rel_err(v, out[0][1][k]) <= 1e-5, k
