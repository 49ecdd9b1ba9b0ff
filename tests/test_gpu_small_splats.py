"""The two sets of compositing kernels (tile-wide ones, and those for small
splats that frames of few pixels take) against each other and the tile-wide
ones against the oracle.  A second view of more pixels than the small-splat
kernels take moves the same view to the tile-wide kernels."""
import numpy as np
import pytest
import torch

import oracle
import scenegen
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

BIG = (2048, 1600)  # 3,276,800 pixels: beyond the small-splat kernels at any splat size


def _run(rast, s, cams, dl, **settings):
    """Per-pixel results of the first view and the gradients of a loss on it."""
    from paper_2412_20522_amd import maskgs as M
    rast.set(**settings)
    dev = U.to_device(s)
    params = {k: dev[k] for k in U.PARAM_KEYS}
    P0, P = cams[0]["width"] * cams[0]["height"], sum(c["width"] * c["height"] for c in cams)
    frame = rast.acquire_frame()
    tfin = torch.empty(P, device="cuda")
    img = rast.forward(frame, params, dev["masks"], cams, t_final=tfin)
    full = torch.zeros(3 * P, device="cuda")
    full[:3 * P0] = torch.from_numpy(dl).cuda()
    g = rast.backward(frame, params, full)
    ex = {k: M.mgs_frame_export(rast.ctx, frame, k) for k in ("last", "stats", "evals")}
    torch.cuda.synchronize()
    rast.release_frame(frame)
    out = {"image": img[:3 * P0], "t_final": tfin[:P0], "last": ex["last"][:P0], "stats": ex["stats"][:4 * P0],
           "evals": ex["evals"][:4 * P0]}
    return {k: v.cpu().numpy() for k, v in out.items()}, g


def _settings(tile, **kw):
    base = dict(sh_degree=1, bg=(0.2, 0.4, 0.6), tile_w=tile[0], tile_h=tile[1], batch_depth=64, fwd_ppt=1, bwd_ppt=1,
                persistent=0, exact_mode=0, wide_tiles=0, tile_cull=1, stats=1, mask_mode=0)
    base.update(kw)
    return base


def _big():
    return scenegen.orbit_camera(4.0, 0.0, 0.0, *BIG)


@pytest.mark.parametrize("tile", [(16, 16), (8, 8), (16, 8), (32, 8)])
@pytest.mark.parametrize("kw", [dict(), dict(wide_tiles=1), dict(wide_tiles=4, persistent=1), dict(tile_cull=0),
                                dict(exact_mode=1), dict(mask_mode=1)],
                         ids=["default", "regions", "persistent", "nocull", "exact", "opacity"])
def test_small_splat_kernels_equal_the_tile_wide_ones(tile, kw):
    """Images, final transmittance, last blended entry and work counters bit
    for bit (every product and sum in the same order), gradients to the
    rounding of differently grouped FP32 partial sums."""
    from paper_2412_20522_amd.raster import Rasterizer
    n = 60 if kw.get("exact_mode") else 3000
    s = scenegen.small_scene(n, 149, 91, seed=811, sh_degree=1, log_scale_mean=-2.4, opacity_mean=1.5)
    s["masks"][::7] = 0.25  # any mask value in [0, 1]
    cam = s["cameras"][0]
    dl = np.random.default_rng(3).normal(size=3 * 149 * 91).astype(np.float32)
    rast = Rasterizer(0)
    a, ga = _run(rast, s, [cam], dl, **_settings(tile, **kw))
    b, gb = _run(rast, s, [cam, _big()], dl, **_settings(tile, **kw))
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    assert (a["t_final"] < 1e-3).mean() > 0.05 or kw.get("exact_mode")  # early stops are among them
    for k in ("means", "log_scales", "quats", "opacity_logits", "sh", "masks"):
        e = U.rel_err(getattr(ga, k).cpu().numpy(), getattr(gb, k).cpu().numpy())
        assert e <= 1e-5, (k, e)


@pytest.mark.parametrize("size", [(1, 1), (8, 8), (17, 3), (65, 33)])
@pytest.mark.parametrize("n", [1, 5, 700])
def test_small_splat_kernels_at_the_edges_of_parts_and_batches(size, n):
    """Views of less than a block, a part and a tile and just beyond; lists
    shorter than a round of four and longer than two batches."""
    from paper_2412_20522_amd.raster import Rasterizer
    w, h = size
    s = scenegen.small_scene(n, w, h, seed=812 + n, sh_degree=1, log_scale_mean=-1.5, opacity_mean=-3.0)
    dl = np.random.default_rng(4).normal(size=3 * w * h).astype(np.float32)
    rast = Rasterizer(0)
    a, ga = _run(rast, s, s["cameras"], dl, **_settings((16, 16)))
    b, gb = _run(rast, s, [s["cameras"][0], _big()], dl, **_settings((16, 16)))
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    for k in ("means", "log_scales", "quats", "opacity_logits", "sh", "masks"):
        x, y = getattr(ga, k).cpu().numpy(), getattr(gb, k).cpu().numpy()
        assert U.rel_err(x, y) <= 1e-5 or np.abs(x - y).max() <= 1e-9, k


@pytest.mark.parametrize("tile,fwd_ppt,bwd_ppt", [((8, 8), 1, 1), ((16, 8), 1, 2), ((16, 8), 2, 1), ((16, 16), 1, 4),
                                                  ((16, 16), 2, 2), ((16, 16), 4, 1), ((32, 8), 1, 2),
                                                  ((32, 8), 2, 4), ((32, 8), 4, 1)])
@pytest.mark.parametrize("wide", [-1, 1])
def test_tile_wide_kernels_match_oracle(tile, fwd_ppt, bwd_ppt, wide):
    from paper_2412_20522_amd.raster import Rasterizer
    s = scenegen.small_scene(3000, 150, 90, seed=813, sh_degree=1, log_scale_mean=-2.6)
    cam = s["cameras"][0]
    dl = np.random.default_rng(5).normal(size=3 * 150 * 90).astype(np.float32)
    rast = Rasterizer(0)
    a, g = _run(rast, s, [cam, _big()], dl, **_settings(tile, fwd_ppt=fwd_ppt, bwd_ppt=bwd_ppt, wide_tiles=wide))
    ost = oracle.RasterSettings(sh_degree=1, bg=(0.2, 0.4, 0.6))
    op = oracle.run_pipeline(s, [cam], s["masks"].astype(np.float64), ost, dl_dimage=dl.astype(np.float64))
    assert U.rel_err(a["image"].astype(np.float64), op.fwd.image) <= 2e-4
    for name, x, y in [("means", g.means, op.grads.means), ("log_scales", g.log_scales, op.grads.log_scales),
                       ("quats", g.quats, op.grads.quats),
                       ("opacity_logits", g.opacity_logits, op.grads.opacity_logits), ("sh", g.sh, op.grads.sh),
                       ("masks", g.masks, op.bwd.d_mask)]:
        e = U.rel_err(x.cpu().numpy(), y)
        assert e <= 2e-3, (name, e)


@pytest.mark.parametrize("n", [1, 64, 1025, 8192, 8193, 16384, 16385, 40_000, 300_000])
@pytest.mark.parametrize("views", [1, 3])
def test_depth_order_and_lists_over_the_sort_variants(n, views):
    """Record order and list entries around the sizes where the sorts change
    between one workgroup with 8 or 16 keys per thread and several blocks."""
    from paper_2412_20522_amd import maskgs as M
    from paper_2412_20522_amd.raster import Rasterizer
    s = scenegen.small_scene(n, 70, 50, seed=900 + n, sh_degree=0, log_scale_mean=-4.0, n_views=views)
    s["means"][: n // 3] = s["means"][n // 3: 2 * (n // 3)]  # equal depths: ties by record id
    rast = Rasterizer(0, **_settings((8, 8), sh_degree=0, wide_tiles=4))
    dev = U.to_device(s)
    frame = rast.acquire_frame()
    rast.forward(frame, {k: dev[k] for k in U.PARAM_KEYS}, dev["masks"], s["cameras"])
    ex = {k: M.mgs_frame_export(rast.ctx, frame, k) for k in ("order", "depth", "tiles", "values", "ranges")}
    torch.cuda.synchronize()
    K = rast.stats(frame)["n_instances"]
    rast.release_frame(frame)
    bits, tiles, order = U.u32(ex["depth"]), U.u32(ex["tiles"]), U.u32(ex["order"])
    key = np.where(tiles > 0, bits, np.uint32(0xffffffff))
    for v in range(views):
        want = np.argsort(key[v * n:(v + 1) * n], kind="stable") + v * n
        assert np.array_equal(order[v * n:(v + 1) * n], want)
    r = U.u32(ex["ranges"]).reshape(-1, 2).astype(np.int64)
    vals = U.u32(ex["values"]).astype(np.int64)[:K]
    r = r[r[:, 1] > r[:, 0]]
    assert (r[:, 1] - r[:, 0]).sum() == K and np.array_equal(r[1:, 0], r[:-1, 1]) and (K == 0 or r[0, 0] == 0)
    step = np.diff(vals) > 0
    step[r[1:, 0] - 1] = True  # positions ascend within a cell
    assert step.all()


@pytest.mark.parametrize("n,views", [(16_385, 1), (500_003, 1), (1_400_001, 3), (4_001_792, 1)])
@pytest.mark.parametrize("dead", ["none", "some", "runs", "last", "all"])
def test_depth_order_with_records_that_reach_no_tile(n, views, dead):
    """Positions of the records with tiles by (depth, record), the others
    behind them by record: below and above the size from which the first pass
    drops the others, over segments of whole and broken tiles of the sort."""
    from paper_2412_20522_amd import maskgs as M
    from paper_2412_20522_amd.raster import Rasterizer
    s = scenegen.small_scene(n, 70, 50, seed=910, sh_degree=0, log_scale_mean=-7.0, n_views=views)
    s["means"][: n // 3] = s["means"][n // 3: 2 * (n // 3)]  # equal depths
    far = np.zeros(n, bool)
    far[{"none": slice(0, 0), "some": slice(0, None, 3), "runs": slice(n // 5, n // 2), "last": slice(n - 5000, None),
         "all": slice(None)}[dead]] = True
    s["means"][far] = (1e4, -1e4, 1e4)  # outside every view
    rast = Rasterizer(0, **_settings((8, 8), sh_degree=0, wide_tiles=4, stats=0))
    dev = U.to_device(s)
    frame = rast.acquire_frame()
    rast.forward(frame, {k: dev[k] for k in U.PARAM_KEYS}, dev["masks"], s["cameras"])
    ex = {k: M.mgs_frame_export(rast.ctx, frame, k) for k in ("order", "depth", "tiles")}
    torch.cuda.synchronize()
    rast.release_frame(frame)
    bits, tiles, order = U.u32(ex["depth"]), U.u32(ex["tiles"]), U.u32(ex["order"])
    assert (tiles.reshape(views, n)[:, far] == 0).all()
    key = np.where(tiles > 0, bits, np.uint32(0xffffffff))
    for v in range(views):
        want = np.argsort(key[v * n:(v + 1) * n], kind="stable") + v * n
        assert np.array_equal(order[v * n:(v + 1) * n], want)


@pytest.mark.parametrize("w,h", [(1928, 2024), (1928, 2032), (2048, 2048)])
@pytest.mark.parametrize("cull", [0, 1])
def test_lists_on_both_sides_of_16_bit_cell_keys(w, h, cull):
    """60,973 and 61,214 tiles of 8x8 with 3,904 regions (64,877 and 65,118
    cells, 16-bit keys), 65,536 tiles with 4,096 (32-bit): every cell's list
    holds the records whose rectangle reaches it."""
    from paper_2412_20522_amd import maskgs as M
    from paper_2412_20522_amd.raster import Rasterizer
    n = 30_000
    s = scenegen.small_scene(n, w, h, seed=940, sh_degree=0, log_scale_mean=-4.0)
    s["means"][::7] *= 3.0  # some near the edges and outside
    dev = U.to_device(s)
    rast = Rasterizer(0, **_settings((8, 8), sh_degree=0, tile_cull=cull, wide_tiles=-1))
    frame = rast.acquire_frame()
    rast.forward(frame, {k: dev[k] for k in U.PARAM_KEYS}, dev["masks"], s["cameras"])
    ex = {k: M.mgs_frame_export(rast.ctx, frame, k) for k in ("records", "radius", "order", "tiles", "values", "ranges")}
    torch.cuda.synchronize()
    K, T = rast.stats(frame)["n_instances"], rast.stats(frame)["total_tiles"]
    rast.release_frame(frame)
    assert K > 16384 and T == ((w + 7) // 8) * ((h + 7) // 8)
    order, tiles = U.u32(ex["order"]), U.u32(ex["tiles"]).astype(np.int64)
    r = U.u32(ex["ranges"]).reshape(-1, 2).astype(np.int64)[:T]
    vals = U.u32(ex["values"]).astype(np.int64)[:K]
    length = r[:, 1] - r[:, 0]
    assert length.sum() == K and (length >= 0).all()
    cell = np.full(K, -1, np.int64)
    for c in np.flatnonzero(length):
        cell[r[c, 0]:r[c, 1]] = c
        assert (np.diff(vals[r[c, 0]:r[c, 1]]) > 0).all()
    assert (cell >= 0).all()
    rec = ex["records"].cpu().numpy().reshape(-1, 12).astype(np.float64)
    rad = ex["radius"].cpu().numpy().astype(np.float64)
    g = order[vals]
    gw, gh = (w + 7) // 8, (h + 7) // 8
    lo = lambda c, k: np.maximum(np.floor((rec[g, c] - rad[g]) / 8), 0)
    hi = lambda c, k: np.minimum(np.floor((rec[g, c] + rad[g]) / 8), k - 1)
    cx, cy = cell % gw, cell // gw
    assert ((cx >= lo(0, gw)) & (cx <= hi(0, gw)) & (cy >= lo(1, gh)) & (cy <= hi(1, gh))).all()
    if not cull:
        assert K == tiles.sum() and np.array_equal(np.bincount(g, minlength=n), tiles)


@pytest.mark.parametrize("size", [(60, 70), (300, 130), (1030, 520)])
@pytest.mark.parametrize("wide", [-1, 4, 40])
@pytest.mark.parametrize("n", [3, 64, 1500])
def test_lists_of_rectangles_around_the_cell_mask(size, wide, n):
    """Splats of a cell to the whole view: rectangles up to 64 cells go from
    the classification to the duplication as a mask, larger ones row by row.
    Without culling every cell of every rectangle is listed; with it the lists
    are the ones of the image: the same bits."""
    from paper_2412_20522_amd import maskgs as M
    from paper_2412_20522_amd.raster import Rasterizer
    w, h = size
    s = scenegen.small_scene(n, w, h, seed=920 + n, sh_degree=0, log_scale_mean=-2.5)
    s["log_scales"] += np.random.default_rng(1).uniform(-2, 3, (n, 1)).astype(np.float32)  # radii over 2 decades
    s["opacity_logits"][:] = -3.0
    dev = U.to_device(s)
    params = {k: dev[k] for k in U.PARAM_KEYS}
    img = []
    for cull in (0, 1):
        rast = Rasterizer(0, **_settings((8, 8), sh_degree=0, tile_cull=cull, wide_tiles=wide))
        frame = rast.acquire_frame()
        img.append(rast.forward(frame, params, dev["masks"], s["cameras"]).clone())
        ex = {k: M.mgs_frame_export(rast.ctx, frame, k) for k in ("tiles", "values", "ranges")}
        torch.cuda.synchronize()
        K = rast.stats(frame)["n_instances"]
        rast.release_frame(frame)
        if wide < 0 and cull == 0:
            assert K == int(U.u32(ex["tiles"]).astype(np.int64).sum())
        r = U.u32(ex["ranges"]).reshape(-1, 2).astype(np.int64)
        vals = U.u32(ex["values"]).astype(np.int64)[:K]
        r = r[r[:, 1] > r[:, 0]]
        assert (r[:, 1] - r[:, 0]).sum() == K
        step = np.diff(vals) > 0
        step[r[1:, 0] - 1] = True  # positions ascend within a cell
        assert step.all()
    assert torch.equal(img[0], img[1])


@pytest.mark.parametrize("n", [1, 255, 1023, 1025, 9000])
@pytest.mark.parametrize("shift", [0, 1])
def test_compaction_over_row_widths(n, shift):
    """Rows of one to four units and wider, of 16-, 8- and 4-byte units (the
    pointers off by one float too), around a workgroup's rows: the bits of
    boolean indexing, and nothing behind the kept rows."""
    from paper_2412_20522_amd import maskgs as M
    from paper_2412_20522_amd.raster import Rasterizer
    rast = Rasterizer(0)
    g = torch.Generator(device="cuda").manual_seed(n)
    keep = (torch.rand(n, generator=g, device="cuda") < 0.4).to(torch.int32)
    ins, outs = [], []
    for w in (1, 2, 3, 4, 5, 6, 8, 16, 20, 48, 49, 1030):
        ins.append(torch.randn(n * w + shift, generator=g, device="cuda")[shift:].view(n, w))
        outs.append(torch.full((n * w + shift,), -7.0, device="cuda")[shift:].view(n, w))
    kept = torch.zeros(1, dtype=torch.int64, device="cuda")
    M.mgs_compact_rows(rast.ctx, keep, ins, outs, n_kept=kept)
    k = int(keep.sum())
    assert int(kept) == k
    for a, b in zip(ins, outs):
        assert torch.equal(b[:k], a[keep.bool()]) and bool((b[k:] == -7.0).all())


@pytest.mark.parametrize("tile,ppt,batch", [((16, 16), 1, 256), ((16, 16), 2, 128), ((16, 8), 1, 32), ((32, 8), 1, 64),
                                            ((32, 8), 2, 128)])
@pytest.mark.parametrize("n", [1, 33, 700])
def test_backward_sums_over_the_waves_of_a_tile(tile, ppt, batch, n):
    """Large splats over 1,575 to 3,150 tiles, where the waves' totals meet in
    LDS, against the same view beside one whose tiles make every wave add its
    own: the same FP32 totals in FP64 sums, so gradients to a few roundings.
    Lists below and above a round of 32 entries and a batch."""
    from paper_2412_20522_amd.raster import Rasterizer
    w, h = 1000, 400
    s = scenegen.small_scene(n, w, h, seed=950 + n, sh_degree=1, log_scale_mean=-0.3, opacity_mean=-3.0)
    s["masks"][::4] = 0.0  # masked entries return dL/dM alone
    away = _big()
    away["viewmat"] = np.array(away["viewmat"], np.float64).reshape(4, 4)
    away["viewmat"][2, 3] -= 1e4  # everything behind this view: the tiles count, nothing is in them
    dl = np.random.default_rng(6).normal(size=3 * w * h).astype(np.float32)
    rast = Rasterizer(0)
    kw = dict(fwd_ppt=ppt, bwd_ppt=ppt, batch_depth=batch, wide_tiles=8)
    a, ga = _run(rast, s, s["cameras"], dl, **_settings(tile, **kw))
    b, gb = _run(rast, s, [s["cameras"][0], away], dl, **_settings(tile, **kw))
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    for k in ("means", "log_scales", "quats", "opacity_logits", "sh", "masks"):
        x, y = getattr(ga, k).cpu().numpy(), getattr(gb, k).cpu().numpy()
        assert U.rel_err(x, y) <= 1e-6 or np.abs(x - y).max() <= 1e-9, (k, U.rel_err(x, y))


@pytest.mark.parametrize("tile,ppt,batch", [((16, 16), 1, 32), ((16, 16), 2, 128), ((16, 16), 4, 256), ((8, 8), 1, 64),
                                            ((32, 8), 2, 64)])
@pytest.mark.parametrize("n", [1, 3, 5, 900])
def test_importance_of_the_tile_wide_kernels(tile, ppt, batch, n):
    """Lists shorter than a round of four entries, with remainders and over
    several batches, one to four waves to a tile: the scores are those of the
    kernels for small splats to FP32 sums in another order (at most 256 weights
    each: 256 x 2^-24), and the maxima the same bits."""
    from paper_2412_20522_amd.raster import Rasterizer
    s = scenegen.small_scene(n, 131, 77, seed=930 + n, sh_degree=0, log_scale_mean=-2.0, opacity_mean=-2.0)
    s["masks"][::5] = 0.5
    away = _big()
    away["viewmat"] = np.array(away["viewmat"], np.float64).reshape(4, 4)
    away["viewmat"][2, 3] -= 1e4  # everything behind this view: the tiles count, nothing is in them
    dev = U.to_device(s)
    params = {k: dev[k] for k in U.PARAM_KEYS}
    rast = Rasterizer(0, **_settings(tile, sh_degree=0, fwd_ppt=ppt, batch_depth=batch, stats=0))
    out = []
    for cams in ([s["cameras"][0]], [s["cameras"][0], away]):
        frame = rast.acquire_frame()
        img, isum, imax = rast.forward_importance(frame, params, dev["masks"], cams)
        torch.cuda.synchronize()
        rast.release_frame(frame)
        out.append((img[:3 * 131 * 77].cpu().numpy(), isum.cpu().numpy(), imax.cpu().numpy()))
    (i0, s0, m0), (i1, s1, m1) = out
    assert np.array_equal(i0, i1) and np.array_equal(m0, m1)
    assert (np.abs(s0 - s1) <= 256 * 2.0 ** -24 * np.abs(s0)).all() and (s0.max() > 0)


@pytest.mark.parametrize("persistent", [0, 1])
def test_tile_setup_in_one_workgroup_equals_several(persistent):
    """2048 tiles take the one-workgroup set-up; one tile more (a second view
    of one pixel) the two-kernel one: same images, also on a workspace fixed
    from each set-up's checkpoint count."""
    from paper_2412_20522_amd.raster import Rasterizer
    s = scenegen.small_scene(20_000, 1024, 512, seed=77, sh_degree=1, log_scale_mean=-2.5)
    dev = U.to_device(s)
    params = {k: dev[k] for k in U.PARAM_KEYS}
    rast = Rasterizer(0, **_settings((16, 16), persistent=persistent, wide_tiles=8))
    one = s["cameras"]
    two = one + [scenegen.orbit_camera(4.0, 10.0, 0.0, 1, 1)]
    out = []
    for cams in (one, two):
        frame = rast.acquire_frame()
        plain = rast.forward(frame, params, dev["masks"], cams)[:3 * 1024 * 512].clone()
        again = rast.forward(frame, params, dev["masks"], cams)[:3 * 1024 * 512].clone()  # measured order
        rast.reserve(frame, 1.0)
        fixed = rast.forward(frame, params, dev["masks"], cams)[:3 * 1024 * 512].clone()
        rast.check(frame)
        rast.reserve(frame, 0)
        rast.release_frame(frame)
        out += [plain, again, fixed]
    torch.cuda.synchronize()
    for x in out[1:]:
        assert torch.equal(x, out[0])


@pytest.mark.parametrize("n", [1, 255, 256, 16_384, 16_385, 300_001])
def test_mask_loss_and_gradient_over_the_reduction_variants(n):
    from paper_2412_20522_amd import maskgs as M
    from paper_2412_20522_amd.raster import Rasterizer
    rng = np.random.default_rng(n)
    m = (rng.uniform(size=n) < 0.6).astype(np.float32)
    y, d = rng.uniform(size=n).astype(np.float32), rng.normal(size=n).astype(np.float32)
    ctx = Rasterizer(0).ctx
    t = {k: torch.from_numpy(v).cuda() for k, v in (("m", m), ("y", y), ("d", d))}
    loss, loss2, out = torch.full((1,), -1.0, device="cuda"), torch.full((1,), -1.0, device="cuda"), \
        torch.empty(n, 2, device="cuda")
    M.mgs_mask_loss(ctx, t["m"], loss)
    M.mgs_mask_grad(ctx, t["d"], t["m"], t["y"], 0.5, 0.3, out, loss_m=loss2)
    torch.cuda.synchronize()
    want = m.astype(np.float64).mean() ** 2
    assert abs(loss.item() - want) <= 2e-7 * want and loss.item() == loss2.item()
    y64 = y.astype(np.float64)
    g = (d + 0.3 * 2.0 * m.sum(dtype=np.float64) / n ** 2) * y64 * (1.0 - y64) / 0.5
    o = out.cpu().numpy().astype(np.float64)
    # a few FP32 roundings of the sum and the product
    assert np.all(np.abs(o[:, 0] - g) <= 1e-6 * (np.abs(g) + np.abs(d) + 1.0)) and np.array_equal(o[:, 1], -o[:, 0])


@pytest.mark.parametrize("away", [False, True], ids=["small-splat", "tile-wide"])
def test_infinite_colours_reach_the_pixels_of_their_splats_only(away):
    """A splat of infinite colour makes the pixels it is blended into infinite,
    or NaN where its mask (its weight) is 0, and no others: in both kernels."""
    from paper_2412_20522_amd.raster import Rasterizer
    n, w, h = 400, 64, 48
    s = scenegen.small_scene(n, w, h, seed=961, sh_degree=1, log_scale_mean=-3.0, opacity_mean=-2.0)
    s["masks"][:] = 1.0
    s["masks"][1::2] = 0.0
    bad = np.array([10, 11, 200, 201])  # two of mask 1, two of mask 0
    cams = [s["cameras"][0]] + ([_big()] if away else [])
    dl = np.random.default_rng(8).normal(size=3 * w * h).astype(np.float32)
    rast = Rasterizer(0)
    ref, _ = _run(rast, s, cams, dl, **_settings((16, 16)))
    reach = []
    for k in bad:  # the pixels a splat is blended into, from the counters without it
        one = dict(s, opacity_logits=s["opacity_logits"].copy())
        one["opacity_logits"][k] = -20.0  # below the alpha filter
        a, _ = _run(rast, one, cams, dl, **_settings((16, 16)))
        reach.append(ref["stats"].reshape(-1, 4)[:, 1] > a["stats"].reshape(-1, 4)[:, 1])
        assert reach[-1].any() and not reach[-1].all()
    s["sh"][bad, 0] = np.inf
    b, _ = _run(rast, s, cams, dl, **_settings((16, 16)))
    img = b["image"].reshape(3, -1)
    nan = reach[1] | reach[3]
    inf = (reach[0] | reach[2]) & ~nan
    assert np.isnan(img[:, nan]).all() and np.isposinf(img[:, inf]).all()
    rest = ~(nan | inf)
    assert np.array_equal(img[:, rest], ref["image"].reshape(3, -1)[:, rest])
    assert np.array_equal(b["t_final"], ref["t_final"]) and np.array_equal(b["last"], ref["last"])


@pytest.mark.parametrize("n", [3, 500])
def test_small_splat_gradients_of_one_part_repeat_to_the_bit(n):
    """A view of one 8x8 part, where every FP64 sum has one term: the FP32 sums
    over the part's four waves do not depend on the order they finish in."""
    from paper_2412_20522_amd.raster import Rasterizer
    s = scenegen.small_scene(n, 8, 8, seed=962, sh_degree=1, log_scale_mean=-1.0, opacity_mean=-3.0)
    dl = np.random.default_rng(9).normal(size=3 * 64).astype(np.float32)
    rast = Rasterizer(0)
    first = None
    for _ in range(40):
        _, g = _run(rast, s, s["cameras"], dl, **_settings((8, 8)))
        got = {k: getattr(g, k).cpu().numpy() for k in ("means", "log_scales", "quats", "opacity_logits", "sh", "masks")}
        first = got if first is None else first
        for k, v in got.items():
            assert np.array_equal(v, first[k]), k


@pytest.mark.parametrize("waves", [4100, 4108, 4612, 4676, 4748, 4936, 4996, 5000, 5060, 5116, 5120, 5124, 9160])
def test_list_offsets_of_a_group_that_ends_within_a_wave(waves):
    """Numbers of positions whose last group of 1024 waves ends in each part of
    a 64-lane row of it, with few lanes there: every slot of the lists is
    filled, each record once per tile of its rectangle."""
    from paper_2412_20522_amd import maskgs as M
    from paper_2412_20522_amd.raster import Rasterizer
    n = 64 * waves - 37
    s = scenegen.small_scene(n, 70, 50, seed=970, sh_degree=0, log_scale_mean=-5.0)
    dev = U.to_device(s)
    rast = Rasterizer(0, **_settings((16, 16), sh_degree=0, tile_cull=0, wide_tiles=-1, stats=0))
    frame = rast.acquire_frame()
    rast.forward(frame, {k: dev[k] for k in U.PARAM_KEYS}, dev["masks"], s["cameras"])
    ex = {k: M.mgs_frame_export(rast.ctx, frame, k) for k in ("order", "tiles", "values", "ranges")}
    torch.cuda.synchronize()
    K = rast.stats(frame)["n_instances"]
    rast.release_frame(frame)
    tiles = U.u32(ex["tiles"]).astype(np.int64)
    vals, order = U.u32(ex["values"]).astype(np.int64)[:K], U.u32(ex["order"])
    assert K == tiles.sum() and vals.max() < n
    assert np.array_equal(np.bincount(order[vals], minlength=n), tiles)
    r = U.u32(ex["ranges"]).reshape(-1, 2).astype(np.int64)
    assert (r[:, 1] - r[:, 0]).sum() == K


@pytest.mark.parametrize("n", [1, 3, 300])
def test_few_records_over_many_tiles_leave_no_range_of_the_forward_before(n):
    """The duplication clears the cells' ranges, with workgroups beyond those
    of the records where there are many cells."""
    from paper_2412_20522_amd import maskgs as M
    from paper_2412_20522_amd.raster import Rasterizer
    w, h = 2000, 1100
    s = scenegen.small_scene(40_000, w, h, seed=980, sh_degree=0, log_scale_mean=-4.0)
    s["means"] *= 2.5  # over the whole view
    dev = U.to_device(s)
    few = {k: v[:n].contiguous() for k, v in dev.items() if torch.is_tensor(v)}
    rast = Rasterizer(0, **_settings((8, 8), sh_degree=0, tile_cull=0, wide_tiles=-1, stats=0))
    frame, fresh = rast.acquire_frame(), M.mgs_frame_create(rast.ctx)
    rast.forward(frame, {k: dev[k] for k in U.PARAM_KEYS}, dev["masks"], s["cameras"])
    r = U.u32(M.mgs_frame_export(rast.ctx, frame, "ranges")).reshape(-1, 2)
    assert (r[:, 1] > r[:, 0]).mean() > 0.5
    out = []
    for f in (frame, fresh):
        img = rast.forward(f, {k: few[k] for k in U.PARAM_KEYS}, few["masks"], s["cameras"])
        r = U.u32(M.mgs_frame_export(rast.ctx, f, "ranges")).reshape(-1, 2).astype(np.int64)
        assert (r[:, 1] - r[:, 0]).sum() == rast.stats(f)["n_instances"]
        out.append((img.cpu().numpy(), r))
    assert np.array_equal(out[0][0], out[1][0])
    assert np.array_equal(out[0][1], out[1][1])
    rast.release_frame(frame)
    rast.release_frame(fresh)
