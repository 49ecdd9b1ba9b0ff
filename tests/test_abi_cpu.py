"""C-ABI checks that need no GPU: the library loads, exports every entry
point the header declares, and rejects bad arguments on the host before
touching a device."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "maskgs.h")


def _declared():
    txt = open(HEADER).read()
    return sorted(set(re.findall(r"MGS_API\s+[\w\s\*]+?\b(mgs_\w+)\s*\(", txt)))


def _lib():
    from paper_2412_20522_amd import maskgs
    return maskgs


def test_header_declares_entry_points():
    names = _declared()
    for must in ("mgs_create", "mgs_forward", "mgs_backward", "mgs_project", "mgs_scan", "mgs_duplicate",
                 "mgs_sort", "mgs_tile_ranges", "mgs_project_backward", "mgs_sample_masks", "mgs_mask_loss",
                 "mgs_mask_grad", "mgs_l1_loss_grad", "mgs_adam_step", "mgs_adam_step_multi", "mgs_scan_noalloc"):
        assert must in names


def test_library_exports_every_declared_symbol():
    M = _lib()
    raw = C.CDLL(M.LIB_PATH)
    for name in _declared():
        assert hasattr(raw, name), name
    # and the binding wraps every declared symbol under the same name
    assert set(_declared()) == set(M.EXPORTED)


def test_default_settings_and_version():
    M = _lib()
    s = M.mgs_default_settings()
    assert (s.tile_w, s.tile_h, s.batch_depth) == (16, 16, 256)
    assert abs(s.alpha_min - 1 / 255) < 1e-9 and abs(s.alpha_max - 0.99) < 1e-7
    assert abs(s.t_min - 1e-4) < 1e-10 and s.q_max == 9.0
    assert M.mgs_version() >= 200


def test_struct_layouts_match_header():
    M = _lib()
    assert C.sizeof(M.mgs_camera) == 16 * 4 + 4 * 4 + 2 * 4
    assert C.sizeof(M.mgs_settings) == 4 * 4 + 8 * 4 + 3 * 4 + 8 * 4
    assert C.sizeof(M.mgs_eval_counts) == 6 * 8
    assert C.sizeof(M.mgs_gaussians) == 6 * 8 + 8
    assert C.sizeof(M.mgs_gradients) == 7 * 8 + 8
    assert C.sizeof(M.mgs_adam_array) == 5 * 8 + 8


def test_host_validation_without_device():
    M = _lib()
    L = M.lib()
    # NULL context / NULL outputs are rejected before any device call
    assert L.mgs_create(0, None) == 1
    assert L.mgs_frame_create(None, None) == 1
    assert L.mgs_scan(None, None, None, 0, None, None, None) == 1
    assert L.mgs_sort(None, None, None, None, 0, 40, None, None, None) == 1
    assert L.mgs_sample_masks(None, None, None, 0, 0.5, 0, 0, None, None, None) == 1
    assert L.mgs_mask_loss(None, None, None, 0, None, None) == 1
    assert L.mgs_adam_step_multi(None, None, None, 0, 0.9, 0.999, 1e-15, 1, None) == 1
    assert L.mgs_step_advance(None, None, None, 1) == 1
    assert L.mgs_scan_noalloc(None, None, None, 0, None, None) == 1
    assert L.mgs_default_settings(None) == 1
    assert L.mgs_scan_scratch_bytes(10_000) > 0
    assert L.mgs_sort_scratch_bytes(1_000_000) > L.mgs_sort_scratch_bytes(1000)


def test_noalloc_scan_limit_matches_its_scratch():
    txt = open(HEADER).read()
    nbytes = int(re.search(r"#define MGS_SCAN_NOALLOC_BYTES (\d+)", txt).group(1))
    max_n = int(re.search(r"#define MGS_SCAN_NOALLOC_MAX_N (\d+)", txt).group(1))
    # (blocks + 1) u64 partial sums and 256 bytes, blocks of 4096 elements
    assert max_n == ((nbytes - 256) // 8 - 1) * 4096
    assert _lib().SCAN_NOALLOC_MAX_N == max_n


def test_create_fails_cleanly_without_gfx950():
    import torch
    if torch.cuda.is_available():
        pytest.skip("a GPU is present")
    M = _lib()
    with pytest.raises(M.MaskGSError):
        M.mgs_create(0)
    assert M.mgs_last_error(None)


def test_library_queues_nothing_on_the_null_stream():
    """Every fill and copy names the caller's stream: one on the null stream is
    not ordered with a caller's non-blocking stream."""
    src = os.path.join(ROOT, "paper_2412_20522_amd", "csrc")
    for name in sorted(os.listdir(src)):
        txt = re.sub(r"//[^\n]*", "", open(os.path.join(src, name)).read())
        assert not re.search(r"\bhip(Memset|Memcpy)(D8|D16|D32|2D|3D|DtoD|DtoH|HtoD|ToSymbol|FromSymbol)?\s*\(", txt), name


@pytest.mark.parametrize("change", [{}, {"fx": 1e39}, {"cy": -1e300}, {"cx": float("nan")}, {"fy": float("inf")},
                                    {"width": 2 ** 33 + 5}, {"height": -2 ** 40}, {"width": -1, "cx": 4e38}])
def test_camera_values_beyond_the_struct_convert_as_ctypes_does(change):
    import numpy as np
    M = _lib()
    rng = np.random.default_rng(3)
    cam = dict(viewmat=rng.normal(size=(4, 4)), fx=100.0, fy=101.5, cx=64.0, cy=32.25, width=128, height=64)
    cam.update(change)
    got, want = M.camera_struct(cam), M.mgs_camera()
    for i, v in enumerate(np.asarray(cam["viewmat"], np.float32).reshape(16)):
        want.viewmat[i] = float(v)
    want.fx, want.fy, want.cx, want.cy = (float(cam[k]) for k in ("fx", "fy", "cx", "cy"))
    want.width, want.height = cam["width"], cam["height"]
    # (the bytes of two NaN may differ)
    assert [np.float32(v).tobytes() if v == v else "nan" for v in [*got.viewmat, got.fx, got.fy, got.cx, got.cy]] == \
           [np.float32(v).tobytes() if v == v else "nan" for v in [*want.viewmat, want.fx, want.fy, want.cx, want.cy]]
    assert (got.width, got.height) == (want.width, want.height)
