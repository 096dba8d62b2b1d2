"""Host-only checks of the PowerSGD plan: which tiles a configuration gets, and in which workspace (CPU only)."""
import ctypes as C
import os

import pytest

from paper_2010_16248_amd import binding as B
from paper_2010_16248_amd import workloads as wl
from tests import helpers as H


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(B.LIB_PATH):
        from paper_2010_16248_amd import build
        build.build(verbose=False)
    return B.load_library()


@pytest.mark.parametrize("name,shapes,W,heights", [
    ("tiny", wl.tiny4_shapes(), 2, (16, 32)),
    ("tiny_w8", wl.tiny4_shapes(), 8, (16, 64)),
    ("tiny_w16", wl.tiny4_shapes(), 16, (16, 128)),
    ("resnet18_w1", wl.resnet18_shapes(), 1, (16, 128)),
    ("resnet18_w4", wl.resnet18_shapes(), 4, (32, 128)),
    ("vgg19_w1", wl.vgg19bn_shapes(), 1, (32, 128)),
    # the lines: 2048 workgroups of 32-row tiles; 256 workgroups of the right product, at 128 and at 64 rows
    ("flat_2048", [(32 * 1024, 4, 1)], 2, (16, 128)),
    ("flat_2049", [(32 * 2049, 4, 1)], 1, (32, 128)),
    ("right_256", [(128 * 256, 4, 1)], 1, (16, 128)),
    ("right_255", [(128 * 255, 4, 1)], 1, (16, 64)),
    ("right_64_256", [(64 * 256, 4, 1), (1, 99, 0)], 1, (16, 64)),
    ("right_64_255", [(64 * 255, 4, 1), (1, 99, 0)], 1, (16, 32)),
    ("one_element", [(1, 1, 1)], 1, (16, 32)),
])
def test_tile_heights(lib, name, shapes, W, heights):
    layers = wl.make_layers(shapes)
    cfg, keep = B.make_config(B.ACC_POWERSGD, layers, W, 4, 1)
    assert B.accordion_workspace_bytes(cfg) == H.powersgd_workspace_bytes(layers, W, 4, *heights), name


@pytest.mark.parametrize("name,shapes,W", [
    ("tiny", wl.tiny4_shapes(), 2), ("resnet18", wl.resnet18_shapes(), 1), ("resnet18_w4", wl.resnet18_shapes(), 4),
    ("ragged", [(r, c, 1) for r, c in ((17, 3), (129, 255), (33, 259), (700, 1300))] + [(1, 1031, 0)], 3),
])
def test_a_workspace_that_holds_only_the_tallest_tiles_is_accepted(lib, name, shapes, W):
    """64 and 128 rows need the least workspace.  The call stops at the missing start of Q, which comes after the
    size of the workspace: no device work."""
    layers = wl.make_layers(shapes)
    cfg, keep = B.make_config(B.ACC_POWERSGD, layers, W, 4, 1)
    least = H.powersgd_workspace_bytes(layers, W, 4, 64, 128)
    assert least < B.accordion_workspace_bytes(cfg)
    ctx = C.c_void_p(None)
    for nbytes, rc, words in ((least, B.ACC_EINVAL, "q_init_host"), (least - 256, B.ACC_ENOSPACE, "too small")):
        assert lib.accordion_init(C.byref(cfg), C.c_void_p(256), nbytes, None, None, C.byref(ctx)) == rc, name
        assert words in lib.accordion_last_error(None).decode()
