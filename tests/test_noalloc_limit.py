"""The most pair slots gsr_rasterize_forward_noalloc takes for some sizes: one
more is refused on the host, before any launch.  The numbers are those of the
bytes a pair, a record and a Gaussian have taken of the library's scratch since
the entry point exists; a path that needs less does not move them."""
import ctypes as C

import pytest

from paper_2410_16978_amd import rasterizer as rz

LIMITS = [
    # n, views, width, height, shared order, slots
    (1000, 1, 64, 48, False, 2793504), (1000, 1, 64, 48, True, 2790208),
    (200_000, 2, 640, 480, False, 2447872), (200_000, 2, 640, 480, True, 1830240),
    (200_000, 2, 1100, 1025, False, 2629696), (200_000, 2, 1100, 1025, True, 1955936),
    (400_000, 1, 800, 800, False, 2447200), (400_000, 1, 800, 800, True, 1612928),
    (400_000, 2, 160, 160, True, 892672), (900_000, 1, 640, 480, True, 161728),
    (600_000, 2, 1832, 1920, False, 1787296), (600_000, 2, 1832, 1920, True, 0),
]


@pytest.mark.parametrize("n,views,width,height,shared,limit", LIMITS)
def test_limit(n, views, width, height, shared, limit):
    import torch
    if torch.cuda.is_available():
        pytest.skip("the buffers here are addresses only")
    tiles = views * ((width + 15) // 16) * ((height + 15) // 16)

    def call(slots):
        model = rz.Model(n, 3, *[256] * 6)
        state = rz.FwdState(*[256] * 11, slots, int(rz.lib().gsr_batch_capacity(slots, tiles)))
        cams, states = (rz.Camera * views)(), (rz.ViewState * views)()
        for cam, vs in zip(cams, states):
            cam.fx, cam.fy, cam.width, cam.height = 500.0, 500.0, width, height
            vs.sort_shared = int(shared)
        return rz.lib().gsr_rasterize_forward_noalloc(C.byref(model), views, cams, states, C.byref(state), 256, 256,
                                                      None, None)

    assert call(limit + 1) == rz.GSR_ENOSPACE
    if limit:
        assert call(limit) == rz.GSR_EHIP  # taken: the first call of the device fails, there being none
