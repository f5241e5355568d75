"""Which path a call takes: records ordered before they are paired, or pairs
sorted by tile.  The stage timer shows it; that both give the same products is
tested elsewhere."""
import numpy as np
import pytest

from paper_2410_16978_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _inputs(n, n_views, W, H, ls, mask):
    from paper_2410_16978_amd import rasterizer as rz
    sc = scenes.shell_scene(max(n, 4), 2, 1, seed=n, log_scale_mu=ls, log_scale_sigma=0.5)
    every = np.linspace(0, sc["layer"].shape[0] - 1, n).astype(int)
    sc = {k: (np.ascontiguousarray(v[..., every]) if isinstance(v, np.ndarray) else v) for k, v in sc.items()}
    rng = np.random.default_rng(n)
    cams = [scenes.orbit_camera(scenes.random_direction(rng), W, H) for _ in range(n_views)]
    vs = scenes.view_state(mask, clips=[([0.3, -0.2, 1.0], 0.4, 0b10)], bg=(0.2, 0.1, 0.3))
    return rz.to_device(sc), cams, [vs] * n_views


@pytest.mark.parametrize("n,n_views,W,H,slots,by_tile", [
    (500, 1, 160, 160, (3 << 16) - 1, True), (500, 1, 160, 160, 2048 * 100, False),  # 100 tiles: full
    (500, 1, 160, 160, 3 << 16, True),                                               # not quite
    (500, 1, 800, 800, (1 << 21) - 1, True), (500, 1, 800, 800, 1 << 21, False),     # 2500 tiles
    (500, 1, 1100, 1000, (1 << 20) - 1, True), (500, 1, 1100, 1000, 1 << 20, False),  # 4347 tiles
    (99_000, 4, 200, 200, 1_142_854, True), (500, 4, 200, 200, 2048 * 676, False),   # 676 tiles of 1691 and 2048 slots
    (200_000, 1, 160, 160, 200_000, True), (200_000, 1, 160, 160, 2048 * 100, False),  # boxes fit from a slot a record
    (500_000, 1, 1100, 1000, 999_999, True), (600_000, 1, 1100, 1000, 1_200_000, False),
])
def test_by_slots(n, n_views, W, H, slots, by_tile):
    from paper_2410_16978_amd import rasterizer as rz
    model, cams, views = _inputs(n, n_views, W, H, -6.0, 3)
    timer = rz.Timer()
    st = rz.make_state(n, n_views, W, H, slots)
    rz.rasterize_forward(model, cams, views, state=st, sync=False, timer=timer)
    assert (timer.read()["duplicate"][1] == 1) == by_tile
