"""Which path a call takes: records ordered before they are paired, or pairs
sorted by tile.  The stage timer shows it.  A call that reads its pair count
back and finds too few pairs for its slots turns from the first path to the
second after the projection: its products - images, last indices, ranges, pair
lists, all gradients - equal those of a call that goes by its slots and of one
that sorts by tile from the start, bit for bit."""
import numpy as np
import pytest

from paper_2410_16978_amd import scenes

pytestmark = pytest.mark.gpu


SMALL_CAP, ORDER_CAP = (3 << 16) - 1, 1 << 21

CASES = [
    # n, views, width, height, log-scale, layer mask
    (1, 1, 400, 240, -2.0, 3),
    (65, 2, 333, 170, -3.0, 3),
    (1025, 3, 130, 250, -3.5, 1),
    (20000, 3, 300, 200, -4.5, 2),
    (4097, 2, 1100, 1000, -4.5, 3),  # more than 4096 tiles: radix passes, their look-back words cleared late
    (9, 1, 1030, 1025, 0.5, 3),      # boxes of the whole image
    (3000, 1, 300, 230, -4.0, 4),    # no layer active: no pair
    (300, 1, 4112, 4100, -5.0, 3),   # 257 x 257 tiles: boxes of eight bytes
    (600, 2, 4112, 4100, -5.0, 3),   # 2 x 66049 tiles
]


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
    (500, 1, 256, 256, 2048 * 256 - 1, True), (500, 1, 256, 256, 2048 * 256, False),  # 256 tiles
    (200_000, 1, 300, 300, 787_326, True), (99_000, 4, 200, 200, 1_142_854, True),   # 361 and 676 tiles
    (500, 4, 200, 200, 3072 * 676 - 1, True), (500, 4, 200, 200, 3072 * 676, False),
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


def _run(model, cams, views, capacity, sync):
    import torch
    from paper_2410_16978_amd import rasterizer as rz
    n, V, W, H = model["layer"].shape[0], len(cams), cams[0]["width"], cams[0]["height"]
    st = rz.make_state(n, V, W, H, capacity)
    st.workspace.fill_(255)
    timer = rz.Timer()
    rgb, alpha, st = rz.rasterize_forward(model, cams, views, state=st, sync=sync, timer=timer)
    K = rz.forward_check(st)
    by_tile = timer.read()["duplicate"][1] == 1
    assert st.capacity == capacity and st.n_pairs == (K if sync else None)
    sel = int(st.sort_sel.item())
    g = torch.Generator(device="cuda").manual_seed(3)
    contrib = torch.zeros(n, device="cuda")
    out = {"rgb": rgb, "alpha": alpha, "last": st.last, "ranges": st.ranges, "offsets": st.offsets,
           "pairs": st.pair_vals[sel * capacity: sel * capacity + K].clone()}
    grads = rz.rasterize_backward(model, cams, views, st, torch.randn(rgb.shape, generator=g, device="cuda"),
                                  torch.randn(alpha.shape, generator=g, device="cuda"), max_contrib=contrib)
    out.update({"grad_" + k: v for k, v in grads.items()}, contrib=contrib)
    return by_tile, K, {k: v.cpu().numpy().view(np.uint8) for k, v in out.items()}


def _assert_same(got, want, label):
    for k, v in want.items():
        np.testing.assert_array_equal(got[k], v, err_msg=f"{label}: {k}")


@pytest.mark.parametrize("n,n_views,W,H,ls,mask", CASES)
def test_a_turned_call(n, n_views, W, H, ls, mask):
    args = _inputs(n, n_views, W, H, ls, mask)
    by_tile, K, turned = _run(*args, ORDER_CAP, True)
    assert by_tile and (K == 0) == (mask == 4)
    by_tile, K1, by_slots = _run(*args, ORDER_CAP, False)
    assert not by_tile and K1 == K
    by_tile, K2, from_start = _run(*args, SMALL_CAP, False)
    assert by_tile and K2 == K
    _assert_same(turned, by_slots, "by slots")
    _assert_same(turned, from_start, "by tile")


@pytest.mark.parametrize("n,n_views,W,H,ls", [
    (4000, 2, 240, 240, 1.0),                           # 450 tiles, full
    (65, 2, 333, 17, -3.0), (500, 1, 256, 256, -3.0)])  # few pairs, but no more than 256 tiles
def test_a_call_that_stays(n, n_views, W, H, ls):
    args = _inputs(n, n_views, W, H, ls, 3)
    by_tile, K, synced = _run(*args, ORDER_CAP, True)
    tiles = n_views * ((W + 15) // 16) * ((H + 15) // 16)
    assert not by_tile and (tiles <= 256 or K >= 3072 * tiles)
    by_tile, _, by_slots = _run(*args, ORDER_CAP, False)
    assert not by_tile
    _assert_same(synced, by_slots, "by slots")


def test_without_a_workspace():
    """The no-allocation forward's layout has no backward behind it."""
    import torch
    from paper_2410_16978_amd import rasterizer as rz
    model, cams, views = _inputs(20000, 2, 300, 150, -4.5, 3)
    cap = 1_200_000  # full by its slots: 380 tiles, two slots a record and more
    got = []
    for sync in (True, False):
        st = rz.make_state(20000, 2, 300, 150, cap)
        out = (torch.empty((2, 3, 150, 300), device="cuda"), torch.empty((2, 150, 300), device="cuda"))
        rgb, alpha, st = rz.rasterize_forward_noalloc(model, cams, views, st, out, n_pairs=sync)
        g = rz.rasterize_backward(model, cams, views, st, torch.ones_like(rgb), torch.ones_like(alpha))
        assert 0 < rz.forward_check(st) < 3 << 16
        got.append({k: v.cpu().numpy().view(np.uint8) for k, v in dict(g, rgb=rgb, alpha=alpha).items()})
    _assert_same(got[0], got[1], "noalloc")
