"""The order-first pair lists (records sorted by depth, then paired and grouped
by tile) against the per-tile path on the same inputs: the pair capacity alone
chooses between them, so every product of the two - images, last indices,
ranges, sorted records and keys, emitted keys, boxes and all gradients - has to
agree bit for bit.  The per-tile path is pinned to the oracle elsewhere; one
case here compares the order-first products with the oracle too.  Sizes sit
at the edges of the kernels: one record, 64 and 1024 records and one more, a
pass block of 4096 records, more than one emission run and pair step, equal
depths, nothing visible, splats over the whole image, 65536 tiles and more."""
import numpy as np
import pytest

from paper_2410_16978_amd import scenes

pytestmark = pytest.mark.gpu

SMALL_CAP, ORDER_CAP = (3 << 16) - 1, 1 << 21


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _scene(n, seed, log_scale=-3.5, equal_depths=False):
    sc = scenes.shell_scene(max(n, 4), 2, 1, seed=seed, log_scale_mu=log_scale, log_scale_sigma=0.5)
    every = np.linspace(0, sc["layer"].shape[0] - 1, n).astype(int)  # of both layers
    sc = {k: (np.ascontiguousarray(v[..., every]) if isinstance(v, np.ndarray) else v) for k, v in sc.items()}
    if equal_depths:  # copies of a few Gaussians: many equal keys, kept in record order
        pick = np.arange(n) % 5
        sc = {k: (np.ascontiguousarray(v[..., pick]) if isinstance(v, np.ndarray) else v) for k, v in sc.items()}
        sc["opacity"] = np.ascontiguousarray(np.linspace(0.02, 0.2, n).astype(np.float32))
    return sc


def _products(model, cams, views, capacity):
    import torch
    from paper_2410_16978_amd import rasterizer as rz
    rgb, alpha, st, dbg = rz.rasterize_forward(model, cams, views, capacity=capacity, debug=True)
    K, kept = st.n_pairs, dbg["n_tiles"] != 0
    assert K <= capacity, "the capacity has to choose the path"
    sel = int(st.sort_sel.item())
    out = {"rgb": rgb, "alpha": alpha, "last": st.last, "ranges": st.ranges, "n_tiles": dbg["n_tiles"],
           "offsets": st.offsets, "records": st.records.view(-1, 12)[kept], "boxes": dbg["tile_box"][kept],
           "pairs": st.pair_vals[sel * st.capacity: sel * st.capacity + K], "keys_emit": dbg["keys_emit"][:K],
           "vals_emit": dbg["vals_emit"][:K], "keys_sorted": dbg["keys_sorted"][:K]}
    g = torch.Generator(device="cuda").manual_seed(3)
    contrib = torch.zeros(model["layer"].shape[0], device="cuda")
    grads = rz.rasterize_backward(model, cams, views, st, torch.randn(rgb.shape, generator=g, device="cuda"),
                                  torch.randn(alpha.shape, generator=g, device="cuda"), max_contrib=contrib)
    assert rz.forward_check(st) == K
    out.update({"grad_" + k: v for k, v in grads.items()}, contrib=contrib)
    return K, {k: v.cpu().numpy().view(np.uint8) for k, v in out.items()}


CASES = [
    # n, views, width, height, log-scale, equal depths, layer mask
    (1, 1, 40, 24, -2.0, False, 3),
    (64, 1, 100, 70, -3.0, False, 3),
    (65, 2, 333, 17, -3.0, False, 3),
    (1024, 1, 200, 120, -3.5, True, 3),
    (1025, 3, 130, 250, -3.5, False, 1),
    (4096, 1, 640, 480, -4.0, False, 3),
    (4097, 2, 1100, 1000, -4.5, False, 3),   # more than 4096 tiles
    (20000, 3, 300, 200, -4.5, False, 2),
    (9, 1, 1030, 1025, 0.5, False, 3),       # boxes of the whole image
    (3000, 1, 300, 200, -4.0, False, 4),     # no layer active: no pair
    (300, 1, 4112, 4100, -5.0, False, 3),    # 257 x 257 tiles: four-byte tile ids
    (600, 2, 4112, 4100, -5.0, False, 3),    # 2 x 66049 tiles: digits of nine bits
    (300, 4, 4112, 4112, -5.0, False, 3),    # 4 x 66049 tiles: three passes
]


@pytest.mark.parametrize("n,n_views,W,H,ls,equal,mask", CASES)
def test_order_first_equals_the_per_tile_path(n, n_views, W, H, ls, equal, mask):
    from paper_2410_16978_amd import rasterizer as rz
    rng = np.random.default_rng(n)
    model = rz.to_device(_scene(n, seed=n, log_scale=ls, equal_depths=equal))
    cams = [scenes.orbit_camera(scenes.random_direction(rng), W, H) for _ in range(n_views)]
    vs = scenes.view_state(mask, clips=[([0.3, -0.2, 1.0], 0.4, 0b10)], bg=(0.2, 0.1, 0.3))
    K0, per_tile = _products(model, cams, [vs] * n_views, SMALL_CAP)
    K1, ordered = _products(model, cams, [vs] * n_views, ORDER_CAP)
    assert K0 == K1 and (K1 == 0) == (mask == 4)
    for k, v in per_tile.items():
        np.testing.assert_array_equal(ordered[k], v, err_msg=f"{k} of n={n}")


def test_full_tiles_with_few_slots_a_record():
    """Full tiles are ordered first from as many pair slots as records, the
    boxes of all records then filling the emission array."""
    from paper_2410_16978_amd import rasterizer as rz
    cap = 3 << 16
    for n in (cap, cap - 1, 150_000):
        model = rz.to_device(_scene(n, seed=4, log_scale=-6.0))
        cam = scenes.orbit_camera(scenes.random_direction(np.random.default_rng(4)), 120, 100)
        vs = scenes.view_state(1, bg=(0.2, 0.1, 0.3))
        K0, per_tile = _products(model, [cam], [vs], cap - 1)
        K1, ordered = _products(model, [cam], [vs], cap)
        assert K0 == K1 > 0
        for k, v in per_tile.items():
            np.testing.assert_array_equal(ordered[k], v, err_msg=f"{k} of n={n}")


def test_order_first_matches_the_oracle(orc):
    from paper_2410_16978_amd import rasterizer as rz
    rng = np.random.default_rng(1)
    sc = _scene(6000, seed=1)
    cams = [scenes.orbit_camera(scenes.random_direction(rng), 320, 200) for _ in range(2)]
    vs = [scenes.view_state(3, bg=(0.2, 0.1, 0.3))] * 2
    rgb, alpha, st, dbg = rz.rasterize_forward(rz.to_device(sc), cams, vs, capacity=ORDER_CAP, debug=True)
    ref = orc.render(sc, cams, vs, pairs=True, n_threads=0)
    K, sel = st.n_pairs, int(st.sort_sel.item())
    assert K == ref["counts"]["K"]
    np.testing.assert_array_equal(dbg["keys_sorted"][:K].cpu().numpy().view(np.uint64), ref["keys"])
    np.testing.assert_array_equal(st.pair_vals.cpu().numpy().view(np.uint32)[sel * st.capacity:][:K], ref["vals"])
    np.testing.assert_array_equal(st.ranges.cpu().numpy().view(np.uint32).reshape(-1, 2), ref["ranges"])
    ok = ref["margin"] >= 1
    assert np.abs(rgb.cpu().numpy() - ref["rgb"]).max(axis=1)[ok].max() <= 1e-4


def test_batch_cut_at_a_request():
    """A batch whose later requests do not fit: order-first and per-tile mark
    the same requests and draw the same images."""
    from paper_2410_16978_amd import rasterizer as rz
    rng = np.random.default_rng(5)
    model = rz.to_device(_scene(30000, seed=5, log_scale=-2.5))
    vs = scenes.view_state(3, bg=(0.1, 0.2, 0.3))
    reqs = [{"model": 0, "cams": [scenes.orbit_camera(scenes.random_direction(rng), 400, 320)], "view": vs}
            for _ in range(6)]
    cap = 1 << 21
    out, status, _ = rz.render_batch([model], reqs, cap)
    fits = status.cpu().numpy()
    assert fits[0] == 0 and fits[-1] == rz.GSR_ENOSPACE, fits
    for q in range(len(reqs)):
        if fits[q]:
            continue
        rgb, alpha, st = rz.rasterize_forward(model, reqs[q]["cams"], [vs], capacity=1_000_000)
        np.testing.assert_array_equal(out[q][0][0].cpu().numpy(), rgb[0].cpu().numpy())
        np.testing.assert_array_equal(out[q][1][0].cpu().numpy(), alpha[0].cpu().numpy())
