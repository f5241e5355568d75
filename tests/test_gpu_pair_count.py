"""What a call reports of its pair count: totals beyond 32 bits are an overflow
of the capacity, not counted modulo 2^32, and a batch marks exactly the
requests whose pairs end beyond the capacity."""
import numpy as np
import pytest

from paper_2410_16978_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _screen_filling(n, W, H):
    """n splats whose boxes are the whole image."""
    import torch
    model = {"mean": torch.zeros((3, n), device="cuda"), "scale": torch.full((3, n), 0.5, device="cuda"),
             "quat": torch.zeros((4, n), device="cuda"), "opacity": torch.full((n,), 0.5, device="cuda"),
             "sh": torch.zeros((1, 3, n), device="cuda"), "layer": torch.zeros(n, dtype=torch.uint8, device="cuda"),
             "sh_degree": 0}
    model["quat"][0] = 1.0
    cam = scenes.orbit_camera(np.array([0.0, 0.0, -1.0]), W, H)
    cam["fx"] = cam["fy"] = 1e6
    return model, cam


# The blocks' totals of the scan are exact powers of two: 8192 records of 2^19
# tiles, and (the longer blocks of calls above 4M records) 32768 of 2^17; the
# third pairs its records unsorted.
@pytest.mark.parametrize("n,W,H,capacity", [(8192, 16384, 8192, 1 << 20), ((1 << 22) + (1 << 15), 8192, 4096, 9 << 20),
                                            (8192, 16384, 8192, 1 << 13)])
def test_totals_beyond_32_bits(n, W, H, capacity):
    from paper_2410_16978_amd import rasterizer as rz
    model, cam = _screen_filling(n, W, H)
    st = rz.make_state(n, 1, W, H, capacity)
    rgb, alpha, st = rz.rasterize_forward(model, [cam], [scenes.view_state()], state=st, sync=False)
    K = int(st.counters[0].item()) & 0xFFFFFFFF
    off = st.offsets.cpu().numpy().view(np.uint32).astype(np.int64)
    with pytest.raises(rz.GsrError) as e:
        rz.forward_check(st)
    assert e.value.status == rz.GSR_ENOSPACE
    assert K == 0xFFFFFFFF  # the count, as far as its word holds it
    tiles = (W // 16) * (H // 16)
    np.testing.assert_array_equal(off, np.minimum(np.arange(n + 1, dtype=np.int64) * tiles, 0xFFFFFFFF))


@pytest.mark.parametrize("capacity", [1 << 20, 1 << 13])
def test_batch_total_beyond_32_bits(capacity):
    from paper_2410_16978_amd import rasterizer as rz
    model, cam = _screen_filling(8192, 16384, 8192)
    small, cam2 = _screen_filling(7, 160, 160)
    reqs = [{"model": 1, "cams": [cam2], "view": scenes.view_state()},
            {"model": 0, "cams": [cam], "view": scenes.view_state()}]
    _, status, _ = rz.render_batch([model, small], reqs, capacity)
    assert status.cpu().tolist() == [0, rz.GSR_ENOSPACE]


@pytest.mark.parametrize("capacity", [1 << 21, 1 << 18])  # records ordered first, pairs sorted by tile
def test_batch_status_is_the_running_sum(capacity):
    from paper_2410_16978_amd import rasterizer as rz
    rng = np.random.default_rng(5)
    n = 30000 if capacity > 1 << 20 else 9000
    sc = scenes.shell_scene(n // 2, 2, 1, seed=5, log_scale_mu=-2.5, log_scale_sigma=0.5)
    model, vs = rz.to_device(sc), scenes.view_state(3, bg=(0.1, 0.2, 0.3))
    reqs, ends = [], []
    for q in range(6):
        W, H = ((400, 320), (160, 90), (333, 200))[q % 3]
        cams = [scenes.orbit_camera(scenes.random_direction(rng), W, H)]
        reqs.append({"model": 0, "cams": cams, "view": vs})
        ends.append((ends[-1] if ends else 0) + rz.rasterize_forward(model, cams, [vs])[2].n_pairs)
    assert ends[0] <= capacity < ends[-1], ends
    _, status, _ = rz.render_batch([model], reqs, capacity)
    assert status.cpu().tolist() == [0 if e <= capacity else rz.GSR_ENOSPACE for e in ends], ends
    exact = ends[2]  # a capacity that a request's pairs fill to the last slot, and one less
    for cap in (exact, exact - 1):
        _, status, _ = rz.render_batch([model], reqs, cap)
        assert status.cpu().tolist() == [0 if e <= cap else rz.GSR_ENOSPACE for e in ends], (cap, ends)
