"""The blend backward's blocks take more than one batch of pairs once more than
32768 batches were evaluated: three equal views whose batches together pass
that number against one of them, which stays below."""
import numpy as np
import pytest

from paper_2410_16978_amd import scenes

pytestmark = pytest.mark.gpu

# Every view adds the same double to each sum; what differs is the rounding of
# three terms and of the result to float32 (the colour terms are summed in
# float32): at most a few 2^-24 of the value, plus double rounding of sums
# that cancel.
RTOL, ATOL_OF_MAX = 2.0 ** -20, 1e-9


@pytest.mark.parametrize("W,H", [(2048, 1760), (1761, 2040)])
def test_more_batches_than_blocks(W, H):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_16978_amd import rasterizer as rz
    sc = scenes.shell_scene(12, 2, 1, seed=5, log_scale_mu=0.5, log_scale_sigma=0.3)
    sc["opacity"] = np.full_like(sc["opacity"], 0.3)
    model = rz.to_device(sc)
    cam = scenes.orbit_camera(scenes.random_direction(np.random.default_rng(2)), W, H)
    vs = scenes.view_state(3, bg=(0.1, 0.2, 0.3))
    gen = torch.Generator(device="cuda").manual_seed(1)
    g_rgb = torch.rand((1, 3, H, W), generator=gen, device="cuda")
    g_alpha = torch.rand((1, H, W), generator=gen, device="cuda")
    got = []
    for n in (1, 3):
        rgb, alpha, st = rz.rasterize_forward(model, [cam] * n, [vs] * n)
        seen = alpha.reshape(n, H, W)[:, ::16, ::16] > 0  # a pixel of each tile: its batch is evaluated
        assert (int(seen.sum()) > 32768) == (n == 3)
        contrib = torch.zeros(model["layer"].shape[0], device="cuda")
        g = rz.rasterize_backward(model, [cam] * n, [vs] * n, st, g_rgb.repeat(n, 1, 1, 1),
                                  g_alpha.repeat(n, 1, 1), max_contrib=contrib)
        got.append(({k: v.cpu().numpy().astype(np.float64) for k, v in g.items()}, contrib.cpu().numpy()))
    assert np.array_equal(got[0][1], got[1][1])
    for k, one in got[0][0].items():
        want = 3.0 * one
        assert np.abs(want).max() > 0, k
        np.testing.assert_allclose(got[1][0][k], want, rtol=RTOL, atol=ATOL_OF_MAX * np.abs(want).max(), err_msg=k)
