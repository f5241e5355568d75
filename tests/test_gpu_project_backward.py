"""The projection backward splits a call's views over the waves of a block up
to 2^17 Gaussians: its gradients and statistics against the sums of the single
views' calls, which do not split."""
import numpy as np
import pytest

from paper_2410_16978_amd import scenes

pytestmark = pytest.mark.gpu

# Both sides round every output to float32 once or twice a call and are double
# inside (the colour gradient of a record is rounded equally on both), so they
# differ by a few 2^-24 of the views' terms; the mean's is a sum of a geometry
# and a colour term, each rounded, which can cancel.
RTOL, ATOL_OF_MAX = 2.0 ** -20, 1e-6


@pytest.mark.parametrize("n,n_views", [(1, 2), (63, 3), (64, 4), (65, 5), (1000, 2), (1000, 8), (1000, 9),
                                       (131072, 3), (131073, 3)])
def test_views_add_up(n, n_views):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_16978_amd import rasterizer as rz
    W, H = 150, 90
    sc = scenes.shell_scene(max(n, 4), 2, 1, seed=n, log_scale_mu=-3.0 if n < 10000 else -5.5, log_scale_sigma=0.4)
    keep = np.linspace(0, sc["layer"].shape[0] - 1, n).astype(int)
    sc = {k: (np.ascontiguousarray(v[..., keep]) if isinstance(v, np.ndarray) else v) for k, v in sc.items()}
    model = rz.to_device(sc)
    rng = np.random.default_rng(n_views)
    cams = [scenes.orbit_camera(scenes.random_direction(rng), W, H) for _ in range(n_views)]
    vs = scenes.view_state(3, bg=(0.1, 0.2, 0.3))
    gen = torch.Generator(device="cuda").manual_seed(1)
    g_rgb = torch.randn((n_views, 3, H, W), generator=gen, device="cuda")
    g_alpha = torch.randn((n_views, H, W), generator=gen, device="cuda")
    trainable = 3 if n == 1 else 2

    def run(first, last):
        c = cams[first:last]
        rgb, alpha, st = rz.rasterize_forward(model, c, [vs] * len(c))
        dens = (torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda"))
        g = rz.rasterize_backward(model, c, [vs] * len(c), st, g_rgb[first:last].reshape(rgb.shape).contiguous(),
                                  g_alpha[first:last].reshape(alpha.shape).contiguous(), trainable=trainable,
                                  densify=dens)
        g = dict(g, dens_grad=dens[0], dens_cnt=dens[1])
        return {k: v.cpu().numpy().astype(np.float64) for k, v in g.items()}

    together, single = run(0, n_views), [run(j, j + 1) for j in range(n_views)]
    for k, got in together.items():
        want, size = sum(s[k] for s in single), sum(np.abs(s[k]) for s in single)
        if k == "dens_cnt":
            assert np.array_equal(got, want)
        assert np.all(np.abs(got - want) <= RTOL * size + ATOL_OF_MAX * np.abs(size).max()), k
    assert max(np.abs(v).max() for v in together.values()) > 0
