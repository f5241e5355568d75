"""A culled Gaussian's record is not written, so what its memory held before a
call must not reach an image or a gradient: with Gaussian 0 hidden, calls on
buffers filled with 0xFF bytes (a NaN in every float) equal calls on zeroed
ones bit for bit, on one tile of N pairs around the 256-pair batches (the last
batch is partial, and so is the last step of four of a wave's list)."""
import numpy as np
import pytest

from paper_2410_16978_amd import scenes
from tests.helpers import axis_camera, make_scene

pytestmark = pytest.mark.gpu

N_PAIRS = (1, 2, 3, 255, 257, 509)
CAPACITIES = (1 << 12, 1 << 21)  # pairs sorted by tile, records ordered first


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _tile(n):
    """Gaussian 0 in layer 0, n faint ones in layer 1, all in one tile."""
    rng = np.random.default_rng(n)
    z = rng.uniform(2.0, 4.0, n + 1)
    xy = rng.uniform(-0.1, 0.1, (n + 1, 2)) * z[:, None]
    cam = axis_camera(16, 16, f=20.0, cx=8.0, cy=8.0)
    sc = make_scene(np.column_stack([xy, z]), np.exp(rng.normal(-2.0, 0.4, (n + 1, 3))),
                    quats=rng.standard_normal((n + 1, 4)), opacity=rng.uniform(0.005, 0.02, n + 1),
                    rgb=rng.uniform(0, 1, (n + 1, 3)))
    sc["layer"] = np.r_[0, np.ones(n)].astype(np.uint8)
    scenes.enforce_distinct_depths(sc, [cam])
    return sc, cam, scenes.view_state(0b10, bg=(0.1, 0.2, 0.3))


@pytest.mark.parametrize("capacity", CAPACITIES)
@pytest.mark.parametrize("n", N_PAIRS)
def test_forward_and_backward(n, capacity):
    import torch
    from paper_2410_16978_amd import rasterizer as rz
    sc, cam, vs = _tile(n)
    model = rz.to_device(sc)
    gen = torch.Generator(device="cuda").manual_seed(n)
    g_rgb = torch.randn((1, 3, 16, 16), generator=gen, device="cuda")
    g_alpha = torch.randn((1, 16, 16), generator=gen, device="cuda")
    rz.rasterize_forward(model, [cam], [scenes.view_state(0b11)])  # leaves longer lists behind
    got = []
    for byte in (0, 255):
        st = rz.make_state(n + 1, 1, 16, 16, capacity)
        st.records.view(torch.uint8).fill_(byte)
        st.workspace.fill_(byte)
        rgb, alpha, st = rz.rasterize_forward(model, [cam], [vs], state=st)
        assert st.n_pairs == n and st.capacity == capacity
        contrib, activity = torch.zeros(n + 1, device="cuda"), torch.zeros(n + 1, device="cuda")
        g = rz.rasterize_backward(model, [cam], [vs], st, g_rgb, g_alpha, max_contrib=contrib, activity=activity)
        out = dict(g, rgb=rgb, alpha=alpha, last=st.last, pixels=st.pixel_state, contrib=contrib, activity=activity)
        got.append({k: v.cpu().numpy() for k, v in out.items()})
    for k, want in got[0].items():
        assert np.isfinite(want).all(), k
        np.testing.assert_array_equal(got[1][k].view(np.uint8), want.view(np.uint8), err_msg=k)


@pytest.mark.parametrize("capacity", CAPACITIES)
def test_batch(capacity):
    import torch
    from paper_2410_16978_amd import rasterizer as rz
    parts = [_tile(n) for n in N_PAIRS]
    models = [rz.to_device(sc) for sc, _, _ in parts]
    reqs = [{"model": q, "cams": [cam], "view": vs} for q, (_, cam, vs) in enumerate(parts)]
    _, _, ws = rz.render_batch(models, reqs, capacity)
    got = []
    for byte in (0, 255):
        ws.fill_(byte)
        outs, status, _ = rz.render_batch(models, reqs, capacity, workspace=ws)
        assert not status.any()
        got.append([t.cpu().numpy() for rgbs, alphas in outs for t in rgbs + alphas])
    for a, b in zip(*got):
        assert np.isfinite(a).all()
        np.testing.assert_array_equal(b.view(np.uint8), a.view(np.uint8))
