"""The sizes the library asks for, on the host: a workspace sized for a call
holds every smaller one (fewer Gaussians, views, pixels or pair slots, whichever
path each takes), and a batch needs no more than its requests alone."""
import ctypes as C
import itertools
import random

import pytest

from paper_2410_16978_amd import rasterizer as rz

# around the sizes at which a call takes another path or another layout
N = (0, 1, 8192, 200_000, 524_288, 1 << 20, 4_194_305, (8 << 20) + 1)
SLOTS = (1, 4095, 4097, (3 << 16) - 1, 3 << 16, (1 << 20) - 1, 1 << 20, (1 << 20) + 1, (1 << 21) - 1, 1 << 21, 1 << 24,
         (1 << 24) + 1, 100_000_000)
IMAGES = ((16, 16), (160, 160), (800, 800), (1024, 1024), (1025, 1025), (1100, 1025), (4080, 4096), (4096, 4097),
          (4112, 4112))


def _ascending(sizes, label):
    for a, b in zip(sizes, sizes[1:]):
        assert 0 < a <= b, label


@pytest.mark.parametrize("shared", [False, True])
def test_more_of_anything_needs_no_less(shared):
    def size(n, views, image, slots):
        return rz.workspace_size(n, views, *image, slots, shared)

    for n, image, slots in itertools.product(N, IMAGES, SLOTS):
        _ascending([size(n, v, image, slots) for v in (1, 2, 3, 17)], (n, image, slots))
    for views, image, slots in itertools.product((1, 2), IMAGES, SLOTS):
        _ascending([size(n, views, image, slots) for n in N], (views, image, slots))
    for n, views, slots in itertools.product(N, (1, 2), SLOTS):
        _ascending([size(n, views, image, slots) for image in IMAGES], (n, views, slots))
    for n, views, image in itertools.product(N, (1, 2), IMAGES):
        _ascending([size(n, views, image, slots) for slots in SLOTS], (n, views, image))


def test_a_shared_order_needs_no_less():
    for n, image, slots in itertools.product(N, IMAGES, SLOTS):
        assert rz.workspace_size(n, 2, *image, slots, True) >= rz.workspace_size(n, 2, *image, slots, False) > 0


def _models(sizes):
    """Models the size function accepts; their arrays are never read."""
    return (rz.Model * len(sizes))(*[rz.Model(n, 3, 256, 256, 256, 256, 256, 256) for n in sizes])


def _request(model, eyes, w, h, shared=False):
    r = rz.Request()
    r.model, r.n_views = model, eyes
    for e in range(eyes):
        r.cam[e].fx = r.cam[e].fy = 500.0
        r.cam[e].width, r.cam[e].height = w, h
        r.rgb[e] = r.alpha[e] = 256
    r.vs.sort_shared = 1 if shared else 0
    return r


def _size(models, reqs, slots):
    return rz.batch_workspace_size(models, (rz.Request * len(reqs))(*reqs), slots)


def test_a_batch_needs_no_more_than_its_requests():
    # one alone is ordered by record, the other by tile, and the two by tile
    models = _models([1_000_000, 2_000_000])
    reqs, slots = [_request(0, 1, 512, 512), _request(1, 1, 1832, 1920)], [1_200_000, 2_500_000]
    assert _size(models, reqs, sum(slots)) <= sum(_size(models, [r], s) for r, s in zip(reqs, slots))
    rng = random.Random(1)
    for _ in range(3000):
        models = _models([int(10 ** rng.uniform(0, 7)) for _ in range(2)])
        reqs, slots = [], []
        for _ in range(rng.randint(2, 12)):
            m, eyes = rng.randint(0, 1), rng.randint(1, 2)
            reqs.append(_request(m, eyes, int(10 ** rng.uniform(1, 3.6)), int(10 ** rng.uniform(1, 3.6)),
                                 eyes == 2 and rng.random() < 0.3))
            slots.append(int(models[m].n * eyes * 10 ** rng.uniform(-2, 1)) % (1 << 26) + 1)
        alone = [_size(models, [r], s) for r, s in zip(reqs, slots)]
        assert 0 < _size(models, reqs, sum(slots)) <= sum(alone)


def test_a_batch_workspace_holds_smaller_batches():
    models = _models([300_000, 1_500_000])
    reqs = [_request(q % 2, 1 + q % 3 // 2, *IMAGES[q % len(IMAGES)], q == 5) for q in range(12)]
    for slots in SLOTS:
        _ascending([_size(models, reqs[:k], slots) for k in range(1, 13)], slots)
    for k in (1, 4, 12):
        _ascending([_size(models, reqs[:k], slots) for slots in SLOTS], k)


def test_a_workspace_below_the_size_is_refused():
    """On the host, before any launch, whichever path the call would take."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("the buffers here are addresses only")
    W = H = 800
    cam, view = rz.Camera(), rz.ViewState()
    cam.fx, cam.fy, cam.width, cam.height = 500.0, 500.0, W, H
    for n, slots in itertools.product((100_000, 600_000), (10_000, 1 << 20, 1 << 21, 1 << 24)):
        model = _models([n])[0]
        state = rz.FwdState(*[256] * 11, slots, int(rz.lib().gsr_batch_capacity(slots, 2500)))
        nbytes = rz.workspace_size(n, 1, W, H, slots) - 1
        args = (C.byref(model), 1, C.byref(cam), C.byref(view), C.byref(state))
        assert rz.lib().gsr_rasterize_forward(*args, 256, nbytes, 256, 256, None, None, None, None) == rz.GSR_ENOSPACE
        grads = rz.Grads(*[256] * 5)
        assert rz.lib().gsr_rasterize_backward(*args, 256, 256, 1, 256, nbytes, C.byref(grads), None, None, None,
                                               None) == rz.GSR_ENOSPACE
        reqs = (rz.Request * 1)(_request(0, 1, W, H))
        nbytes = rz.batch_workspace_size(_models([n]), reqs, slots) - 1
        assert rz.lib().gsr_render_batch(_models([n]), 1, reqs, 1, slots, 256, nbytes, 256, None,
                                         None) == rz.GSR_ENOSPACE
