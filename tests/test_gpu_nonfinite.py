"""Values that are not finite reach only the pixels and Gaussians that they belong to.

The colour rasterisers multiply by a weight of zero where a lane has nothing to
blend, and 0 * Inf is NaN: a colour, a weight or an upstream gradient that is not
finite must not get into such a product with another pixel's sums.  One small
view alone takes the rasterisers' way by 4x4 blocks, 63 equal views in one call
(over 8192 8x8 regions) the way by regions.
"""
import numpy as np
import pytest

import gpu_helpers as G
import helpers as H
from paper_2412_03378_amd import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _setup():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2412_03378_amd import Renderer
    return Renderer(0), torch.device("cuda", 0)


@pytest.mark.parametrize("model,tile,batch", [
    ("volumetric", (8, 8), 64), ("volumetric", (16, 16), 64), ("volumetric", (32, 8), 64),
    ("splat", (8, 8), 64), ("splat", (8, 8), 32), ("splat", (16, 8), 64), ("splat", (16, 16), 32),
    ("splat", (32, 8), 64)])
def test_leftovers_of_another_frame(model, tile, batch):
    """A frame of short lists after one whose staged colours were all infinite: what
    the kernels before it left in the LDS does not show."""
    R, dev = _setup()
    from paper_2412_03378_amd import Settings
    w, h = 1280, 1024            # 20480 regions of 8x8
    cam = scenes.axis_camera(3.0, w, h, 45.0)
    st = Settings(tile=tile, batch=batch, alpha_model=model, bg=(0.2, 0.1, 0.3))
    rng = np.random.default_rng(5)
    # 96 faint Gaussians over the whole frame, infinite colours
    n = 96
    faint = 0.01 if model == "splat" else 0.002
    full = H.scene(np.c_[rng.uniform(-0.1, 0.1, (n, 2)), rng.uniform(0.0, 0.5, n)], 2.0, faint)
    full.sh[:] = np.inf
    # a few entries per list
    m = 4000
    few = H.scene(np.c_[rng.uniform(-1.2, 1.2, (m, 2)), rng.uniform(-0.2, 0.2, m)],
                  rng.uniform(0.005, 0.02, (m, 3)),
                  rng.uniform(0.1, 0.9, m) if model == "splat" else rng.uniform(5.0, 60.0, m),
                  quats=rng.standard_normal((m, 4)), rgb=rng.uniform(0, 1, (m, 3)))
    t_full, t_few = G.device_scene(full, dev), G.device_scene(few, dev)
    for _ in range(4):
        flood = R.forward(*t_full, [cam], st)[0]
        img = R.forward(*t_few, [cam], st)[0]
        torch.cuda.synchronize()
        assert torch.isinf(flood).all()
        assert torch.isfinite(img).all(), int((~torch.isfinite(img)).sum())


def _settings(tile, option):
    from paper_2412_03378_amd import Settings
    return Settings(tile=tile, bg=(0.2, 0.1, 0.3), near_segment=option == "near",
                    kernel="epanechnikov" if option == "epanechnikov" else "gaussian",
                    alpha_model="splat" if option == "splat" else "volumetric")


def _cloud(rng, n, bad_color):
    """Lists of several batches that no pixel leaves early; every fiftieth Gaussian is
    small and of the given colour."""
    means = rng.normal(0.0, 0.3, (n, 3))
    scales = np.exp(rng.uniform(np.log(0.01), np.log(0.05), (n, 3)))
    dens = np.exp(rng.uniform(np.log(0.2), np.log(2.0), n))
    rgb = rng.uniform(0.1, 1, (n, 3))
    quats = rng.standard_normal((n, 4))
    scales[::50] = 0.008
    dens[::50] = 20.0
    rgb[::50] = bad_color
    return H.scene(means, scales, dens, quats=quats, rgb=rgb)


@pytest.mark.parametrize("views", [1, 63])
@pytest.mark.parametrize("option", ["gaussian", "near", "epanechnikov", "splat"])
@pytest.mark.parametrize("tile", [(8, 8), (16, 16), (32, 8)])
def test_infinite_colours(tile, option, views):
    """Pixels that blend none of the infinite colours equal the image with finite ones."""
    R, dev = _setup()
    w, h, n = 123, 91, 3000
    cam = scenes.axis_camera(3.0, w, h, 45.0)
    st = _settings(tile, option)

    def image(color):
        sc = _cloud(np.random.default_rng(n), n, color)
        if option == "splat":
            sc.dens[:] = 1.0 - np.exp(-0.05 * sc.dens)
        return R.forward(*G.device_scene(sc, dev), [cam] * views, st)[-1].clone()

    far, img, bad = image(100.0), image(0.7), image(np.inf)
    blends = (far != img).any(0)               # pixels that blend one of them
    assert 0 < int(blends.sum()) < blends.numel() // 2
    assert torch.equal(bad[:, ~blends], img[:, ~blends])
    assert not torch.isfinite(bad[:, blends]).any()


@pytest.mark.parametrize("views", [1, 63])
@pytest.mark.parametrize("front", [1, 2, 3, 4])
def test_overflow_behind_a_stopped_pixel(front, views):
    """Opaque Gaussians stop every pixel; behind them one whose line integral overflows
    to Inf * 0.  Its place in the step of four in which the pixels stop does not
    matter."""
    R, dev = _setup()
    from paper_2412_03378_amd import Settings
    w, h = 123, 91
    cam = scenes.axis_camera(3.0, w, h, 45.0)
    st = Settings(tile=(8, 8), bg=(0.2, 0.1, 0.3), T_min=0.02)
    # front - 1 faint ones, one that leaves T = 0.01 < T_min, the one that overflows
    n = front + 1
    means = np.c_[np.zeros((n, 2)), np.linspace(0.0, 0.5, n)]
    dens = np.full(n, 0.01)
    dens[front - 1] = 1e4
    dens[front] = 3e38
    scales = np.full((n, 3), 3.0)
    scales[front] = 0.05
    t = G.device_scene(H.scene(means, scales, dens, rgb=np.linspace(0.2, 0.9, n)[:, None]), dev)
    want = R.forward(*[x[:front].contiguous() for x in t], [cam] * views, st)[-1].clone()
    img = R.forward(*t, [cam] * views, st)[-1]
    torch.cuda.synchronize()
    assert torch.isfinite(want).all()
    assert torch.equal(img, want)


@pytest.mark.parametrize("views", [1, 63])
@pytest.mark.parametrize("option", ["gaussian", "near", "epanechnikov"])
@pytest.mark.parametrize("tile", [(8, 8), (16, 16)])
def test_gradients_beside_infinite_colours(tile, option, views):
    """Gaussians that share no pixel with the infinite colours have the gradients of
    the scene with finite ones."""
    R, dev = _setup()
    w, h, n = 123, 91, 3000
    cam = scenes.axis_camera(3.0, w, h, 45.0)
    st = _settings(tile, option)

    def forward(color):
        t = G.device_scene(_cloud(np.random.default_rng(n), n, color), dev)
        return t, R.forward(*t, [cam] * views, st)[-1].clone()

    def grads(t, dL):
        g = [torch.zeros_like(x) for x in t]
        R.backward([dL] * views, *g)
        return [x.cpu().numpy().reshape(n, -1).astype(np.float64) for x in g]

    _, far = forward(100.0)
    t, img = forward(0.7)
    blends = (far != img).any(0)
    # Gaussians that some such pixel blends (their colours get a gradient from it)
    ones = blends.float()[None].expand(3, -1, -1).contiguous()
    apart = (grads(t, ones)[4] == 0.0).all(1)
    assert 0 < int(apart.sum()) < n
    rng = np.random.default_rng(1)
    dL = torch.from_numpy(rng.standard_normal((3, h, w)).astype(np.float32)).to(dev) * ~blends
    want = grads(t, dL)
    t, _ = forward(np.inf)
    got = grads(t, dL)
    for k, a, b in zip(G.GRAD_KEYS, got, want):
        # (the FP32 sums of a Gaussian's pixels in another order)
        assert np.isfinite(a[apart]).all(), k
        assert np.all(np.abs(a - b)[apart] <= G.GRAD_REL * np.abs(b[apart]).max()), k


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("views", [1, 63])
@pytest.mark.parametrize("option", ["gaussian", "near", "epanechnikov"])
def test_upstream_gradient_of_one_pixel(option, views, value):
    """Two Gaussians of one pixel each in every 8x8 region, both in its first 4x4
    block.  An upstream gradient that is not finite at the first one's pixel leaves
    the gradients of the second alone."""
    R, dev = _setup()
    w, h = 123, 91
    cam = scenes.axis_camera(3.0, w, h, 45.0)
    st = _settings((8, 8), option)
    px, py = np.meshgrid(np.arange(0, w - 7, 8), np.arange(0, h - 7, 8))
    first = np.c_[px.ravel(), py.ravel()]
    pix = np.r_[first, first + [2, 3]]
    mean = np.c_[(pix + 0.5 - [cam.cx, cam.cy]) * 3.0 / [cam.fx, cam.fy], np.zeros(len(pix))]
    # sigma 0.2 pixels, alpha 0.3 at the centre: no other pixel centre reaches 1/255
    s = 0.2 * 3.0 / cam.fx
    sc = H.scene(mean, s, 0.36 / (s * np.sqrt(2 * np.pi)), rgb=(0.6, 0.3, 0.8))
    t = G.device_scene(sc, dev)
    dL = torch.ones((3, h, w), device=dev)

    def grads(dL):
        imgs = R.forward(*t, [cam] * views, st)
        assert int((imgs[0][0] != imgs[0][0, 1, 1]).sum()) == len(pix)
        g = [torch.zeros_like(x) for x in t]
        R.backward([dL] * views, *g)
        return [x.cpu().numpy().reshape(len(pix), -1).astype(np.float64) for x in g]

    want = grads(dL)
    dL[:, first[:, 1], first[:, 0]] = value
    got = grads(dL)
    m = len(first)
    for k, a, b in zip(G.GRAD_KEYS, got, want):
        # one pixel a view: the sums differ in the order of equal terms only
        assert np.allclose(a[m:], b[m:], rtol=1e-5, atol=1e-5 * np.abs(b).max()), k
    assert not np.isfinite(got[3][:m]).any()
