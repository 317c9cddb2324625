"""The colour rasterisers' two ways through a tile's list: a wave per 4x4 pixel
block (every tile of a small frame, the longest lists of a large one) and a
wave per 8x8 region or tile (the rest of a large one).

A small view alone takes the first; 63 times over in one call (over 8192 8x8
regions, more than 2048 of them not empty) most of its tiles take the second and
the longest the first.  The image may not depend on the route (bitwise); the
gradients of both, the second's divided by the number of views, are held to the
oracle with the suite's bound (GRAD_REL, ERR_K), whose slack covers any order of
the FP32 sums: m terms stay within about sqrt(m) u of their summed magnitudes,
63 views of a thousand terms each 1.5e-5.
"""
import numpy as np
import pytest

import gpu_helpers as G
import helpers as H
import oracle
from paper_2412_03378_amd import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _scene(rng, n, spread):
    """n small Gaussians in a cloud of the given spread, a few opaque ones
    (clamped pairs) and a few large faint ones."""
    means = rng.normal(0.0, spread, (n, 3))
    scales = np.exp(rng.uniform(np.log(0.01), np.log(0.06), (n, 3)))
    dens = np.exp(rng.uniform(np.log(2.0), np.log(40.0), n))
    dens[: n // 16] = 4000.0
    scales[n // 16: n // 8] = 0.4
    dens[n // 16: n // 8] = 0.05
    return H.scene(means, scales, dens, quats=rng.standard_normal((n, 4)),
                   rgb=rng.uniform(0, 1, (n, 3)))


# ragged frames; one Gaussian, lists about a batch of 64 long, lists of several
# batches
@pytest.mark.parametrize("near", [False, True])
@pytest.mark.parametrize("tile", [(8, 8), (16, 8), (16, 16), (32, 8)])
@pytest.mark.parametrize("n,w,h,spread", [(1, 121, 90, 0.0), (700, 123, 91, 0.3),
                                          (2500, 97, 113, 0.25)])
def test_routes_agree(tile, n, w, h, spread, near):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2412_03378_amd import Renderer, Settings
    R, dev = Renderer(0), torch.device("cuda", 0)
    rng = np.random.default_rng(7 * n + w + tile[0])
    sc = _scene(rng, n, spread)
    cam = scenes.axis_camera(3.0, w, h, 45.0)
    st = Settings(tile=tile, bg=(0.2, 0.1, 0.3), near_segment=near)
    t = G.device_scene(sc, dev)
    ref = oracle.render(sc, cam, oracle.Settings(bg=st.bg, near_segment=near))
    dL = torch.from_numpy(G.upstream(rng, ref, 3).astype(np.float32)).to(dev)

    def run(views):
        imgs = R.forward(*t, [cam] * views, st)
        grads = [torch.zeros_like(x) for x in t]
        R.backward([dL] * views, *grads)
        torch.cuda.synchronize()
        return [i.cpu().numpy() for i in imgs], [g.cpu().numpy().astype(np.float64) for g in grads]

    views = 63
    (one,), g1 = run(1)
    many, gn = run(views)
    G.check_image(one, ref)
    for img in many:
        assert np.array_equal(img, one)
    gref = oracle.render_backward(sc, cam, oracle.Settings(bg=st.bg, near_segment=near),
                                  dL.cpu().numpy().astype(np.float64))
    summed = G.sum_backward([gref], G.GRAD_KEYS)
    # exactly zero where the three scales are equal (the oracle leaves FP64 rounding)
    summed["quats"][0][n // 16: n // 8] = 0.0
    G.check_grads(dict(zip(G.GRAD_KEYS, g1)), summed)
    G.check_grads({k: g / views for k, g in zip(G.GRAD_KEYS, gn)}, summed)
