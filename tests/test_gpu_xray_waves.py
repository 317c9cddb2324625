"""X-ray rasterisers: a tile's list split over one to eight waves (by the number
of tiles of the call), entries packed 64 at a time per 8x8 region, ragged
regions.  One view alone has the most waves per tile, 63 equal views in one call
the fewest.  Image and gradients of both against the oracle with the suite's
bounds (XRAY_REL, GRAD_REL, ERR_K; the gradients of equal views divided by their
number), whose slack covers any order of the FP32 sums; the number of terms per
pixel, decided pair by pair, is the same on both.
"""
import functools

import numpy as np
import pytest

import gpu_helpers as G
import helpers as H
import oracle
from paper_2412_03378_amd import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@functools.lru_cache(maxsize=None)
def _case(n, w, h, option):
    """Scene, camera, options, upstream gradient and the oracle's results."""
    rng = np.random.default_rng(11 * n)
    sc = H.scene(rng.normal(0.0, 0.25, (n, 3)),
                 np.exp(rng.uniform(np.log(0.01), np.log(0.2), (n, 3))),
                 np.exp(rng.uniform(np.log(0.1), np.log(5.0), n)),
                 quats=rng.standard_normal((n, 4)), rgb=rng.uniform(0, 1, (n, 3)))
    cam = scenes.axis_camera(1.2 if option == "near" else 3.0, w, h, 45.0)
    opts = dict(near_segment=option == "near",
                kernel="epanechnikov" if option == "epanechnikov" else "gaussian")
    ost = oracle.Settings(mode="xray", **opts)
    ref = oracle.render(sc, cam, ost)
    dL = G.upstream(rng, ref, 1, xray=True)[0].astype(np.float32)
    up = dL[None].astype(np.float64)
    part = oracle.render_backward(sc, cam, ost, up)
    flip = oracle.render_backward(sc, cam, ost, up, near_threshold=G.MARGIN_X)
    return sc, cam, opts, ref, dL, G.sum_backward([part], G.GRAD_KEYS[:4], [flip])


# one entry; a few batches of 64 with a partial one; lists long enough for every wave
@pytest.mark.parametrize("option", ["gaussian", "near", "epanechnikov"])
@pytest.mark.parametrize("tile", [(8, 8), (16, 8), (16, 16), (32, 8)])
@pytest.mark.parametrize("n,w,h", [(1, 139, 125), (200, 133, 129), (1000, 129, 131)])
def test_split_lists(tile, n, w, h, option):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2412_03378_amd import Renderer, Settings
    R, dev = Renderer(0), torch.device("cuda", 0)
    sc, cam, opts, ref, dL, gref = _case(n, w, h, option)
    st = Settings(mode="xray", tile=tile, **opts)
    keys = G.GRAD_KEYS[:4]
    t = G.device_scene(sc, dev)
    terms = []
    for views in (1, 63):
        imgs = R.forward(*t, [cam] * views, st)
        terms.append(R.aux(views - 1, h, w)[1].cpu().numpy())
        grads = [torch.zeros_like(x) for x in t[:4]]
        R.backward([torch.from_numpy(dL).to(dev)] * views, *grads, None)
        torch.cuda.synchronize()
        G.check_image(imgs[-1].cpu().numpy()[None], ref, xray=True, label=f"{views} views: ")
        G.check_grads({k: g.cpu().numpy().astype(np.float64) / views for k, g in zip(keys, grads)}, gref)
    assert np.array_equal(terms[0], terms[1])
    assert terms[0].max() > 0
