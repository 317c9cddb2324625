"""The X-ray cut in the forward and in the backward: the cut value is set to one
pixel's line integral and a few units in the last place around it, where the
forms of the integral that the kernels use round to either side.  The terms of
the image (R.aux counts them) and of the gradient have to be the same ones:
dL/ddens * dens summed over the pixels is the image summed over the pixels.
"""
import numpy as np
import pytest

import gpu_helpers as G
import helpers as H
from paper_2412_03378_amd import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("option", ["gaussian", "near", "epanechnikov"])
@pytest.mark.parametrize("tile", [(8, 8), (16, 16)])
def test_same_terms(tile, option):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2412_03378_amd import Renderer, Settings
    R, dev = Renderer(0), torch.device("cuda", 0)
    w, h = 48, 40
    rng = np.random.default_rng(3)
    # (near: the Gaussian's near side is cut off)
    cam = scenes.axis_camera(0.5 if option == "near" else 3.0, w, h, 45.0)
    size = 0.06 if option == "near" else 0.25
    sc = H.scene([[0.01, -0.02, 0.03]], size * np.array([1.0, 0.6, 1.4]), 2.0,
                 quats=rng.standard_normal((1, 4)))
    t = G.device_scene(sc, dev)
    opts = dict(mode="xray", tile=tile, near_segment=option == "near",
                kernel="epanechnikov" if option == "epanechnikov" else "gaussian")
    dL = torch.ones((h, w), device=dev)
    img0 = R.forward(*t, [cam], Settings(x_min_xray=1e-6, **opts))[0].cpu().numpy()
    # pixels in the flank, where one term is a good part of the sum
    vals = np.sort(img0[(img0 > 0.02 * img0.max()) & (img0 < 0.5 * img0.max())])
    vals = vals[:: max(1, len(vals) // 40)]
    assert len(vals) >= 20
    split = 0
    for v in vals:
        counts = set()
        for step in range(-4, 5):
            x = np.float32(v)
            for _ in range(abs(step)):
                x = np.nextafter(x, np.float32(np.sign(step) * np.inf), dtype=np.float32)
            st = Settings(x_min_xray=float(x), **opts)
            img = R.forward(*t, [cam], st)[0]
            counts.add(int(R.aux(0, h, w)[1].sum()))
            g = [torch.zeros_like(a) for a in t[:4]]
            R.backward([dL], *g, None)
            total = float(img.double().sum())
            # the sums agree to rounding (some hundred terms of 2^-22 each); one term
            # more or less is x
            assert abs(float(g[3][0]) * 2.0 - total) <= 1e-5 * total + 0.1 * float(x) * 0.1, (v, step)
        split += len(counts) > 1
    assert split > 0   # the cut did move across the pixels' values
