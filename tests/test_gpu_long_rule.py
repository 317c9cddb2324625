"""Which tiles the colour rasterisers walk by 4x4 blocks and which by 8x8 regions:
frames around 2048 and 4096 regions, with lists around the shortest that counts
as long and sparse and dense ones together.  The route may not show: image and
gradients against the oracle with the suite's bounds."""
import numpy as np
import pytest

import gpu_helpers as G
import helpers as H
import oracle
from paper_2412_03378_amd import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# 45 and 46 x 45 regions (2025, 2070), 64 and 65 x 64 (4096, 4160)
@pytest.mark.parametrize("tile", [(8, 8), (16, 16)])
@pytest.mark.parametrize("w,h", [(360, 360), (368, 360), (512, 512), (520, 512)])
def test_frames_around_the_limits(w, h, tile):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2412_03378_amd import Renderer, Settings
    R, dev = Renderer(0), torch.device("cuda", 0)
    rng = np.random.default_rng(w + tile[0])
    # a few entries almost everywhere, a knot of about a hundred, one of 40 to 60 entries
    n = 900
    means = np.r_[np.c_[rng.uniform(-1.2, 1.2, (700, 2)), rng.uniform(-0.3, 0.3, 700)],
                  np.c_[rng.normal(0.4, 0.02, (150, 2)), rng.uniform(-0.3, 0.3, 150)],
                  np.c_[rng.normal(-0.5, 0.02, (50, 2)), rng.uniform(-0.3, 0.3, 50)]]
    sc = H.scene(means, np.exp(rng.uniform(np.log(0.01), np.log(0.03), (n, 3))),
                 np.exp(rng.uniform(np.log(0.5), np.log(10.0), n)), quats=rng.standard_normal((n, 4)),
                 rgb=rng.uniform(0, 1, (n, 3)))
    cam = scenes.axis_camera(3.0, w, h, 45.0)
    st = Settings(tile=tile, bg=(0.2, 0.1, 0.3))
    ref = oracle.render(sc, cam, oracle.Settings(bg=st.bg))
    t = G.device_scene(sc, dev)
    img = R.forward(*t, [cam], st)[0].cpu().numpy()
    G.check_image(img, ref)
    dL = G.upstream(rng, ref, 3).astype(np.float32)
    g = [torch.zeros_like(x) for x in t]
    R.backward([torch.from_numpy(dL).to(dev)], *g)
    gref = oracle.render_backward(sc, cam, oracle.Settings(bg=st.bg), dL.astype(np.float64))
    G.check_grads({k: x.cpu().numpy().astype(np.float64) for k, x in zip(G.GRAD_KEYS, g)},
                  G.sum_backward([gref], G.GRAD_KEYS))
