"""Emission by waves that own instances: items that reach into several waves' shares,
several items per wave, and more than 64; long tile rows, written by the whole
wave, beside short ones, around the length at which that begins and longer than
the window of the instances.  The image against the oracle on sampled pixels with
the suite's bounds; every item has to emit the tiles that the preprocess counted."""
import numpy as np
import pytest

import gpu_helpers as G
import helpers as H
import oracle
from paper_2412_03378_amd import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# (extent in tiles of the wide ones, frame)
@pytest.mark.parametrize("n", [3, 64, 9000])
@pytest.mark.parametrize("tiles,w,h", [(31, 400, 24), (33, 400, 24), (65, 800, 40), (900, 8000, 16)])
def test_long_rows(tiles, w, h, n):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2412_03378_amd import Renderer, Settings
    R, dev = Renderer(0), torch.device("cuda", 0)
    rng = np.random.default_rng(n + tiles)
    f = 600.0
    cam = scenes.Camera(np.eye(3, dtype=np.float32), np.array([0.0, 0.0, 4.0], np.float32),
                        f, f, w / 2, h / 2, w, h, 0.2)
    means = np.c_[rng.uniform(-0.5, 0.5, n) * w * 4 / f, rng.uniform(-0.5, 0.5, n) * h * 4 / f,
                  rng.uniform(-0.3, 0.3, n)]
    scales = np.exp(rng.uniform(np.log(0.005), np.log(0.02), (n, 3)))
    # every third one wide: about 3 sigma each way span the tiles
    scales[::3, 0] = 8.0 * tiles * 4 / f / 6 * rng.uniform(0.9, 1.2, len(scales[::3]))
    dens = rng.uniform(0.02, 0.2, n) / scales.max(1) * 0.2
    dens[1::3] *= 20
    dens[2::3] *= 20
    sc = H.scene(means, scales, dens, rgb=rng.uniform(0, 1, (n, 3)))
    st = Settings(tile=(8, 8), bg=(0.1, 0.2, 0.3))
    img = R.forward(*G.device_scene(sc, dev), [cam], st)[0].cpu().numpy()
    s = R.stats()
    assert s["emit_mismatch"] == 0 and s["instances"] >= s["visible"] > 0
    pix = np.c_[rng.integers(0, w, 80), rng.integers(0, h, 80)].astype(np.int32)
    ref = oracle.render(sc, cam, oracle.Settings(bg=st.bg), pixels=pix)
    G.check_image(img[:, pix[:, 1], pix[:, 0]], ref)
