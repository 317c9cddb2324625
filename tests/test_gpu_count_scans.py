"""Scans of the preprocess's counts around the longest array that 256 threads take
(4096: 16 views of 256 blocks), short, exact and just over: a call of several
views gives every view the image and the instances of a call of its own."""
import numpy as np
import pytest

import gpu_helpers as G
import helpers as H
from paper_2412_03378_amd import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [256, 65280, 65536, 65537])
def test_views_together_and_alone(n):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2412_03378_amd import Renderer, Settings
    R, dev = Renderer(0), torch.device("cuda", 0)
    rng = np.random.default_rng(n)
    sc = H.scene(rng.normal(0.0, 0.8, (n, 3)), np.exp(rng.uniform(np.log(0.002), np.log(0.02), (n, 3))),
                 np.exp(rng.uniform(np.log(0.5), np.log(20.0), n)), quats=rng.standard_normal((n, 4)),
                 rgb=rng.uniform(0, 1, (n, 3)))
    cams = [scenes.axis_camera(2.0 + 0.1 * v, 64 + 8 * (v % 5), 80 - 8 * (v % 4), 50.0) for v in range(16)]
    st = Settings(tile=(8, 8))
    t = G.device_scene(sc, dev)
    many = [x.cpu().numpy() for x in R.forward(*t, cams, st)]
    total = R.stats()["instances"]
    alone = 0
    for v, cam in enumerate(cams):
        one = R.forward(*t, [cam], st)[0].cpu().numpy()
        alone += R.stats()["instances"]
        assert np.array_equal(one, many[v]), v
    assert total == alone > 0
