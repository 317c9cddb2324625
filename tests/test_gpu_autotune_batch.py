"""The autotuner and the records per batch: where the batch does not change the
kernels (every mode but the splatting opacity), the 32-record candidates are not
run a second time under another name, and 64 is what it reports."""
import numpy as np
import pytest

import gpu_helpers as G
import helpers as H
from paper_2412_03378_amd import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("mode", ["color", "xray", "splat"])
def test_candidates(mode):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2412_03378_amd import Renderer, Settings
    R, dev = Renderer(0), torch.device("cuda", 0)
    rng = np.random.default_rng(2)
    n = 2000
    sc = H.scene(rng.normal(0.0, 0.4, (n, 3)), np.exp(rng.uniform(np.log(0.01), np.log(0.05), (n, 3))),
                 rng.uniform(0.1, 0.9, n), quats=rng.standard_normal((n, 4)), rgb=rng.uniform(0, 1, (n, 3)))
    cams = [scenes.axis_camera(3.0, 160, 120, 45.0)]
    t = G.device_scene(sc, dev)
    st = Settings(mode="xray" if mode == "xray" else "color",
                  alpha_model="splat" if mode == "splat" else "volumetric")
    shape = (120, 160) if mode == "xray" else (3, 120, 160)
    outs, dL = [torch.empty(shape, device=dev)], [torch.ones(shape, device=dev)]
    grads = [torch.zeros_like(x) for x in t]
    best, batch, ms = R.autotune(t, cams, st, outs, dL, grads, iters=2)
    assert all(m > 0 for m in ms)
    if mode == "splat":
        assert len(set(ms)) > 4
    else:
        assert batch == 64 and ms[4:] == ms[:4]
    assert ms[[(8, 8), (16, 8), (16, 16), (32, 8)].index(best) + (4 if batch == 32 else 0)] == min(ms)
