"""Frames whose colour rasterisers have more workgroups than one row of their grid
(2^20): every region of an 8192x8200 view is rendered, and its gradients arrive,
also from the last rows.  Small Gaussians at the frame's corners and middle
against crops of the same camera, which fit into one row."""
import numpy as np
import pytest

import gpu_helpers as G
import helpers as H
from paper_2412_03378_amd import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("tile", [(8, 8), (16, 16)])
def test_more_than_one_row(tile):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2412_03378_amd import Renderer, Settings
    R, dev = Renderer(0), torch.device("cuda", 0)
    w, h, f, side = 8192, 8200, 8000.0, 64
    rng = np.random.default_rng(1)
    corners = [(0, 0), (w - side, 0), (0, h - side), (w - side, h - side), (w // 2, h // 2)]
    n = 40 * len(corners)
    pix = np.concatenate([rng.uniform(8, side - 8, (40, 2)) + c for c in corners])
    z = rng.uniform(3.0, 3.5, n)
    cam = lambda cx, cy, cw, ch: scenes.Camera(np.eye(3, dtype=np.float32), np.zeros(3, np.float32),
                                               f, f, cx, cy, cw, ch, 0.2)
    means = np.c_[(pix - [w / 2, h / 2]) / f * z[:, None], z]
    sc = H.scene(means, rng.uniform(0.5, 2.0, (n, 3)) * 3.0 / f, rng.uniform(200.0, 900.0, n),
                 quats=rng.standard_normal((n, 4)), rgb=rng.uniform(0, 1, (n, 3)))
    t = G.device_scene(sc, dev)
    st = Settings(tile=tile, bg=(0.2, 0.1, 0.3))
    img = R.forward(*t, [cam(w / 2, h / 2, w, h)], st)[0]
    dL = torch.zeros_like(img)
    ups = [torch.from_numpy(rng.standard_normal((3, side, side)).astype(np.float32)).to(dev)
           for _ in corners]
    for (x, y), u in zip(corners, ups):
        dL[:, y:y + side, x:x + side] = u
    g = [torch.zeros_like(x) for x in t]
    R.backward([dL], *g)
    bg = torch.tensor(st.bg, device=dev)[:, None, None]
    assert int((img != bg).any(0).sum()) == sum(
        int((img[:, y:y + side, x:x + side] != bg).any(0).sum()) for x, y in corners)
    want = [torch.zeros_like(x) for x in t]
    for (x, y), u in zip(corners, ups):
        crop = R.forward(*t, [cam(w / 2 - x, h / 2 - y, side, side)], st)[0]
        # (the same pixels, but for the rounding of their coordinates)
        assert (crop != bg).any()
        assert (crop - img[:, y:y + side, x:x + side]).abs().max() < 2e-3
        R.backward([u], *want)
    for k, a, b in zip(G.GRAD_KEYS, g, want):
        a, b = a.reshape(n, -1).cpu().numpy(), b.reshape(n, -1).cpu().numpy()
        assert np.abs(b).max(1).min() > 0 and np.abs(a - b).max() <= 2e-2 * np.abs(b).max(), k
