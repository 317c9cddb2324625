"""Sorts by one workgroup (up to 8192 pairs) against numpy's stable sort: around
the rounds of 1024 keys and the largest size, one to four passes, passes that
leave every key in place."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("kind", ["random", "one digit", "equal"])
@pytest.mark.parametrize("bits", [1, 8, 9, 17, 32])
@pytest.mark.parametrize("n", [1, 63, 65, 1023, 1024, 1025, 5000, 8191, 8192, 8193])
def test_sort_one_workgroup(n, bits, kind):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2412_03378_amd import Renderer
    R, dev = Renderer(0), torch.device("cuda", 0)
    rng = np.random.default_rng(n * 33 + bits)
    k = rng.integers(0, 1 << bits, n, dtype=np.uint64).astype(np.uint32)
    if kind == "one digit":
        k = (k & np.uint32(0xFF00FF)) | np.uint32(0x3A005A00 & ((1 << bits) - 1))
        k &= np.uint32((1 << bits) - 1)
    elif kind == "equal":
        k[:] = k[0]
    v = np.arange(n, dtype=np.uint32)[::-1].copy()
    kt = torch.from_numpy(k.view(np.int32).copy()).to(dev)
    vt = torch.from_numpy(v.view(np.int32).copy()).to(dev)
    R.sort_pairs(kt, vt, bits)
    torch.cuda.synchronize()
    order = np.argsort(k, kind="stable")
    assert np.array_equal(kt.cpu().numpy().view(np.uint32), k[order])
    assert np.array_equal(vt.cpu().numpy().view(np.uint32), v[order])


@pytest.mark.parametrize("skip", [0, 1, 3])
@pytest.mark.parametrize("n", [10241, 1048577, 4198403, 8388609])
def test_sort_unaligned_keys(n, skip):
    """Tables of counts from keys that do and do not start at 16 bytes, in all tile
    sizes, with a last tile that is not whole."""
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2412_03378_amd import Renderer
    R, dev = Renderer(0), torch.device("cuda", 0)
    rng = np.random.default_rng(n + skip)
    k = rng.integers(0, 1 << 20, n, dtype=np.uint64).astype(np.int32)
    buf = torch.zeros(n + skip, dtype=torch.int32, device=dev)
    kt = buf[skip:]
    kt.copy_(torch.from_numpy(k))
    vt = torch.arange(n, dtype=torch.int32, device=dev)
    R.sort_pairs(kt, vt, 20)
    torch.cuda.synchronize()
    order = np.argsort(k, kind="stable")
    assert np.array_equal(kt.cpu().numpy(), k[order])
    assert np.array_equal(vt.cpu().numpy(), order.astype(np.int32))
