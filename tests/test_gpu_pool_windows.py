"""The row-band pool kernel over its windows and steps, against maxima taken
with numpy: identity layers around one pool make every output an exact copy of
a pooled value, so the map is compared bit for bit."""
import numpy as np
import pytest

from oracle import index as ix
from paper_1302_1700_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fsb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1302_1700_amd import fragscan
    fragscan.load()
    return fragscan


@pytest.mark.parametrize("ky,kx", [(2, 2), (3, 3), (4, 4), (2, 3), (3, 2)])
@pytest.mark.parametrize("sy,sx", [(1, 1), (2, 2), (3, 2), (3, 3), (1, 5), (5, 4)])
def test_windows_and_steps(fsb, monkeypatch, ky, kx, sy, sx):
    monkeypatch.setenv("FRAGSCAN_POOL_FUSE", "0")
    rng = np.random.default_rng(ky * 100 + kx * 10 + sy + sx)
    for c, dt, rows in ((3, "f32", "4"), (8, "f32", "8"), (12, "f32", "4"), (16, "bf16", "8"), (3, "bf16", "4")):
        layers = [wl.conv(1, c, c, "none"), wl.pool(ky, c, kx=kx, stride=sy, stride_x=sx), wl.fc(1, c, c, "none")]
        eye = (np.eye(c, dtype=np.float32)[:, :, None, None], np.zeros(c, np.float32))
        # one row and column more than the window, odd sizes, several bands of rows
        for H, W in ((ky, kx), (ky + 1, kx + 40), (41, kx + 29)):
            img = rng.integers(-128, 128, (2, H, W, c)).astype(np.float32)  # exact in bf16
            monkeypatch.setenv("FRAGSCAN_POOL_ROWS", rows)
            net = fsb.Net(layers, [eye, None, eye], c, 0, dt)
            names = [L["name"] for L in net.launches(2, H, W)]
            print("pool", (ky, kx), (sy, sx), c, dt, (H, W), names, flush=True)
            got = net.scan(torch.from_numpy(img).cuda())
            torch.cuda.synchronize()
            net.close()
            name = "pool_frag_rows<%d, %s," % (ky, rows) if ky == kx == sy == sx else \
                "pool_frag<%d, %d, %s," % (ky, kx, rows)
            assert any(n.startswith(name) for n in names), names
            want = np.full((2, H - ky + 1, W - kx + 1, c), -np.inf, np.float32)
            for i in range(ky):
                for j in range(kx):
                    want = np.maximum(want, img[:, i:i + H - ky + 1, j:j + W - kx + 1])
            assert (H - ix.patch_hw(layers)[0] + 1, W - ix.patch_hw(layers)[1] + 1) == want.shape[1:3]
            assert np.array_equal(got.cpu().numpy(), want)
