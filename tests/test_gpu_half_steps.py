"""The convolution's half-step K walk on the GPU: float32 layers with inputs
bounded by a tanh, whose products run on the f16 matrix cores with operands
split into f16 pairs, and bf16 layers with an odd multiple of 16 input
channels.  Sizes at the walk's edges: one K step, odd and even counts of
16-channel groups, steps that span two taps, K split over waves, padded
channel blocks, run tiles, fused pools and heads."""
import numpy as np
import pytest

import oracle
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


def _scan(fsb, layers, params, img, dt):
    net = fsb.Net(layers, params, img.shape[3], 0, dt)
    names = [L["name"] for L in net.launches(*img.shape[:3])]
    out = net.scan(torch.from_numpy(np.ascontiguousarray(img, np.float32)).cuda())
    torch.cuda.synchronize()
    net.close()
    return out.cpu().numpy().astype(np.float64), names


def _half(name):
    return name.split(">")[0].endswith("true")


def _net(cin, ky, kx, cout, pooled):
    layers = [wl.conv(2, 3, cin), wl.conv(ky, cin, cout, kx=kx)]
    if pooled:
        layers.append(wl.pool(2, cout))
    return layers + [wl.fc(2, cout, 20), wl.fc(1, 20, 3, "none")]


EDGES = [(16, 1, 1, 16, False), (16, 2, 1, 33, True), (16, 3, 3, 16, True), (32, 1, 2, 100, False),
         (48, 1, 1, 48, False), (48, 3, 3, 200, False), (48, 4, 4, 48, True), (48, 5, 5, 48, True),
         (80, 2, 3, 64, True), (112, 1, 3, 17, False), (256, 1, 1, 32, False)]


@pytest.mark.parametrize("cin,ky,kx,cout,pooled", EDGES)
def test_split_float32(fsb, monkeypatch, cin, ky, kx, cout, pooled):
    """Scores against float64: the split products are no further off than the
    float32 ones (three f16 products of 23-bit operands, 32 K indices per
    accumulation, against 4), and both within 2^-24 per accumulated term."""
    layers = _net(cin, ky, kx, cout, pooled)
    h0, w0 = ix.patch_hw(layers)
    params = wl.make_weights(layers, cin + ky, 1.0 / np.sqrt(cin * ky * kx))
    img = wl.make_image(cin + 1, 2, h0 + 37, w0 + 52, 3)
    ref = oracle.frag_cpu.frag_scan(layers, params, img, (h0, w0))
    off = {}
    for mode in ("1", "0"):
        monkeypatch.setenv("FRAGSCAN_SPLIT", mode)
        print("split", (cin, ky, kx, cout, pooled), mode, flush=True)
        got, names = _scan(fsb, layers, params, img, "f32")
        assert not _half(names[0]) and _half(names[1]) == (mode == "1"), names
        off[mode] = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    bound = 2.0 ** -24 * 4 * np.sqrt(cin * ky * kx + 4 * cout)
    assert off["1"] <= min(1.2 * off["0"] + 2e-8, bound), off


@pytest.mark.parametrize("cin,ky,kx,cout,pooled", [e for e in EDGES if e[0] % 32 == 16])
def test_bf16_half_steps(fsb, cin, ky, kx, cout, pooled):
    layers = _net(cin, ky, kx, cout, pooled)
    h0, w0 = ix.patch_hw(layers)
    params = wl.make_weights(layers, cin + ky, 1.0 / np.sqrt(cin * ky * kx))
    img = wl.make_image(cin + 2, 2, h0 + 37, w0 + 52, 3)
    ref = oracle.frag_cpu.frag_scan(layers, params, img, (h0, w0))
    print("bf16 half steps", (cin, ky, kx, cout, pooled), flush=True)
    got, names = _scan(fsb, layers, params, img, "bf16")
    assert _half(names[1]), names
    # a handful of roundings to 8 significand bits per value, averaged by the sums
    assert np.linalg.norm(got - ref) <= 2.0 ** -6 * np.linalg.norm(ref)


@pytest.mark.parametrize("env", [{"FRAGSCAN_RUN": "1"}, {"FRAGSCAN_ROWTILES": "1", "FRAGSCAN_POOL_FUSE": "0"},
                                 {"FRAGSCAN_POOL_FUSE": "1"}, {"FRAGSCAN_STORE": "lds", "FRAGSCAN_POOL_FUSE": "0"},
                                 {"FRAGSCAN_NO_FUSED_HEAD": "1"}, {"FRAGSCAN_LDS_PAD": "0"}])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_same_values_on_every_tile_path(fsb, monkeypatch, env, dt):
    """Run tiles, row tiles, fused pools and restaged stores leave each
    output's products and their order alone: bit for bit the same map (the
    separate head sums in another order)."""
    layers = [wl.conv(3, 1, 48), wl.pool(2, 48), wl.conv(3, 48, 48), wl.pool(2, 48), wl.fc(2, 48, 200),
              wl.fc(1, 200, 2, "softmax")]
    w0 = ix.patch_size(layers)
    params = wl.make_weights(layers, 9, 0.08)
    img = wl.make_image(10, 2, w0 + 121, w0 + 108, 1)
    base, names = _scan(fsb, layers, params, img, dt)
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    got, other = _scan(fsb, layers, params, img, dt)
    print("tile paths", dt, env, other, flush=True)
    assert any(_half(n) for n in names) and any(_half(n) for n in other)
    if "FRAGSCAN_NO_FUSED_HEAD" in env:
        assert np.abs(got - base).max() <= (1e-5 if dt == "f32" else 2e-2) * np.abs(base).max()
    else:
        assert np.array_equal(got, base)


@pytest.mark.parametrize("H,W,B", [(95, 95, 1), (96, 103, 1), (103, 110, 2), (128, 128, 1), (140, 333, 1),
                                   (180, 180, 1), (230, 210, 1)])
def test_small_grids(fsb, H, W, B):
    """N4 on images whose grids leave the device part empty: 16- to 64-pixel
    tiles, pools fused where the grid is smallest, fragments
    of one to a few pixels (and empty ones); the whole map against the CPU
    fragment method, and the profiled scan's map bit for bit."""
    w = wl.WORKLOADS[2]
    params, img = wl.workload_inputs(2, batch=B, height=H, width=W)
    ref = oracle.frag_cpu.frag_scan(w.layers, params, img, w.patch)
    net = fsb.Net(w.layers, params, 1)
    print("small grid", (B, H, W), [L["name"] for L in net.launches(B, H, W)], flush=True)
    x = torch.from_numpy(img).cuda()
    got = net.scan(x).clone()
    again = torch.full_like(got, float("nan"))
    net.profile(x, reps=2, out=again)
    torch.cuda.synchronize()
    net.close()
    assert torch.equal(got, again)
    assert np.abs(got.cpu().numpy() - ref).max() <= 2e-6  # probabilities; float32 sums of 1200 terms behind a tanh


@pytest.mark.parametrize("H,W,tile", [(512, 480, (100, 130)), (300, 333, (40, 240)), (260, 260, (9, 11))])
def test_tiles_of_other_sizes_give_the_same_sums(fsb, H, W, tile):
    """A tiled scan whose tiles take other register tiles (and fuse other
    pools) than the whole image's scan gives its map bit for bit."""
    w = wl.WORKLOADS[2]
    params, img = wl.workload_inputs(2, height=H, width=W)
    net = fsb.Net(w.layers, params, 1)
    x = torch.from_numpy(img).cuda()
    ref = net.scan(x).clone()
    whole = [L["name"] for L in net.launches(1, H, W)]
    part = [L["name"] for L in net.launches(1, tile[0] + 94, tile[1] + 94)]
    assert whole != part
    print("tiled sums", (H, W), tile, whole, part, flush=True)
    got = net.scan_tiled(x, tile)
    torch.cuda.synchronize()
    net.close()
    assert torch.equal(got, ref)


def test_channels_of_any_scale(fsb, monkeypatch):
    """Every output channel is scaled by its own largest weight: channels from
    1e-12 to 1e12 times the others keep float32's accuracy (read out one at a
    time through a linear last layer), as do zero channels."""
    monkeypatch.setenv("FRAGSCAN_SPLIT", "1")
    layers = [wl.conv(2, 1, 48), wl.conv(2, 48, 16, "none"), wl.fc(1, 16, 16, "none")]
    params = wl.make_weights(layers, 5, 0.3)
    gain = np.float32(10.0) ** np.linspace(-12, 12, 16).astype(np.float32)
    w, b = params[1]
    w, b = w * gain[:, None, None, None], b * gain
    w[7], b[7] = 0, 0
    params[1] = (w, b)
    params[2] = (np.eye(16, dtype=np.float32)[:, :, None, None], np.zeros(16, np.float32))
    img = wl.make_image(6, 1, 40, 45, 1)
    ref = oracle.frag_cpu.frag_scan(layers, params, img, 3)
    got, names = _scan(fsb, layers, params, img, "f32")
    assert _half(names[1]), names
    rms = np.sqrt((ref ** 2).mean(axis=(0, 1, 2)))
    assert rms[7] == 0 and (got[..., 7] == 0).all()
    err = np.sqrt(((got - ref) ** 2).mean(axis=(0, 1, 2)))
    assert (err <= 1e-6 * rms).all(), err / rms


def test_scores_keep_the_float32_products(fsb, monkeypatch):
    """A net without a softmax at the end keeps its map bit for bit."""
    layers = _net(48, 3, 3, 48, True)
    params = wl.make_weights(layers, 3, 0.1)
    img = wl.make_image(4, 1, 60, 71, 3)
    base, names = _scan(fsb, layers, params, img, "f32")
    assert not any(_half(n) for n in names), names
    monkeypatch.setenv("FRAGSCAN_SPLIT", "0")
    off, _ = _scan(fsb, layers, params, img, "f32")
    assert np.array_equal(base, off)


@pytest.mark.parametrize("bad", [np.inf, np.nan, 1e30])
def test_weights_out_of_range_stay_float32(fsb, bad):
    """A weight that is not finite, or a channel whose range the f16 pairs
    cannot take, keeps the layer on the float32 products."""
    layers = [wl.conv(2, 1, 16), wl.conv(2, 16, 16), wl.fc(1, 16, 2, "softmax")]
    params = wl.make_weights(layers, 5, 0.3)
    params[1][0][3, 2, 1, 0] = bad
    img = wl.make_image(6, 1, 30, 31, 1)
    got, names = _scan(fsb, layers, params, img, "f32")
    assert not any(_half(n) for n in names), names
    if np.isfinite(bad):
        assert np.abs(got - oracle.frag_cpu.frag_scan(layers, params, img, 3)).max() <= 1e-4
    else:
        assert got.shape == (1, 28, 29, 2)


def test_non_finite_pixels_stay_in_their_windows(fsb):
    """A NaN pixel reaches exactly the windows that hold it; an infinite one
    saturates the first layer's tanh and stays finite after it."""
    layers = [wl.conv(2, 1, 48), wl.pool(2, 48), wl.conv(3, 48, 48), wl.fc(1, 48, 2, "softmax")]
    w0 = ix.patch_size(layers)
    params = wl.make_weights(layers, 15, 0.1)
    img = wl.make_image(16, 1, w0 + 40, w0 + 33, 1)
    img[0, 20, 17, 0] = np.inf
    got, names = _scan(fsb, layers, params, img, "f32")
    assert _half(names[-1]) or _half(names[-2]), names
    assert np.isfinite(got).all()
    img[0, 20, 17, 0] = np.nan
    got, _ = _scan(fsb, layers, params, img, "f32")
    Y, X = np.meshgrid(np.arange(got.shape[1]), np.arange(got.shape[2]), indexing="ij")
    clean = (Y > 20) | (Y + w0 - 1 < 20) | (X > 17) | (X + w0 - 1 < 17)
    assert np.isfinite(got[0][clean]).all()


@pytest.mark.parametrize("net", [2, 3, 5])
def test_nan_pixels_lose_in_every_pool(fsb, monkeypatch, net):
    """A NaN pixel makes NaN of the outputs whose pools hold nothing else: the
    same windows in float32 and bf16, with pools fused and separate."""
    layers = wl.WORKLOADS[net].layers
    w0 = ix.patch_size(layers)
    rng = np.random.default_rng(net)
    params = []
    for L in layers:
        if L["kind"] == "pool":
            params.append(None)
        else:
            shape = (L["c_out"], L["c_in"], L["k"], L["k"])
            params.append((rng.normal(0.0, 1.0 / np.sqrt(np.prod(shape[1:])), shape).astype(np.float32),
                           np.zeros(L["c_out"], np.float32)))
    c = layers[0]["c_in"]
    img = wl.make_image(net, 1, w0 + 60, w0 + 71, c)
    img[0, 60, 70, 0] = img[0, 61, 3, c - 1] = np.nan
    img[0, 5, 77, 0] = np.uint32(0xffc00000).view(np.float32)  # its sign bit set
    masks = {}
    for dt in ("f32", "bf16"):
        for fuse in ("1", "0"):
            monkeypatch.setenv("FRAGSCAN_POOL_FUSE", fuse)
            print("NaN pixels", net, dt, fuse, flush=True)
            got, _ = _scan(fsb, layers, params, img, dt)
            masks[dt, fuse] = np.isnan(got)
    assert 0 < masks["f32", "0"].sum() < masks["f32", "0"].size
    for k, m in masks.items():
        assert np.array_equal(m, masks["f32", "0"]), (k, m.sum(), masks["f32", "0"].sum())


@pytest.mark.parametrize("cout", [97, 112, 48])
@pytest.mark.parametrize("mb", [2, 4])
def test_bf16_padding_blocks_of_paired_tiles(fsb, monkeypatch, cout, mb):
    """A forced 4 x 2 channel tile whose last block is past an odd count of
    output blocks: in a pair of bf16 blocks that block still holds channels
    (8g + 4 .. 8g + 7 of the pair's 32), and none may be dropped."""
    layers = [wl.conv(2, 3, 48), wl.conv(2, 48, cout), wl.conv(1, cout, 16), wl.fc(1, 16, 3, "none")]
    w0 = ix.patch_size(layers)
    params = wl.make_weights(layers, cout, 0.1)
    img = wl.make_image(cout + 1, 1, w0 + 33, w0 + 40, 3)
    base, _ = _scan(fsb, layers, params, img, "bf16")
    monkeypatch.setenv("FRAGSCAN_TILE", "1:%d,4,2" % mb)
    got, names = _scan(fsb, layers, params, img, "bf16")
    print("paired tiles", cout, mb, names, flush=True)
    assert names[1].startswith("conv_frag_mfma<%d, 4, 2, 1, " % mb) and _half(names[1]), names
    assert np.array_equal(got, base)
