"""Scans whose layers fall back to another tiling (or stay off a slower one):
maps against the CPU fragment method."""
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


def _check(fsb, layers, dt, more, seed):
    """Probabilities against the oracle: float32 sums of up to ~1000 terms
    behind a tanh, or a few roundings to 8 significand bits per value."""
    h0, w0 = ix.patch_hw(layers)
    sigma = [1.0 / np.sqrt(L["c_in"] * L["k"] * (L.get("kx") or L["k"])) for L in layers if L["kind"] != "pool"]
    params = wl.make_weights(layers, seed, float(np.mean(sigma)))
    img = wl.make_image(seed + 1, 2, h0 + more[0], w0 + more[1], layers[0]["c_in"])
    ref = oracle.frag_cpu.frag_scan(layers, params, img, (h0, w0))
    net = fsb.Net(layers, params, layers[0]["c_in"], 0, dt)
    names = [L["name"] for L in net.launches(*img.shape[:3])]
    print("fallback", dt, img.shape, names, flush=True)
    got = net.scan(torch.from_numpy(img).cuda())
    torch.cuda.synchronize()
    net.close()
    assert np.abs(got.cpu().numpy() - ref).max() <= (2e-6 if dt == "f32" else 3e-2)
    return names


@pytest.mark.parametrize("dt,cin,cout,ky,kx", [("f32", 48, 48, 8, 8), ("f32", 48, 48, 9, 9), ("f32", 48, 40, 3, 22),
                                               ("f32", 48, 48, 2, 33), ("bf16", 16, 128, 12, 12),
                                               ("bf16", 48, 200, 17, 9)])
def test_pools_beyond_a_fused_tile(fsb, dt, cin, cout, ky, kx):
    layers = [wl.conv(2, 1, cin), wl.conv(3, cin, cout), wl.pool(ky, cout, kx=kx), wl.fc(1, cout, 20),
              wl.fc(1, 20, 3, "softmax")]
    names = _check(fsb, layers, dt, (21, 30), ky + kx)
    if ky * kx > 64:
        assert any(n.startswith("pool_") for n in names), names


@pytest.mark.parametrize("dt,cin,k,cout", [("f32", 192, 3, 100), ("f32", 256, 2, 112), ("f32", 240, 2, 97),
                                           ("bf16", 336, 3, 112), ("bf16", 240, 5, 100)])
def test_seven_channel_blocks_in_64_pixel_tiles(fsb, dt, cin, k, cout):
    layers = [wl.conv(1, 3, cin), wl.fc(k, cin, cout), wl.fc(1, cout, 3, "softmax")]
    names = _check(fsb, layers, dt, (40, 53), cin + k)
    assert any("<1, 7, 1, 1, " in n and n.split(">")[0].endswith("true") for n in names), names


@pytest.mark.parametrize("cin,cout,p,more", [(16, 176, 3, (60, 51)), (48, 200, 5, (70, 61)), (16, 144, 8, (90, 97)),
                                             (32, 129, 10, (12, 15))])
def test_wide_layers_with_pools_on_small_grids(fsb, cin, cout, p, more):
    """Every tile size the planner may take there."""
    layers = [wl.conv(2, 1, cin), wl.conv(1, cin, cout), wl.pool(p, cout), wl.fc(1, cout, 20), wl.fc(1, 20, 3, "softmax")]
    names = _check(fsb, layers, "f32", more, p)
    assert any(", 7, 2, 1, " in n and "+pool" in n for n in names), names


def test_head_grids_that_take_a_cu_each(fsb):
    """Float32 fused heads run one workgroup per CU where a quarter of the
    tiles hold no pixel, or where two would leave half a round empty; on other
    grids as many as fit."""
    layers = [wl.conv(4, 1, 32), wl.pool(8, 32, stride=5), wl.pool(2, 32), wl.conv(4, 32, 208), wl.pool(3, 208),
              wl.fc(1, 208, 100), wl.fc(1, 100, 2, "none")]
    params = wl.make_weights(layers, 7, 0.05)
    net = fsb.Net(layers, params, 1)
    sparse, dense = net.launches(1, net.patch + 8, net.patch + 11)[-1], net.launches(4, 400, 400)[-1]
    net.close()
    assert sparse["name"] == dense["name"] and "+head" in sparse["name"], (sparse, dense)
    assert (sparse["per_cu"], dense["per_cu"]) == (1, 2), (sparse, dense)
    layers = [wl.conv(2, 1, 48), wl.pool(3, 48), wl.fc(3, 48, 100), wl.fc(1, 100, 2, "none")]
    net = fsb.Net(layers, wl.make_weights(layers, 7, 0.05), 1)
    heads = {H: net.launches(1, H, H + 3)[-1] for H in (300, 420, 510)}
    net.close()
    rounds = {H: -(-L["grid"] // 256) for H, L in heads.items()}
    assert [rounds[H] for H in (300, 420, 510)] == [2, 3, 5], rounds
    assert {H: L["per_cu"] for H, L in heads.items()} == {300: 2, 420: 1, 510: 2}, heads


@pytest.mark.parametrize("act", ["tanh", "none"])
@pytest.mark.parametrize("cout,ky,kx", [(20, 2, 2), (33, 3, 3), (100, 5, 5), (100, 4, 3), (100, 2, 5), (39, 1, 4), (17, 3, 1)])
def test_fused_pools_of_odd_channel_counts(fsb, monkeypatch, act, cout, ky, kx):
    """bf16 outputs not in whole 16-byte chunks, even and odd window columns:
    the fused pool's values are the separate one's bit for bit."""
    layers = [wl.conv(2, 3, 32), wl.conv(2, 32, cout, act), wl.pool(ky, cout, kx=kx), wl.fc(1, cout, 16),
              wl.fc(1, 16, 3, "none")]
    h0, w0 = ix.patch_hw(layers)
    params = wl.make_weights(layers, cout, 0.1)
    img = torch.from_numpy(wl.make_image(cout + 1, 2, h0 + 37, w0 + 50, 3)).cuda()
    got = {}
    for fuse in ("1", "0"):
        monkeypatch.setenv("FRAGSCAN_POOL_FUSE", fuse)
        net = fsb.Net(layers, params, 3, 0, "bf16")
        names = [L["name"] for L in net.launches(*img.shape[:3])]
        print("odd channels", act, cout, (ky, kx), names, flush=True)
        assert ("+pool" in names[1]) == (fuse == "1"), names
        got[fuse] = net.scan(img).clone()
        torch.cuda.synchronize()
        net.close()
    assert torch.equal(got["1"], got["0"])
