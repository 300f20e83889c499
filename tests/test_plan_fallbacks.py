"""Planner rules with more than one way to run a layer: the way that has no
tile must not refuse the net (CPU, planning-only handles: 256 CUs)."""
import numpy as np
import pytest

from oracle import index as ix
from paper_1302_1700_amd import fragscan as fsb
from paper_1302_1700_amd import workloads as wl


@pytest.fixture(autouse=True)
def _no_switches(monkeypatch):
    for v in ("FRAGSCAN_TILE", "FRAGSCAN_RUN", "FRAGSCAN_POOL_FUSE", "FRAGSCAN_SPLIT", "FRAGSCAN_WIDE",
              "FRAGSCAN_STORE", "FRAGSCAN_LDS_PAD", "FRAGSCAN_ROWTILES", "FRAGSCAN_NO_FUSED_HEAD"):
        monkeypatch.delenv(v, raising=False)


def _net(layers, dt="f32"):
    return fsb.Net(layers, wl.make_weights(layers, 0, 0.1), layers[0]["c_in"], 0, dt, plan_only=True)


WIDE_POOLS = [(8, 8), (9, 9), (10, 10), (12, 12), (16, 16), (3, 22), (2, 33)]


@pytest.mark.parametrize("ky,kx", WIDE_POOLS)
@pytest.mark.parametrize("side", [60, 100, 130, 400])
def test_wide_pools_at_every_size(ky, kx, side):
    """A pool whose window holds more outputs than a small grid's 64-pixel
    tile runs by itself, as on larger images: the same net plans at every
    size that holds its window."""
    layers = [wl.conv(4, 1, 48), wl.conv(3, 48, 48), wl.pool(ky, 48, kx=kx), wl.fc(2, 48, 200),
              wl.fc(1, 200, 2, "softmax")]
    h0, w0 = ix.patch_hw(layers)
    H, W = max(side, h0), max(side, w0)
    net = _net(layers)
    ls = net.launches(1, H, W)
    assert net.plan(1, H, W)["out_h"] == H - h0 + 1
    net.close()
    if ky * kx > 64:
        assert [L["kind"] for L in ls][-2:] == [1, 0] and "+pool" not in ls[-3]["name"], ls


@pytest.mark.parametrize("dt,cin,k,cout,p", [("bf16", 112, 2, 144, 17), ("bf16", 16, 1, 128, 12), ("f32", 16, 1, 16, 30),
                                             ("bf16", 32, 1, 64, 17), ("f32", 1, 3, 48, 17)])
def test_pool_windows_beyond_any_fused_tile(dt, cin, k, cout, p):
    """Layers that fuse their pools by the work rule: a window of more outputs
    than their largest tile is pooled by itself."""
    layers = ([wl.conv(2, 3, cin)] if cin > 1 else []) + [wl.conv(k, cin, cout), wl.pool(p, cout), wl.fc(1, cout, 16),
                                                          wl.fc(1, 16, 3, "softmax")]
    h0, w0 = ix.patch_hw(layers)
    net = _net(layers, dt)
    ls = net.launches(2, h0 + 90, w0 + 71)
    net.close()
    assert sum(L["kind"] == 1 for L in ls) == 1, ls


def test_tilings_that_do_not_fit_leave_no_error_message():
    layers = [wl.conv(4, 1, 48), wl.conv(3, 48, 48), wl.pool(9, 48), wl.fc(2, 48, 200), wl.fc(1, 200, 2, "softmax")]
    net = _net(layers)
    with pytest.raises(fsb.FsError, match="smaller than the window"):
        net.plan(1, 9, 60)
    before = fsb.load().fs_last_error()
    net.plan(1, 60, 60)
    assert fsb.load().fs_last_error() == before
    net.close()


@pytest.mark.parametrize("cin", [16, 48, 96, 128, 192, 256])
@pytest.mark.parametrize("k", [1, 2, 3, 5])
def test_half_steps_refuse_no_layer(monkeypatch, cin, k):
    """Every float32 layer that plans on the float32 products plans on the
    split ones too, whatever its outputs: the largest windows fit only in the
    64-pixel tiles."""
    taken = 0
    for cout in (20, 48, 100, 112, 128, 200, 300):
        layers = [wl.conv(1, 1, cin), wl.conv(k, cin, cout), wl.fc(1, cout, 2, "softmax")]
        net = _net(layers)
        for H, W in ((300, 300), (k + 60, k + 6)):
            with monkeypatch.context() as m:
                m.setenv("FRAGSCAN_SPLIT", "0")
                try:
                    net.plan(1, H, W)
                except fsb.FsError:
                    continue
            half = [L["name"].split(">")[0].endswith("true") for L in net.launches(1, H, W)]
            assert half[1], (cin, k, cout, H, W)
            taken += 1
        net.close()
    assert taken or (cin, k) in ((192, 5), (256, 5))  # (no tile holds a 5x5 window of these)


@pytest.mark.parametrize("dt,layers,H,W", [
    ("f32", [wl.conv(2, 1, 16, kx=1), wl.conv(1, 16, 144), wl.fc(3, 144, 100), wl.fc(1, 100, 3, "softmax")], 504, 8),
    ("f32", [wl.conv(1, 1, 192), wl.fc(3, 192, 100), wl.fc(1, 100, 2, "softmax")], 300, 300),
    ("f32", [wl.conv(1, 1, 256), wl.fc(3, 256, 112), wl.fc(1, 112, 2, "softmax")], 300, 300),
    ("bf16", [wl.conv(9, 1, 304), wl.pool(2, 304, kx=3), wl.fc(3, 304, 100), wl.fc(1, 100, 3, "softmax")], 74, 37),
    ("bf16", [wl.conv(1, 1, 240), wl.fc(5, 240, 100), wl.fc(1, 100, 2, "softmax")], 300, 300),
    ("bf16", [wl.conv(1, 1, 336), wl.fc(3, 336, 112), wl.fc(1, 112, 2, "softmax")], 300, 300)])
def test_seven_channel_blocks_in_64_pixel_tiles(dt, layers, H, W):
    """65 to 112 outputs behind windows that leave LDS for 64 pixels only."""
    net = _net(layers, dt)
    names = [L["name"] for L in net.launches(1, H, W)]
    net.close()
    assert any("<1, 7, 1, 1, " in n and n.split(">")[0].endswith("true") for n in names), names


@pytest.mark.parametrize("p,side,fused", [(2, 60, True), (2, 130, True), (3, 130, True), (4, 64, True), (4, 130, False),
                                          (5, 96, True), (6, 96, True), (6, 130, False), (7, 130, False),
                                          (8, 60, False), (8, 130, False)])
def test_small_grid_pools_by_fused_tiles(monkeypatch, p, side, fused):
    """A pool behind a 64-pixel tile is fused while the fused grid stays near
    one round of workgroups: never the thousands of one-value tiles of a wide
    window (8x8 on 130^2: 14520)."""
    layers = [wl.conv(3, 1, 48), wl.conv(3, 48, 48), wl.pool(p, 48), wl.fc(2, 48, 200), wl.fc(1, 200, 2, "softmax")]
    net = _net(layers)
    mid = [L for L in net.launches(1, side, side + 3) if L["layer"] == 1]
    assert len(mid) == 1 and mid[0]["name"].startswith("conv_frag_mfma<2, 3, 1, 2, "), mid
    assert ("+pool" in mid[0]["name"]) == fused, mid
    assert mid[0]["grid"] <= 1024, mid
    monkeypatch.setenv("FRAGSCAN_POOL_FUSE", "1")
    assert "+pool" in [L for L in net.launches(1, side, side + 3) if L["layer"] == 1][0]["name"]
    net.close()


@pytest.mark.parametrize("cin,cout,p,px,side,fused", [
    (16, 80, 2, 2, 300, True), (16, 224, 3, 3, 300, True), (48, 128, 4, 4, 300, False), (48, 128, 2, 3, 300, False), (48, 128, 4, 4, 90, True),
    (48, 100, 2, 2, 300, False), (48, 100, 8, 8, 300, False), (80, 112, 5, 5, 300, True), (80, 112, 5, 5, 90, True),
    (80, 112, 8, 8, 300, True), (16, 224, 10, 10, 300, False), (48, 128, 10, 10, 90, False), (16, 64, 4, 4, 300, True)])
def test_wide_half_step_pools(monkeypatch, cin, cout, p, px, side, fused):
    """bf16 half-step layers of more than 64 outputs (a separate pool before
    they took the vector path) fuse only the pools that run faster so; up to
    64 outputs the work rule alone decides."""
    layers = [wl.conv(3, 1, cin), wl.conv(2, cin, cout), wl.pool(p, cout, kx=px), wl.fc(1, cout, 16),
              wl.fc(1, 16, 2, "softmax")]
    net = _net(layers, "bf16")
    mid = lambda: [L for L in net.launches(1, side, side + 3) if L["layer"] == 1][0]["name"]
    assert ("+pool" in mid()) == fused, mid()
    monkeypatch.setenv("FRAGSCAN_POOL_FUSE", "1")
    assert "+pool" in mid()
    net.close()


@pytest.mark.parametrize("cin,k,cout", [(16, 2, 176), (48, 1, 200)])
@pytest.mark.parametrize("p,side", [(2, 60), (3, 90), (5, 90), (5, 128), (8, 30), (8, 128), (10, 30)])
def test_small_grid_pools_of_wide_layers(monkeypatch, cin, k, cout, p, side):
    """129 to 224 outputs on a small grid: the pool stays fused, in the small
    tile only while its halo leaves the tiles near a round of workgroups."""
    layers = [wl.conv(3, 1, cin), wl.conv(k, cin, cout), wl.pool(p, cout), wl.fc(1, cout, 16),
              wl.fc(1, 16, 2, "softmax")]
    net = _net(layers)
    mid = lambda: [L for L in net.launches(1, side, side + 3) if L["layer"] == 1][0]
    got = mid()
    assert "+pool" in got["name"], got
    mb = int(got["name"].split("<")[1].split(",")[0])
    assert got["grid"] <= {1: 512, 2: 1024, 4: 1 << 24}[mb], got
    assert mb == {(2, 60): 1, (8, 30): 2, (8, 128): 4, (10, 30): 4}.get((p, side), mb), got
    monkeypatch.setenv("FRAGSCAN_RUN", "0")  # keeps the layer's own tile
    assert mid()["name"].startswith("conv_frag_mfma<4, 7, 2, 1, ")
    net.close()


def test_pool_kernels_have_names_of_their_own(monkeypatch):
    """Launch names (the profiler's) tell the row-band kernels from the one
    that takes a child row per workgroup."""
    monkeypatch.setenv("FRAGSCAN_POOL_FUSE", "0")
    for (p, s), want in {(3, 3): "pool_frag_rows<", (3, 2): "pool_frag<", (5, 5): "pool_frag_child_row<",
                         (5, 2): "pool_frag_child_row<"}.items():
        net = _net([wl.conv(2, 1, 16), wl.pool(p, 16, stride=s), wl.fc(1, 16, 2, "softmax")])
        assert net.launches(1, 60, 60)[1]["name"].startswith(want)
        net.close()


def test_wide_half_step_pools_by_work():
    """A halo of many tiles is not recomputed over a long K walk."""
    layers = [wl.conv(2, 1, 80), wl.pool(3, 80), wl.conv(3, 80, 176, kx=5), wl.pool(8, 176), wl.fc(1, 176, 48),
              wl.fc(1, 48, 2, "softmax")]
    net = _net(layers, "bf16")
    names = {L["layer"]: L["name"] for L in net.launches(1, 451, 458)}
    net.close()
    assert "+pool" not in names[2] and names[3].startswith("pool_frag_child_row<"), names
