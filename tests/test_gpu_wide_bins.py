"""Tile lists of wide segments, whose tiles are found row by row as exact intervals: axis-parallel,
steep, slanted and pixel-short segments with radii on both sides of the 2 px where the footprint is
looked at, and of many tiles, across all image edges, against the oracle's test per tile."""
import numpy as np
import pytest
import torch

import hairsynth as hs
from oracle import render as R

pytestmark = pytest.mark.gpu

FY = float(np.float32(150.0))


@pytest.fixture(scope="module")
def ctx(hip):
    c = hip.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("hw_px", [1.4, 1.5, 1.6, 8.0, 75.0, 400.0])
@pytest.mark.parametrize("size", [(16, 16), (331, 245)])
def test_wide_segments_tiles(hip, ctx, hw_px, size):
    W, H = size
    K = 240
    rng = np.random.default_rng(int(hw_px * 10) + W)
    d = 1.0 + 0.5 * rng.random(K)
    mid = np.stack([(rng.random(K) - 0.5) * 1.4 * W, (rng.random(K) - 0.5) * 1.4 * H], -1) * d[:, None] / FY
    ang = rng.random(K) * 2.0 * np.pi
    ang[:60] = rng.integers(0, 4, 60) * 0.5 * np.pi        # axis-parallel
    half = (np.where(rng.random(K) < 0.3, 0.2, 60.0 * rng.random(K)) * d / FY)[:, None]
    step = half * np.stack([np.cos(ang), np.sin(ang)], -1)
    xyz = np.empty((3, 2 * K), dtype=np.float32)
    for e, s in ((0, -1.0), (1, 1.0)):
        p = mid + s * step
        xyz[0, e::2], xyz[1, e::2], xyz[2, e::2] = p[:, 0], p[:, 1], -d
    sig = np.repeat(np.array([0.3, 0.6, 1.2], dtype=np.float32)[:, None], K, axis=1)
    asset = hs.Asset(K, 1, xyz, np.full(K, 8e-6, dtype=np.float32), np.ascontiguousarray(sig))
    axes = (hw_px * (0.8 + 0.4 * rng.random(K)) * d / FY).astype(np.float32)
    lod = {"centers": xyz.T.reshape(K, 2, 3).copy(), "ahat": np.tile(np.array([0.0, 0.0, 1.0], np.float32), (K, 1, 1)),
           "axes": np.stack([axes, axes], -1)[:, None, :].copy(), "n_total": np.full(K, 6, np.int32),
           "sigma_a": sig.copy(), "r": np.full(K, 4e-6, np.float32)}
    cam = hs.Camera(np.zeros(3, np.float32), np.eye(3, dtype=np.float32), FY, FY, W / 2.0, H / 2.0, W, H, 0.01)
    aid = ctx.upload_asset(asset)
    ctx.set_lod(aid, 1, lod)
    ws = ctx.workspace()
    _, st, _ = ctx.render(aid, 1, cam, hs.default_lights(asset, with_point=False), ws=ws)
    torch.cuda.synchronize()
    c, XA, YA, XB, YB, izA, izB, hw, hw_fx, vis = R.segment_records(R.cluster_level(lod), cam)
    tid, sid, _ = R.rs.bins(XA, YA, XB, YB, hw_fx, vis, W, H, 16)
    T = -(-W // 16) * -(-H // 16)
    print(f"case: half-width {hw_px} px at {W} x {H}: {len(tid)} pairs", flush=True)
    assert st["pairs"] == len(tid) and vis.sum() > K // 4
    ts, segs = ctx.debug_bins(ws, T, int(st["pairs"]))
    start = np.searchsorted(tid, np.arange(T + 1))
    assert np.array_equal(ts.astype(np.int64), start)
    for t in range(T):
        assert np.array_equal(np.sort(segs[ts[t]:ts[t + 1]]), sid[start[t]:start[t + 1]]), t
    ws.close()
    ctx.release(aid)
