"""Batch sizes chosen per tile and frame: tiles whose fragments just fit one LDS batch, just do
not, and pixels around the smallest batch's 256 fragments, against the oracle; a frame of tiles on
both sides renders the same bits twice."""
import numpy as np
import pytest
import torch

import hairsynth as hs
from oracle import render as R

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(hip):
    c = hip.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n", [1, 16, 95, 96, 97, 255, 256, 257, 511, 1536, 1537])
def test_tiles_around_the_batch_sizes(hip, ctx, n):
    """n strands across pixel row 20 of a 40 x 40 image: a tile's 16 pixels of that row hold 16 n
    fragments (1536 at n = 96), a pixel n."""
    fy = float(np.float32(74.6))
    d = np.linspace(1.0, 2.0, n)
    xyz = np.empty((3, 2 * n), dtype=np.float32)
    xyz[0, 0::2], xyz[0, 1::2] = -0.2 * d, 0.2 * d
    xyz[1, 0::2] = xyz[1, 1::2] = -0.5 * d / fy
    xyz[2, 0::2] = xyz[2, 1::2] = -d
    sig = np.repeat(np.array([0.3, 0.6, 1.2], dtype=np.float32)[:, None], n, axis=1)
    asset = hs.Asset(n, 1, xyz, np.full(n, 2e-3, dtype=np.float32), np.ascontiguousarray(sig))
    cam = hs.Camera(np.zeros(3, np.float32), np.eye(3, dtype=np.float32), fy, fy, 20.0, 20.0, 40, 40, 0.01)
    lights = hs.default_lights(asset, with_point=False)
    aid = ctx.upload_asset(asset)
    ws = ctx.workspace()
    img, st, _ = ctx.render(aid, 0, cam, lights, ws=ws)
    torch.cuda.synchronize()
    first = img.clone()
    img, _, _ = ctx.render(aid, 0, cam, lights, ws=ws)
    torch.cuda.synchronize()
    ref, ras = R.render(R.strand_level(asset), cam, lights, tuple(float(v) for v in asset.material.as_array()))
    depth = np.bincount(ras.pix)
    print(f"case: {n} strands: {len(ras.seg)} fragments, {st['batches']} batches", flush=True)
    assert depth.max() == n and st["fragments"] == len(ras.seg)
    assert st["deep_pixels"] == int((depth > hip.HAIR_PIXEL_CAPACITY).sum())
    assert torch.equal(first.view(torch.int32), img.view(torch.int32))
    err = np.abs(img.cpu().numpy().astype(np.float64) - ref) - (1e-4 * np.abs(ref) + 1e-7)
    assert int((err > 0).sum()) == 0, float(err.max())
    ws.close()
    ctx.release(aid)
