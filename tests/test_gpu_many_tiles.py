"""Images of more tiles than one binning pass counts in LDS (36,864) and than the single-block scans
take (65,536): the tile lists of wide thick hairs, binned with eight lanes each in two passes, and
the frames' fragment counts and pixels, against the oracle."""
import dataclasses

import numpy as np
import pytest
import torch

import hairsynth as hs
from oracle import lod as OL
from oracle import render as R
from test_gpu_wide_bins import ctx, test_wide_segments_tiles as wide_segments_tiles   # noqa: F401

pytestmark = pytest.mark.gpu

SIZES = [(3216, 2960), (4112, 4112)]    # 201 x 185 and 257 x 257 tiles


@pytest.mark.parametrize("hw_px", [8.0, 400.0])
@pytest.mark.parametrize("size", SIZES)
def test_tile_lists(hip, ctx, hw_px, size):                                          # noqa: F811
    wide_segments_tiles(hip, ctx, hw_px, size)


@pytest.mark.parametrize("level", [0, 1])
@pytest.mark.parametrize("size", SIZES)
def test_frames(hip, ctx, level, size):                                              # noqa: F811
    asset = hs.make_asset(60, 6, 90.0, seed=5)
    lod = OL.build_level(asset, np.arange(60) % 7)
    cam, lights = hs.camera_for(asset, *size), hs.default_lights(asset, with_point=True)
    geom = R.strand_level(asset) if level == 0 else R.cluster_level(lod)
    aid = ctx.upload_asset(asset)
    ctx.set_lod(aid, 1, lod)
    ws = ctx.workspace()
    rect = (size[0] // 2 - 200, size[1] // 2 - 200, 400, 400)
    geom = R.split_long(geom, cam)
    part = R.rasterize(geom, cam, rect=rect)
    alpha, L = R.fragment_radiance(geom, part, cam, lights, R.material(asset.material))
    x, y, w, h = rect
    local = (part.pix // part.W - y) * w + part.pix % part.W - x
    want = R.composite(dataclasses.replace(part, pix=local, W=w, H=h), alpha, L).numpy()
    n = len(R.rasterize(geom, cam).seg)
    for frame in range(2):                                   # (a first and a warm one)
        img, st, _ = ctx.render(aid, level, cam, lights, ws=ws)
        torch.cuda.synchronize()
        print(f"case: level {level} at {size[0]} x {size[1]}, frame {frame}: {st['fragments']} fragments", flush=True)
        assert st["fragments"] == n and len(part.seg) > 1000
        got = img[y:y + h, x:x + w].cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - want) <= 1e-4 * np.abs(want) + 1e-7)
    ws.close()
    ctx.release(aid)
