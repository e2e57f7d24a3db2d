"""Light views with few and with many work items (one and four chunks of a tile's list per block), on
a fresh workspace and on one that drew a larger frame before: the maps are the same bits, and the
chunks per block follow the view, not what the workspace has room for."""
import numpy as np
import pytest
import torch

import hairsynth as hs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("strands, res", [(3000, 64), (40000, 1024)])
def test_maps_after_larger_frames(hip, strands, res):
    ctx = hip.Context(0)
    asset = hs.make_asset(strands, 16, 90.0, seed=3)
    lights = hs.default_lights(asset, with_point=False)
    aid = ctx.upload_asset(asset)
    cam, big = hs.camera_for(asset, 320, 240), hs.camera_for(asset, 1920, 1080)
    fresh, used = ctx.workspace(), ctx.workspace()
    ctx.render_shadowed(aid, 0, big, lights, (2048, 2, 0.02), ws=used)
    maps = []
    for ws in (fresh, used):
        for _ in range(2):
            ctx.render_shadowed(aid, 0, cam, lights, (res, 4, 0.02), ws=ws)
            torch.cuda.synchronize()
            maps.append(ctx.debug_dom(ws, 0, res)[0])
    print(f"case: {strands} strands, map {res}: {int((maps[0][:, 0] > 0).sum())} texels with hair", flush=True)
    for m in maps[1:]:
        assert np.array_equal(m.view(np.uint32), maps[0].view(np.uint32))
    ctx.close()
