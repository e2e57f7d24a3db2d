"""Shadow maps whose layers are so thin that the quotient of a depth and the layer depth leaves the
float range: everything behind the first hit lies in the last layer, as with layers that are merely
thin."""
import dataclasses

import numpy as np
import pytest
import torch

import hairsynth as hs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("thin", [1e-30, 8e-31, 1e-37])
def test_infinite_layer_quotients(hip, thin):
    print(f"case: layers of {thin} in a groom 1e10 across", flush=True)
    small = hs.make_asset(300, 8, 60.0, seed=5)
    k = np.float32(1e11)
    asset = dataclasses.replace(small, xyz=small.xyz * k, width=small.width * k)
    cam, lights = hs.camera_for(asset, 120, 90), hs.default_lights(asset, with_point=False)
    ctx = hip.Context(0)
    aid = ctx.upload_asset(asset)
    ws = ctx.workspace()
    out = []
    for delta in (1e-20, thin):
        img, _, _ = ctx.render_shadowed(aid, 0, cam, lights, (64, 4, delta), ws=ws)
        torch.cuda.synchronize()
        out.append((img.cpu().numpy().copy(), ctx.debug_dom(ws, 0, 64)[0]))
    (img0, tex0), (img1, tex1) = out
    hit = tex0[:, 0] > 0
    extent = float((tex0[hit, 0]).max())
    assert extent / thin > 3.5e38 and hit.sum() > 100
    assert (tex0[hit, 4] > tex0[hit, 1]).any()             # hairs behind the first layer
    assert np.array_equal(tex0.view(np.uint32), tex1.view(np.uint32))
    assert np.array_equal(img0.view(np.uint32), img1.view(np.uint32))
    assert np.isfinite(img1).all() and img1[..., 3].max() > 0
    ctx.close()
