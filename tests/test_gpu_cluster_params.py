"""Level parameters set on the device, any subset of the three arrays in one copy, and gradients that
start from cleared arrays whatever those held before."""
import numpy as np
import pytest
import torch

import hairsynth as hs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("clusters", [1, 7, 300])
@pytest.mark.parametrize("which", [(1, 1, 1), (1, 0, 0), (0, 1, 0), (0, 0, 1), (0, 0, 0)])
def test_set_cluster_params(hip, clusters, which):
    ctx = hip.Context(0)
    asset = hs.make_asset(400, 5, 60.0, seed=3)
    aid = ctx.upload_asset(asset)
    ctx.build_lod(aid, [(np.arange(400) % clusters).astype(np.int32)])
    old = ctx.get_lod(aid, 1)
    old = [np.array(a) for a in (old.axes, old.r, old.sigma_a)]
    new = [(1.5 * a + 1e-4).astype(np.float32) for a in old]
    args = [torch.tensor(n, device="cuda:0") if w else None for n, w in zip(new, which)]
    print(f"case: {clusters} clusters, arrays {which}", flush=True)
    ctx.set_cluster_params(aid, 1, *args)
    torch.cuda.synchronize()
    got = ctx.get_lod(aid, 1)
    for g, o, n, w in zip((got.axes, got.r, got.sigma_a), old, new, which):
        assert np.array_equal(np.array(g), n if w else o)
    ctx.close()
