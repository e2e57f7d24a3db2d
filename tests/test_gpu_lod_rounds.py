"""Per-group levels where a wave's 64 lanes just hold a group's owners, just do not, and hold several
levels at once; and the selection's row counts on both sides of its one-block limit, with entries out
of range refused on both, against the oracle."""
import numpy as np
import pytest
import torch

import hairsynth as hs
from oracle import mixed as M
from test_gpu_mixed import oracle_levels

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(hip):
    c = hip.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("mid", [1, 2, 62, 63, 64, 65, 127, 128])
def test_initial_levels_over_several_rounds(hip, ctx, mid):
    """Three groups; per group one coarse owner, `mid` and about 140 finer ones."""
    asset = hs.make_asset(900, 4, 60.0, seed=31, sigma_spread=True)
    i = np.arange(asset.n_strands)
    g, j = i % 3, i // 3
    m = j % mid
    fine = np.unique(g * 100000 + m * 200 + (j // mid) % max(1, 140 // mid), return_inverse=True)[1]
    assigns = [fine.astype(np.int32), (g * mid + m).astype(np.int32), g.astype(np.int32)]
    aid = ctx.upload_asset(asset)
    lods = oracle_levels(ctx, aid, asset, assigns)
    geoms, grps = M.level_geoms(asset, lods), M.groups(assigns)
    cam = hs.camera_for(asset, 90, 70)
    G, S = 3, asset.segs
    seen = set()
    w = np.concatenate([M.level_widths(geoms[l], grps[l], G, S, cam).ravel() for l in (1, 2, 3)])
    for eps in [float(x) for x in np.quantile(w[w > 0], [0.0, 0.3, 0.6, 0.9])] + [1e6]:
        lev = torch.empty((G, S), dtype=torch.int32, device="cuda:0")
        ctx.lod_init(aid, cam, eps, lev)
        ref = M.init_levels(geoms, grps, cam, eps)
        print(f"case: {mid} middle owners, eps {eps:.3f}", flush=True)
        assert np.array_equal(lev.cpu().numpy(), ref)
        seen |= set(np.unique(ref).tolist())
    assert len(seen) >= 2
    ctx.release(aid)


@pytest.mark.parametrize("clusters, segs", [(1, 1), (1023, 64), (1024, 64), (1025, 64)])
def test_selection_counts(hip, ctx, clusters, segs):
    n = clusters + 40
    asset = hs.make_asset(n, segs, 60.0, seed=32)
    a = (np.arange(n) % clusters).astype(np.int32)
    aid = ctx.upload_asset(asset)
    ctx.build_lod(aid, [a])
    G = ctx.lod_groups(aid)
    assert G == clusters
    cam = hs.camera_for(asset, 48, 40)
    lights = hs.default_lights(asset, with_point=False)
    rng = np.random.default_rng(clusters)
    levels = rng.integers(0, 2, size=(G, segs)).astype(np.int32)
    want = int(np.where(levels == 1, 1, np.bincount(a, minlength=G)[:, None]).sum())
    ws = ctx.workspace()
    lev = torch.tensor(levels, device="cuda:0")
    print(f"case: {G} groups x {segs}: {want} rows", flush=True)
    _, st, _ = ctx.render_mixed(aid, cam, lights, lev, eps_w=0.0, ws=ws)
    assert st["segments"] == want
    levels[0, 0], levels[-1, -1] = 7, -1
    with pytest.raises(hip.HairError, match=f"{2 if G * segs > 1 else 1} entries"):
        ctx.render_mixed(aid, cam, lights, torch.tensor(levels, device="cuda:0"), eps_w=0.0, ws=ws)
    ws.close()
    ctx.release(aid)
