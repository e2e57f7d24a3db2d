"""Frames on workspaces that hold just what the frame cannot do without.  Some buffers are there
for speed (a shadow map's layer sums of all layers at once) or larger for it (the table of small
batches); where they do not fit the workspace's limit or the context's budget, the frame starts
over without headroom and without the layer sums, and gives the same result, bit for bit, as
without a limit.  The static scratch keeps the batch table where the binning matrix was, and
falls back to full batches where that is too small.

The limits of the shadowed strand and mixed frames are what a workspace holds whose light views
have the per-pixel tables of a camera frame and nothing more, those of plain frames what it holds
with full batches."""
import numpy as np
import pytest
import torch

import hairsynth as hs

pytestmark = pytest.mark.gpu

MAP = (1024, 7, 0.02)
LIMITS = {"strands": 80_851_412, "thick hairs": 131_000_000, "mixed": 100_861_268}


class Scene:
    def __init__(self, hip, budget=0):
        self.ctx = hip.Context(0, budget)
        self.asset = hs.make_asset(2500, 10, 90.0, seed=23, sigma_spread=True)
        self.lights = hs.default_lights(self.asset, with_point=True)
        self.aid = self.ctx.upload_asset(self.asset)
        self.ctx.build_lod(self.aid, hs.kmeans_hierarchy(self.asset, (400, 80, 12), seed=23))
        gs = (self.ctx.lod_groups(self.aid), self.asset.segs)
        self.levels = torch.tensor(np.random.default_rng(7).integers(0, 4, size=gs).astype(np.int32), device="cuda:0")

    def shadowed(self, kind, ws, width=640, height=480, shadow=MAP, **more):
        cam = hs.camera_for(self.asset, width, height)
        if kind == "mixed":
            return self.ctx.render_mixed_shadowed(self.aid, cam, self.lights, self.levels, shadow, ws=ws, **more)
        return self.ctx.render_shadowed(self.aid, 0 if kind == "strands" else 1, cam, self.lights, shadow, ws=ws, **more)


@pytest.fixture(scope="module")
def scene(hip):
    s = Scene(hip)
    yield s
    s.ctx.close()


def _same(a, b):
    torch.cuda.synchronize()
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("kind", ["strands", "thick hairs", "mixed"])
def test_shadowed_frames_within_a_limit(hip, scene, kind):
    free = scene.ctx.workspace()
    ref, _, _ = scene.shadowed(kind, free)
    ref_map = scene.ctx.debug_dom(free, 0, MAP[0])
    print(f"case: shadowed {kind}: {free.memory()[0]} bytes without a limit, {LIMITS[kind]} with one", flush=True)
    assert free.memory()[0] > LIMITS[kind]
    ws = scene.ctx.workspace(LIMITS[kind])
    for _ in range(2):                                     # (a first and a warm frame)
        img, _, _ = scene.shadowed(kind, ws)
        assert _same(img, ref)
        tex, grid = scene.ctx.debug_dom(ws, 0, MAP[0])
        assert np.array_equal(tex.view(np.uint32), ref_map[0].view(np.uint32))
        assert ws.memory()[0] <= LIMITS[kind]
    # another number of layers, a larger and a smaller map and image on the same workspaces
    for size, shadow in (((320, 200), (1024, 1, 0.02)), ((640, 480), (512, 4, 0.05)), ((640, 480), (1000, 7, 1e-4))):
        ref, _, _ = scene.shadowed(kind, free, *size, shadow)
        img, _, _ = scene.shadowed(kind, ws, *size, shadow)
        assert _same(img, ref)
    # no more limit: the buffer for all layers again
    ws.set_limit(0)
    img, _, _ = scene.shadowed(kind, ws)
    ref, _, _ = scene.shadowed(kind, free)
    assert _same(img, ref) and ws.memory()[0] > LIMITS[kind]
    # far too little is still refused
    small = scene.ctx.workspace(1 << 20)
    with pytest.raises(hip.HairError) as e:
        scene.shadowed(kind, small)
    assert e.value.code == hip.HAIR_ENOMEM
    for w in (free, ws, small):
        w.close()


def _first(asset, n):
    x = np.asarray(asset.xyz).reshape(3, asset.n_strands, asset.segs + 1)[:, :n]
    return hs.Asset(n, asset.segs, np.ascontiguousarray(x.reshape(3, -1)), np.asarray(asset.width)[:n].copy(),
                    np.ascontiguousarray(np.asarray(asset.sigma_a)[:, :n]))


FULL_BATCHES = 67_072_229


@pytest.mark.parametrize("what", ["workspace", "budget"])
def test_plain_frames_within_a_limit(hip, what):
    print(f"case: 20,000 strands at 400 x 400, limited {what}", flush=True)
    asset = hs.make_asset(20000, 16, 90.0, seed=3)
    cam, lights = hs.camera_for(asset, 400, 400), hs.default_lights(asset, with_point=True)
    ctx = hip.Context(0)
    aid = ctx.upload_asset(asset)
    used = ctx.memory()[0]
    free = ctx.workspace()
    ref, st, _ = ctx.render(aid, 0, cam, lights, ws=free)
    assert free.memory()[0] > FULL_BATCHES
    if what == "budget":
        tight = hip.Context(0, used + FULL_BATCHES)
        aid2, ws = tight.upload_asset(asset), tight.workspace()
    else:
        tight, aid2, ws = ctx, aid, ctx.workspace(FULL_BATCHES)
    for _ in range(3):
        img, st2, _ = tight.render(aid2, 0, cam, lights, ws=ws)
        assert _same(img, ref)
        assert all(st2[k] == st[k] for k in ("batches", "fragments", "pairs", "deep_pixels"))
        assert ws.memory()[0] <= FULL_BATCHES
    # the deferred frame on the same workspace
    out = torch.empty_like(ref)
    tight.render_async(aid2, 0, cam, lights, out, ws)
    ws.finish()
    assert _same(out, ref)
    ws.close()
    free.close()
    if tight is not ctx:
        tight.close()
    ctx.close()


def test_static_scratch_keeps_the_batch_table_in_the_binning_matrix(hip):
    """20,062 strands at 896 x 640 fill the scratch to within a few hundred bytes."""
    asset = _first(hs.make_asset(21000, 16, 90.0, seed=3), 20062)
    lights = hs.default_lights(asset, with_point=False)
    cam = hs.camera_for(hs.make_asset(21000, 16, 90.0, seed=3), 896, 640)
    ctx = hip.Context(0)
    out = torch.empty((640, 896, 4), device="cuda:0")
    aid = ctx.upload_asset(asset)
    print("case: 20,062 strands at 896 x 640 in the static scratch", flush=True)
    _, st, rc = ctx.render_noalloc(aid, 0, cam, lights, out, raise_on_error=False)
    assert rc == hip.HAIR_OK
    ref, st2, _ = ctx.render(aid, 0, cam, lights)
    assert _same(out, ref) and st["batches"] == st2["batches"]
    ctx.close()


@pytest.mark.parametrize("n", [3900, 3970])
def test_static_scratch_with_few_wide_segments(hip, n):
    """One-segment strands some 40 px wide: 6.8 M fragments, a binning matrix of 74 KB, and small
    batches whose table (34 k) does not fit beside 3,970 of them."""
    whole = hs.make_asset(4000, 1, 90.0, seed=3)
    asset = _first(whole, n)
    asset.width[:] = 6e-2
    lights = hs.default_lights(asset, with_point=False)
    cam = hs.camera_for(whole, 900, 700)
    ctx = hip.Context(0)
    out = torch.empty((700, 900, 4), device="cuda:0")
    aid = ctx.upload_asset(asset)
    print(f"case: {n} wide segments in the static scratch", flush=True)
    _, st, rc = ctx.render_noalloc(aid, 0, cam, lights, out, raise_on_error=False)
    assert rc == hip.HAIR_OK
    ref, st2, _ = ctx.render(aid, 0, cam, lights)
    assert st["fragments"] == st2["fragments"]
    if n == 3900:
        assert _same(out, ref) and st["batches"] == st2["batches"]
    else:
        assert st["batches"] < st2["batches"]
        assert torch.allclose(out, ref, rtol=1e-4, atol=1e-7)
    ctx.close()


def test_thick_hairs_within_a_budget(hip):
    """2,000 x 16 narrow thick-hair segments at 1280 x 720: binned by eight lanes each where memory
    allows (a count matrix of 9 MB), by one lane where it does not (2.3 MB)."""
    asset = hs.make_asset(2000, 16, 90.0, seed=3)
    cam, lights = hs.camera_for(asset, 1280, 720), hs.default_lights(asset, with_point=True)
    held = []
    for budget in (0, 30_087_522):
        print(f"case: 2,000 thick hairs, budget {budget}", flush=True)
        ctx = hip.Context(0, budget)
        aid = ctx.upload_asset(asset)
        ctx.build_lod(aid, [np.arange(2000).astype(np.int32)])
        ws = ctx.workspace()
        for _ in range(2):
            img, st, _ = ctx.render(aid, 1, cam, lights, ws=ws)
            if not budget:
                ref = img
            assert _same(img, ref)
        held.append(ws.memory()[0])
        ctx.close()
    assert held[1] < held[0] - 4 * (500 - 62) * 80 * 45
