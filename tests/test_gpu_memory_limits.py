"""Frames on workspaces that hold just what the frame cannot do without.  Some buffers are there
for speed (a shadow map's layer sums of all layers at once); where they do not fit the
workspace's limit, the frame starts over without them and gives the same result, bit for bit,
as on a workspace without a limit.

The limits of the strand and mixed frames are what a workspace holds whose light views have the
per-pixel tables of a camera frame and nothing more."""
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
