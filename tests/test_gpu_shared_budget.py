"""Several workspaces and assets within one context's budget.  What a workspace keeps for speed alone
(a shadow map's layer sums, a wide binning matrix) is given back when another workspace or an asset
of the context needs the memory: one workspace's shadowed frames take no other's room."""
import threading

import pytest
import torch

import hairsynth as hs

pytestmark = pytest.mark.gpu

MAP = (1024, 7, 0.02)
HELD = 80_851_412    # a workspace whose light views have the per-pixel tables of a camera frame and nothing more


class Scene:
    def __init__(self, hip, budget=0):
        self.ctx = hip.Context(0, budget)
        self.asset = hs.make_asset(2500, 10, 90.0, seed=23, sigma_spread=True)
        self.lights = hs.default_lights(self.asset, with_point=True)
        self.aid = self.ctx.upload_asset(self.asset)
        self.cam = hs.camera_for(self.asset, 320, 200)

    def shadowed(self, ws):
        img = self.ctx.render_shadowed(self.aid, 0, self.cam, self.lights, MAP, ws=ws)[0]
        torch.cuda.synchronize()
        return img


@pytest.fixture(scope="module")
def alone(hip):
    """The image, the asset's bytes and those of a workspace in a context without a budget."""
    s = Scene(hip)
    asset = s.ctx.memory()[0]
    ws = s.ctx.workspace()
    ref = s.shadowed(ws)
    most = ws.memory()[0]
    ws.close()
    s.ctx.close()
    print(f"case: asset {asset} bytes, workspace {most}", flush=True)
    assert most > 1.5 * HELD
    return ref, asset, most


def _same(a, b):
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


def test_two_workspaces_in_a_budget_for_two(hip, alone):
    ref, asset, most = alone
    s = Scene(hip, asset + 2 * HELD)
    a, b = s.ctx.workspace(), s.ctx.workspace()
    for ws in (a, b, a, b, b, a):
        assert _same(s.shadowed(ws), ref)
        assert s.ctx.memory()[0] == asset + a.memory()[0] + b.memory()[0] <= asset + 2 * HELD
    a.close()
    b.close()
    s.ctx.close()


def test_an_asset_beside_a_shadowed_frame(hip, alone):
    ref, asset, most = alone
    s = Scene(hip, 2 * asset + most - 1)
    ws = s.ctx.workspace()
    assert _same(s.shadowed(ws), ref)
    assert s.ctx.memory()[0] == asset + most
    other = s.ctx.upload_asset(s.asset)      # (does not fit beside the layer sums)
    assert other != s.aid
    assert _same(s.shadowed(ws), ref)
    with pytest.raises(hip.HairError) as e:  # (until the workspace has no more to give)
        while True:
            s.ctx.upload_asset(s.asset)
    assert e.value.code == hip.HAIR_ENOMEM
    for _ in range(2):                       # what its own frames need it has kept
        assert _same(s.shadowed(ws), ref)
    ws.close()
    s.ctx.close()


def test_threads_on_their_own_workspaces(hip, alone):
    """Frames of two threads beside a third workspace, in a budget for three: each equals the frame
    alone, and none is refused."""
    ref, asset, most = alone
    s = Scene(hip, asset + 3 * HELD)
    idle = s.ctx.workspace()
    assert _same(s.shadowed(idle), ref)
    bad = []

    def frames():
        ws = s.ctx.workspace()
        try:
            for _ in range(8):
                if not _same(s.shadowed(ws), ref):
                    bad.append("another image")
        except Exception as e:               # noqa: BLE001 (reported by the test's own thread)
            bad.append(repr(e))
        finally:
            ws.close()

    print("case: two threads and an idle workspace in a budget for three", flush=True)
    threads = [threading.Thread(target=frames) for _ in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad
    assert _same(s.shadowed(idle), ref)
    idle.close()
    s.ctx.close()
