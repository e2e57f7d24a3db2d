"""Mixed frames with the opaque pass never, always and where it pays: the frames against the oracle by
the tests of mixed frames (small frames have no pass of their own accord), with fragments without
coverage left out too, and the device's choice against the areas that it is made from."""
import types

import numpy as np
import pytest
import torch

import hairsynth as hs
from paper_2405_10565_amd import binding
from test_gpu_mixed import (scene, test_far_view_lod_frame_matches_oracle,                    # noqa: F401
                            test_mixed_frame_matches_oracle_and_updates_levels,
                            test_mixed_frame_with_few_thick_cells_matches_oracle,
                            test_uniform_mixed_equals_level_render)
from test_gpu_rttd import test_rttd_mixed_frame                                              # noqa: F401
from test_gpu_shadow import test_shadowed_mixed_frame                                        # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[(None, 0), (None, 1), (0, 1)],
                ids=["no opaque pass", "opaque pass", "opaque pass and trimming"])
def hip(request):
    trim, mode = request.param

    class Context(binding.Context):
        def __init__(self, device=0, budget_bytes=0):
            super().__init__(device, budget_bytes)
            self._passes(None)

        def _passes(self, ws):
            self.debug_opaque(mode, ws)
            if trim is not None:
                self.debug_trim_rows(trim, ws)

        def workspace(self, max_bytes=0):
            ws = super().workspace(max_bytes)
            self._passes(ws)
            return ws

    return types.SimpleNamespace(**{**vars(binding), "Context": Context})


@pytest.fixture(scope="module")
def ctx(hip):
    c = hip.Context(0)
    yield c
    c.close()


def _groom(n, segs, clumps):
    return hs.make_asset(n, segs, 90.0, seed=1002, sigma_spread=True, clumps=clumps, flow=0.99)


def _pays(ctx, ws, st, W, H):
    """The device's areas and choice from the frame's own records: hairs' opaque cores and footprints on
    the tiles that hold any segment."""
    ri, rf = ctx.debug_segments(ws, st["segments"])
    T = -(-W // 16) * -(-H // 16)
    ts, segs = ctx.debug_bins(ws, T, int(st["pairs"]))
    tiles = int((np.diff(ts.astype(np.int64)) > 0).sum())
    per_seg = np.bincount(segs, minlength=len(ri))
    on = ((ri[:, 5] & 1) != 0) & (per_seg > 0)
    length = np.hypot(*(ri[on, 2:4] - ri[on, 0:2]).T.astype(np.float64)) / 16
    hw, cap = rf[on, 2].astype(np.float64), 256.0 * per_seg[on]
    core = np.minimum(2 * np.maximum(hw - 0.5 - 2.0**-6, 0) * length, cap).sum()
    whole = np.minimum((2 * hw + 1) * length, cap).sum()
    m = core / (256 * tiles)
    return m, (1 - (1 - np.exp(-m)) / m) * whole if m > 0 else 0.0


@pytest.mark.parametrize("eps, size, expect", [(1.5, (1280, 720), False), (9.0, (1280, 720), True),
                                               (9.0, (4112, 4112), True), (2.0, (4112, 4112), False)])
def test_the_device_chooses(eps, size, expect):
    """(4112 x 4112: the tiles are counted outside the single-block scans)"""
    W, H = size
    ctx = binding.Context(0)
    asset = _groom(20000, 24, 1250)
    aid = ctx.upload_asset(asset)
    ctx.build_lod(aid, hs.kmeans_hierarchy(asset, [1250, 156], seed=3, iters=5, features="path"))
    lights = hs.default_lights(asset, with_point=True)
    cam = hs.camera_occupancy(asset, W, H, 0.5 if W < 4000 else 0.05)
    lev = torch.empty((ctx.lod_groups(aid), asset.segs), dtype=torch.int32, device="cuda:0")
    ctx.lod_init(aid, cam, eps, lev)
    img, stored = {}, {}
    for mode in (0, 1, -1):
        ws = ctx.workspace()
        ctx.debug_opaque(mode, ws)
        for frame in range(3):                               # (a first and warm frames)
            out, st, _ = ctx.render_mixed(aid, cam, lights, lev, ws=ws)
            torch.cuda.synchronize()
            if frame:
                assert torch.equal(out.view(torch.int32), img[mode].view(torch.int32))
            img[mode] = out
        stored[mode] = ctx.debug_stored(ws)
        if mode == -1:
            m, hidden = _pays(ctx, ws, st, W, H)
        ws.close()
    print(f"case: thick hairs up to {eps} px at {W} x {H}: {st['fragments']} fragments, stored {stored}, "
          f"cores cover the tiles {m:.3f} times, {hidden:.0f} fragments hidden by estimate", flush=True)
    assert (m >= 0.5 and hidden >= 180000) == expect
    assert stored[-1] == stored[1 if expect else 0] and stored[1] < stored[0]
    for mode in (1, -1):
        a, b = img[mode].cpu().numpy().astype(np.float64), img[0].cpu().numpy().astype(np.float64)
        assert np.all(np.abs(a - b) <= 1e-4 * np.abs(b) + 1e-6)
    ctx.close()
