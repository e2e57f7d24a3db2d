"""The benchmark prices its shading kernels by the fragments that a frame stores and shades, not by
those that it counts (a frame leaves out fragments without coverage and hidden ones)."""
import types

import bench
import hairsynth as hs

COUNTED, STORED = 10_000, 700


class _Ctx:
    """Frames of COUNTED fragments, STORED of them shaded in one millisecond."""

    def _frame(self, *args, **kw):
        return None, {"fragments": COUNTED, "ms_total": 2.0, "ms_tile": 1.0}, 0

    render = render_shadowed = _frame

    def upload_asset(self, asset):
        return 0

    def build_lod(self, *args):
        pass

    def release(self, aid):
        pass

    def debug_stored(self, ws):
        return STORED


def _check(frame, kind, lights):
    ops, trans = bench.ops_per_fragment(kind, lights)
    r = frame["roofline"]
    assert r["fragments"] == STORED
    assert r["ops_per_launch"] == int(STORED * (ops + bench.TRANS_WEIGHT * trans))
    assert abs(r["frac"] - r["ops_per_launch"] / 1e-3 / bench.PEAK_LANE_OPS) < 1e-4


def test_shadowed_frame():
    asset = hs.make_asset(10, 2, 60.0, seed=1)
    lights = hs.default_lights(asset, with_point=True)
    frame = bench.shadowed_frame(_Ctx(), 0, None, lights, None, frames=2)
    _check(frame, "strand_shadowed_100k_1080p", lights)


def test_thick_frame(monkeypatch):
    asset = hs.make_asset(10, 2, 60.0, seed=1)
    lights = hs.default_lights(asset, with_point=True)
    monkeypatch.setattr(hs, "config", lambda i: (asset, types.SimpleNamespace(), lights))
    monkeypatch.setattr(hs, "kmeans_assign", lambda *args, **kw: None)
    frame = bench.thick_frame(_Ctx(), None, frames=2)
    assert frame["fragments"] == COUNTED
    _check(frame, "thick_1080p", lights)
