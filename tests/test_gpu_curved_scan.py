"""Rows of curved levels whose segment counts lie on both sides of what one block scans in a launch,
and on the edges of the chunks beyond: every row against the oracle's tessellation."""
import numpy as np
import pytest

import hairsynth as hs
from oracle import curve as CV
from oracle import lod as OL
from oracle import render as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("clusters, segs", [(255, 64), (256, 64), (257, 64), (321, 64), (819, 25)])
def test_rows(hip, clusters, segs):
    ctx = hip.Context(0)
    n = 2 * clusters
    asset = hs.make_asset(n, segs, 60.0, seed=41)
    cam = hs.camera_for(asset, 200, 160)
    lod = OL.build_level(asset, (np.arange(n) % clusters).astype(np.int32))
    aid = ctx.upload_asset(asset)
    ctx.set_lod(aid, 1, lod)
    ws = ctx.workspace()
    _, st, _ = ctx.render_curved(aid, 1, cam, hs.default_lights(asset, with_point=False), 1, 4, ws=ws)
    geom = CV.curved_geometry(lod, cam, 1, 4)
    rows = geom.pA.shape[1]
    print(f"case: {clusters * segs} segments, {rows} rows", flush=True)
    assert st["segments"] == rows > clusters * segs
    c, XA, YA, XB, YB, izA, izB, hw, hw_fx, vis = R.segment_records(geom, cam)
    ri, _ = ctx.debug_segments(ws, rows)
    assert np.array_equal((ri[:, 5] & 1).astype(bool), vis)
    for col, ref in enumerate((XA, YA, XB, YB)):
        assert np.array_equal(ri[vis, col], ref[vis]), col
    ctx.close()
