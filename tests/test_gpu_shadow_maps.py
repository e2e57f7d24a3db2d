"""Shadow maps at the ends of their ranges: one and seven layers, the smallest map (long lists in
one tile), maps of several tiles per side, and a layer depth whose reciprocal is not used, for
strands and thick hairs, against the oracle."""
import numpy as np
import pytest
import torch

import hairsynth as hs
from oracle import render as R
from test_gpu_shadow import _check, _dom_parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(hip):
    c = hip.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("R_, K, delta", [(16, 1, 0.02), (16, 7, 0.02), (17, 3, 0.02), (200, 7, 0.002), (300, 4, 1e31)])
def test_strand_maps(hip, ctx, R_, K, delta):
    print(f"case: strands, map {R_}, {K} layers of {delta}", flush=True)
    asset, cam, _ = hs.config(1)
    lights = hs.default_lights(asset, with_point=True)
    aid = ctx.upload_asset(asset)
    ws = ctx.workspace()
    img, st, _ = ctx.render_shadowed(aid, 0, cam, lights, (R_, K, delta), ws=ws)
    torch.cuda.synchronize()
    geom = R.strand_level(asset)
    _dom_parity(ctx, ws, geom, lights[0], 0, R_, K, np.float32(delta), "strands")
    ref, ras = R.render(geom, cam, lights, R.material(asset.material), shadow=(R_, K, np.float32(delta)))
    assert st["fragments"] == len(ras.seg)
    _check(img.cpu().numpy(), ref, "shadowed strands")
    first = img.clone()
    img, _, _ = ctx.render_shadowed(aid, 0, cam, lights, (R_, K, delta), ws=ws)   # (a warm frame)
    assert torch.equal(first.view(torch.int32), img.view(torch.int32))
    ws.close()
    ctx.release(aid)


@pytest.mark.parametrize("R_, K", [(16, 7), (130, 4)])
def test_thick_maps(hip, ctx, R_, K):
    asset, cam, _ = hs.config(1)
    lights = hs.default_lights(asset, with_point=True)
    n = 300
    S = asset.n_segments // asset.n_strands
    cen = np.asarray(asset.xyz).T.reshape(asset.n_strands, S + 1, 3)[:n].astype(np.float32)
    rng = np.random.default_rng(7)
    u = cen[:, 1:] - cen[:, :-1]
    a = np.cross(u, rng.normal(size=u.shape))
    a /= np.linalg.norm(a, axis=-1, keepdims=True)
    ext = float(np.linalg.norm(cen.reshape(-1, 3).max(0) - cen.reshape(-1, 3).min(0)))
    ax = (ext * (0.002 + 0.01 * rng.random((n, S)))).astype(np.float32)
    lod = {"centers": cen.copy(), "ahat": a.astype(np.float32),
           "axes": np.stack([ax, 0.6 * ax], -1), "n_total": rng.integers(1, 60, n).astype(np.int32),
           "sigma_a": np.ascontiguousarray(np.asarray(asset.sigma_a)[:, :n]), "r": np.full(n, 0.0004 * ext, np.float32)}
    aid = ctx.upload_asset(asset)
    ctx.set_lod(aid, 1, lod)
    ws = ctx.workspace()
    delta = np.float32(0.02 * ext)
    print(f"case: thick hairs, map {R_}, {K} layers", flush=True)
    img, st, _ = ctx.render_shadowed(aid, 1, cam, lights, (R_, K, float(delta)), ws=ws)
    torch.cuda.synchronize()
    geom = R.cluster_level(lod)
    _dom_parity(ctx, ws, geom, lights[0], 0, R_, K, delta, "thick hairs")
    ref, ras = R.render(geom, cam, lights, R.material(asset.material), shadow=(R_, K, delta))
    assert st["fragments"] == len(ras.seg)
    _check(img.cpu().numpy(), ref, "shadowed thick hairs")
    ws.close()
    ctx.release(aid)
