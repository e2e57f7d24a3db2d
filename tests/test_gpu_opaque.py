"""Frames whose thick hairs hide what lies behind them: the fragments behind an opaque one (alpha
exactly 1) are counted but neither stored nor shaded.  Half-widths on both sides of the narrowest
opaque hair (a pixel centre within hw - 1/2 of the centre line), hairs that share the opaque
one's depth key, stacks deeper than a batch, and the gradients, against the oracle."""
import numpy as np
import pytest
import torch

import hairsynth as hs
from oracle import grad as OG
from oracle import render as R

pytestmark = pytest.mark.gpu

W, H, FY = 37, 40, float(np.float32(74.6))


@pytest.fixture(scope="module")
def ctx(hip):
    c = hip.Context(0)
    yield c
    c.close()


def _stack(hw_px, depths, n_hairs=6):
    """One horizontal one-segment thick hair per depth across pixel row 20, each with a circular
    cross-section of half-width hw_px pixels at its own depth."""
    d = np.asarray(depths, dtype=np.float64)
    K = len(d)
    xyz = np.empty((3, 2 * K), dtype=np.float32)
    xyz[0, 0::2], xyz[0, 1::2] = -0.2 * d, 0.2 * d
    xyz[1, 0::2] = xyz[1, 1::2] = -0.5 * d / FY
    xyz[2, 0::2] = xyz[2, 1::2] = -d
    rng = np.random.default_rng(5)
    sig = (np.array([0.3, 0.6, 1.2])[:, None] * np.exp(0.2 * rng.normal(size=(1, K)))).astype(np.float32)
    asset = hs.Asset(K, 1, xyz, np.full(K, 8e-6, dtype=np.float32), np.ascontiguousarray(sig))
    axes = (np.asarray(hw_px) * d / FY).astype(np.float32)
    lod = {"centers": xyz.T.reshape(K, 2, 3).copy(), "ahat": np.tile(np.array([0.0, 1.0, 0.0], np.float32), (K, 1, 1)),
           "axes": np.stack([axes, axes], -1)[:, None, :].copy(), "n_total": np.full(K, n_hairs, np.int32),
           "sigma_a": sig.copy(), "r": np.full(K, 4e-6, np.float32)}
    cam = hs.Camera(np.zeros(3, np.float32), np.eye(3, dtype=np.float32), FY, FY, W / 2.0, H / 2.0, W, H, 0.01)
    return asset, lod, cam


def _check(ctx, asset, lod, cam, what):
    lights = hs.default_lights(asset, with_point=True)
    aid = ctx.upload_asset(asset)
    ctx.set_lod(aid, 1, lod)
    ws = ctx.workspace()
    img, st, _ = ctx.render(aid, 1, cam, lights, ws=ws)
    torch.cuda.synchronize()
    geom = R.cluster_level(lod)
    mat = tuple(float(v) for v in asset.material.as_array())
    ref, ras = R.render(geom, cam, lights, mat)
    depth = np.bincount(ras.pix)
    print(f"case: {what}: {len(ras.seg)} fragments, deepest pixel {depth.max()}", flush=True)
    assert st["fragments"] == len(ras.seg)
    assert st["deep_pixels"] == int((depth > 1536).sum()) and st["overflow_pixels"] == 0
    err = np.abs(img.cpu().numpy().astype(np.float64) - ref) - (1e-4 * np.abs(ref) + 1e-7)
    assert int((err > 0).sum()) == 0, float(err.max())
    return aid, ws, lights, geom, mat, ras


@pytest.mark.parametrize("hw_px", [0.02, 0.4, 0.5, 0.515625, 0.52, 0.75, 1.0, 2.3, 30.0])
def test_hidden_fragments_change_nothing(hip, ctx, hw_px):
    depths = np.concatenate([np.linspace(1.0, 2.0, 60), np.full(20, 1.3)])
    rng = np.random.default_rng(int(hw_px * 100))
    asset, lod, cam = _stack(hw_px * (0.9 + 0.2 * rng.random(len(depths))), rng.permutation(depths))
    aid, ws, *_ = _check(ctx, asset, lod, cam, f"half-width {hw_px} px")
    ws.close()
    ctx.release(aid)


def test_opaque_hair_inside_a_deep_stack(hip, ctx):
    """2,000 narrow hairs, one opaque hair in their middle, 2,000 more behind it: the pixels it
    covers store the front half, deeper than a batch."""
    depths = np.concatenate([np.linspace(1.0, 1.4, 2000), [1.5], np.linspace(1.6, 2.0, 2000)])
    hw = np.full(len(depths), 1e-3)
    hw[2000] = 1.5
    asset, lod, cam = _stack(hw, depths)
    aid, ws, *_ = _check(ctx, asset, lod, cam, "deep stack with an opaque hair")
    ws.close()
    ctx.release(aid)


@pytest.mark.parametrize("hw_px", [0.6, 2.3])
def test_gradients_behind_opaque_hairs(hip, ctx, hw_px):
    rng = np.random.default_rng(3)
    asset, lod, cam = _stack(hw_px * (0.8 + 0.4 * rng.random(40)), rng.permutation(np.linspace(1.0, 2.0, 40)))
    aid, ws, lights, geom, mat, ras = _check(ctx, asset, lod, cam, f"gradients at half-width {hw_px} px")
    K = asset.n_strands
    d = rng.normal(size=(H, W, 4))
    ref = OG.cluster_vjp(geom, cam, lights, mat, d, K, 1, ras=ras)[:3]
    out = [torch.empty(s, dtype=torch.float32, device="cuda:0") for s in ((K, 1, 2), (K,), (3, K))]
    ctx.render_backward(aid, 1, cam, lights, torch.tensor(d, dtype=torch.float32, device="cuda:0"), *out, ws=ws)
    torch.cuda.synchronize()
    for g, r in zip(out, ref):
        r = r.reshape(g.shape)
        assert np.allclose(g.cpu().numpy(), r, rtol=1e-3, atol=1e-5 * max(1.0, float(np.abs(r).max())))
    ws.close()
    ctx.release(aid)
