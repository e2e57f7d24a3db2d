"""Scattering over the materials' range: refractive indices on both sides of the one from which a
single arcsine polynomial serves the refracted offsets, and azimuthal widths from narrow lobes to
ones that fill the circle, for strands and thick hairs, against the oracle."""
import dataclasses

import numpy as np
import pytest
import torch

import hairsynth as hs
from oracle import render as R

pytestmark = pytest.mark.gpu

FY = float(np.float32(90.0))


@pytest.fixture(scope="module")
def ctx(hip):
    c = hip.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("eta", [1.2, 1.4705, 1.4707, 1.55, 2.5])
@pytest.mark.parametrize("beta_n", [0.1, 0.3, 3.0])
def test_materials(hip, ctx, eta, beta_n):
    W, H, K = 49, 37, 120
    rng = np.random.default_rng(int(1e4 * eta) + int(10 * beta_n))
    d = 1.0 + 0.5 * rng.random(K)
    xyz = np.empty((3, 2 * K), dtype=np.float32)
    mid = np.stack([(rng.random(K) - 0.5) * W, (rng.random(K) - 0.5) * H], -1) * d[:, None] / FY
    ang = 2.0 * np.pi * rng.random(K)
    step = 0.1 * np.stack([np.cos(ang), np.sin(ang), rng.random(K) - 0.5], -1)
    for e, s in ((0, -1.0), (1, 1.0)):
        xyz[0, e::2], xyz[1, e::2] = mid[:, 0] + s * step[:, 0], mid[:, 1] + s * step[:, 1]
        xyz[2, e::2] = -d + s * step[:, 2]
    sig = np.repeat(np.array([0.3, 0.6, 1.2], dtype=np.float32)[:, None], K, axis=1)
    asset = hs.Asset(K, 1, xyz, np.full(K, 4e-3, dtype=np.float32), np.ascontiguousarray(sig))
    asset = dataclasses.replace(asset, material=hs.Material(eta=eta, beta_n=beta_n))
    u = (xyz[:, 1::2] - xyz[:, 0::2]).T.astype(np.float64)
    a = np.cross(u, rng.normal(size=(K, 3)))
    a /= np.linalg.norm(a, axis=1, keepdims=True)
    axes = np.stack([8e-3 * (1.0 + rng.random(K)), 8e-3 * np.ones(K)], -1).astype(np.float32)
    lod = {"centers": xyz.T.reshape(K, 2, 3).copy(), "ahat": a.astype(np.float32), "axes": axes[:, None, :].copy(),
           "n_total": rng.integers(1, 40, K).astype(np.int32), "sigma_a": sig.copy(), "r": np.full(K, 1e-3, np.float32)}
    cam = hs.Camera(np.zeros(3, np.float32), np.eye(3, dtype=np.float32), FY, FY, W / 2.0, H / 2.0, W, H, 0.01)
    lights = hs.default_lights(asset, with_point=True)
    aid = ctx.upload_asset(asset)
    ctx.set_lod(aid, 1, lod)
    mat = tuple(float(v) for v in asset.material.as_array())
    ws = ctx.workspace()
    for level, geom in ((0, R.strand_level(asset)), (1, R.cluster_level(lod))):
        img, st, _ = ctx.render(aid, level, cam, lights, ws=ws)
        torch.cuda.synchronize()
        ref, ras = R.render(geom, cam, lights, mat)
        err = np.abs(img.cpu().numpy().astype(np.float64) - ref) - (1e-4 * np.abs(ref) + 1e-7)
        print(f"case: eta {eta}, beta_n {beta_n}, level {level}: {len(ras.seg)} fragments", flush=True)
        assert st["fragments"] == len(ras.seg) > 0
        assert int((err > 0).sum()) == 0, float(err.max())
    ws.close()
    ctx.release(aid)
