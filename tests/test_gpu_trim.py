"""Frames that leave out the fragments without coverage, as the largest do (2^21 rows), at small
sizes with the threshold at 0: strands, thick hairs with and without hidden fragments, curved,
mixed, split and shadowed frames and the gradients, against the oracle, by the tests that render
these frames untrimmed; and how many fragments are left out, against the oracle's coverage."""
import types

import numpy as np
import pytest
import torch

import hairsynth as hs
from oracle import lod as OL
from oracle import render as R
from paper_2405_10565_amd import binding
from test_gpu_backward import (test_backward_long_tile_lists_matches_oracle_gradient,        # noqa: F401
                               test_backward_matches_oracle_gradient,
                               test_backward_pixels_deeper_than_a_batch_match_oracle_gradient)
from test_gpu_curved import test_curved_rows_and_radiance                                     # noqa: F401
from test_gpu_mixed import (scene, test_mixed_frame_matches_oracle_and_updates_levels,        # noqa: F401
                            test_mixed_frame_with_few_thick_cells_matches_oracle,
                            test_uniform_mixed_equals_level_render)
from test_gpu_opaque import (test_gradients_behind_opaque_hairs, test_hidden_fragments_change_nothing,  # noqa: F401
                             test_opaque_hair_inside_a_deep_stack)
from test_gpu_rttd import test_rttd_mixed_frame, test_rttd_strand_level, test_rttd_thick_hair_level     # noqa: F401
from test_gpu_shadow import test_shadowed_mixed_frame, test_shadowed_strands, test_shadowed_thick_hairs  # noqa: F401
from test_gpu_split import curtain, test_long_strands_drawn_as_pieces, test_mixed_frame_drawn_as_pieces  # noqa: F401

pytestmark = pytest.mark.gpu


class TrimmingContext(binding.Context):
    def __init__(self, device=0, budget_bytes=0):
        super().__init__(device, budget_bytes)
        self.debug_trim_rows(0)

    def workspace(self, max_bytes=0):
        ws = super().workspace(max_bytes)
        self.debug_trim_rows(0, ws)
        return ws


@pytest.fixture(scope="module")
def hip():
    return types.SimpleNamespace(**{**vars(binding), "Context": TrimmingContext})


@pytest.fixture(scope="module")
def ctx(hip):
    c = hip.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("level", [0, 1])
@pytest.mark.parametrize("scale", [0.02, 1.0, 30.0])
def test_what_is_left_out(hip, ctx, level, scale):
    """Every fragment with coverage is stored (but for the hidden ones of a level of thick hairs), and
    few without: those within the safety of the strip's float estimate, one unit of the cross
    product, of which a pixel has 16 times the segment's length."""
    small = hs.make_asset(500, 6, 90.0, seed=5)
    asset = hs.Asset(small.n_strands, small.segs, small.xyz, small.width * np.float32(scale), small.sigma_a)
    lod = OL.build_level(asset, np.arange(500))
    cam, lights = hs.camera_for(asset, 200, 150), hs.default_lights(asset, with_point=False)
    geom = R.strand_level(asset) if level == 0 else R.cluster_level(lod)
    aid = ctx.upload_asset(asset)
    ctx.set_lod(aid, 1, lod)
    ws, plain = ctx.workspace(), ctx.workspace()
    ctx.debug_trim_rows(1 << 30, plain)
    img, st, _ = ctx.render(aid, level, cam, lights, ws=ws)
    ref, st2, _ = ctx.render(aid, level, cam, lights, ws=plain)
    torch.cuda.synchronize()
    ras = R.rasterize(geom, cam)
    hw = torch.as_tensor(np.asarray(ras.hw)[ras.seg].astype(np.float64))
    alpha = R.fragment_alpha_h(ras, hw)[0].numpy()
    covered, n = int((alpha > 0).sum()), len(ras.seg)
    stored, all_stored = ctx.debug_stored(ws), ctx.debug_stored(plain)
    print(f"case: level {level}, widths x {scale}: {n} fragments, {covered} with coverage, {stored} stored, "
          f"{all_stored} without trimming", flush=True)
    assert st["fragments"] == st2["fragments"] == n
    if level == 0:
        assert all_stored == n and covered <= stored < n
        assert stored - covered <= max(2, n // 200)
    else:
        assert stored <= all_stored <= n and stored < n
    # the same fragments in other runs of the blend: a pixel's transmittance is rounded once per
    # fragment and scan step, its colour (a sum of positive terms) three times as often
    steps = int(np.bincount(ras.pix).max()) + 8
    a, b = img.cpu().numpy().astype(np.float64), ref.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(a[..., 3] - b[..., 3]) <= 2 * steps * 2.0**-24)
    assert np.all(np.abs(a[..., :3] - b[..., :3]) <= 6 * steps * 2.0**-24 * b[..., :3])
    ws.close()
    plain.close()
    ctx.release(aid)
