"""The work that programs built on this renderer have it do, as cases that can be timed.

A case is a dict of plain values; listed() names the ones every measurement takes, draw() makes
more over the same ranges.  prepare() builds what such a program holds before its frame loop (a
context with the groom resident, its LoD levels, a workspace, the output image, camera, lights),
run() is one pass through the public entry points, work() the bytes and operations of a pass
that no implementation can do without, and exact() the pass's results in float64, from plain
torch and the renderer's definitions alone.

Sizes are those of this repository's workloads (hairsynth.CONFIGS, bench.py, experiments.py):
grooms of 1k to 300k strands with 16 to 64 segments, images of 256 x 256 to 3840 x 2160, 1 to 3
lights, views from the whole groom in a corner of the image to one that fills it.  The grooms
are the same random walks (or locks of 16 strands following a smooth flow), drawn on the GPU.

Kinds of pass:
  strands          hair_render at the strand level; material "rttrt" or "rttd"
  shadowed         hair_render_shadowed at the strand level (deep opacity map per directional light)
  thick            hair_render at one thick-hair level
  curved           hair_render_curved at one thick-hair level
  mixed            hair_lod_init and hair_render_mixed, what a served request does
  mixed_shadowed   the same with hair_render_mixed_shadowed
  fit              one view of LoD fitting: the differentiable render and its gradients
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2405_10565_amd import binding as B
from paper_2405_10565_amd.autograd import render_lod

DEV = "cuda" if torch.cuda.is_available() else "cpu"
F64 = torch.float64
F32 = torch.float32
PI = math.pi
TAN_HALF_FOV = math.tan(math.radians(15.0))
EPS_W = 2.0          # pixels: a thick hair stands in for its strands while no wider than this


# ---------------------------------------------------------------------------------------
# The cases.
def _case(kind, strands, segs, width, height, occupancy, lights=2, **more):
    c = dict(kind=kind, strands=strands, segs=segs, width=width, height=height, occupancy=occupancy, lights=lights,
             material="rttrt", locks=False, clusters=0, shadow_res=0, shadow_layers=0, max_px=0)
    c.update(more)
    return c


def listed():
    return [
        # a preview or thumbnail: the smallest call, latency and launches
        dict(name="strands_1k_256", **_case("strands", 1_000, 16, 256, 256, 0.6, 1)),
        # a served request for the small asset at 720p, middle view
        dict(name="strands_10k_720p", **_case("strands", 10_000, 16, 1280, 720, 0.1)),
        # the headline frame: a full groom at 1080p (the groom's sphere over 90% of the height)
        dict(name="strands_100k_1080p", **_case("strands", 100_000, 32, 1920, 1080, 0.36)),
        # the largest served request: the dense asset filling a 4K image
        dict(name="strands_300k_2160p", **_case("strands", 300_000, 48, 3840, 2160, 0.6)),
        # the second material on sizes that divide nothing, three lights
        dict(name="rttd_33k_odd", **_case("strands", 33_333, 23, 1277, 717, 0.3, 3, material="rttd")),
        # the headline frame with shadows
        dict(name="shadowed_100k_1080p", **_case("shadowed", 100_000, 32, 1920, 1080, 0.36, shadow_res=1024,
                                                 shadow_layers=4)),
        # a level of the LoD sweep: 150k strands as 1000 wide thick hairs
        dict(name="thick_1k_1080p", **_case("thick", 150_000, 64, 1920, 1080, 0.36, clusters=1_000)),
        # the same groom with spline centre lines in steps of at most 2 pixels
        dict(name="curved_1k_1080p", **_case("curved", 150_000, 64, 1920, 1080, 0.36, clusters=1_000, max_px=2)),
        # per-group LoD on a combed groom, middle view: strands and thick hairs in one frame
        dict(name="mixed_middle_1080p", **_case("mixed", 100_000, 32, 1920, 1080, 0.1, locks=True, clusters=6_250)),
        # the same groom far away, nearly all of it thick hairs
        dict(name="mixed_far_1080p", **_case("mixed", 100_000, 32, 1920, 1080, 0.003, locks=True, clusters=6_250)),
        # a served request with shadows on
        dict(name="mixed_shadowed_720p", **_case("mixed_shadowed", 40_000, 32, 1280, 720, 0.1, locks=True,
                                                 clusters=2_500, shadow_res=512, shadow_layers=4)),
        # LoD fitting, forward and backward: 50k strands as 500 thick hairs at 512 x 512
        dict(name="fit_500_512", **_case("fit", 50_000, 32, 512, 512, 0.6, 1, clusters=500)),
    ]


def _between(rng, lo, hi):
    """A whole number between lo and hi, even over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["strands", "strands", "strands", "shadowed", "thick", "curved", "mixed", "mixed",
                       "mixed_shadowed", "fit"])
    height = _between(rng, 240, 2160 if kind == "strands" else 1080)
    width = max(160, min(3840, int(height * rng.uniform(0.8, 1.8))))
    segs = rng.randint(12, 64)
    lights = rng.randint(1, 3)
    occupancy = round(math.exp(rng.uniform(math.log(0.02), math.log(0.6))), 4)
    if kind == "strands":
        n = _between(rng, 1_000, min(300_000, 14_000_000 // segs))
        return _case(kind, n, segs, width, height, occupancy, lights, material=rng.choice(["rttrt", "rttrt", "rttd"]))
    if kind == "shadowed":
        n = _between(rng, 1_000, 100_000)
        return _case(kind, n, segs, width, height, occupancy, lights, shadow_res=_between(rng, 200, 1200),
                     shadow_layers=rng.randint(1, 7))
    if kind in ("thick", "curved"):
        n = _between(rng, 10_000, 150_000)
        return _case(kind, n, segs, width, height, min(occupancy, 0.36), min(lights, 2),
                     clusters=_between(rng, 100, 1_000), max_px=rng.choice([1, 2, 4]) if kind == "curved" else 0)
    if kind == "fit":
        n = _between(rng, 5_000, 50_000)
        side = _between(rng, 128, 512)
        return _case(kind, n, rng.randint(12, 40), side, side, 0.6, min(lights, 2), clusters=_between(rng, 50, 500))
    n = 16 * _between(rng, 200, 6_000)
    more = dict(shadow_res=_between(rng, 200, 1024), shadow_layers=rng.randint(2, 6)) if kind == "mixed_shadowed" else {}
    return _case(kind, n, min(segs, 40), width, height, round(min(occupancy, 0.2), 4), lights, locks=True,
                 clusters=n // 16, **more)


# ---------------------------------------------------------------------------------------
# Scenes: the groom, its clusters, camera and lights, from the seed alone.
def _unit(v):
    return v / v.norm(dim=-1, keepdim=True)


def _cap(u, v):
    """Points of the unit half sphere about +y, even over its area."""
    c = 1.0 - u
    s = torch.sqrt((1.0 - c * c).clamp_min(0.0))
    return torch.stack([s * torch.cos(2.0 * PI * v), c, s * torch.sin(2.0 * PI * v)], -1)


def _groom(case, gen):
    """Strand vertices float32 [n, segs + 1, 3] and, of a combed groom, each strand's lock."""
    n, S = case["strands"], case["segs"]
    rand = lambda *s: torch.rand(*s, generator=gen, device=DEV, dtype=F64)
    randn = lambda *s: torch.randn(*s, generator=gen, device=DEV, dtype=F64)
    drift = torch.tensor([0.0, -0.2, 0.0], device=DEV, dtype=F64)
    lock = None
    if case["locks"]:
        K, modes = max(1, n // 16), 8
        guide = _cap(rand(K), rand(K))
        lock = torch.arange(n, device=DEV) * K // n
        wave = (0.1 * guide) @ _unit(randn(modes, 3)).T * (2.0 * PI / 0.15)
        amp, phase = randn(S, modes, 3) / math.sqrt(modes), 2.0 * PI * rand(S, modes)
        ref = torch.where(guide[:, 1:2].abs() < 0.9, drift.new_tensor([[0.0, 1.0, 0.0]]), drift.new_tensor([[1.0, 0.0, 0.0]]))
        t1 = _unit(torch.linalg.cross(guide, ref))
        t2 = torch.linalg.cross(guide, t1)
        rad, ang = 1e-3 * torch.sqrt(rand(n)), 2.0 * PI * rand(n)
        normal = _unit(0.1 * guide[lock] + (rad * torch.cos(ang))[:, None] * t1[lock]
                       + (rad * torch.sin(ang))[:, None] * t2[lock])
        dg = guide
    else:
        normal = _cap(rand(n), rand(n))
    x, d = 0.1 * normal, normal
    out = torch.empty(n, S + 1, 3, device=DEV, dtype=F32)
    out[:, 0] = x
    for k in range(S):
        if lock is not None:
            flow = (torch.cos(wave + phase[k])[:, :, None] * amp[k]).sum(1)
            dg = _unit(dg + 0.3 * (math.sqrt(1.0 - 0.99 ** 2) * randn(K, 3) + 0.99 * math.sqrt(2.0) * flow) + drift)
            d = _unit(dg[lock] + 0.02 * randn(n, 3))
        else:
            d = _unit(d + 0.3 * randn(n, 3) + drift)
        x = x + 0.01 * d
        out[:, k + 1] = x
    return out, lock


def _means(labels, K, values):
    """Mean of the rows of values by label (float64 sums in row order)."""
    lab = labels.cpu()
    s = torch.zeros(K, values.shape[1], dtype=F64).index_add_(0, lab, values.double().cpu())
    return s / torch.bincount(lab, minlength=K)[:, None]


def _clusters(feats, k, gen, rounds=3):
    """Dense k-means labels (k rows drawn as centres, then Lloyd rounds)."""
    k = min(k, feats.shape[0])
    pick = torch.randperm(feats.shape[0], generator=gen, device=DEV)[:k]
    centres, lab = feats[pick], None
    for r in range(rounds + 1):
        c2 = (centres * centres).sum(1)
        lab = torch.cat([(c2 - 2.0 * f @ centres.T).argmin(1) for f in feats.split(max(1, 40_000_000 // k))])
        lab = torch.unique(lab, return_inverse=True)[1]
        if r < rounds:
            centres = _means(lab, int(lab.max()) + 1, feats).to(DEV)
    return lab


def _scene(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    xyz, lock = _groom(case, gen)
    n, V = xyz.shape[:2]
    sig = (torch.tensor([[0.3, 0.6, 1.2]], device=DEV, dtype=F64)
           * torch.exp(0.2 * torch.randn(n, 1, generator=gen, device=DEV, dtype=F64))).float()
    assigns = []
    if case["clusters"]:
        pts = xyz[:, torch.linspace(0, V - 1, 4).round().long()].reshape(n, 12).double()
        if lock is None:
            assigns = [_clusters(torch.cat([xyz[:, 0] / 0.1, _unit((xyz[:, 1] - xyz[:, 0]).double())], 1).double(),
                                 case["clusters"], gen)]
        else:   # one thick hair per lock, then per 4 and per 16 locks, nested
            assigns = [lock]
            for k in (case["clusters"] // 4, case["clusters"] // 16):
                m = _means(assigns[-1], int(assigns[-1].max()) + 1, pts).to(DEV)
                assigns.append(_clusters(m, max(1, k), gen)[assigns[-1]])
    box = xyz.reshape(-1, 3)
    lo, hi = (v.double().cpu().numpy() for v in (box.min(0)[0], box.max(0)[0]))
    centre, radius = 0.5 * (lo + hi), 0.5 * float(np.linalg.norm(hi - lo))
    W, H = case["width"], case["height"]
    fill = math.sqrt(case["occupancy"] * W * H / PI) / (H / 2.0)
    az = 0.4
    back = np.array([math.sin(az), 0.0, math.cos(az)])
    right = np.cross([0.0, 1.0, 0.0], back)
    f = float(np.float32(H / 2.0 / TAN_HALF_FOV))
    cam = SimpleNamespace(pos=(centre + radius / (fill * TAN_HALF_FOV) * back).astype(np.float32),
                          rot=np.stack([right, np.cross(back, right), back]).astype(np.float32), fx=f, fy=f,
                          cx=W / 2.0, cy=H / 2.0, width=W, height=H, z_near=0.01)
    toward = np.array([0.5, 0.6, 0.6])
    lights = [SimpleNamespace(kind=0, vec=(toward / np.linalg.norm(toward)).astype(np.float32), rgb=np.ones(3, np.float32)),
              SimpleNamespace(kind=1, vec=(centre + [-0.3, 0.1, -0.4]).astype(np.float32), rgb=np.full(3, 0.25, np.float32)),
              SimpleNamespace(kind=1, vec=(centre + [0.4, 0.3, -0.2]).astype(np.float32),
                              rgb=np.array([0.1, 0.08, 0.06], np.float32))][: case["lights"]]
    if case["material"] == "rttd":
        mat = SimpleNamespace(eta=1.55, alpha=0.0, beta_m=0.3, beta_n=0.3, model=1, beta_r=0.1, beta_tt=0.2, gamma_tt=0.3,
                              a_r=(0.1, 0.1, 0.1), a_tt=(0.3, 0.2, 0.12), a_d=(0.3, 0.16, 0.09))
    else:
        mat = SimpleNamespace(eta=1.55, alpha=math.radians(-3.0), beta_m=0.3, beta_n=0.3, model=0)
    d_rgba = torch.randn(H, W, 4, generator=gen, device=DEV) if case["kind"] == "fit" else None
    return SimpleNamespace(xyz=xyz, width=torch.full((n,), 80e-6, device=DEV), sig=sig, assigns=assigns, cam=cam,
                           lights=lights, mat=mat, d_rgba=d_rgba,
                           shadow=(case["shadow_res"], case["shadow_layers"], 0.02) if case["shadow_res"] else None)


# ---------------------------------------------------------------------------------------
# One pass of a program.
def prepare(case, seed):
    s = _scene(case, seed)
    n, V = s.xyz.shape[:2]
    ctx = B.Context(0)
    aid = ctx.upload(n, V, s.xyz.reshape(n * V, 3).T.contiguous().cpu().numpy(), s.width.cpu().numpy(),
                     s.sig.T.contiguous().cpu().numpy(), s.mat)
    if s.assigns:
        ctx.build_lod(aid, [a.cpu().numpy() for a in s.assigns])
    state = SimpleNamespace(case=case, ctx=ctx, aid=aid, ws=ctx.workspace(), cam=s.cam, lights=s.lights,
                            shadow=s.shadow, d_rgba=s.d_rgba,
                            out=torch.empty(case["height"], case["width"], 4, device=DEV))
    if case["kind"].startswith("mixed"):
        state.levels = torch.zeros(ctx.lod_groups(aid), case["segs"], device=DEV, dtype=torch.int32)
    if case["kind"] == "fit":
        lod = ctx.get_lod(aid, 1)
        state.params = [torch.tensor(p, device=DEV, requires_grad=True) for p in (lod.axes, lod.r, lod.sigma_a)]
    return state


def run(s):
    kind = s.case["kind"]
    if kind == "fit":
        img = render_lod(*s.params, s.ctx, s.aid, 1, s.cam, s.lights, s.ws)
        grads = torch.autograd.grad(img, s.params, s.d_rgba)
        return {"rgba": img.detach(), "d_axes": grads[0], "d_r": grads[1], "d_sigma_a": grads[2]}
    where = dict(out=s.out, ws=s.ws)
    if kind.startswith("mixed"):
        s.ctx.lod_init(s.aid, s.cam, EPS_W, s.levels, ws=s.ws)
        if s.shadow:
            out, st, _ = s.ctx.render_mixed_shadowed(s.aid, s.cam, s.lights, s.levels, s.shadow, **where)
        else:
            out, st, _ = s.ctx.render_mixed(s.aid, s.cam, s.lights, s.levels, **where)
        return {"rgba": out, "fragments": st["fragments"], "levels": s.levels}
    if kind == "shadowed":
        out, st, _ = s.ctx.render_shadowed(s.aid, 0, s.cam, s.lights, s.shadow, **where)
    elif kind == "curved":
        out, st, _ = s.ctx.render_curved(s.aid, 1, s.cam, s.lights, max_px=s.case["max_px"], **where)
    else:
        out, st, _ = s.ctx.render(s.aid, 1 if kind == "thick" else 0, s.cam, s.lights, **where)
    return {"rgba": out, "fragments": st["fragments"]}


# ---------------------------------------------------------------------------------------
# What a pass cannot do without.  Bytes: the level's vertices and attributes read, the image
# written (the gradients too).  Operations: the fragments, from the screen lengths and widths of
# the segments, times the operations of one fragment's definition (transcendentals count 4):
# position, frame and blending, then each light.
def work(case):
    kind, S, W, H = case["kind"], case["segs"], case["width"], case["height"]
    px_per_m = math.sqrt(case["occupancy"] * W * H / PI) / (0.255 + 0.0077 * S)   # over the groom's radius
    step = 0.01 * 0.785 * px_per_m
    K = case["clusters"]
    rows = (K if kind in ("thick", "curved", "fit") else case["strands"]) * S
    strand_px = 1.125 * step
    if kind in ("thick", "curved", "fit"):   # clusters of K over the groom: half-widths grow as 1 / sqrt(K)
        frags = rows * step * px_per_m * 5.2 / math.sqrt(K)
        frags = min(frags, rows * W * H)
        base, light = 129 + 6 * 4 + 15, 1090 + 4 * 108
    else:
        frags = rows * strand_px
        base, light = 105 + 5 * 4 + 18, 190 + 22 * 4
        if kind == "strands" and case["material"] == "rttd":
            light = 110 + 12 * 4
    per = base + light * case["lights"]
    if case["shadow_res"]:   # one directional light: most of its fragments lie behind others
        per += 185 + 765 + 4 * 85
    if kind == "fit":
        per *= 4
    nbytes = 16.0 * W * H + rows * (12.0 if K == 0 else 44.0) + 16.0 * rows / S
    if kind == "fit":
        nbytes += 32.0 * W * H + 8.0 * rows
    return {"bytes": nbytes, "flops": frags * per}


# ---------------------------------------------------------------------------------------
# The results in float64.  What decides which fragments exist and their order (projection,
# snapping to 1/16 pixel, half-widths, depth keys, the shadow map's grid) is by definition
# float32 with one rounding per operation; everything after that is float64 here.
_DISTINCT = 1 << 32


def _dot(a, b):
    return (a[..., 0] * b[..., 0] + a[..., 1] * b[..., 1]) + a[..., 2] * b[..., 2]


def _cross(a, b):
    return torch.stack([a[..., 1] * b[..., 2] - a[..., 2] * b[..., 1], a[..., 2] * b[..., 0] - a[..., 0] * b[..., 2],
                        a[..., 0] * b[..., 1] - a[..., 1] * b[..., 0]], -1)


def _len(a):
    return torch.sqrt(_dot(a, a))


def _strand_rows(s):
    S = s.xyz.shape[1] - 1
    rep = lambda t: t.repeat_interleave(S, 0)
    return SimpleNamespace(pA=s.xyz[:, :-1].reshape(-1, 3), pB=s.xyz[:, 1:].reshape(-1, 3), sig=rep(s.sig),
                           width=rep(s.width), thick=None)


def _level_rows(s, assign):
    """One thick hair per cluster: centre line, cross-section ellipses, hair count, radius."""
    n, V = s.xyz.shape[:2]
    S, K = V - 1, int(assign.max()) + 1
    means = lambda v: _means(assign, K, v).to(DEV)
    ctr = means(s.xyz.reshape(n, -1)).float().reshape(K, V, 3)
    count = torch.bincount(assign, minlength=K)
    r = (means(s.width[:, None])[:, 0] * 0.5).float()
    c = ctr.double()
    u = _unit(c[:, 1:] - c[:, :-1])
    e1 = torch.zeros_like(u).scatter_(-1, u.abs().argmin(-1, keepdim=True), 1.0)
    e1 = _unit(e1 - _dot(e1, u)[..., None] * u)
    e2 = _cross(u, e1)
    mid = 0.5 * (s.xyz[:, 1:].double() + s.xyz[:, :-1].double())
    q = mid - (0.5 * (c[:, 1:] + c[:, :-1]))[assign]
    q1, q2 = _dot(q, e1[assign]), _dot(q, e2[assign])
    c11, c12, c22 = means(q1 * q1), means(q1 * q2), means(q2 * q2)
    hm, hd = 0.5 * (c11 + c22), 0.5 * (c11 - c22)
    rad = torch.sqrt(hd * hd + c12 * c12)
    l1, l2 = (hm + rad).clamp_min(0.0), (hm - rad).clamp_min(0.0)
    first = (l1 - c22) ** 2 + c12 ** 2 >= c12 ** 2 + (l1 - c11) ** 2
    v = torch.stack([torch.where(first, l1 - c22, c12), torch.where(first, c12, l1 - c11)], -1)
    v = torch.where(((l1 - l2) <= 1e-12 * (l1 + l2))[..., None], v.new_tensor([1.0, 0.0]), _unit(v))
    rep = lambda t: t.repeat_interleave(S, 0)
    rows = SimpleNamespace(pA=ctr[:, :-1].reshape(-1, 3), pB=ctr[:, 1:].reshape(-1, 3), sig=rep(means(s.sig).float()),
                           width=torch.zeros(K * S, device=DEV), thick=torch.ones(K * S, dtype=torch.bool, device=DEV),
                           ahat=(v[..., :1] * e1 + v[..., 1:] * e2).float().reshape(-1, 3),
                           a=(r.double()[:, None] + 2.0 * torch.sqrt(l1)).float().reshape(-1),
                           b=(r.double()[:, None] + 2.0 * torch.sqrt(l2)).float().reshape(-1),
                           n=rep(count.float()), r=rep(r), ctr=ctr)
    return rows


def _pick(rows, i, **more):
    return SimpleNamespace(**{**{k: v[i] for k, v in vars(rows).items() if k != "ctr" and v is not None}, **more})


def _curved_rows(rows, cam, max_px, max_sub=16):
    """Catmull-Rom centre lines in steps of at most max_px pixels."""
    K, V = rows.ctr.shape[:2]
    XA, YA, _, _, okA = _project(rows.pA, cam)
    XB, YB, _, _, okB = _project(rows.pB, cam)
    d2 = (XB - XA) ** 2 + (YB - YA) ** 2
    m = torch.ones_like(d2)
    for j in range(1, max_sub):
        m += ((m == j) & ((16 * j * max_px) ** 2 < d2)).long()
    m = torch.where(okA & okB, m, 1)
    par = torch.arange(K * (V - 1), device=DEV).repeat_interleave(m)
    j = torch.arange(par.numel(), device=DEV) - (torch.cumsum(m, 0) - m)[par]
    cl, k = par // (V - 1), par % (V - 1)

    def point(jj):
        u = jj.float() / m[par].float()
        u2 = u * u
        u3 = u2 * u
        w = [0.5 * ((2.0 * u2 - u3) - u), 0.5 * ((3.0 * u3 - 5.0 * u2) + 2.0), 0.5 * ((4.0 * u2 - 3.0 * u3) + u),
             0.5 * (u3 - u2)]
        c = [rows.ctr[cl, (k + o).clamp(0, V - 1)] for o in (-1, 0, 1, 2)]
        p = ((w[0][:, None] * c[0] + w[1][:, None] * c[1]) + w[2][:, None] * c[2]) + w[3][:, None] * c[3]
        return torch.where((jj == 0)[:, None], c[1], torch.where((jj == m[par])[:, None], c[2], p))

    return _pick(rows, par, pA=point(j), pB=point(j + 1))


def _project(p, cam):
    pos, R = [float(v) for v in cam.pos], [float(v) for v in np.asarray(cam.rot, np.float32).reshape(9)]
    fx, fy, cx, cy = (float(np.float32(v)) for v in (cam.fx, cam.fy, cam.cx, cam.cy))
    d = [p[:, i] - pos[i] for i in range(3)]
    vx, vy, vz = ((d[0] * R[3 * i] + d[1] * R[3 * i + 1]) + d[2] * R[3 * i + 2] for i in range(3))
    z = -vz
    X = 16.0 * (cx + fx * (vx / z))
    Y = 16.0 * (cy - fy * (vy / z))
    ok = ((z >= float(np.float32(cam.z_near))) & (X >= -16384) & (X <= 16 * cam.width + 16384)
          & (Y >= -16384) & (Y <= 16 * cam.height + 16384))
    snap = lambda v: torch.where(ok, v, 0.0).round().long()
    return snap(X), snap(Y), z, 1.0 / z, ok


def _support(rows, i, toward):
    """Half-width across the direction `toward` of the ellipses of rows i (float32, fixed order)."""
    t = rows.pB[i] - rows.pA[i]
    u = t / _len(t)[:, None]
    w = toward
    wp = w - _dot(w, u)[:, None] * u
    wl = _len(wp)
    yh = _cross(u, wp / wl[:, None])
    pa, pb = rows.a[i] * _dot(rows.ahat[i], yh), rows.b[i] * _dot(_cross(u, rows.ahat[i]), yh)
    return torch.where(wl > 1e-7, torch.sqrt(pa * pa + pb * pb), torch.maximum(rows.a[i], rows.b[i]))


def _visible(r, ok):
    c16 = torch.ceil(16.0 * r.hw)
    r.vis = ok & torch.isfinite(c16) & (c16 >= 0)
    r.fx = torch.where(r.vis, c16, 0.0).long()
    r.vis &= ((r.XB - r.XA).abs() <= 16384) & ((r.YB - r.YA).abs() <= 16384) & (r.fx <= 32768)
    return r


def _records(rows, cam):
    XA, YA, zA, iA, okA = _project(rows.pA, cam)
    XB, YB, zB, iB, okB = _project(rows.pB, cam)
    fy, zm = float(np.float32(cam.fy)), (zA + zB) * 0.5
    pos = torch.tensor(np.asarray(cam.pos, np.float32), device=DEV)
    hw = ((0.5 * rows.width) * fy) / zm
    if rows.thick is not None:
        i = rows.thick.nonzero()[:, 0]
        w = pos - (rows.pA[i] + rows.pB[i]) * 0.5
        hw[i] = (_support(rows, i, w / _len(w)[:, None]) * fy) / zm[i]
    r = _visible(SimpleNamespace(XA=XA, YA=YA, XB=XB, YB=YB, iA=iA, iB=iB, hw=hw), okA & okB)
    # the side on which the cross-section offset is positive (toward u x x^)
    A, Bp = rows.pA.double(), rows.pB.double()
    u, m = _unit(Bp - A), 0.5 * (A + Bp)
    w = _unit(pos.double() - m)
    yh = _cross(u, _unit(w - _dot(w, u)[:, None] * u))
    R = torch.tensor(np.asarray(cam.rot, np.float32), device=DEV).double()
    yv, mv = yh @ R.T, (m - pos.double()) @ R.T
    sx = yv[:, 0] - (mv[:, 0] / mv[:, 2]) * yv[:, 2]
    sy = -(yv[:, 1] - (mv[:, 1] / mv[:, 2]) * yv[:, 2])
    r.sign = torch.where(sx * (YB - YA) - sy * (XB - XA) >= 0.0, 1.0, -1.0).double()
    return r


def _fragments(r, W, H):
    """Every fragment (segment, pixel) with t_num, t_den and cross, by pixel, depth key, segment."""
    R = r.fx + 8
    lox, hix = torch.minimum(r.XA, r.XB) - R, torch.maximum(r.XA, r.XB) + R
    loy, hiy = torch.minimum(r.YA, r.YB) - R, torch.maximum(r.YA, r.YB) + R
    i0, j0 = ((lox - 8).div(16, rounding_mode="floor") + 1).clamp_min(0), ((loy - 8).div(16, rounding_mode="floor") + 1).clamp_min(0)
    i1 = (-(8 - hix).div(16, rounding_mode="floor") - 1).clamp_max(W - 1)
    j1 = (-(8 - hiy).div(16, rounding_mode="floor") - 1).clamp_max(H - 1)
    nx = (i1 - i0 + 1).clamp_min(0)
    cnt = torch.where(r.vis, nx * (j1 - j0 + 1).clamp_min(0), 0)
    end = torch.cumsum(cnt, 0)
    total, got, at = int(end[-1]) if end.numel() else 0, [], 0
    cuts = torch.searchsorted(end, torch.arange(1, total // 20_000_000 + 2, device=DEV) * 20_000_000).tolist()
    for to in sorted(set(min(c + 1, end.numel()) for c in cuts) | {end.numel()}):
        if to <= at:
            continue
        s = torch.arange(at, to, device=DEV).repeat_interleave(cnt[at:to])
        loc = torch.arange(s.numel(), device=DEV) - (end[s] - cnt[s] - (end[at] - cnt[at]))
        pi, pj = i0[s] + loc % nx[s].clamp_min(1), j0[s] + loc // nx[s].clamp_min(1)
        dx, dy = r.XB[s] - r.XA[s], r.YB[s] - r.YA[s]
        ex, ey = 16 * pi + 8 - r.XA[s], 16 * pj + 8 - r.YA[s]
        tn, td, cr = ex * dx + ey * dy, dx * dx + dy * dy, ex * dy - ey * dx
        ok = (td > 0) & (tn >= 0) & (tn < td) & (cr * cr < R[s] * R[s] * td)
        got.append([v[ok] for v in (s, pj * W + pi, tn, td, cr)])
        at = to
    s, pix, tn, td, cr = (torch.cat(v) for v in zip(*got)) if got else (torch.zeros(0, dtype=torch.long, device=DEV),) * 5
    t = tn.float() / td.float()
    iz = r.iA[s] + t * (r.iB[s] - r.iA[s])
    key = 0xFFFFFFFF - (iz.view(torch.int32).long() & 0xFFFFFFFF)
    order = torch.sort(pix * _DISTINCT + key, stable=True)[1]
    return SimpleNamespace(s=s[order], pix=pix[order], tn=tn[order], td=td[order], cr=cr[order], iz=iz[order])


def _gauss(beta, x):
    return torch.exp(-(x * x) / (2.0 * beta * beta)) / (math.sqrt(2.0 * PI) * beta)


def _wrap(x):
    return x - 2.0 * PI * torch.floor((x + PI) / (2.0 * PI))


def _fiber(xd, h, sig, eta):
    """Attenuations [..., lobe, rgb] of R, TT, TRT and the lobes' exit azimuths."""
    sx, cx = torch.sin(xd), torch.cos(xd)
    go, sgt = torch.asin(h), h * cx / torch.sqrt(eta * eta - sx * sx)
    gt, cgt = torch.asin(sgt), torch.sqrt(1.0 - sgt * sgt)
    ci = cx * torch.sqrt((1.0 - h) * (1.0 + h))
    ct = torch.sqrt(1.0 - (1.0 - ci * ci) / (eta * eta))
    rs, rp = (ci - eta * ct) / (ci + eta * ct), (eta * ci - ct) / (eta * ci + ct)
    F = (0.5 * (rs * rs + rp * rp))[..., None]
    T = torch.exp(-sig * (2.0 * cgt / torch.sqrt(1.0 - (sx / eta) ** 2))[..., None])
    A = torch.stack([F.expand_as(T), (1.0 - F) ** 2 * T, (1.0 - F) ** 2 * F * T * T], -2)
    return A, [2.0 * p * gt - 2.0 * go + p * PI for p in range(3)]


def _logistic(x, s):
    e = torch.exp(-x.abs() / s)
    return e / (s * (1.0 + e) ** 2) / torch.tanh(PI / (2.0 * s))


def _f_single(th, xd, phi, h, sig, m):
    A, mu = _fiber(xd, h, sig, m.eta)
    s = torch.tensor(math.sqrt(3.0) * m.beta_n / PI, dtype=F64, device=DEV)
    return sum(A[..., p, :] * (0.5 * _gauss(m.bp[p], th - m.ap[p]) * _logistic(_wrap(phi - mu[p]), s))[..., None]
               for p in range(3))


def _f_rttd(th, phi, m):
    mn = [0.5 * _gauss(m.beta_r, th) / (2.0 * PI), 0.5 * _gauss(m.beta_tt, th) * _gauss(m.gamma_tt, _wrap(phi - PI)),
          torch.full_like(th, 1.0 / (2.0 * PI * PI))]
    return sum(v[..., None] * th.new_tensor(a) for v, a in zip(mn, (m.a_r, m.a_tt, m.a_d)))


_GL = np.polynomial.legendre.leggauss(8)


def _f_ours(th, xd, phi, h, sig, m, n, rho, nF, nB):
    """The aggregated scattering of a thick hair of n hairs (nF toward, nB away from the light)."""
    s = torch.tensor(math.sqrt(3.0) * m.beta_n / PI, dtype=F64, device=DEV)
    lo, hi = 1.0 / (1.0 + torch.exp(PI / s)), 1.0 / (1.0 + torch.exp(-PI / s))

    def cdf(x):
        k = torch.floor((x + PI) / (2.0 * PI))
        return k + (1.0 / (1.0 + torch.exp(-(x - 2.0 * PI * k) / s)) - lo) / (hi - lo)

    node = th.new_tensor(_GL[0]).expand(*xd.shape, 8)
    A, mu = _fiber(xd[..., None].expand_as(node), node, sig[..., None, :], m.eta)
    back = torch.stack([cdf(0.5 * PI - v) - cdf(-0.5 * PI - v) for v in mu], -1)[..., None]
    wk = 0.5 * th.new_tensor(_GL[1])[:, None, None]
    front, behind = (wk * A * (1.0 - back)).sum(-3), (wk * A * back).sum(-3)
    aF, aB, b2 = front.sum(-2), behind.sum(-2), th.new_tensor([b * b for b in m.bp])
    vf = (front.mean(-1) * b2).sum(-1) / front.mean(-1).sum(-1)
    vb = (behind.mean(-1) * b2).sum(-1) / behind.mean(-1).sum(-1)
    A, mu = _fiber(xd, h, sig, m.eta)
    extra = (nF - 1.0) * vf
    sb = math.sqrt(3.0) * torch.sqrt(m.beta_n ** 2 + extra) / PI
    f = sum(A[..., p, :] * (0.5 * _gauss(torch.sqrt(m.bp[p] ** 2 + extra), th - m.ap[p])
                            * _logistic(_wrap(phi - mu[p]), sb))[..., None] for p in range(3))
    f = aF ** (nF - 1.0)[..., None] * f
    aF2 = aF * aF
    A1, A3 = aB * aF2 / (1.0 - aF2), aB ** 3 * aF2 / (1.0 - aF2) ** 3
    A1p = 0.6 * aB * aF * (1.0 - aF ** (2.0 * nB[..., None])) / (1.0 - aF2)
    m1, m3, m1p = A1.mean(-1), A3.mean(-1), A1p.mean(-1)
    var = (m1 * (vb + 2.0 * vf) + m3 * (3.0 * vb + 2.0 * vf) + m1p * (vb + (2.0 * nB - 1.0) * vf)) / (m1 + m3 + m1p)
    near = phi.abs() < 0.5 * PI
    many = near & (n >= 2)
    f = f + torch.where(many, 0.5 * _gauss(torch.sqrt(var), th) / PI, 0.0)[..., None] * (A1 + A3 + A1p)
    Ps = (1.0 - rho) * (1.0 - torch.cos(phi))
    Pn = (1.0 - 0.2 * (1.0 - rho) - Ps).clamp_min(0.0)
    return torch.where(many[..., None], Ps[..., None] * aF + Pn[..., None], 1.0) * f


def _shade(rows, r, fr, cam, lights, m, thick, ns, par=None):
    """Coverage alpha [F] and radiance L [F, 3] of fragments fr, all strands or all thick hairs;
    ns: per light the hairs in front (or None); par: a, b, r, sig, hw to differentiate by."""
    s = fr.s
    pos = torch.tensor(np.asarray(cam.pos, np.float32), device=DEV).double()
    A, Bp = rows.pA[s].double(), rows.pB[s].double()
    t = fr.tn.double() / fr.td.double()
    iA, iB = r.iA[s].double(), r.iB[s].double()
    x = A + (t * iB / (iA + t * (iB - iA)))[:, None] * (Bp - A)
    u, wo = _unit(Bp - A), _unit(pos - x)
    so = _dot(wo, u)
    xh = _unit(wo - so[:, None] * u)
    yh = _cross(u, xh)
    hw = r.hw[s].double() if par is None else par.hw[s]
    sig = rows.sig[s].double() if par is None else par.sig[s]
    dist = fr.cr.double().abs() / torch.sqrt(fr.td.double()) / 16.0
    alpha = ((dist + hw).clamp_max(0.5) - (dist - hw).clamp_min(-0.5)).clamp(0.0, 1.0)
    edge = 1.0 if par is None else 1.0 - 1e-14     # (h = 1 only where alpha = 0; its derivative is not finite)
    h = (torch.sign(fr.cr) * r.sign[s] * dist / (hw + 0.5)).clamp(-edge, edge)
    if thick:
        ah = rows.ahat[s].double()
        bh = _cross(u, ah)
        a, b, rad = (v[s].double() for v in ((rows.a, rows.b, rows.r) if par is None else (par.a, par.b, par.r)))
        n = rows.n[s].double()
        sup = torch.sqrt((a * _dot(ah, yh)) ** 2 + (b * _dot(bh, yh)) ** 2)
    L = torch.zeros(s.numel(), 3, dtype=F64, device=DEV)
    for li, light in enumerate(lights):
        vec = torch.tensor(light.vec, device=DEV).double()
        E = torch.tensor(light.rgb, device=DEV).double()
        if light.kind == 0:
            wi = vec.expand_as(x)
        else:
            d2 = _dot(vec - x, vec - x)
            wi, E = (vec - x) / torch.sqrt(d2)[:, None], E / d2[:, None]
        si = _dot(wi, u)
        phi = -torch.atan2(_dot(wi, yh), _dot(wi, xh))
        ti, to = torch.asin(si.clamp(-1.0, 1.0)), torch.asin(so.clamp(-1.0, 1.0))
        th, xd = 0.5 * (ti + to), 0.5 * (ti - to).abs()
        if not thick:
            f = _f_rttd(th, phi, m) if m.model == 1 else _f_single(th, xd, phi, h, sig, m)
            if ns is not None and ns[li] is not None:
                one = torch.ones_like(th)
                f = torch.where((ns[li] > 0)[:, None], _f_ours(th, xd, phi, h, sig, m, one, one, 1.0 + ns[li], one), f)
        else:
            D = wi - si[:, None] * u
            D = D / _len(D)[:, None]
            oa, ob = h * sup * _dot(yh, ah) / a, h * sup * _dot(yh, bh) / b
            xa, xb = _dot(xh, ah) / a, _dot(xh, bh) / b
            qa, qb, qc = xa * xa + xb * xb, oa * xa + ob * xb, oa * oa + ob * ob - 1.0
            disc = qb * qb - qa * qc
            tt = (qb - torch.where(disc > 0, torch.sqrt(disc.clamp_min(1e-30)), 0.0)) / qa
            da, db = _dot(D, ah) / a, _dot(D, bh) / b
            chord = -2.0 * ((oa - tt * xa) * da + (ob - tt * xb) * db) / (da * da + db * db)
            rho = (n * rad * rad / (a * b)).clamp(0.0, 1.0)
            per = rho * torch.sqrt(n / (PI * a * b))
            nF = torch.where((phi.abs() < 0.5 * PI) | (n < 2), 1.0, (per * chord).clamp_min(1.0))
            nB = (per * -chord).clamp_min(1.0)
            if ns is not None and ns[li] is not None:
                nF = nF + ns[li]
            f = _f_ours(th, xd, phi, h, sig, m, n, rho, nF, nB)
        L = L + E * f * torch.sqrt((1.0 - si) * (1.0 + si)).clamp_min(0.0)[:, None]
    return alpha, L


def _part(fr, i):
    return SimpleNamespace(**{k: v[i] for k, v in vars(fr).items()})


def _alpha_radiance(rows, r, fr, cam, lights, m, ns):
    alpha = torch.zeros(fr.s.numel(), dtype=F64, device=DEV)
    L = torch.zeros(fr.s.numel(), 3, dtype=F64, device=DEV)
    kinds = [(False, None)] if rows.thick is None else [(False, ~rows.thick[fr.s]), (True, rows.thick[fr.s])]
    for thick, mask in kinds:
        every = torch.arange(fr.s.numel(), device=DEV) if mask is None else mask.nonzero()[:, 0]
        for i in every.split(400_000 if thick or ns is not None else 3_000_000):
            sub = None if ns is None else [None if v is None else v[i] for v in ns]
            alpha[i], L[i] = _shade(rows, r, _part(fr, i), cam, lights, m, thick, sub)
    return alpha, L


def _ranks(fr):
    """Per pixel (deepest first) its id and first fragment; per rank the number of pixels that deep."""
    pix, cnt = torch.unique_consecutive(fr.pix, return_counts=True)
    start = torch.cumsum(cnt, 0) - cnt
    cnt, o = torch.sort(cnt, descending=True)
    deep = torch.bincount(cnt).flip(0).cumsum(0).flip(0)[1:].tolist() if cnt.numel() else []
    return pix[o], start[o], deep


def _composite(fr, alpha, L, W, H):
    pix, start, deep = _ranks(fr)
    C = torch.zeros(pix.numel(), 3, dtype=F64, device=DEV)
    T = torch.ones(pix.numel(), dtype=F64, device=DEV)
    for k, n in enumerate(deep):
        i = start[:n] + k
        C[:n] += (T[:n] * alpha[i])[:, None] * L[i]
        T[:n] *= 1.0 - alpha[i]
    rgba = torch.zeros(H * W, 4, dtype=F64, device=DEV)
    rgba[pix] = torch.cat([C, (1.0 - T)[:, None]], 1)
    return rgba.reshape(H, W, 4)


def _composite_adjoint(fr, alpha, L, d):
    """d sum(d * rgba) / d alpha and / d L, per fragment."""
    pix, start, deep = _ranks(fr)
    d = d.reshape(-1, 4).double()[pix]
    T = torch.ones(pix.numel(), dtype=F64, device=DEV)
    before = torch.zeros_like(alpha)
    for k, n in enumerate(deep):
        i = start[:n] + k
        before[i] = T[:n]
        T[:n] *= 1.0 - alpha[i]
    C, rest = torch.zeros(pix.numel(), 3, dtype=F64, device=DEV), torch.ones(pix.numel(), dtype=F64, device=DEV)
    d_alpha, d_L = torch.zeros_like(alpha), torch.zeros_like(L)
    for k in range(len(deep) - 1, -1, -1):
        n = deep[k]
        i = start[:n] + k
        a, t = alpha[i], before[i]
        d_alpha[i] = t * ((d[:n, :3] * (L[i] - C[:n])).sum(1) + d[:n, 3] * rest[:n])
        d_L[i] = d[:n, :3] * (t * a)[:, None]
        C[:n] = a[:, None] * L[i] + (1.0 - a)[:, None] * C[:n]
        rest[:n] *= 1.0 - a
    return d_alpha, d_L


def _shadow_counts(rows, r, fr, lights, shadow):
    """Per light the hairs in front of every fragment, from a deep opacity map of the rows."""
    R, K, delta = shadow
    thick = torch.zeros_like(rows.width, dtype=torch.bool) if rows.thick is None else rows.thick
    ti = thick.nonzero()[:, 0]
    t = fr.tn.float() / fr.td.float()
    tw = (t * r.iB[fr.s]) / (r.iA[fr.s] + t * (r.iB[fr.s] - r.iA[fr.s]))
    pA = rows.pA[fr.s]
    x = pA + tw[:, None] * (rows.pB[fr.s] - pA)
    f32 = lambda v: torch.tensor(np.asarray(v, np.float32), device=DEV)
    out = []
    for light in lights:
        if light.kind != 0:
            out.append(None)
            continue
        w = np.asarray(light.vec, np.float64)
        w = w / math.sqrt(float(w @ w))
        e1 = np.cross([0.0, 1.0, 0.0] if abs(w[1]) < 0.9 else [1.0, 0.0, 0.0], w)
        e1 = e1 / math.sqrt(float(e1 @ e1))
        e1, e2, d, om = f32(e1), f32(np.cross(w, e1)), f32(-w), f32(w)
        pad = 0.5 * rows.width
        if ti.numel():
            pad[ti] = torch.maximum(rows.a[ti], rows.b[ti])
        (uA, uB), (vA, vB), (zA, zB) = ([_dot(p, e) for p in (rows.pA, rows.pB)] for e in (e1, e2, d))
        low = lambda a, b: torch.minimum((a - pad).min(), (b - pad).min())
        high = lambda a, b: torch.maximum((a + pad).max(), (b + pad).max())
        u0, v0 = low(uA, uB), low(vA, vB)
        s = torch.maximum(high(uA, uB) - u0, high(vA, vB) - v0).clamp_min(1e-6) / float(R - 2)
        u0, v0, k16, zref = u0 - s, v0 - s, 16.0 / s, torch.maximum(zA.max(), zB.max()) + 1.0
        hw = (0.5 * rows.width) / s
        if ti.numel():
            hw[ti] = _support(rows, ti, om.expand(ti.numel(), 3)) / s
        snap = lambda v, o: ((v - o) * k16).round().long()
        lr = _visible(SimpleNamespace(XA=snap(uA, u0), YA=snap(vA, v0), XB=snap(uB, u0), YB=snap(vB, v0),
                                      iA=zref - zA, iB=zref - zB, hw=hw), torch.ones_like(thick))
        lf = _fragments(lr, R, R)
        first = torch.zeros(R * R, device=DEV).scatter_reduce_(0, lf.pix, lf.iz, "amax")
        layer = torch.floor((first[lf.pix] - lf.iz) / delta).long().clamp_max(K - 1)
        dist = lf.cr.double().abs() / torch.sqrt(lf.td.double()) / 16.0
        h2 = lr.hw[lf.s].double()
        c = ((dist + h2).clamp_max(0.5) - (dist - h2).clamp_min(-0.5)).clamp(0.0, 1.0)
        i = thick[lf.s].nonzero()[:, 0]
        if i.numel():
            q = lf.s[i]
            a, b, n, rad = (v[q].double() for v in (rows.a, rows.b, rows.n, rows.r))
            h = (dist[i] / h2[i]).clamp_max(1.0)
            c[i] *= (n * rad * rad / (a * b)).clamp(0.0, 1.0) * torch.sqrt(n / (PI * a * b)) \
                * (2.0 * a * b / (h2[i] * s.double())) * torch.sqrt(1.0 - h * h)
        C = torch.zeros(R * R * K, dtype=F64, device=DEV).index_add_(0, lf.pix * K + layer, c).reshape(-1, K).cumsum(1)
        C = torch.cat([torch.zeros_like(C[:, :1]), C], 1).reshape(-1)          # C_-1 = 0, C_0 .. C_K-1
        tx, ty = (_dot(x, e1) - u0) / s - 0.5, (_dot(x, e2) - v0) / s - 0.5
        izp = zref - _dot(x, d)
        bx, by = torch.floor(tx), torch.floor(ty)
        gx, gy = (tx - bx).double(), (ty - by).double()
        n = torch.zeros(x.shape[0], dtype=F64, device=DEV)
        for ox, oy, wt in ((0, 0, (1 - gx) * (1 - gy)), (1, 0, gx * (1 - gy)), (0, 1, (1 - gx) * gy), (1, 1, gx * gy)):
            qx, qy = bx.long() + ox, by.long() + oy
            q = torch.where((qx >= 0) & (qy >= 0) & (qx < R) & (qy < R), qy * R + qx, -1)
            z0 = torch.where(q >= 0, first[q], 0.0)
            xl = ((z0 - izp) / delta).double() - 1.0
            j = torch.floor(xl).clamp(0, K - 1).long()
            o = q.clamp_min(0) * (K + 1) + j
            val = torch.where(xl >= K, C[q.clamp_min(0) * (K + 1) + K], C[o] + (xl - j) * (C[o + 1] - C[o]))
            n += torch.where((z0 > 0) & (xl >= 0), wt * val, 0.0)
        out.append(n)
    return out


def _mixed_rows(s, cam):
    """The levels of every (group, segment) and the rows of the mixed frame, by group, segment, owner."""
    S = s.xyz.shape[1] - 1
    lv = [_strand_rows(s)] + [_level_rows(s, a) for a in s.assigns]
    G, top = int(s.assigns[-1].max()) + 1, s.assigns[-1]
    groups = [top] + [torch.zeros(int(a.max()) + 1, dtype=torch.long, device=DEV).scatter_(0, a, top) for a in s.assigns]
    level = torch.zeros(G, S, dtype=torch.long, device=DEV)
    for l in range(1, len(lv)):      # the coarsest level that is narrow enough wins
        r = _records(lv[l], cam)
        w = torch.where(r.vis, 2.0 * r.hw, 0.0).reshape(-1, S)
        wide = torch.zeros(G, S, device=DEV).scatter_reduce_(0, groups[l][:, None].expand_as(w), w, "amax")
        level = torch.where(wide <= EPS_W, l, level)
    parts, order = [], []
    for l, rows in enumerate(lv):
        N = rows.pA.shape[0]
        owner, k = torch.arange(N, device=DEV) // S, torch.arange(N, device=DEV) % S
        g = groups[l][owner]
        i = (level[g, k] == l).nonzero()[:, 0]
        if l == 0:
            one = torch.ones(i.numel(), device=DEV)
            part = _pick(rows, i, thick=one < 0, ahat=one[:, None].expand(-1, 3), a=one, b=one, n=one, r=one)
        else:
            part = _pick(rows, i)
        parts.append(part)
        order.append((g[i] * S + k[i]) * _DISTINCT + owner[i])
    o = torch.sort(torch.cat(order))[1]
    return level, SimpleNamespace(**{k: torch.cat([getattr(p, k) for p in parts])[o] for k in vars(parts[0])})


def _halfwidth(rows, cam, a, b):
    """The half-width of thick hairs in float64, differentiable by a and b."""
    pos = torch.tensor(np.asarray(cam.pos, np.float32), device=DEV).double()
    A, Bp = rows.pA.double(), rows.pB.double()
    u, w = _unit(Bp - A), _unit(pos - 0.5 * (A + Bp))
    yh, ah = _cross(u, _unit(w - _dot(w, u)[:, None] * u)), rows.ahat.double()
    zm = 0.5 * (_project(rows.pA, cam)[2].double() + _project(rows.pB, cam)[2].double())
    return torch.sqrt((a * _dot(ah, yh)) ** 2 + (b * _dot(_cross(u, ah), yh)) ** 2) * float(np.float32(cam.fy)) / zm


def _fit_gradients(s, rows, r, fr, m, alpha, L, S):
    K = rows.ctr.shape[0]
    d_alpha, d_L = _composite_adjoint(fr, alpha, L, s.d_rgba)
    leaf = lambda t: t.double().detach().requires_grad_(True)
    a, b, rad, sig = leaf(rows.a), leaf(rows.b), leaf(rows.r[::S]), leaf(rows.sig[::S])
    grads = [torch.zeros_like(t) for t in (a, b, rad, sig)]
    for i in torch.arange(fr.s.numel(), device=DEV).split(200_000):
        par = SimpleNamespace(a=a, b=b, r=rad.repeat_interleave(S), sig=sig.repeat_interleave(S, 0),
                              hw=_halfwidth(rows, s.cam, a, b))
        al, l = _shade(rows, r, _part(fr, i), s.cam, s.lights, m, True, None, par)
        for g, v in zip(grads, torch.autograd.grad((al * d_alpha[i]).sum() + (l * d_L[i]).sum(), (a, b, rad, sig))):
            g += v
    return torch.stack([grads[0].reshape(K, S), grads[1].reshape(K, S)], -1), grads[2], grads[3].T.contiguous()


def exact(case, seed):
    s = _scene(case, seed)
    kind, cam = case["kind"], s.cam
    m = SimpleNamespace(**{k: float(np.float32(v)) if isinstance(v, float) else v for k, v in vars(s.mat).items()})
    for k in ("a_r", "a_tt", "a_d"):
        if hasattr(m, k):
            setattr(m, k, [float(np.float32(v)) for v in getattr(m, k)])
    m.ap, m.bp = (m.alpha, -0.5 * m.alpha, -1.5 * m.alpha), (m.beta_m, 0.5 * m.beta_m, 2.0 * m.beta_m)
    if kind.startswith("mixed"):
        _, rows = _mixed_rows(s, cam)
    elif kind in ("strands", "shadowed"):
        rows = _strand_rows(s)
    else:
        rows = _level_rows(s, s.assigns[0])
    if kind == "curved":
        rows = _curved_rows(rows, cam, case["max_px"])
    r = _records(rows, cam)
    fr = _fragments(r, cam.width, cam.height)
    ns = _shadow_counts(rows, r, fr, s.lights, s.shadow) if s.shadow else None
    alpha, L = _alpha_radiance(rows, r, fr, cam, s.lights, m, ns)
    rgba = _composite(fr, alpha, L, cam.width, cam.height)
    if kind == "fit":
        d_axes, d_r, d_sig = _fit_gradients(s, rows, r, fr, m, alpha, L, case["segs"])
        return {"rgba": rgba, "d_axes": d_axes, "d_r": d_r, "d_sigma_a": d_sig}
    out = {"rgba": rgba, "fragments": None}
    if kind.startswith("mixed"):
        out["levels"] = None
    return out
