"""A CPU model of the float estimates that bound the integer coverage (k_bin_count, k_scatter,
k_opaque, k_count, k_emit), at the largest radii, segments and images that the kernels admit
(half-widths up to 2048 px, segments of up to 1024 px per axis, images of 16384 px):

  * strip_vis and strip_opaque against the exact coverage (alpha = 0 outside the one, alpha = 1
    inside the other), in exact integers and by the shading pass's float formula;
  * the box of cov_setup, narrowed to a strip's own reach: no pixel centre inside the strip and
    the slab lies outside it, for all three strips;
  * the row intervals of FootprintRows against the test of every tile's four corner centres.

The hardware reciprocal and square root err by at most one ulp; the model takes them one ulp either
side of the rounded ones."""
import math
import random
from fractions import Fraction

import numpy as np
import pytest

F32 = np.float32
TILE = 16
MAX_HW_FX, MAX_AXIS = 32768, 16384


def _ulps(x, n):
    x = F32(x)
    for _ in range(abs(n)):
        x = np.nextafter(x, F32(np.inf if n > 0 else -np.inf), dtype=np.float32)
    return x


def _rcp(d, n):
    return _ulps(F32(1.0) / F32(d), n)


def _sqrt(x, n):
    return _ulps(np.sqrt(F32(x)), n)


def _smax(R, tden):
    return min(math.isqrt(R * R * tden - 1), 0x7FFFFFFF)


def _strip_vis(hw, tden, smax, n, margin=F32(1.0) + F32(2.0**-18)):
    s = (((hw + F32(0.5)) * F32(16.0)) * _sqrt(tden, n)) * margin + F32(1.0)
    return min(int(min(s, F32(2147483520.0))), smax)


def _strip_opaque(hw, tden, n, margin=F32(2.0**-6)):
    w = (hw - F32(0.5)) - margin
    return int(min((w * F32(16.0)) * _sqrt(tden, n), F32(1073741824.0))) if w > 0 else -1


def _segment(rng):
    """(dx, dy, hw, R): a visible segment, the extremes often."""
    top = rng.choice((16, 256, 2048, MAX_AXIS))
    while True:
        dx, dy = rng.randint(-top, top), rng.randint(-top, top)
        if rng.random() < 0.1:
            dx = rng.choice((0, 1, -1, MAX_AXIS, -MAX_AXIS))
        if dx or dy:
            break
    hw = F32(rng.choice((rng.uniform(0, 0.1), rng.uniform(0, 2), rng.uniform(0, 60), rng.uniform(0, 2048),
                         2048.0, 0.5 + 2.0**-6, 0.0)))
    if rng.random() < 0.2:
        hw = _ulps(F32(rng.randint(1, 16 * 64)) / F32(16.0), rng.choice((-1, 1)))
    return dx, dy, hw, math.ceil(16 * Fraction(float(hw))) + 8


def _thick_alpha(cr, tden, hw):
    """The shading pass's alpha of a thick hair (the strand's is the same formula in double)."""
    dd = abs(cr) / math.sqrt(tden) * 0.0625
    delta = F32(dd)
    dlo = F32(dd - float(delta))
    d_minus, d_plus = (delta - hw) + dlo, (hw + delta) + dlo
    return min(max(min(d_plus, F32(0.5)) - max(d_minus, F32(-0.5)), F32(0.0)), F32(1.0))


def _strips_fail(rng, n, vis=_strip_vis, opaque=_strip_opaque):
    bad = 0
    for _ in range(n):
        dx, dy, hw, R = _segment(rng)
        tden = dx * dx + dy * dy
        smax = _smax(R, tden)
        h, e = Fraction(float(hw)), rng.choice((-1, 0, 1))
        sv, so = vis(hw, tden, smax, e), opaque(hw, tden, e)
        # |cross| / (16 sqrt(t_den)) < hw + 1/2 holds nowhere beyond the strip of what is visible
        if sv < smax:
            bad += (sv + 1) ** 2 < ((h + Fraction(1, 2)) * 16) ** 2 * tden or _thick_alpha(sv + 1, tden, hw) != 0
        # ... and delta <= hw - 1/2 everywhere inside the opaque one, which lies inside the other
        if so >= 0:
            bad += Fraction(so) ** 2 > ((h - Fraction(1, 2)) * 16) ** 2 * tden or _thick_alpha(so, tden, hw) != 1
            bad += so > sv
    return bad


def test_strips_bound_the_coverage():
    assert _strips_fail(random.Random(11), 20000) == 0


def test_the_strip_model_fails_with_a_planted_mistake():
    short = lambda hw, tden, smax, n: min(int(((hw + F32(0.5)) * F32(16.0)) * _sqrt(tden, n)) - 1, smax)   # noqa: E731
    assert _strips_fail(random.Random(12), 4000, vis=short) > 0
    wide = lambda hw, tden, n: _strip_opaque(hw, tden, n, margin=F32(-(2.0**-10)))                          # noqa: E731
    assert _strips_fail(random.Random(12), 4000, opaque=wide) > 0


def _box_fail(rng, n, slack=2):
    bad = inside = 0
    for _ in range(n):
        dx, dy, hw, R = _segment(rng)
        tden = dx * dx + dy * dy
        e = rng.choice((-1, 0, 1))
        sms = [_smax(R, tden)]
        sms += [_strip_vis(hw, tden, sms[0], e), _strip_opaque(hw, tden, e)]
        for sm in sms:
            if sm < 0:
                continue
            il = _rcp(tden, e) * F32(sm)
            rx = min(R, int(min(F32(abs(dy)) * il, F32(2147483520.0))) + slack)
            ry = min(R, int(min(F32(abs(dx)) * il, F32(2147483520.0))) + slack)
            # points of the plane in the strip's corners: foot at t in [0, 1), cross = +-sm
            for t in (0.0, rng.random(), 1.0):
                for s in (-1, 1):
                    q = s * sm / tden
                    fx, fy = t * dx + q * dy, t * dy - q * dx
                    for ex in (math.floor(fx), math.ceil(fx)):
                        for ey in (math.floor(fy), math.ceil(fy)):
                            tn, cr = ex * dx + ey * dy, ex * dy - ey * dx
                            if not (0 <= tn < tden and abs(cr) <= sm):
                                continue
                            inside += 1
                            # the kernel's columns are those whose centre lies strictly inside
                            bad += not (min(0, dx) - rx < ex < max(0, dx) + rx)
                            bad += not (min(0, dy) - ry < ey < max(0, dy) + ry)
    assert inside > n
    return bad


def test_narrowed_boxes_hold_the_strip():
    assert _box_fail(random.Random(21), 12000) == 0


def test_the_box_model_fails_with_a_planted_mistake():
    assert _box_fail(random.Random(22), 4000, slack=0) > 0


def _floordiv(n, d, rd, lo, hi, correct=True):
    q = math.floor(min(max(F32(n) * rd, F32(lo)), F32(hi)))
    if correct:
        if q * d > n:
            q -= 1
        elif q * d + d <= n:
            q += 1
    return min(max(q, lo), hi)


def _rows_fail(rng, n, **fd):
    bad = hits = misses = 0
    for _ in range(n):
        dx, dy, hw, R = _segment(rng)
        if R <= 32:
            hw = F32(rng.uniform(1.6, 2048.0))
            R = math.ceil(16 * Fraction(float(hw))) + 8
        ntx = rng.choice((1, 7, 120, 1024))
        xa, ya = rng.randint(-4096, 256 * ntx + 4096), rng.randint(-4096, 256 * ntx + 4096)
        if rng.random() < 0.3:   # corner centres exactly on the slab's ends and the strip's edges
            dx, dy = rng.choice(((dx or 1, 0), (0, dy or 1), (dx or 1, dx or 1)))
            xa, ya = 256 * rng.randint(0, ntx) + rng.choice((8, 248)), 256 * rng.randint(0, ntx) + rng.choice((8, 248))
        tden, xb, yb = dx * dx + dy * dy, xa + dx, ya + dy
        smax = _smax(R, tden)
        tx0, tx1 = max((min(xa, xb) - R) >> 8, 0), min((max(xa, xb) + R) >> 8, ntx - 1)
        ty0, ty1 = max((min(ya, yb) - R) >> 8, 0), min((max(ya, yb) + R) >> 8, ntx - 1)
        if tx0 > tx1 or ty0 > ty1:
            continue
        K, span = tx1 - tx0, 16 * (TILE - 1)
        rdx, rdy = _rcp(256 * max(abs(dx), 1), rng.choice((-1, 0, 1))), _rcp(256 * max(abs(dy), 1), rng.choice((-1, 0, 1)))

        def bound(v, w, c0, c1, a, ra, k0, k1):
            if a > 0:
                k0 = max(k0, -_floordiv(v - c0, a, ra, -K - 1, 1, **fd))
                k1 = min(k1, _floordiv(c1 - w, a, ra, -1, K + 1, **fd))
            elif a < 0:
                k1 = min(k1, _floordiv(v - c0, -a, ra, -1, K + 1, **fd))
                k0 = max(k0, -_floordiv(c1 - w, -a, ra, -K - 1, 1, **fd))
            elif v < c0 or w > c1:
                k1 = -1
            return k0, k1

        for ty in {ty0, ty1, rng.randint(ty0, ty1)}:
            ex, ey = 256 * tx0 + 8 - xa, 256 * ty + 8 - ya
            t, c = ex * dx + ey * dy, ex * dy - ey * dx
            k0, k1 = bound(t + max(0, span * dx) + max(0, span * dy), t + min(0, span * dx) + min(0, span * dy), 0, tden,
                           256 * dx, rdx, 0, K)
            k0, k1 = bound(c + max(0, span * dy) + max(0, -span * dx), c + min(0, span * dy) + min(0, -span * dx), -smax,
                           smax, 256 * dy, rdy, k0, k1)
            for k in {0, K, max(k0 - 1, 0), min(max(k0, 0), K), min(max(k1, 0), K), min(k1 + 1, K), rng.randint(0, K)}:
                if k < 0:
                    continue
                ts, cs = [], []
                for cx in (ex + 256 * k, ex + 256 * k + span):
                    for cy in (ey, ey + span):
                        ts.append(cx * dx + cy * dy)
                        cs.append(cx * dy - cy * dx)
                want = not (max(ts) < 0 or min(ts) > tden or min(cs) > smax or max(cs) < -smax)
                bad += want != (k0 <= k <= k1)
                hits += want
                misses += not want
    assert hits > n and misses > n // 2
    return bad


def test_row_intervals_equal_the_corner_test():
    assert _rows_fail(random.Random(31), 6000) == 0


def test_the_row_model_fails_with_a_planted_mistake():
    assert _rows_fail(random.Random(32), 3000, correct=False) > 0


@pytest.mark.parametrize("d", [256, 256 * 16384, 256 * 3, 256 * 9973])
def test_floor_quotients_at_their_edges(d):
    for q in list(range(-1025, 1026, 41)) + [-1, 0, 1]:
        for off in (-1, 0, 1):
            for e in (-1, 0, 1):
                n = q * d + off
                want = min(max(n // d, -1025), 1025)
                assert _floordiv(n, d, _rcp(d, e), -1025, 1025) == want, (n, d)
