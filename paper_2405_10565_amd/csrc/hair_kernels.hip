// Device kernels of the LoD hair renderer (gfx950 / MI355X).
//
// Frame pipeline, all on the caller's stream:
//   k_project        one thread per segment: float32 projection and 1/16-pixel snapping, screen
//                    half-width (Sec. 5.2, hair width calculation), culling.
//   k_bin_count      per block of consecutive segments: tile counts in LDS (no device atomics);
//   k_bin_offsets    column scan of the per-block count matrix -> each block's place in every list;
//   k_lists_scan     exclusive prefix sums: tile list offsets and work items.
//   k_scatter        per block: append its segments' ids to the overlapped tiles' lists, and clear
//                    what the later passes accumulate into.
//   k_opaque         frames with thick hairs: per pixel the nearest opaque fragment's depth key.
//   k_count          per (tile, list chunk): exact integer coverage -> per-pixel fragment counts
//                    (LDS-aggregated, then one global atomic per pixel).
//   k_tile_prep      per tile: pixel offsets, and whole pixels packed into batches of <= kCap.
//   k_emit           per (tile, list chunk): (key, local index) records into the fragment buffer
//                    and each pixel's depth-key range.
//   k_batch          one workgroup per batch, all in LDS: exact per-pixel order (bucket map over
//                    each pixel's key range, then each record's rank in its bucket), one lane per
//                    fragment for shading, front-to-back blending by a two-level segmented scan,
//                    coalesced RGBA stores.
// The integer-deciding steps (projection, snapping, half-width, depth key) are float32 with
// one rounding per operation and no contraction, so they match a float32 reference bit for bit.
#include <algorithm>
#include <type_traits>

#include "hair_internal.h"
#include "hair_shading.h"
#include "hair_dual.h"

#pragma clang fp contract(off)

namespace hair {
namespace {

constexpr int kNT = 256;                   // threads per tile block (= pixels per tile)
constexpr int kPerThread = kCap / kNT;     // LDS batch fragments per thread
static_assert(kCap % kNT == 0, "a batch is kPerThread fragments per thread");

static_assert(kTile == 16, "the shifts below assume 16-pixel tiles in 1/16-pixel units");

__device__ inline int wave_max(int v) {
    for (int off = 32; off >= 1; off >>= 1) v = max(v, __shfl_xor(v, off));
    return v;
}

// Inclusive prefix sum of x over the 64 lanes of a wave, in lane order, with DPP moves: shifts
// by 1, 2, 4 and 8 lanes inside each row of 16 (lanes shifted in from outside the row add 0),
// then the last lane of rows 0 and 2 added to rows 1 and 3, and lane 31 added to rows 2 and 3.
// (No LDS permutes: six adds with a moved operand.)
__device__ inline uint32_t row_inclusive_sum(uint32_t x) {   // over each row of 16 lanes
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);   // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);   // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);   // row_shr:8
    return x;
}
__device__ inline uint32_t wave_inclusive_sum(uint32_t x) {
    x = row_inclusive_sum(x);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);   // row_bcast:15 -> rows 1, 3
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);   // row_bcast:31 -> rows 2, 3
    return x;
}

// Workgroups are dealt to the 8 XCDs round-robin (block b runs on XCD b % 8).  Map block b to
// work index w so that each XCD takes one contiguous range of work: neighbouring work units
// (batches of one tile, chunks of one list) then share that XCD's L2.
__device__ inline uint32_t xcd_contiguous(uint32_t b, uint32_t nb) {
    const uint32_t q = nb / 8, rem = nb % 8, x = b % 8, slot = b / 8;
    return x * q + min(x, rem) + slot;
}

// Its inverse on [0, nb): the block that xcd_contiguous sends to index r.
__device__ inline uint32_t xcd_block_of(uint32_t r, uint32_t nb) {
    const uint32_t q = nb / 8, rem = nb % 8, big = rem * (q + 1);
    uint32_t x, slot;
    if (r < big) {
        x = r / (q + 1);
        slot = r - x * (q + 1);
    } else {   // here q >= 1
        x = rem + (r - big) / q;
        slot = (r - big) - (x - rem) * q;
    }
    return slot * 8 + x;
}

// One LDS batch of the shading pass: tile, pixels [p0, p1), oversized (one pixel deeper than
// a batch), the frame-wide index of its first fragment and its fragment count.  The table is
// stored in launch order (record b is processed by block b, which keeps the tiles of an XCD
// contiguous), so a block reads its record without first reading the batch count.
struct BatchRec {
    int tile, p0, p1;
    bool over;
    uint32_t frag0, nfrag;
    bool thick;   // mixed frames: a pixel of the batch holds a thick-hair fragment
};
__device__ inline uint4 pack_batch(int tile, int p0, int p1, bool over, uint32_t frag0, uint32_t nfrag,
                                   bool thick = false) {
    return make_uint4((uint32_t)tile,
                      (uint32_t)p0 | ((uint32_t)p1 << 9) | (over ? 1u << 18 : 0u) | (thick ? 1u << 19 : 0u), frag0,
                      nfrag);
}
__device__ inline BatchRec unpack_batch(const uint4 r) {
    return BatchRec{(int)r.x, (int)(r.y & 511u), (int)((r.y >> 9) & 511u), ((r.y >> 18) & 1u) != 0, r.z, r.w,
                    ((r.y >> 19) & 1u) != 0};
}

// ---------------------------------------------------------------------------------------
// Projection (float32, fixed operation order).
struct PPoint {
    float X16, Y16, z, iz;
    bool ok;
};

__device__ inline PPoint project_point(const CamConst& c, float px, float py, float pz) {
    const float d0 = px - c.pos[0];
    const float d1 = py - c.pos[1];
    const float d2 = pz - c.pos[2];
    const float vx = (c.rot[0] * d0 + c.rot[1] * d1) + c.rot[2] * d2;
    const float vy = (c.rot[3] * d0 + c.rot[4] * d1) + c.rot[5] * d2;
    const float vz = (c.rot[6] * d0 + c.rot[7] * d1) + c.rot[8] * d2;
    PPoint p;
    p.z = -vz;
    const float xs = c.cx + c.fx * (vx / p.z);
    const float ys = c.cy - c.fy * (vy / p.z);
    p.iz = 1.0f / p.z;
    p.X16 = 16.0f * xs;
    p.Y16 = 16.0f * ys;
    p.ok = (p.z >= c.z_near) && (p.X16 >= -16384.0f) && (p.X16 <= (float)(16 * c.W + kGuard)) &&
           (p.Y16 >= -16384.0f) && (p.Y16 <= (float)(16 * c.H + kGuard));
    return p;
}

__device__ inline float norm3f(float x, float y, float z) { return sqrtf((x * x + y * y) + z * z); }
__device__ inline float dot_e(const float e[3], float x, float y, float z) { return (x * e[0] + y * e[1]) + z * e[2]; }

// Thick-hair half-width: support of the ellipse across the view at the segment midpoint.
__device__ inline float cluster_halfwidth(const CamConst& c, float ax, float ay, float az, float bx, float by,
                                          float bz, float zA, float zB, float hx, float hy, float hz, float a_len,
                                          float b_len) {
    const float tx = bx - ax, ty = by - ay, tz = bz - az;
    const float tl = norm3f(tx, ty, tz);
    const float ux = tx / tl, uy = ty / tl, uz = tz / tl;
    const float mx = (ax + bx) * 0.5f, my = (ay + by) * 0.5f, mz = (az + bz) * 0.5f;
    float wx = c.pos[0] - mx, wy = c.pos[1] - my, wz = c.pos[2] - mz;
    const float wl = norm3f(wx, wy, wz);
    wx = wx / wl;
    wy = wy / wl;
    wz = wz / wl;
    const float dwu = (wx * ux + wy * uy) + wz * uz;
    const float px = wx - dwu * ux, py = wy - dwu * uy, pz = wz - dwu * uz;
    const float pl = norm3f(px, py, pz);
    const float xx = px / pl, xy = py / pl, xz = pz / pl;
    const float yx = uy * xz - uz * xy, yy = uz * xx - ux * xz, yz = ux * xy - uy * xx;
    const float bhx = uy * hz - uz * hy, bhy = uz * hx - ux * hz, bhz = ux * hy - uy * hx;
    const float pa = a_len * ((hx * yx + hy * yy) + hz * yz);
    const float pb = b_len * ((bhx * yx + bhy * yy) + bhz * yz);
    float W = sqrtf(pa * pa + pb * pb);
    if (!(pl > 1e-7f)) W = fmaxf(a_len, b_len);
    const float zm = (zA + zB) * 0.5f;
    return (W * c.fy) / zm;
}

struct TileRect {
    int tx0, tx1, ty0, ty1;
};

// Tiles overlapped by the segment's integer box widened by its radius (x >> 8 = floor(x / 256),
// a 16-pixel tile in 1/16-pixel units; coordinates of a visible segment fit 32 bits).
__device__ inline TileRect tile_rect(const SegRec& s, int ntx, int nty) {
    const int R = (s.hwfx & kHwMask) + 8;
    const int lox = min(s.xa, s.xb) - R, hix = max(s.xa, s.xb) + R;
    const int loy = min(s.ya, s.yb) - R, hiy = max(s.ya, s.yb) + R;
    TileRect r;
    r.tx0 = max(lox >> 8, 0);
    r.tx1 = min(hix >> 8, ntx - 1);
    r.ty0 = max(loy >> 8, 0);
    r.ty1 = min(hiy >> 8, nty - 1);
    return r;
}

// The shading record of a strand segment in a strand-level frame: everything the shading pass
// reads for one fragment in one aligned 64-byte line (the screen record's coverage geometry,
// inverse depths and half-width, whose sign bit carries the side flag, then the world
// endpoints and the strand's absorption):
//   q0 = (xa, ya, xb, yb as int bits)  q1 = (iza, izb, +-hw, pA.x)  q2 = (pA.y, pA.z, pB.x, pB.y)
//   q3 = (pB.z, sigma_r, sigma_g, sigma_b)
__device__ inline void pack_strand_shade(const SegRec& r, float ax, float ay, float az, float bx, float by, float bz,
                                         float sr_, float sg_, float sb_, ShadeRec* sr) {
    const float shw = __uint_as_float(__float_as_uint(r.hw) | ((r.hwfx & kFlagNegSide) ? 0x80000000u : 0u));
    sr->q0 = make_float4(__int_as_float(r.xa), __int_as_float(r.ya), __int_as_float(r.xb), __int_as_float(r.yb));
    sr->q1 = make_float4(r.iza, r.izb, shw, ax);
    sr->q2 = make_float4(ay, az, bx, by);
    sr->q3 = make_float4(bz, sr_, sg_, sb_);
}

// Segment g of level lv, drawn between (ax, ay, az) and (bx, by, bz): its screen record
// (projection, snapping, half-width, culling, side of h > 0) and, when sr is given, its
// shading record (packed: the strand-level layout above; otherwise q0..q3 as ShadeRec states).
// The endpoints are the level's vertices, or points of a curved thick hair.
__device__ inline SegRec project_segment_at(const LevelDev& lv, int g, float ax, float ay, float az, float bx, float by,
                                            float bz, const CamConst& cam, ShadeRec* sr, bool packed = false) {
    const int owner = g / lv.S;
    const PPoint A = project_point(cam, ax, ay, az);
    const PPoint B = project_point(cam, bx, by, bz);
    if (sr && !packed) {   // whole float4 stores (q3 only for thick hairs)
        const float sb = lv.sig[2 * lv.n_owner + owner];
        float4 q2 = make_float4(0.f, 0.f, 0.f, sb);
        if (lv.kind != 0) q2 = make_float4(lv.ahat[g], lv.ahat[lv.nseg + g], lv.ahat[2 * lv.nseg + g], sb);
        sr->q0 = make_float4(ax, ay, az, lv.sig[owner]);
        sr->q1 = make_float4(bx, by, bz, lv.sig[lv.n_owner + owner]);
        sr->q2 = q2;
        if (lv.kind != 0)
            sr->q3 = make_float4(lv.axes[2 * g], lv.axes[2 * g + 1], (float)lv.n_total[owner], lv.r[owner]);
    }
    float hw;
    if (lv.kind == 0) {
        const float zm = (A.z + B.z) * 0.5f;
        hw = ((0.5f * lv.width[owner]) * cam.fy) / zm;
    } else {
        hw = cluster_halfwidth(cam, ax, ay, az, bx, by, bz, A.z, B.z, lv.ahat[g], lv.ahat[lv.nseg + g],
                               lv.ahat[2 * lv.nseg + g], lv.axes[2 * g], lv.axes[2 * g + 1]);
    }
    const float hw16 = 16.0f * hw;
    SegRec r;
    r.xa = r.ya = r.xb = r.yb = 0;
    r.hwfx = 0;
    r.iza = A.iz;
    r.izb = B.iz;
    r.hw = hw;
    if (A.ok && B.ok && isfinite(hw16) && hw16 >= 0.0f) {
        r.xa = (int)rintf(A.X16);
        r.ya = (int)rintf(A.Y16);
        r.xb = (int)rintf(B.X16);
        r.yb = (int)rintf(B.Y16);
        const float c16 = ceilf(hw16);
        const bool too_long = abs(r.xb - r.xa) > kMaxAxis || abs(r.yb - r.ya) > kMaxAxis;
        if (too_long || c16 > (float)kMaxHwFx) {
            // (a segment too long but not too wide is drawn again as pieces)
            r.hwfx = kFlagCulledLong | (too_long && c16 <= (float)kMaxHwFx ? kFlagSplit : 0);
        } else {
            r.hwfx = (int)c16 | kFlagVisible;
            // side of the screen normal (dY, -dX) on which h > 0 (toward y^ = u x x^)
            const float tx = bx - ax, ty = by - ay, tz = bz - az;
            const float tl = norm3f(tx, ty, tz);
            const float ux = tx / tl, uy = ty / tl, uz = tz / tl;
            const float mx = (ax + bx) * 0.5f, my = (ay + by) * 0.5f, mz = (az + bz) * 0.5f;
            float wx = cam.pos[0] - mx, wy = cam.pos[1] - my, wz = cam.pos[2] - mz;
            const float wl = norm3f(wx, wy, wz);
            wx /= wl; wy /= wl; wz /= wl;
            const float dwu = (wx * ux + wy * uy) + wz * uz;
            float px = wx - dwu * ux, py = wy - dwu * uy, pz = wz - dwu * uz;
            const float pl = fmaxf(norm3f(px, py, pz), 1e-30f);
            px /= pl; py /= pl; pz /= pl;
            const float yx = uy * pz - uz * py, yy = uz * px - ux * pz, yz = ux * py - uy * px;
            const float yvx = (cam.rot[0] * yx + cam.rot[1] * yy) + cam.rot[2] * yz;
            const float yvy = (cam.rot[3] * yx + cam.rot[4] * yy) + cam.rot[5] * yz;
            const float yvz = (cam.rot[6] * yx + cam.rot[7] * yy) + cam.rot[8] * yz;
            const float d0 = mx - cam.pos[0], d1 = my - cam.pos[1], d2 = mz - cam.pos[2];
            const float mvx = (cam.rot[0] * d0 + cam.rot[1] * d1) + cam.rot[2] * d2;
            const float mvy = (cam.rot[3] * d0 + cam.rot[4] * d1) + cam.rot[5] * d2;
            const float mvz = (cam.rot[6] * d0 + cam.rot[7] * d1) + cam.rot[8] * d2;
            const float Z = -mvz;
            const float sx = cam.fx * (yvx + (mvx / Z) * yvz);
            const float sy = -cam.fy * (yvy + (mvy / Z) * yvz);
            const float side = sx * (float)(r.yb - r.ya) - sy * (float)(r.xb - r.xa);
            if (side < 0.0f) r.hwfx |= kFlagNegSide;
        }
    }
    if (sr && packed)
        pack_strand_shade(r, ax, ay, az, bx, by, bz, lv.sig[owner], lv.sig[lv.n_owner + owner],
                          lv.sig[2 * lv.n_owner + owner], sr);
    return r;
}

__device__ inline SegRec project_segment(const LevelDev& lv, int g, const CamConst& cam, ShadeRec* sr,
                                         bool packed = false) {
    const int owner = g / lv.S, k = g - owner * lv.S;
    const int va = owner * (lv.S + 1) + k;
    return project_segment_at(lv, g, lv.vx[va], lv.vy[va], lv.vz[va], lv.vx[va + 1], lv.vy[va + 1], lv.vz[va + 1], cam,
                              sr, packed);
}

// A frame of one level: strand levels write the packed strand shading record.  The block's
// records are staged in LDS and stored as consecutive 16-byte words, so that every store
// instruction writes whole contiguous lines.
__global__ __launch_bounds__(256) void k_project(LevelDev lv, CamConst cam, SegRec* __restrict__ seg,
                                                 ShadeRec* __restrict__ shade) {
    __shared__ float4 s_seg[2 * 256];
    __shared__ float4 s_sh[4 * 256];
    const int t = threadIdx.x, g0 = blockIdx.x * 256, g = g0 + t;
    if (g < lv.nseg) {
        ShadeRec sr;
        sr.q3 = make_float4(0.f, 0.f, 0.f, 0.f);
        const SegRec r = project_segment(lv, g, cam, &sr, lv.kind == 0);
        s_seg[2 * t] = make_float4(__int_as_float(r.xa), __int_as_float(r.ya), __int_as_float(r.xb), __int_as_float(r.yb));
        s_seg[2 * t + 1] = make_float4(__int_as_float(r.hwfx), r.iza, r.izb, r.hw);
        s_sh[4 * t] = sr.q0;
        s_sh[4 * t + 1] = sr.q1;
        s_sh[4 * t + 2] = sr.q2;
        s_sh[4 * t + 3] = sr.q3;
    }
    __syncthreads();
    const int n = min(256, lv.nseg - g0);
    float4* dseg = reinterpret_cast<float4*>(seg + g0);
    for (int i = t; i < 2 * n; i += 256) dseg[i] = s_seg[i];
    float4* dsh = reinterpret_cast<float4*>(shade + g0);
    for (int i = t; i < 4 * n; i += 256) dsh[i] = s_sh[i];
}

// ---------------------------------------------------------------------------------------
// Per-group, per-segment LoD (Sec. 5.1 step 5; Sec. 5.2, eq. lod_select).  Groups are the
// clusters of the coarsest level; every finer level's owners (clusters, or strands at level
// 0) are listed per group in h.grp_owner[l] (CSR h.grp_start[l]).  The width of (g, k) at
// level l is the largest 2 hw over the visible k-th segments of level l's owners in g (0 if
// none is visible).  One wave per (g, k).

// Level of (g, k); levels outside [0, n_levels] are read as 0 (the selection counts them, and the
// caller checks before rendering).
__device__ inline int level_at(const HierDev& h, const int32_t* levels, int gk) {
    const int L = levels[gk];
    return (L < 0 || L > h.n_levels) ? 0 : L;
}

// width bits of (g, k) at level l (non-negative float bits order like the floats)
__device__ inline uint32_t group_width_bits(const HierDev& h, int l, int g, int k, const CamConst& cam) {
    const LevelDev& lv = h.lv[l];
    const int b = h.grp_start[l][g], e = h.grp_start[l][g + 1];
    uint32_t w = 0;
    for (int i = b + (int)__lane_id(); i < e; i += 64) {
        const SegRec r = project_segment(lv, h.grp_owner[l][i] * lv.S + k, cam, nullptr);
        if (r.hwfx & kFlagVisible) w = max(w, __float_as_uint(2.0f * r.hw));
    }
    for (int off = 32; off >= 1; off >>= 1) w = max(w, (uint32_t)__shfl_xor((int)w, off));
    return w;
}

// Initial levels: the coarsest l >= 1 whose width is <= eps_w, else 0 (the strands).  The wave's
// lanes take the owners of all levels, coarsest first, 64 at a time, and stop at the level that
// passes: a coarse level has one owner per group or a few, and one after the other the levels are a
// chain of gathers (bound by their latency: 100k strands, three levels, 30 -> 21 us).
__global__ __launch_bounds__(256) void k_lod_init(HierDev h, CamConst cam, float eps_w, int32_t* __restrict__ levels) {
    const int gk = (int)(blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6));
    if (gk >= h.G * h.S) return;
    const int g = gk / h.S, k = gk - g * h.S;
    auto owners = [&](int l) { return h.grp_start[l][g + 1] - h.grp_start[l][g]; };
    int pick = 0, l = h.n_levels, done = 0;   // the first unfinished level and its owners already seen
    uint32_t w_l = 0;                         // their width
    while (l >= 1 && pick == 0) {
        int mine = 0, x = (int)__lane_id() + done;
        uint32_t w = 0;
        for (int q = l; q >= 1 && mine == 0; --q) {
            const int c = owners(q);
            if (x < c) mine = q;
            else x -= c;
        }
        if (mine) {
            const LevelDev& lv = h.lv[mine];
            const SegRec r = project_segment(lv, h.grp_owner[mine][h.grp_start[mine][g] + x] * lv.S + k, cam, nullptr);
            if (r.hwfx & kFlagVisible) w = __float_as_uint(2.0f * r.hw);
        }
        for (int left = 64; l >= 1;) {        // the levels of this round
            uint32_t m = mine == l ? w : 0u;
            for (int off = 32; off >= 1; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
            w_l = max(w_l, m);
            const int c = owners(l) - done;
            if (c > left) {
                done += left;
                break;
            }
            left -= c;
            if (__uint_as_float(w_l) <= eps_w) {
                pick = l;
                break;
            }
            --l;
            done = 0;
            w_l = 0;
        }
    }
    if (__lane_id() == 0) levels[gk] = pick;
}

// Deferred update from this frame's level L, with w_cur its width and w_c the width one
// level coarser: finer if w_cur > eps_w, coarser if w_c <= eps_w, else unchanged.
__global__ __launch_bounds__(256) void k_lod_update(HierDev h, CamConst cam, float eps_w, int32_t* __restrict__ levels) {
    const int gk = (int)(blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6));
    if (gk >= h.G * h.S) return;
    const int g = gk / h.S, k = gk - g * h.S;
    const int L = level_at(h, levels, gk);
    const float w_cur = __uint_as_float(group_width_bits(h, L, g, k, cam));
    int next = L;
    if (w_cur > eps_w) {
        next = max(L - 1, 0);
    } else if (L < h.n_levels) {
        const float w_c = __uint_as_float(group_width_bits(h, L + 1, g, k, cam));
        if (w_c <= eps_w) next = L + 1;
    }
    if (__lane_id() == 0) levels[gk] = next;
}

// Selection of a mixed frame: for every (g, k) the k-th segments of the owners of level
// L(g, k) in g, in (g, k, owner) order; entry = level << 28 | segment id of that level.  start[G S] is
// the number of rows, start[G S + 1] that of entries of levels out of range, start[G S + 2] that of the
// rows that are strands.
__device__ inline uint32_t selected(const HierDev& h, const int32_t* levels, int gk, uint32_t& bad, uint32_t& strands) {
    const int g = gk / h.S, raw = levels[gk], L = level_at(h, levels, gk);
    if (raw != L) ++bad;
    const uint32_t n = (uint32_t)(h.grp_start[L][g + 1] - h.grp_start[L][g]);
    if (L == 0) strands += n;
    return n;
}
// (more than kScanOneBlock (g, k): sums, the last two words of start, is zeroed before)
__global__ __launch_bounds__(256) void k_sel_count(HierDev h, const int32_t* __restrict__ levels,
                                                   uint32_t* __restrict__ cnt, uint32_t* __restrict__ sums) {
    const int gk = blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t bad = 0, strands = 0;
    if (gk < h.G * h.S) cnt[gk] = selected(h, levels, gk, bad, strands);
    if (bad) atomicAdd(&sums[0], 1u);
    strands = wave_inclusive_sum(strands);
    if ((threadIdx.x & 63) == 63 && strands) atomicAdd(&sums[1], strands);
}

__global__ __launch_bounds__(256) void k_sel_fill(HierDev h, const int32_t* __restrict__ levels,
                                                  const uint32_t* __restrict__ sel_start, uint32_t* __restrict__ sel) {
    const int gk = (int)(blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6));
    if (gk >= h.G * h.S) return;
    const int g = gk / h.S, k = gk - g * h.S, L = level_at(h, levels, gk);
    const int b = h.grp_start[L][g], e = h.grp_start[L][g + 1];
    const uint32_t o = sel_start[gk];
    for (int i = b + (int)__lane_id(); i < e; i += 64)
        sel[o + (uint32_t)(i - b)] = ((uint32_t)L << 28) | (uint32_t)(h.grp_owner[L][i] * h.S + k);
}

// (records staged in LDS and stored as consecutive 16-byte words, as in k_project)
__global__ __launch_bounds__(256) void k_project_mixed(HierDev h, const uint32_t* __restrict__ sel, int nsel,
                                                       CamConst cam, SegRec* __restrict__ seg,
                                                       ShadeRec* __restrict__ shade) {
    __shared__ float4 s_seg[2 * 256];
    __shared__ float4 s_sh[4 * 256];
    const int t = threadIdx.x, i0 = blockIdx.x * 256, i = i0 + t;
    if (i < nsel) {
        const uint32_t e = sel[i];
        const int L = (int)(e >> 28), g = (int)(e & 0x0FFFFFFFu);
        ShadeRec sr;
        sr.q3 = make_float4(0.f, 0.f, 0.f, 0.f);
        SegRec r = project_segment(h.lv[L], g, cam, &sr);
        if (h.lv[L].kind == 1) r.hwfx |= kFlagThick;
        // (a strand row's q3 is otherwise unused: its world radius, and -1 marking a strand, for
        // the shadow pass, which reads the rows' world data from these records)
        else sr.q3 = make_float4(0.5f * h.lv[L].width[g / h.lv[L].S], 0.0f, 0.0f, -1.0f);
        s_seg[2 * t] = make_float4(__int_as_float(r.xa), __int_as_float(r.ya), __int_as_float(r.xb), __int_as_float(r.yb));
        s_seg[2 * t + 1] = make_float4(__int_as_float(r.hwfx), r.iza, r.izb, r.hw);
        s_sh[4 * t] = sr.q0;
        s_sh[4 * t + 1] = sr.q1;
        s_sh[4 * t + 2] = sr.q2;
        s_sh[4 * t + 3] = sr.q3;
    }
    __syncthreads();
    const int n = min(256, nsel - i0);
    float4* dseg = reinterpret_cast<float4*>(seg + i0);
    for (int k = t; k < 2 * n; k += 256) dseg[k] = s_seg[k];
    float4* dsh = reinterpret_cast<float4*>(shade + i0);
    for (int k = t; k < 4 * n; k += 256) dsh[k] = s_sh[k];
}

// Exclusive scan of n counts by one 1024-thread block in coalesced chunks of 4096 (four
// consecutive counts per lane, wave shuffles, one LDS step across the 16 waves); start[n] =
// total.  For n up to kScanOneBlock.
constexpr int kScanOneBlock = 1 << 16;
__global__ __launch_bounds__(1024) void k_scan1(const uint32_t* __restrict__ cnt, uint32_t* __restrict__ start, int n) {
    __shared__ uint32_t s_w[16];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    uint32_t carry = 0;
    for (int base = 0; base < n; base += 4096) {
        const int i0 = base + 4 * t;
        uint32_t v[4], sum = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = i0 + k < n ? cnt[i0 + k] : 0u;
            sum += v[k];
        }
        uint32_t x = sum;
        x = wave_inclusive_sum(x);
        if (lane == 63) s_w[w] = x;
        __syncthreads();
        uint32_t wbase = 0, total = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const uint32_t a = s_w[k];
            if (k < w) wbase += a;
            total += a;
        }
        uint32_t run = carry + wbase + (x - sum);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (i0 + k < n) start[i0 + k] = run;
            run += v[k];
        }
        carry += total;
        __syncthreads();
    }
    if (t == 0) start[n] = carry;
}

// Single-block exclusive scan of n values get(i) into put(i, prefix); returns the total.  The
// caller's block has 1024 threads; n up to kScanOneBlock.
template <class G, class P>
__device__ inline uint32_t block_scan_1024(int n, G get, P put, uint32_t* s_w) {
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    uint32_t carry = 0;
    for (int base = 0; base < n; base += 4096) {
        const int i0 = base + 4 * t;
        uint32_t v[4], sum = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = i0 + k < n ? get(i0 + k) : 0u;
            sum += v[k];
        }
        uint32_t x = sum;
        x = wave_inclusive_sum(x);
        if (lane == 63) s_w[w] = x;
        __syncthreads();
        uint32_t wbase = 0, total = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const uint32_t a = s_w[k];
            if (k < w) wbase += a;
            total += a;
        }
        uint32_t run = carry + wbase + (x - sum);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (i0 + k < n) put(i0 + k, run);
            run += v[k];
        }
        carry += total;
        __syncthreads();
    }
    return carry;
}

// The selection's counts and their scan in one block (up to kScanOneBlock (g, k)): one launch
// instead of a clear, a count and a scan, and one readback instead of two.
__global__ __launch_bounds__(1024) void k_select(HierDev h, const int32_t* __restrict__ levels,
                                                 uint32_t* __restrict__ start) {
    __shared__ uint32_t s_w[16], s_bad, s_strands;
    if (threadIdx.x == 0) s_bad = s_strands = 0u;
    __syncthreads();
    const int n = h.G * h.S;
    uint32_t bad = 0, strands = 0;
    const uint32_t total = block_scan_1024(
        n, [&](int i) { return selected(h, levels, i, bad, strands); }, [&](int i, uint32_t x) { start[i] = x; }, s_w);
    if (bad) atomicAdd(&s_bad, bad);
    strands = wave_inclusive_sum(strands);
    if ((threadIdx.x & 63) == 63) atomicAdd(&s_strands, strands);
    __syncthreads();
    if (threadIdx.x == 0) {
        start[n] = total;
        start[n + 1] = s_bad;
        start[n + 2] = s_strands;
    }
}

// Whether a mixed frame looks for what opaque fragments hide.  Hairs whose opaque cores cover the tiles
// that hold any segment m times over hide, lying anywhere in the depth of the groom, a fraction
// 1 - (1 - e^-m) / m of the fragments.  The pass costs a frame what a quarter of its fragments cost the
// later passes (100k strands in locks that fill half the screen, 3% of them hidden: 1.68 ms without it,
// 1.91 with it), and 12 us at least, so: m >= 1/2, and 180,000 hidden fragments.  249 views of five
// grooms with thick hairs up to 1.5 .. 25 px wide take, in the geometric mean, 0.940 of the time that they
// take without the pass (0.35 at best, 29 us of 1.09 ms more at worst) and 0.938 of that with it in every
// view (0.74 at best, 9 us more at worst).
__device__ inline bool opaque_pays(unsigned long long area_opaque, unsigned long long area_all, uint32_t tiles) {
    const float m = (float)area_opaque * (1.0f / 65536.0f) / (float)max(tiles, 1u);
    if (!(m >= 0.5f)) return false;
    const float hidden = 1.0f - (1.0f - expf(-m)) / m;
    return hidden * ((float)area_all * (1.0f / 256.0f)) >= 180000.0f;
}
// The tiles' list offsets (exclusive scan of their list lengths, block 0) and their work items of
// the count and emit passes (kNT list entries each, scanned by block 1), each with its part of the
// first capacity check: the work of k_tile_items, k_scan1 twice and k_check_caps stage 1 for up to
// kScanOneBlock tiles.
__global__ __launch_bounds__(1024) void k_lists_scan(const uint32_t* __restrict__ tot, int T,
                                                     uint32_t* __restrict__ tile_start,
                                                     uint32_t* __restrict__ item_start, Counters* ctr, uint32_t cap_pairs,
                                                     uint32_t cap_items) {
    __shared__ uint32_t s_w[16], s_tiles;
    const bool items = blockIdx.x == 1;
    uint32_t* start = items ? item_start : tile_start;
    uint32_t tiles = 0;   // that hold any segment
    if (threadIdx.x == 0) s_tiles = 0u;
    const uint32_t n = block_scan_1024(
        T, [&](int i) {
            tiles += tot[i] != 0u;
            return items ? (tot[i] + kNT - 1) / kNT : tot[i];
        },
        [&](int i, uint32_t v) { start[i] = v; }, s_w);
    if (items) {
        tiles = wave_inclusive_sum(tiles);
        if ((threadIdx.x & 63) == 63) atomicAdd(&s_tiles, tiles);
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        start[T] = n;
        ctr->sizes[items ? 1 : 0] = n;
        if (n > (items ? cap_items : cap_pairs)) ctr->cap_overflow = 1u;
        if (items) ctr->hides = opaque_pays(ctr->area_opaque, ctr->area_all, s_tiles);
    }
}

// *out = the sum of v[0 .. n) by one 1024-thread block.
__device__ inline void block_sum_u64(const uint32_t* __restrict__ v, int n, unsigned long long* out) {
    __shared__ unsigned long long s_sum[16];
    unsigned long long a = 0;
    for (int i = threadIdx.x; i < n; i += 1024) a += v[i];
    for (int off = 32; off >= 1; off >>= 1) a += (unsigned long long)__shfl_xor((long long)a, off);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) a += s_sum[w];
        *out = a;
    }
}

// (frames of more tiles than the single-block scans take)
__global__ __launch_bounds__(1024) void k_sum_tiles(FrameBufs f) { block_sum_u64(f.tile_all, f.T, &f.ctr->fragments); }

// The tiles' fragment and batch offsets (exclusive scans of tile_tot and tile_nb, block 0 and 1)
// with the second capacity check (k_scan1 twice and k_check_caps stage 2), and the frame's number
// of all fragments (block 2).  A block each: the three are latency (8160 tiles: 12.5 us in one
// block after the other, 5 us side by side).
__global__ __launch_bounds__(1024) void k_tile_scans(const uint32_t* __restrict__ tile_tot,
                                                     uint32_t* __restrict__ frag_base, const uint32_t* __restrict__ tile_nb,
                                                     uint32_t* __restrict__ batch_start, int T, Counters* ctr,
                                                     uint32_t cap_frags, uint32_t cap_batches,
                                                     const uint32_t* __restrict__ tile_all) {
    __shared__ uint32_t s_w[16];
    if (blockIdx.x == 2) {
        block_sum_u64(tile_all, T, &ctr->fragments);
        return;
    }
    const bool fr = blockIdx.x == 0;
    const uint32_t* v = fr ? tile_tot : tile_nb;
    uint32_t* start = fr ? frag_base : batch_start;
    const uint32_t n = block_scan_1024(
        T, [&](int i) { return v[i]; }, [&](int i, uint32_t x) { start[i] = x; }, s_w);
    if (threadIdx.x == 0) {
        start[T] = n;
        ctr->sizes[fr ? 2 : 3] = n;
        if (n > (fr ? cap_frags : cap_batches)) ctr->cap_overflow = 1u;
    }
}

// Multi-block exclusive scan: each 1024-thread block scans kScanChunk counts and leaves its
// total; the totals are scanned by k_scan1; k_scan_add adds each block's base.
__global__ __launch_bounds__(1024) void k_scan_local(const uint32_t* __restrict__ cnt, uint32_t* __restrict__ out,
                                                      uint32_t* __restrict__ part, int n) {
    __shared__ uint32_t s_part[1024];
    const int t = threadIdx.x;
    const int b0 = blockIdx.x * kScanChunk + t * 4;
    uint32_t v[4], sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = b0 + k < n ? cnt[b0 + k] : 0u;
        sum += v[k];
    }
    s_part[t] = sum;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const uint32_t x = t >= off ? s_part[t - off] : 0u;
        __syncthreads();
        s_part[t] += x;
        __syncthreads();
    }
    uint32_t run = s_part[t] - sum;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (b0 + k < n) out[b0 + k] = run;
        run += v[k];
    }
    if (t == 1023) part[blockIdx.x] = s_part[1023];
}

__global__ __launch_bounds__(1024) void k_scan_add(uint32_t* __restrict__ out, const uint32_t* __restrict__ base,
                                                    int n, int nblocks) {
    const int i = blockIdx.x * kScanChunk + threadIdx.x * 4;
    const uint32_t b = base[blockIdx.x];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (i + k < n) out[i + k] += b;
    if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = base[nblocks];
}

// The largest s with s^2 < R^2 t_den (R^2 t_den >= 64): a square root, corrected in 64-bit
// integers, so that |cross| <= s_max is exactly cross^2 < R^2 t_den.  Below 2^48 (every
// strand) the float square root is within 3 of s (relative error under 2^-22 on s < 2^24),
// above it the double one.
__device__ inline int strip_smax(int R, int tden) {
    const unsigned long long lim = (unsigned long long)(unsigned)(R * R) * (unsigned)tden - 1ull;
    unsigned long long s = lim < (1ull << 48) ? (unsigned long long)__builtin_amdgcn_sqrtf((float)lim)
                                              : (unsigned long long)sqrt((double)lim);
    while (s * s > lim) --s;
    while ((s + 1) * (s + 1) <= lim) ++s;
    return (int)min(s, 0x7FFFFFFFull);
}

// Tile binning without device-wide atomics.  Block b owns the contiguous segment range
// [b per_block, (b + 1) per_block) and counts, in LDS, its segments per tile of the range
// [t0, t0 + nt) (the whole image unless it has more than kMaxLdsTiles tiles); the counts form
// row b of M [nb][T].  A column-wise exclusive scan of M gives each block its place inside
// every tile list, and the scatter pass appends each segment at its block's LDS cursors.
// A tile of the box of a wide segment (radius above 2 px) is kept only if the rectangle of its
// pixel centres meets the segment's footprint (the slab 0 <= t_num <= t_den and the strip
// |cross| <= s_max, the largest s with s^2 < R^2 t_den): projected on the segment's direction and
// normal, its four corner centres must overlap both.  For short, wide segments (thick hairs) this
// drops the many box tiles beyond the segment's ends.  Thin segments keep their box's tiles.
//
// Along a row of tiles the projections' ends grow by 256 dx and 256 dy per tile, so each of the
// four conditions bounds the tile's index by an exact floor division, and the row's tiles are one
// interval: a hair of 75 px half-width, whose box has over a hundred tiles and whose footprint
// meets a sixth of them, costs a dozen rows instead of a test per tile (64 k such segments at
// 1080p: count and scatter 68 + 91 -> 32 + 43 us).  Exact in integers (corner offsets below
// 2^15 + 2^18, products below 2^33: 64 bits; a row has at most 2^10 tiles, so a float quotient,
// off by at most one, is settled by one exact test).
struct FootprintRows {
    bool wide;
    int xa, ya, dx, dy, smax;
    int K;                // the box's last tile column, from its first
    float rdx, rdy;       // reciprocals of 256 |dx|, 256 |dy|

    __device__ FootprintRows(const SegRec& r, const TileRect& rc) {
        const int R = (r.hwfx & kHwMask) + 8;
        xa = r.xa; ya = r.ya;
        dx = r.xb - r.xa; dy = r.yb - r.ya;
        const int tden = dx * dx + dy * dy;
        wide = R > 32 && tden > 0;
        smax = wide ? strip_smax(R, tden) : 0;
        K = rc.tx1 - rc.tx0;
        rdx = __builtin_amdgcn_rcpf(256.0f * (float)max(abs(dx), 1));
        rdy = __builtin_amdgcn_rcpf(256.0f * (float)max(abs(dy), 1));
    }
    // floor(n / d), clamped to [lo, hi] (|lo|, |hi| <= 2^11; rd = 1 / d)
    __device__ static int floordiv(long long n, long long d, float rd, int lo, int hi) {
        int q = (int)floorf(fminf(fmaxf((float)n * rd, (float)lo), (float)hi));
        const long long p = (long long)q * d;
        if (p > n) --q;
        else if (p + d <= n) ++q;
        return min(max(q, lo), hi);
    }
    // the k in [0, K] with c0 <= v + a k and w + a k <= c1, kept from [k0, k1]
    __device__ void bound(long long v, long long w, long long c0, long long c1, long long a, float ra, int& k0,
                          int& k1) const {
        if (a > 0) {          // k >= ceil((c0 - v) / a), k <= floor((c1 - w) / a)
            k0 = max(k0, -floordiv(v - c0, a, ra, -K - 1, 1));
            k1 = min(k1, floordiv(c1 - w, a, ra, -1, K + 1));
        } else if (a < 0) {   // k <= floor((v - c0) / |a|), k >= ceil((w - c1) / |a|)
            k1 = min(k1, floordiv(v - c0, -a, ra, -1, K + 1));
            k0 = max(k0, -floordiv(c1 - w, -a, ra, -K - 1, 1));
        } else if (v < c0 || w > c1) {
            k1 = -1;
        }
    }
    // the tiles of row ty that meet the footprint, from the box's [lo, hi] = [tx0, tx1]
    __device__ void clip(int ty, int tx0, int& lo, int& hi) const {
        if (!wide) return;
        constexpr int kSpan = 16 * (kTile - 1);
        const long long ex = 16 * kTile * tx0 + 8 - xa, ey = 16 * kTile * ty + 8 - ya;
        const long long tden = (long long)dx * dx + (long long)dy * dy;
        // at the box's first tile: t_num and cross over the corners
        const long long t = ex * dx + ey * dy, c = ex * dy - ey * dx;
        const long long tmin = t + min(0, kSpan * dx) + min(0, kSpan * dy);
        const long long tmax = t + max(0, kSpan * dx) + max(0, kSpan * dy);
        const long long cmin = c + min(0, kSpan * dy) + min(0, -kSpan * dx);
        const long long cmax = c + max(0, kSpan * dy) + max(0, -kSpan * dx);
        int k0 = 0, k1 = K;
        bound(tmax, tmin, 0, tden, 16ll * kTile * dx, rdx, k0, k1);
        bound(cmax, cmin, -(long long)smax, smax, 16ll * kTile * dy, rdy, k0, k1);
        lo = tx0 + k0;
        hi = tx0 + k1;
    }
};

// (row0, step: the tile rows ty0 + row0, ty0 + row0 + step, ... of the segment)
template <class F>
__device__ inline void for_each_tile_in_range(const SegRec& r, int ntx, int nty, int t0, int nt, int row0, int step,
                                              F&& f) {
    if (!(r.hwfx & kFlagVisible)) return;
    const TileRect rc = tile_rect(r, ntx, nty);
    if ((r.hwfx & kHwMask) + 8 <= 32) {
        for (int ty = rc.ty0 + row0; ty <= rc.ty1; ty += step)
            for (int tx = rc.tx0; tx <= rc.tx1; ++tx) {
                const int l = ty * ntx + tx - t0;
                if ((unsigned)l < (unsigned)nt) f(l);
            }
        return;
    }
    const FootprintRows fp(r, rc);
    for (int ty = rc.ty0 + row0; ty <= rc.ty1; ty += step) {
        int lo = rc.tx0, hi = rc.tx1;
        fp.clip(ty, rc.tx0, lo, hi);
        for (int tx = lo; tx <= hi; ++tx) {
            const int l = ty * ntx + tx - t0;
            if ((unsigned)l < (unsigned)nt) f(l);
        }
    }
}

// (alpha is exactly 1 at delta <= hw - 1/2 - kOpaqueMargin, see strip_opaque)
constexpr float kOpaqueMargin = 0x1p-6f;
// The first pass also leaves per-block segment statistics in blk[b] for k_bin_offsets to reduce.
// AREAS: with the areas that decide about a mixed frame's opaque pass (whole numbers, so that their sums
// and the decision do not depend on an order).
//
// LANES: lanes that share a segment, one tile row each in turn.  One for strands (a strand's box has
// a row or two).  A thick-hair level has few segments of many rows: with one lane each, 16 k of them
// fill 32 blocks, and each lane walks a dozen rows (count and scatter of 1000 hairs of 64 segments at
// 1080p with one and with eight lanes: 32 + 43 -> 20 + 30 us, k_bin_offsets 6 -> 12).
template <int LANES, bool AREAS>
__global__ __launch_bounds__(kBinThreads) void k_bin_count(const SegRec* __restrict__ seg, int nseg, int per_block,
                                                           int ntx, int nty, int t0, int nt,
                                                           uint32_t* __restrict__ M, BlockStats* __restrict__ blk) {
    static_assert(!AREAS || LANES == 1, "");
    extern __shared__ uint32_t s_tc[];
    __shared__ uint32_t s_maxhw;
    const int T = ntx * nty;
    for (int i = threadIdx.x; i < nt; i += kBinThreads) s_tc[i] = 0;
    if (threadIdx.x == 0) s_maxhw = 0;
    __syncthreads();
    const int g0 = blockIdx.x * per_block, g1 = min(nseg, g0 + per_block);
    uint32_t nvis = 0, nlong = 0, nsplit = 0, maxhw = 0;
    unsigned long long core = 0, all = 0;
    const int row0 = (int)threadIdx.x % LANES;
    for (int g = g0 + (int)threadIdx.x / LANES; g < g1; g += kBinThreads / LANES) {
        const SegRec r = seg[g];
        if (LANES == 1 || row0 == 0) {
            if (r.hwfx & kFlagVisible) {
                ++nvis;
                maxhw = max(maxhw, __float_as_uint(r.hw));
            }
            nlong += (r.hwfx & kFlagCulledLong) ? 1u : 0u;
            nsplit += (r.hwfx & kFlagSplit) ? 1u : 0u;
        }
        int tiles = 0;
        for_each_tile_in_range(r, ntx, nty, t0, nt, row0, LANES, [&](int l) {
            atomicAdd(&s_tc[l], 1u);
            if (AREAS) ++tiles;
        });
        if (AREAS && tiles) {   // (2^-8 pixels; at most the tiles' own area)
            const float dx = (float)(r.xb - r.xa), dy = (float)(r.yb - r.ya);
            const float len = 16.0f * __builtin_amdgcn_sqrtf(dx * dx + dy * dy);
            const float cap = 65536.0f * (float)min(tiles, 1 << 15);
            core += (uint32_t)fminf(2.0f * fmaxf(r.hw - 0.5f - kOpaqueMargin, 0.0f) * len, cap);
            all += (uint32_t)fminf((2.0f * r.hw + 1.0f) * len, cap);
        }
    }
    if (AREAS) {
        __shared__ unsigned long long s_core[kBinThreads / 64], s_all[kBinThreads / 64];
        for (int off = 32; off >= 1; off >>= 1) {
            core += (unsigned long long)__shfl_xor((long long)core, off);
            all += (unsigned long long)__shfl_xor((long long)all, off);
        }
        if ((threadIdx.x & 63) == 0) {
            s_core[threadIdx.x >> 6] = core;
            s_all[threadIdx.x >> 6] = all;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < kBinThreads / 64; ++w) {
                core += s_core[w];
                all += s_all[w];
            }
            // (one range of tiles after the other)
            blk[blockIdx.x].area_opaque = core + (t0 ? blk[blockIdx.x].area_opaque : 0ull);
            blk[blockIdx.x].area_all = all + (t0 ? blk[blockIdx.x].area_all : 0ull);
        }
    }
    if (t0 == 0) {
        if (maxhw) atomicMax(&s_maxhw, maxhw);
        uint32_t v = nvis, c = nlong, sp = nsplit;
        for (int off = 32; off >= 1; off >>= 1) {
            v += __shfl_xor(v, off);
            c += __shfl_xor(c, off);
            sp += __shfl_xor(sp, off);
        }
        __shared__ uint32_t s_v[kBinThreads / 64], s_c[kBinThreads / 64], s_sp[kBinThreads / 64];
        if ((threadIdx.x & 63) == 0) {
            s_v[threadIdx.x >> 6] = v;
            s_c[threadIdx.x >> 6] = c;
            s_sp[threadIdx.x >> 6] = sp;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t tv = 0, tc = 0, ts = 0;
            for (int w = 0; w < kBinThreads / 64; ++w) {
                tv += s_v[w];
                tc += s_c[w];
                ts += s_sp[w];
            }
            BlockStats& b = blk[blockIdx.x];
            b.visible = tv;
            b.culled_long = tc;
            b.max_hw_bits = s_maxhw;
            b.split = ts;
        }
    }
    __syncthreads();
    uint32_t* row = M + (size_t)blockIdx.x * T + t0;
    for (int i = threadIdx.x; i < nt; i += kBinThreads) row[i] = s_tc[i];
}

// Column-wise exclusive scan of M: M[b][t] <- sum of M[b'][t] over b' < b, tot[t] = column sum.
// A block takes 64 tiles (one per lane) and its 16 waves split the rows into 16 ranges: each
// wave sums its range, the range offsets come from LDS, and a second walk writes the prefixes.
// Block 0 also clears the frame's counters (nothing before uses them) and reduces the per-block
// segment statistics into them.
__global__ __launch_bounds__(1024) void k_bin_offsets(uint32_t* __restrict__ M, int nb, int T,
                                                      uint32_t* __restrict__ tot, const BlockStats* __restrict__ blk,
                                                      Counters* __restrict__ ctr, bool areas) {
    __shared__ uint32_t s_part[16][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int t = blockIdx.x * 64 + lane;
    const int rows = (nb + 15) / 16, r0 = min(nb, w * rows), r1 = min(nb, r0 + rows);
    uint32_t sum = 0;
    if (t < T) {
#pragma unroll 8
        for (int b = r0; b < r1; ++b) sum += M[(size_t)b * T + t];
    }
    s_part[w][lane] = sum;
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < (int)(sizeof(Counters) / 4); i += 1024) reinterpret_cast<uint32_t*>(ctr)[i] = 0u;
    __syncthreads();
    uint32_t run = 0, total = 0;
    for (int w2 = 0; w2 < 16; ++w2) {
        const uint32_t v = s_part[w2][lane];
        if (w2 < w) run += v;
        total += v;
    }
    if (t < T) {
        for (int b = r0; b < r1; ++b) {
            const size_t q = (size_t)b * T + t;
            const uint32_t v = M[q];
            M[q] = run;
            run += v;
        }
        if (w == 0) tot[t] = total;
    }
    if (blockIdx.x == 0 && w == 0) {
        uint32_t v = 0, c = 0, m = 0, sp = 0;
        unsigned long long core = 0, all = 0;
        for (int b = lane; b < nb; b += 64) {
            v += blk[b].visible;
            c += blk[b].culled_long;
            m = max(m, blk[b].max_hw_bits);
            sp += blk[b].split;
            if (areas) {
                core += blk[b].area_opaque;
                all += blk[b].area_all;
            }
        }
        for (int off = 32; off >= 1; off >>= 1) {
            v += __shfl_xor(v, off);
            c += __shfl_xor(c, off);
            m = max(m, (uint32_t)__shfl_xor((int)m, off));
            sp += __shfl_xor(sp, off);
            core += (unsigned long long)__shfl_xor((long long)core, off);
            all += (unsigned long long)__shfl_xor((long long)all, off);
        }
        if (lane == 0) {
            ctr->area_opaque = core;
            ctr->area_all = all;
            ctr->visible = v;
            ctr->culled_long = c;
            ctr->max_hw_bits = m;
            ctr->split_needed = sp;
        }
    }
}

// What the passes after the scatter expect cleared: the per-pixel counters (counts, stored and left
// out, 0; key minima ~0, key maxima 0, or ~0 before an opaque pass), the frame's image (transparent
// black, when one is given) and the work-item table (item i of tile t: its list chunk
// i - item_start[t], for the items within the table's capacity).
struct FillArgs {
    uint32_t* cnt;
    uint32_t* off;
    uint32_t* kmin;
    uint32_t* kmax;
    uint32_t kmax0;
    uint8_t* thick;
    float4* rgba;
    size_t n_rgba;
    uint4* acc;               // a shadow map's layer sums (its frame has no other per-pixel table than kmin)
    size_t n_acc;
    const uint32_t* item_start;
    uint2* item_tab;
    uint32_t cap_items;
};
__device__ inline void fill_frame(const FillArgs& a, int T) {
    const size_t n = (size_t)T * kTilePix / 4, step = (size_t)gridDim.x * blockDim.x;
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint4 zero = make_uint4(0u, 0u, 0u, 0u), ones = make_uint4(~0u, ~0u, ~0u, ~0u);
    const uint4 k0 = make_uint4(a.kmax0, a.kmax0, a.kmax0, a.kmax0);
    for (size_t i = i0; i < a.n_acc; i += step) a.acc[i] = zero;
    for (size_t i = i0; i < n; i += step) {
        reinterpret_cast<uint4*>(a.kmin)[i] = ones;
        if (!a.cnt) continue;
        reinterpret_cast<uint4*>(a.cnt)[i] = zero;
        reinterpret_cast<uint4*>(a.off)[i] = zero;
        reinterpret_cast<uint4*>(a.kmax)[i] = k0;
        if (a.thick) reinterpret_cast<uint32_t*>(a.thick)[i] = 0u;
    }
    for (size_t i = i0; i < a.n_rgba; i += step) a.rgba[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    // (one wave per tile, its lanes taking the tile's items in turn: a tile can hold thousands
    // of items when a whole groom falls into a few tiles)
    const int lane = threadIdx.x & 63;
    for (int t = (int)(i0 >> 6); t < T; t += (int)(step >> 6)) {
        const uint32_t b = a.item_start[t], e = min(a.item_start[t + 1], a.cap_items);
        for (uint32_t i = b + lane; i < e; i += 64) a.item_tab[i] = make_uint2((uint32_t)t, i - b);
    }
}

// The blocks b < nb append their segments; every block (more are launched where the image is large
// for its segments) then does its share of fill_frame, which saves a launch.
template <int LANES>
__global__ __launch_bounds__(kBinThreads) void k_scatter(const SegRec* __restrict__ seg, int nseg, int per_block,
                                                         int nb, int ntx, int nty, int t0, int nt,
                                                         const uint32_t* __restrict__ tile_start,
                                                         const uint32_t* __restrict__ M, uint32_t* __restrict__ list,
                                                         const Counters* __restrict__ ctr, FillArgs fill) {
    extern __shared__ uint32_t s_tc[];
    const int T = ntx * nty;
    if (t0 == 0) fill_frame(fill, T);
    if (ctr->cap_overflow || (int)blockIdx.x >= nb) return;
    const uint32_t* row = M + (size_t)blockIdx.x * T + t0;
    for (int i = threadIdx.x; i < nt; i += kBinThreads) s_tc[i] = tile_start[t0 + i] + row[i];
    __syncthreads();
    const int g0 = blockIdx.x * per_block, g1 = min(nseg, g0 + per_block);
    for (int g = g0 + (int)threadIdx.x / LANES; g < g1; g += kBinThreads / LANES)
        for_each_tile_in_range(seg[g], ntx, nty, t0, nt, (int)threadIdx.x % LANES, LANES,
                               [&](int l) { list[atomicAdd(&s_tc[l], 1u)] = (uint32_t)g; });
}

// The frame's sizes against the buffers' capacities (one thread).
__global__ void k_check_caps(FrameBufs f, FrameCaps caps, int stage) {
    if (threadIdx.x != 0) return;
    uint32_t over = 0;
    if (stage == 1) {
        const uint32_t pairs = f.tile_start[f.T], items = f.item_start[f.T];
        f.ctr->sizes[0] = pairs;
        f.ctr->sizes[1] = items;
        over = (pairs > caps.pairs) || (items > caps.items);
        f.ctr->hides = opaque_pays(f.ctr->area_opaque, f.ctr->area_all, f.ctr->tiles);
    } else {
        const uint32_t frags = f.frag_base[f.T], batches = f.batch_start[f.T];
        f.ctr->sizes[2] = frags;
        f.ctr->sizes[3] = batches;
        over = (frags > caps.frags) || (batches > caps.batches);
    }
    if (over) f.ctr->cap_overflow = 1u;
}

__global__ void k_fill_u32(uint32_t* p, uint32_t v, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}
__global__ void k_fill_f32(float* p, float v, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}
// Three arrays copied (src set) or cleared in one launch: a fitting step's parameters and gradients
// are small, and each copy or clear of its own costs the host and the stream more than its bytes.
__global__ void k_set3(Arrays3 a) {
    const size_t i0 = blockIdx.x * (size_t)blockDim.x + threadIdx.x, step = (size_t)gridDim.x * blockDim.x;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        for (size_t i = i0; i < a.n[k]; i += step) a.dst[k][i] = a.src[k] ? a.src[k][i] : 0.0f;
}

// ---------------------------------------------------------------------------------------
// Coverage: every fragment of a tile's segments, with the work shared across a wave.  A
// segment's pixels are taken one line at a time along its major axis (rows when |dy| >= |dx|,
// else columns; u names the major axis, v the minor one), and the lanes of a wave share out all
// its (segment, line) pairs, 64 per round, so that a wave does not run as long as its longest
// segment.  On a line the covered pixels are exactly those of the segment's box (widened by the
// radius, clipped to the tile and the image) whose centre passes the integer predicate
// 0 <= t_num < t_den and cross^2 < R^2 t_den.  Along a line both t_num and cross are linear in
// the minor index (steps 16 dv and 16 du per pixel; t_num and |cross| are symmetric under the
// exchange of x and y, so one predicate serves both orientations), so each condition holds on
// an interval of the minor index, and the line's fragments are the intersection of three
// intervals: no candidate is tested one by one.
//
// 32-bit integers are exact here: endpoints lie inside the guard band, |dx|, |dy| <= kMaxAxis
// (longer segments are drawn as pieces), the radius is <= kMaxHwFx + 8 and every pixel centre
// of the widened box lies within kMaxAxis + kMaxHwFx + 24 < 2^16 sub-pixels of the first
// endpoint on each axis, so each product e dv, e du is below 2^30 and t_num, cross are below
// 2^31 (the products take the 24-bit multiplier: operands below 2^23); s_max < 2^30 and
// t_den < 2^30.  cross^2 < R^2 t_den is decided as |cross| <= s_max =
// floor(sqrt(R^2 t_den - 1)), found per segment in 64-bit integers.  x >> 4 is floor(x / 16).
//
// The interval ends are floor divisions n / d with d = 16 |du| or 16 |dv| (<= 2^18), exact:
// only quotients in [-17, 17] matter (a line has at most 16 pixels in a tile), and there n is
// below 2^23 in magnitude, so float(n) is exact; q = floor(n / d - 2^-16) from the hardware
// reciprocal is then floor(n / d) or one less (the reciprocal and the fused multiply-add err by
// under 3e-6 on quotients of that size, less than the 2^-16 bias), and one exact integer test,
// (q + 1) d <= n, settles it.  Quotients beyond [-17, 17] are clamped to +-17 before the test
// and stay on their side.
struct CovSetup {
    int4 g0;     // (c0, t0, dc, dt): cross and t_num at the box's first minor pixel of line l = 0
                 // and their steps per line, each sign-normalised (c by the sign of du, t by
                 // that of dv) so that both grow with the minor index at 16 |du| and 16 |dv|
    int4 g1;     // (s_max, lo, hi, first line - lines before this lane in the wave): the slab
                 // lo <= t <= hi is 0 <= t_num <= t_den - 1 after the sign normalisation
    float4 g2;   // (1 / (16 |du|), 1 / max(16 |dv|, 1), bits of 16 |du|,
                 //  bits of 16 |dv| | first pixel (8 bits) << 19 | last minor offset (4 bits) << 27 | steep << 31)
};

constexpr int kCovLinesPerWave = 64 * kTile;   // a segment has at most kTile lines in a tile

// The strip |cross| <= strip_vis holds every fragment whose coverage alpha is not exactly zero
// (delta < hw + 1/2; the integer radius ceil(16 hw) + 8 reaches up to 1/16 px further), and
// |cross| <= strip_opaque only fragments whose alpha is exactly 1 (delta <= hw - 1/2 - 2^-6;
// negative where the segment has none).  Both are float estimates with their error (a few
// 2^-24 relative) on the safe side.
__device__ inline int strip_vis(float hw, int tden, int smax) {
    const float s = (hw + 0.5f) * 16.0f * __builtin_amdgcn_sqrtf((float)tden) * (1.0f + 0x1p-18f) + 1.0f;
    return min((int)fminf(s, 2147483520.0f), smax);   // (the largest float below 2^31)
}
__device__ inline int strip_opaque(float hw, int tden) {
    const float w = hw - 0.5f - kOpaqueMargin;
    return w > 0.0f ? (int)fminf(w * 16.0f * __builtin_amdgcn_sqrtf((float)tden), 1073741824.0f) : -1;
}
// The smallest depth key a segment's fragments can have (its nearer end; 8 ulps of slack for the
// rounding of the interpolation between the ends).
__device__ inline uint32_t nearest_key(const float4 iz) {
    return 0xFFFFFFFFu - __float_as_uint(fmaxf(iz.x, iz.y)) - 8u;
}
__device__ inline uint32_t nearest_key(const SegRec& s) { return nearest_key(make_float4(s.iza, s.izb, 0.0f, 0.0f)); }

// floor(n / d) for 1 <= d <= 2^18 where it lies in [-17, 17]; a quotient beyond that range
// comes back beyond [-17, 16] on its own side.  rd: the hardware reciprocal of d.
__device__ inline int floordiv_small(int n, int d, float rd) {
    float qf = floorf(fmaf((float)n, rd, -0x1p-16f));
    qf = fminf(fmaxf(qf, -17.0f), 17.0f);
    const int q = (int)qf;
    return q + ((__mul24(q, d) + d <= n) ? 1 : 0);
}

// Stages lane t's segment (valid: the lane holds one) in s_cov[t], numbers the wave's lines
// and records each line's lane in s_own (kCovLinesPerWave bytes per wave); returns the wave's
// line count.  Ends with a block barrier (all threads must call it).  BOUND: the strip whose
// pixels are enumerated: every fragment (kAll), those with coverage (kVisible) or the opaque
// ones (kOpaque).
// drop(i0, i1, j0, j1): the segment's box in the tile (pixel columns and rows); true leaves it out.
enum CovBound { kAll, kVisible, kOpaque };
struct KeepAll {
    __device__ bool operator()(int, int, int, int) const { return false; }
};
template <CovBound BOUND, class D = KeepAll>
__device__ inline uint32_t cov_setup(const SegRec& s, bool valid, int px0, int py0, int W, int H, CovSetup* s_cov,
                                     uint8_t* s_own, D&& drop = D{}) {
    const int t = threadIdx.x, lane = t & 63;
    uint32_t nl = 0;
    CovSetup c{};
    if (valid) {
        const int dx = s.xb - s.xa, dy = s.yb - s.ya;
        const int tden = dx * dx + dy * dy;
        const int R = (s.hwfx & kHwMask) + 8;
        int sm = -1, i0 = 0, i1 = -1, j0 = 0, j1 = -1;
        if (tden > 0) {
            sm = BOUND == kOpaque ? strip_opaque(s.hw, tden) : strip_smax(R, tden);
            if (BOUND == kVisible) sm = strip_vis(s.hw, tden, sm);
            // the footprint's own box: across the segment it reaches sm / sqrt(t_den), which adds
            // sm |dy| / t_den along x and sm |dx| / t_den along y (rounded up; at most the radius)
            const float il = __builtin_amdgcn_rcpf((float)tden) * (float)sm;
            const int rx = min(R, (int)((float)abs(dy) * il) + 2), ry = min(R, (int)((float)abs(dx) * il) + 2);
            i0 = max(px0, ((min(s.xa, s.xb) - rx - 8) >> 4) + 1);
            i1 = min(min(px0 + kTile, W) - 1, ((max(s.xa, s.xb) + rx - 8 + 15) >> 4) - 1);
            j0 = max(py0, ((min(s.ya, s.yb) - ry - 8) >> 4) + 1);
            j1 = min(min(py0 + kTile, H) - 1, ((max(s.ya, s.yb) + ry - 8 + 15) >> 4) - 1);
        }
        if (sm >= 0 && i0 <= i1 && j0 <= j1 && !drop(i0 - px0, i1 - px0, j0 - py0, j1 - py0)) {
            const bool steep = abs(dy) >= abs(dx);
            const int au = steep ? s.ya : s.xa, av = steep ? s.xa : s.ya;
            const int du = steep ? dy : dx, dv = steep ? dx : dy;
            nl = (uint32_t)(steep ? j1 - j0 + 1 : i1 - i0 + 1);
            const int vmin = steep ? i0 : j0, vmax = steep ? i1 : j1;
            const int u0 = steep ? j0 : i0;
            const int eu = 16 * u0 + 8 - au, ev = 16 * vmin + 8 - av;
            const int tn = __mul24(ev, dv) + __mul24(eu, du);   // t_num at (u0, vmin)
            const int cr = __mul24(ev, du) - __mul24(eu, dv);   // cross at (u0, vmin)
            // per line eu grows by 16: t_num by 16 du, cross by -16 dv
            const int sgu = du < 0 ? -1 : 1, sgv = dv < 0 ? -1 : 1;
            const int B = 16 * abs(du), A = 16 * abs(dv);
            const int lu = u0 - (steep ? py0 : px0), lv = vmin - (steep ? px0 : py0);   // 0..15
            const int pix0 = steep ? lu * kTile + lv : lv * kTile + lu;
            c.g0 = make_int4(sgu * cr, sgv * tn, -16 * sgu * dv, 16 * sgv * du);
            c.g1 = make_int4(sm, dv < 0 ? 1 - tden : 0, dv < 0 ? 0 : tden - 1, 0);
            c.g2 = make_float4(__builtin_amdgcn_rcpf((float)B), __builtin_amdgcn_rcpf((float)max(A, 1)),
                               __int_as_float(B),
                               __int_as_float(A | pix0 << 19 | (vmax - vmin) << 27 | (steep ? (int)0x80000000u : 0)));
        }
    }
    uint32_t x = nl;
    x = wave_inclusive_sum(x);
    const uint32_t excl = x - nl;
    c.g1.w = -(int)excl;     // line index = g1.w + the wave-wide line number
    s_cov[t] = c;
    uint8_t* own = s_own + (t >> 6) * kCovLinesPerWave;
    for (uint32_t r = 0; r < nl; ++r) own[excl + r] = (uint8_t)lane;
    const uint32_t total = __shfl(x, 63);
    __syncthreads();
    return total;
}

// Calls f(p, tnum, tden, owner, cross) for every fragment of the wave's segments in this tile
// (p: the pixel's index in the tile; owner: the block thread whose segment it is; cross up to
// its sign).  total and the staging from cov_setup.  line(owner, p, n, steep) sees each line first
// (its first pixel and number of pixels, along the row when steep, else along the column) and may
// take it whole by returning true.
template <class F, class L>
__device__ inline void wave_coverage(const CovSetup* s_cov, const uint8_t* s_own, uint32_t total, F&& f, L&& line) {
    const int t = threadIdx.x, lane = t & 63, wbase = t & ~63;
    const uint8_t* own = s_own + (t >> 6) * kCovLinesPerWave;
    for (uint32_t g = (uint32_t)lane; g < total; g += 64) {
        const int o = wbase + own[g];
        const CovSetup c = s_cov[o];
        const int l = c.g1.w + (int)g;                       // line within the box, 0..15
        const int cl = c.g0.x + __mul24(l, c.g0.z);          // at the box's first minor pixel
        const int tl = c.g0.y + __mul24(l, c.g0.w);
        const int smax = c.g1.x, lo = c.g1.y, hi = c.g1.z;
        const int B = __float_as_int(c.g2.z);
        const int bits = __float_as_int(c.g2.w);
        const int A = bits & 0x7FFFF;
        // strip: -s_max <= cl + x B <= s_max; slab: lo <= tl + x A <= hi.  Values that leave
        // a condition false on all of x = 0..15 are clamped to just beyond that range first, so
        // that the numerators stay below 2^31.
        const int m = smax + 16 * B;
        const int cc = min(max(cl, -m), m);
        int x0 = max(0, -floordiv_small(smax + cc, B, c.g2.x));
        int x1 = min((bits >> 27) & 15, floordiv_small(smax - cc, B, c.g2.x));
        if (A > 0) {
            const int tc = min(max(tl, lo - 16 * A), hi + 1);
            x0 = max(x0, -floordiv_small(tc - lo, A, c.g2.y));
            x1 = min(x1, floordiv_small(hi - tc, A, c.g2.y));
        } else if (tl < lo || tl > hi) {
            x1 = -1;
        }
        if (x0 > x1) continue;
        const int tden = hi - lo + 1;
        const int sv = bits < 0 ? 1 : kTile;                  // pixel step along the minor axis
        int p = ((bits >> 19) & 0xFF) + __mul24(l, bits < 0 ? kTile : 1) + __mul24(x0, sv);
        if (line(o, p, x1 - x0 + 1, bits < 0)) continue;
        // t_num itself: the normalised t times the sign of dv (lo < 0 exactly when dv < 0, as
        // then t_den >= 2)
        const int sgn = lo < 0 ? -1 : 1;
        int tnum = sgn * (tl + __mul24(x0, A));
        const int tstep = sgn * A;
        int cr = cl + __mul24(x0, B);
        for (int xx = x0; xx <= x1; ++xx, p += sv, tnum += tstep, cr += B) f(p, tnum, tden, o, cr);
    }
}

// a / b, correctly rounded, from the correctly rounded reciprocal rb of a divisor that many
// fragments share (Markstein: a quotient within one ulp, which the first correction gives, and one
// more step with the exact remainder): 5 instructions instead of the general division's 11.  The
// steps need a finite quotient (an infinite one comes out NaN), so rb = 0, a divisor outside
// [2^-60, 2^60], takes the general one: no scene is 2^67 across, squared lengths overflow first.
__device__ inline float div_rcp(float a, float b, float rb) {
    float q = a * rb;
    q = __builtin_fmaf(__builtin_fmaf(-q, b, a), rb, q);
    return __builtin_fmaf(__builtin_fmaf(-q, b, a), rb, q);
}
__device__ inline float div_by(float a, float b, float rb) { return rb == 0.0f ? a / b : div_rcp(a, b, rb); }

// A fragment's depth key: its inverse depth, affine on screen, as descending float bits.  rtd: 1 / t_den
// correctly rounded (once per segment; the quotient is that of the plain division).
__device__ inline uint32_t depth_key_iz(float iza, float izb, int tnum, int tden, float rtd) {
    const float t = div_rcp((float)tnum, (float)tden, rtd);
    const float iz = iza + t * (izb - iza);
    return 0xFFFFFFFFu - __float_as_uint(iz);
}
// What the passes that need keys stage of a segment: (izA, izB, 1 / t_den, 0)
__device__ inline float4 key_inputs(const SegRec& s) {
    const int dx = s.xb - s.xa, dy = s.yb - s.ya;
    return make_float4(s.iza, s.izb, 1.0f / (float)(dx * dx + dy * dy), 0.0f);
}

// A cheap upper bound of a fragment's inverse depth, for the tests against the opaque keys: the
// reciprocal product in place of the division errs by under 2^-21 of the nearer end, and the bound
// adds 2^-20 of it.  Most fragments of a stack of thick hairs lie clearly behind and need no more.
__device__ inline float iz_bound(const float4 iz, int tnum) {
    const float t = (float)tnum * iz.z;
    return (iz.x + t * (iz.y - iz.x)) + fmaxf(iz.x, iz.y) * 0x1p-20f;
}
// The inverse depth of an opaque key (0 for none: nothing lies behind it).
__device__ inline float iz_of_key(uint32_t key) { return __uint_as_float(0xFFFFFFFFu - key); }

// The global segment id of a fragment record's second word (see FrameBufs::gid): the record
// holds it, or the index of the segment in the tile's list.
__device__ inline uint32_t seg_of(uint32_t y, const uint32_t* list, bool gid) {
    return gid ? (y & 0xFFFFFFu) : list[y & 0xFFFFFFu];
}

struct ShadeArgs {
    CamConst cam;
    LightsConst lights;
    MatConst mat;
    const SegRec* seg;
    const ShadeRec* shade;
};

// Deep opacity map lookup (the shadow pass's count of hairs in front of a point toward a
// light).  Both helpers round every operation once, in this order, so the lookup position and
// its texel weights are the ones the integer raster parameter fixes (fragment's point on the
// centre line: t from the integer parameter, perspective-correct t_w, x = pA + t_w (pB - pA)).
__device__ inline void dom_point(const SegRec& s, const float4& q0, const float4& q1, int tnum, int tden, float& x,
                                 float& y, float& z) {
    const float t = (float)tnum / (float)tden;
    const float iz = s.iza + t * (s.izb - s.iza);
    const float tw = (t * s.izb) / iz;
    x = q0.x + tw * (q1.x - q0.x);
    y = q0.y + tw * (q1.y - q0.y);
    z = q0.z + tw * (q1.z - q0.z);
}

// delta = |cross| / (16 sqrt(t_den)), the pixel centre's distance from the centre line in pixels,
// in double: the hardware reciprocal square root refined by one Newton step (relative error
// near 2^-46).
__device__ inline double delta_d(int cr, int tden) {
    const double x = (double)tden;
    double r = __builtin_amdgcn_rsq(x);
    const double hx = 0.5 * x * r;
    r = fma(r, fma(-hx, r, 0.5), r);
    return fabs((double)cr) * r * 0.0625;
}

// A strand's coverage alpha = min(hw + delta, 1/2) - max(delta - hw, -1/2), clamped to [0, 1]:
// at an edge pixel of low coverage it is a small difference of numbers near 1/2, so it is
// evaluated in double and rounded to float once, and its relative error stays at float
// precision however small the coverage.
__device__ inline float strand_alpha(int cr, int tden, float hw, float& delta) {
    const double dd = delta_d(cr, tden);
    delta = (float)dd;
    const double h = (double)hw;
    return (float)fmin(fmax(fmin(h + dd, 0.5) - fmax(dd - h, -0.5), 0.0), 1.0);
}

// Hairs in front of (x, y, z): per texel, x_l = (iz0 - iz) / delta - 1 layers behind the first
// hit (one layer of bias), C_{j-1} + (x_l - j)(C_j - C_{j-1}) inside layer j, C_{K-1} beyond;
// bilinear over the four nearest texel centres; outside the grid or on empty texels 0.
// Bound by VALU issue with the rest of the shading: of a texel's eight floats (iz0, C_0 .. C_6) only
// iz0 and the two that bound the layer are loaded (at the layer's address, not selected from all
// eight), the four texels' loads are issued together, and the quotients share their divisors (100k
// strands at 1080p: k_batch 1375 -> 1365 us).
__device__ inline float dom_count(const DomView& dv, float x, float y, float z) {
    const DomGrid& g = *dv.grid;
    const float u = dot_e(g.b.e1, x, y, z), v = dot_e(g.b.e2, x, y, z);
    const float izp = g.z_ref - dot_e(g.b.d, x, y, z);
    const float Tx = div_by(u - g.u0, g.s, g.rs) - 0.5f, Ty = div_by(v - g.v0, g.s, g.rs) - 0.5f;
    const float i0f = floorf(Tx), j0f = floorf(Ty);
    const float fx = Tx - i0f, fy = Ty - j0f;
    const int i0 = (int)i0f, j0 = (int)j0f;
    const float* texel[4];
    float iz0[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int i = i0 + (c & 1), j = j0 + (c >> 1);
        const bool in = i >= 0 && j >= 0 && i < g.R && j < g.R;
        texel[c] = reinterpret_cast<const float*>(dv.tex) + (in ? 8 * ((size_t)j * g.R + i) : 0);
        const float A = *texel[c];
        iz0[c] = in ? A : 0.0f;
    }
    float n = 0.0f;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float xl = div_by(iz0[c] - izp, dv.delta, dv.rdelta) - 1.0f;
        if (!(iz0[c] > 0.0f) || !(xl >= 0.0f)) continue;
        // C_{j-1} and C_j lie at floats j and j + 1, the last pair (j = K) at K - 1 and K
        const int jl = (int)fminf(floorf(xl), (float)dv.K), jr = min(jl, dv.K - 1);
        const float lo = texel[c][jr], Cj = texel[c][jr + 1];
        const float Cp = jl == 0 ? 0.0f : lo;
        const float val = jl == jr ? Cp + (xl - (float)jl) * (Cj - Cp) : Cj;
        const float w = ((c & 1) ? fx : 1.0f - fx) * ((c >> 1) ? fy : 1.0f - fy);
        n += w * val;
    }
    return n;
}

// Radiance (RGB), coverage alpha and cross-section offset h of one fragment, written once over
// the scalar type T: float for rendering, Dual<N> for the backward pass.  T carries the
// fitted parameters (half-width hw, semi-axes |a|, |b|, hair radius r, absorption); the view
// geometry (frame, angles) does not depend on them and stays float.
template <int KIND, int MODEL, class T, bool SHADOW = false>
__device__ inline void shade_core(const ShadeArgs& a, const SegRec& s, const float4& q0, const float4& q1,
                                  const float4& q2, float n_total, int pxg, int pyg, const T& hw, const T& a_len,
                                  const T& b_len, const T& rr, const T sig[3], T& alpha, T& hoff, T L[3]) {
#pragma clang fp contract(fast)
    // integer coverage geometry; 32 bits suffice because a covered pixel centre lies within
    // the segment's box widened by its radius and longer segments (kMaxAxis) are culled
    const int ex = 16 * pxg + 8 - s.xa, ey = 16 * pyg + 8 - s.ya;
    const int dx = s.xb - s.xa, dy = s.yb - s.ya;
    const int tnum = ex * dx + ey * dy, tden = dx * dx + dy * dy;
    const int cr = ex * dy - ey * dx;
    // (the coverage decision was taken exactly when the fragment was emitted; what follows is
    // continuous, so it uses the hardware reciprocal and reciprocal square root)
    float delta;
    if constexpr (KIND == 1) {
        // a thick hair is many pixels wide, so at its footprint's edge alpha = 1/2 - (delta - hw)
        // is a small difference of large numbers; delta is carried as a float pair (hi + lo) from
        // a double evaluation, and hi - hw is exact there (Sterbenz), which keeps alpha's
        // absolute error at the level of a strand's instead of an ulp of the hair width
        const double dd = delta_d(cr, tden);
        delta = (float)dd;
        const float dlo = (float)(dd - (double)delta);
        const T d_minus = (delta - hw) + dlo, d_plus = (hw + delta) + dlo;
        alpha = m_min(m_max(m_min(d_plus, T(0.5f)) - m_max(d_minus, T(-0.5f)), T(0.0f)), T(1.0f));
    } else {
        alpha = strand_alpha(cr, tden, hw, delta);
    }
    float sgn = cr > 0 ? 1.0f : (cr < 0 ? -1.0f : 0.0f);
    if (s.hwfx & kFlagNegSide) sgn = -sgn;
    const T h = m_min(m_max((sgn * delta) * m_rcp(hw + 0.5f), T(-1.0f)), T(1.0f));
    hoff = h;
    // the world parameter of the fragment's screen parameter t = t_num / t_den: inverse depth is
    // affine on screen, so t_w = t izB / (izA + t (izB - izA)), here with t_den cleared
    const float ftn = (float)tnum;
    const float tw = ftn * s.izb * m_rcp((float)tden * s.iza + ftn * (s.izb - s.iza));

    // fibre frame at the fragment's world point
    const V3<float> pA = v3(q0.x, q0.y, q0.z);
    const V3<float> d = sub(v3(q1.x, q1.y, q1.z), pA);
    const V3<float> u = scale(d, m_rsqrt(dot(d, d)));
    const V3<float> xw = v3(pA.x + tw * d.x, pA.y + tw * d.y, pA.z + tw * d.z);
    V3<float> wo = sub(v3(a.cam.pos[0], a.cam.pos[1], a.cam.pos[2]), xw);
    wo = scale(wo, m_rsqrt(dot(wo, wo)));
    const float dwu = dot(wo, u);
    V3<float> wp = sub(wo, scale(u, dwu));
    float wpn2 = dot(wp, wp);
    // the longitudinal angle from both of its legs: atan2(sin, |w_perp|) stays accurate where
    // asin(sin) loses digits (views and lights close to the fibre axis, where the narrow
    // longitudinal lobes are most sensitive to theta)
    float r_wp = m_rsqrt(wpn2);
    const float cos_to = wpn2 > 0.0f ? wpn2 * r_wp : 0.0f;   // |w_perp|
    const bool degen = wpn2 < 1e-14f;
    if (degen) {  // view along the fibre: any normal direction; phi is set to 0
        const float ax = fabsf(u.x), ay = fabsf(u.y), az = fabsf(u.z);
        V3<float> e = (ax <= ay && ax <= az) ? v3(1.f, 0.f, 0.f) : (ay <= az ? v3(0.f, 1.f, 0.f) : v3(0.f, 0.f, 1.f));
        wp = sub(e, scale(u, dot(e, u)));
        wpn2 = dot(wp, wp);
        r_wp = m_rsqrt(wpn2);
    }
    const V3<float> xh = scale(wp, r_wp);
    const V3<float> yh = cross(u, xh);
    const float sin_to = fminf(fmaxf(dwu, -1.0f), 1.0f);
    const T gamma_o = m_asin(h);
    const T cgo = m_sqrt((1.0f - h) * (1.0f + h));
    const T sigl[3] = {sig[0] * kLog2e, sig[1] * kLog2e, sig[2] * kLog2e};

    ClusterFrag<T> cf;
    T W, ia, ib;
    V3<float> ah{}, bh{};
    if (KIND == 1) {
        ah = v3(q2.x, q2.y, q2.z);
        bh = cross(u, ah);
        const T pa = a_len * dot(ah, yh), pb = b_len * dot(bh, yh);
        W = m_sqrt(pa * pa + pb * pb);
        ia = m_rcp(a_len);
        ib = m_rcp(b_len);
        cf.n_total = T(n_total);
        cf.rho = m_min(m_max(n_total * rr * rr * (ia * ib), T(0.0f)), T(1.0f));
    }
    float dpx = 0.f, dpy = 0.f, dpz = 0.f;
    if (SHADOW) dom_point(s, q0, q1, tnum, tden, dpx, dpy, dpz);
    L[0] = L[1] = L[2] = T(0.0f);
    for (int li = 0; li < a.lights.n; ++li) {
        const LightConst& lc = a.lights.l[li];
        V3<float> wi;
        float E[3];
        if (lc.kind == 0) {
            wi = v3(lc.vec[0], lc.vec[1], lc.vec[2]);
            E[0] = lc.rgb[0]; E[1] = lc.rgb[1]; E[2] = lc.rgb[2];
        } else {
            const V3<float> dl = sub(v3(lc.vec[0], lc.vec[1], lc.vec[2]), xw);
            const float inv = m_rsqrt(dot(dl, dl));
            wi = scale(dl, inv);
            const float i2 = inv * inv;
            E[0] = lc.rgb[0] * i2; E[1] = lc.rgb[1] * i2; E[2] = lc.rgb[2] * i2;
        }
        const float sin_ti = dot(wi, u);
        const LightView v = light_view(sin_ti, sin_to, cos_to, dot(wi, xh), dot(wi, yh), degen, a.mat);
        // hairs between the light and this fragment (shadow pass), added to the forward count
        const float ns = (SHADOW && a.lights.dom[li].grid) ? dom_count(a.lights.dom[li], dpx, dpy, dpz) : 0.0f;
        T f[3];
        if (KIND == 0 && SHADOW && ns > 0.0f) {
            ClusterFrag<T> c1;
            c1.n_total = T(1.0f);
            c1.rho = T(1.0f);
            c1.n_F = T(1.0f + ns);
            c1.n_B = T(1.0f);
            if (MODEL == 0)
                f_ours(v, h, gamma_o, cgo, sigl, a.mat, c1, f);
            else
                f_ours_rttd(v, a.mat, c1, f);
        } else if (KIND == 0) {
            if (MODEL == 0)
                f_single(v, h, gamma_o, cgo, sigl, a.mat, f);
            else
                f_single_rttd(v, a.mat, f);
        } else {
            // chord of the view ray's entry point toward the light, in the cross-section
            const V3<float> Dp = sub(wi, scale(u, sin_ti));
            const float dn2 = dot(Dp, Dp);
            T s_star(0.0f);
            if (dn2 > 1e-14f) {
                const V3<float> D = scale(Dp, m_rsqrt(dn2));
                const T oa = h * W * dot(yh, ah) * ia, ob = h * W * dot(yh, bh) * ib;
                const T xa = dot(xh, ah) * ia, xb = dot(xh, bh) * ib;
                const T qa = xa * xa + xb * xb, qb = oa * xa + ob * xb, qc = oa * oa + ob * ob - 1.0f;
                const T disc = m_max(qb * qb - qa * qc, T(0.0f));
                const T tt = (qb - m_sqrt(disc)) * m_rcp(qa);
                const T Pa = oa - tt * xa, Pb = ob - tt * xb;
                const T Da = dot(D, ah) * ia, Db = dot(D, bh) * ib;
                s_star = -2.0f * (Pa * Da + Pb * Db) * m_rcp(Da * Da + Db * Db);
            }
            const T kappa = m_sqrt(n_total * (1.0f / kPi) * (ia * ib));
            const T lF = m_max(s_star, T(0.0f)), lB = m_max(-s_star, T(0.0f));
            const bool back = fabsf(v.phi) < 0.25f;
            cf.n_F = (back || n_total < 2.0f) ? T(1.0f) : m_max(cf.rho * kappa * lF, T(1.0f));
            cf.n_B = m_max(cf.rho * kappa * lB, T(1.0f));
            if (SHADOW) cf.n_F = cf.n_F + ns;
            if (MODEL == 0)
                f_ours(v, h, gamma_o, cgo, sigl, a.mat, cf, f);
            else
                f_ours_rttd(v, a.mat, cf, f);
        }
        L[0] = L[0] + (E[0] * v.cos_ti) * f[0];
        L[1] = L[1] + (E[1] * v.cos_ti) * f[1];
        L[2] = L[2] + (E[2] * v.cos_ti) * f[2];
    }
}

// KIND 0: strands, 1: thick hairs, 2: a mixed frame (the segment's flag decides).
// MODEL 0: near-field R / TT / TRT, 1: R / TT / D.
// A fragment's segment inputs (integer record and shading record), fetched ahead of use.
struct SegInputs {
    SegRec s;
    float4 q0, q1, q2, q3;
};

// KIND 0 (a strand-level frame) reads the packed strand record alone; the others read the
// screen record and the ShadeRec.
template <int KIND>
__device__ inline SegInputs fetch_segment(const ShadeArgs& a, uint32_t gseg) {
    SegInputs r;
    const ShadeRec& sr = a.shade[gseg];
    if (KIND == 0) {
        const float4 p0 = sr.q0, p1 = sr.q1, p2 = sr.q2, p3 = sr.q3;
        r.s.xa = __float_as_int(p0.x);
        r.s.ya = __float_as_int(p0.y);
        r.s.xb = __float_as_int(p0.z);
        r.s.yb = __float_as_int(p0.w);
        r.s.iza = p1.x;
        r.s.izb = p1.y;
        r.s.hw = fabsf(p1.z);
        r.s.hwfx = (__float_as_uint(p1.z) >> 31) ? kFlagNegSide : 0;
        r.q0 = make_float4(p1.w, p2.x, p2.y, p3.y);
        r.q1 = make_float4(p2.z, p2.w, p3.x, p3.z);
        r.q2 = make_float4(0.f, 0.f, 0.f, p3.w);
        r.q3 = make_float4(0.f, 0.f, 0.f, 0.f);
        return r;
    }
    r.s = a.seg[gseg];
    r.q0 = sr.q0;
    r.q1 = sr.q1;
    r.q2 = sr.q2;
    r.q3 = sr.q3;
    return r;
}

template <int KIND, int MODEL, bool SHADOW = false>
__device__ inline void shade_inputs(const ShadeArgs& a, const SegInputs& in, int pxg, int pyg, float& alpha,
                                    float& hoff, float L[3]) {
    const float sig[3] = {in.q0.w, in.q1.w, in.q2.w};
    if (KIND == 0 || KIND == 3 || (KIND == 2 && !(in.s.hwfx & kFlagThick))) {
        shade_core<0, MODEL, float, SHADOW>(a, in.s, in.q0, in.q1, in.q2, 1.0f, pxg, pyg, in.s.hw, 0.f, 0.f, 0.f, sig, alpha,
                                    hoff, L);
    } else {
        shade_core<1, MODEL, float, SHADOW>(a, in.s, in.q0, in.q1, in.q2, in.q3.z, pxg, pyg, in.s.hw, in.q3.x, in.q3.y, in.q3.w,
                                    sig, alpha, hoff, L);
    }
}

template <int KIND, int MODEL>
__device__ inline void shade_fragment(const ShadeArgs& a, uint32_t gseg, int pxg, int pyg, float& alpha, float& hoff,
                                      float L[3]) {
    shade_inputs<KIND, MODEL>(a, fetch_segment<KIND>(a, gseg), pxg, pyg, alpha, hoff, L);
}

// Block-wide exclusive scan of one uint per thread (256 threads); returns the total.
__device__ inline uint32_t block_exscan_u32(uint32_t v, uint32_t* s_tmp, uint32_t& excl) {
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    uint32_t x = v;
    x = wave_inclusive_sum(x);
    if (lane == 63) s_tmp[wv] = x;
    __syncthreads();
    uint32_t base = 0, total = 0;
#pragma unroll
    for (int w2 = 0; w2 < kNT / 64; ++w2) {
        const uint32_t a = s_tmp[w2];
        if (w2 < wv) base += a;
        total += a;
    }
    __syncthreads();
    excl = base + x - v;
    return total;
}

#ifdef HAIR_PHASE_STATS
#define PHASE_BEGIN() unsigned long long ph_t0 = wall_clock64()
// (the barrier here only makes the timing cover the whole block; correctness never relies on it)
#define PHASE_END(ctr, i)                                                      \
    do {                                                                       \
        __syncthreads();                                                       \
        if (threadIdx.x == 0) atomicAdd(&(ctr)->phase[i], wall_clock64() - ph_t0); \
        ph_t0 = wall_clock64();                                                \
    } while (0)
#define PHASE_RESET() ph_t0 = wall_clock64()
#define PHASE_ADD(ctr, i, v) do { if (threadIdx.x == 0) atomicAdd(&(ctr)->phase[i], (unsigned long long)(v)); } while (0)
#else
#define PHASE_BEGIN() do {} while (0)
#define PHASE_END(ctr, i) do {} while (0)
#define PHASE_RESET() do {} while (0)
#define PHASE_ADD(ctr, i, v) do {} while (0)
#endif

// Work items of the count and emit kernels: chunks of kNT consecutive entries of a tile list.
__global__ __launch_bounds__(256) void k_tile_items(const uint32_t* __restrict__ tile_start, int T,
                                                    uint32_t* __restrict__ items, Counters* ctr) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t n = t < T ? tile_start[t + 1] - tile_start[t] : 0u;
    const unsigned long long full = __ballot(n > 0u);
    if ((threadIdx.x & 63) == 0 && full) atomicAdd(&ctr->tiles, (uint32_t)__popcll(full));
    if (t < T) items[t] = (n + kNT - 1) / kNT;
}

// What is known to hide in a tile: each pixel's opaque key and the largest key of every run of four
// pixels along the rows and the columns, so that a segment or a line of one that lies behind all it
// could cover is recognised without a test per pixel.
struct HideLds {
    uint32_t z[kTilePix];
    uint4 row[kTile], col[kTile];   // [line]: its four runs
    uint4 cell[4];                  // [row of 4 x 4 cells]: its four cells
};
struct NoHide {   // (frames without an opaque pass)
    uint32_t z[1];
    uint4 row[1], col[1], cell[1];
};
template <bool ZC> using HideOf = std::conditional_t<ZC, HideLds, NoHide>;
// Sets h from the block's pixel keys z0 (0 for pixels off the image).  All threads call it; ends
// with a barrier.
__device__ inline void hide_setup(HideLds& h, uint32_t z0) {
    const int t = threadIdx.x;
    h.z[t] = z0;
    const uint32_t a = max(z0, (uint32_t)__shfl_xor((int)z0, 1));
    const uint32_t r = max(a, (uint32_t)__shfl_xor((int)a, 2));
    const uint32_t b = max(z0, (uint32_t)__shfl_xor((int)z0, 16));
    const uint32_t c = max(b, (uint32_t)__shfl_xor((int)b, 32));   // (a wave holds four rows)
    const uint32_t d = max(r, (uint32_t)__shfl_xor((int)r, 16));
    const uint32_t e = max(d, (uint32_t)__shfl_xor((int)d, 32));
    if ((t & 3) == 0) reinterpret_cast<uint32_t*>(h.row)[t >> 2] = r;
    if ((t & 63) < 16) reinterpret_cast<uint32_t*>(h.col)[4 * (t & 15) + (t >> 6)] = c;
    if ((t & 0x33) == 0) reinterpret_cast<uint32_t*>(h.cell)[4 * (t >> 6) + ((t >> 2) & 3)] = e;
    __syncthreads();
}
// The largest of a line's four runs (or cells) that its pixels [a, b] touch.
__device__ inline uint32_t runs_max(const uint4 g, int a, int b) {
    uint32_t m = a < 4 ? g.x : 0u;
    m = max(m, a < 8 && b >= 4 ? g.y : 0u);
    m = max(m, a < 12 && b >= 8 ? g.z : 0u);
    return max(m, b >= 12 ? g.w : 0u);
}
// Whether a box of the tile's pixels lies behind all its cells, with nearest the smallest key its
// segment can have.
template <class H>
__device__ inline bool box_hidden(const H& h, uint32_t nearest, int i0, int i1, int j0, int j1) {
    uint32_t m = 0u;
    for (int r = j0 >> 2; r <= j1 >> 2; ++r) m = max(m, runs_max(h.cell[r], i0, i1));
    return nearest > m;
}
// Whether a line of n pixels from p (see wave_coverage) does.
template <class H>
__device__ inline bool line_hidden(const H& h, uint32_t nearest, int p, int n, bool steep) {
    const int a = steep ? p & 15 : p >> 4;
    return nearest > runs_max(steep ? h.row[p >> 4] : h.col[p & 15], a, a + n - 1);
}

// Opaque pass (frames that can hold thick hairs): per pixel the smallest depth key among its
// fragments of alpha exactly 1.  A fragment behind it (a larger key) composites with T = 0 and
// changes nothing, so the count and emit passes leave it out: the frame stores, orders and
// shades only what can be seen.  Only segments wider than a pixel have such fragments; frames
// without one skip the pass, and a segment that lies behind the keys already found for the
// whole tile (a stale read only costs work: keys fall, never rise) is skipped.  The keys live in
// pix_kmax, which the emit pass needs only later: a pixel with an opaque fragment stores it as
// its farthest one, so its key maximum is that key already, and k_tile_prep clears the others
// (see kmax_seen for how the emit pass tells them apart).
// 150k x 64 strands as 1000 thick hairs at 1080p: 99.7% of its 43 M fragments are hidden, and the
// frame takes 0.27 ms instead of 3.5 (this pass 0.06, the shading 0.03 instead of 1.97).  Mixed
// frames have the pass where opaque_pays says so: locks of 100k strands at a middle view, thick
// hairs up to 4 px wide, 78% of 12 M fragments hidden: 0.53 instead of 0.81 ms.  Bound by the
// per-line coverage arithmetic (VALU).
// first: only 4 kFirstLanes segments of every tile, spread over its list (a contiguous run of it
// would hold the segments of a few neighbouring hairs, which may lie at the back).  A block is
// bound by the latency of its lines' pixels, so this launch is short, and what it finds hides most
// segments of the second one, which takes them all: 43 M fragments in 5 k chunks, 119 -> 20 + 45 us.
constexpr int kFirstLanes = 16;
__device__ inline void opaque_item(const FrameBufs& f, const CamConst& cam, int first, uint32_t item) {
    __shared__ HideLds s_hide;
    __shared__ CovSetup s_cov[kNT];
    __shared__ uint8_t s_own[kNT / 64 * kCovLinesPerWave];
    __shared__ float4 s_iz[kNT];
    const int t = threadIdx.x;
    const uint2 it = f.item_tab[item];
    if (first && it.y > 0) return;
    const int tile = (int)it.x;
    const int px0 = (tile % f.ntx) * kTile, py0 = (tile / f.ntx) * kTile;
    const uint32_t lstart = f.tile_start[tile];
    const uint32_t n = f.tile_start[tile + 1] - lstart;
    const uint32_t j = first && n > (uint32_t)kNT ? (uint32_t)((unsigned long long)t * n / kNT) : it.y * kNT + t;
    SegRec s{};
    if (j < n) s = f.seg[f.list[lstart + j]];
    const size_t q = (size_t)tile * kTilePix + t;
    const int gx = px0 + (t % kTile), gy = py0 + (t / kTile);
    const uint32_t z0 = gx < cam.W && gy < cam.H ? f.pix_kmax[q] : 0u;
    hide_setup(s_hide, z0);
    uint32_t* s_z = s_hide.z;
    s_iz[t] = key_inputs(s);
    const bool valid = j < n && s.hw > 0.5f + kOpaqueMargin && (!first || (t & 63) % (64 / kFirstLanes) == 0);
    const uint32_t total = cov_setup<kOpaque>(
        s, valid, px0, py0, cam.W, cam.H, s_cov, s_own,
        [&](int i0, int i1, int j0, int j1) { return box_hidden(s_hide, nearest_key(s), i0, i1, j0, j1); });
    float4 iz;   // (the line's segment)
    wave_coverage(s_cov, s_own, total, [&](int p, int tnum, int tden, int, int) {
        const uint32_t z = s_z[p];
        if (iz_bound(iz, tnum) < iz_of_key(z)) return;
        const uint32_t key = depth_key_iz(iz.x, iz.y, tnum, tden, iz.z);
        if (key < z) atomicMin(&s_z[p], key);
    }, [&](int o, int p, int n, bool steep) {
        iz = s_iz[o];
        return line_hidden(s_hide, nearest_key(iz), p, n, steep);
    });
    __syncthreads();
    // (kmax_key: whatever the key, the count and emit passes take the same word for hiding)
    if (s_z[t] < z0) atomicMin(&f.pix_kmax[q], kmax_key(s_z[t]));
}
// An item per block, or (CHOICE: the device chose whether the frame has the pass, f.opaque == 2) several in
// turn, see launch_count.
template <bool CHOICE> __global__ __launch_bounds__(kNT) void k_opaque(FrameBufs f, CamConst cam, int first) {
    if (!(__uint_as_float(f.ctr->max_hw_bits) > 0.5f + kOpaqueMargin)) return;
    const uint32_t n_items = f.item_start[f.T];
    if (blockIdx.x >= n_items || f.ctr->cap_overflow) return;
    if constexpr (!CHOICE) {
        opaque_item(f, cam, first, xcd_contiguous(blockIdx.x, n_items));
    } else {
        if (!f.ctr->hides) return;
        for (uint32_t b = blockIdx.x; b < n_items; b += gridDim.x) {
            if (b != blockIdx.x) __syncthreads();
            opaque_item(f, cam, first, xcd_contiguous(b, n_items));
        }
    }
}

// Count pass: per pixel the fragments that the frame stores and, in pix_off until k_tile_prep
// writes the offsets, those it leaves out.  Each item adds its LDS-aggregated counts (stored in
// the low half word, left out in the high one: an item has at most kNT fragments per pixel) to
// the tile's pixels and keeps the returned base (its slice of every pixel's range).
// ZC: the frame has an opaque pass, and leaves out what an opaque fragment hides (see launch_count).
// TRIM: fragments without coverage are left out too (FrameBufs::trim).
// CHOICE: the device has chosen whether it has (f.opaque == 2).
template <bool TRIM, bool ZC, bool CHOICE>
__global__ __launch_bounds__(kNT) void k_count(FrameBufs f, CamConst cam) {
    __shared__ uint32_t s_cnt[kTilePix];
    __shared__ HideOf<ZC> s_hide[1];
    __shared__ uint32_t s_dr[ZC ? kTilePix : 1], s_dc[ZC ? kTilePix : 1];   // see below
    __shared__ float4 s_iz[ZC ? kNT : 1];
    __shared__ CovSetup s_cov[kNT];
    __shared__ int s_vis[TRIM ? kNT : 1];   // |cross| up to which the segment's fragments have coverage
    __shared__ uint8_t s_own[kNT / 64 * kCovLinesPerWave];
    PHASE_BEGIN();
    const uint32_t n_items = f.item_start[f.T];
    if (blockIdx.x >= n_items || f.ctr->cap_overflow) return;
    const bool hides = ZC && (!CHOICE || f.ctr->hides != 0);
    const uint32_t item = xcd_contiguous(blockIdx.x, n_items);
    const int t = threadIdx.x;
    const uint2 it = f.item_tab[item];
    const int tile = (int)it.x;
    s_cnt[t] = 0;
    const int px0 = (tile % f.ntx) * kTile, py0 = (tile / f.ntx) * kTile;
    const uint32_t lstart = f.tile_start[tile];
    const uint32_t n = f.tile_start[tile + 1] - lstart;
    const uint32_t j = it.y * kNT + t;
    SegRec s{};
    if (j < n) s = f.seg[f.list[lstart + j]];
    const size_t q = (size_t)tile * kTilePix + t;
    if constexpr (ZC) {
        if (hides) {
            s_dr[t] = s_dc[t] = 0u;
            s_iz[t] = key_inputs(s);
            const int gx = px0 + (t % kTile), gy = py0 + (t / kTile);
            hide_setup(s_hide[0], gx < cam.W && gy < cam.H ? f.pix_kmax[q] : 0u);
        }
    }
    if constexpr (TRIM) {
        const int dx = s.xb - s.xa, dy = s.yb - s.ya;
        s_vis[t] = strip_vis(s.hw, dx * dx + dy * dy, 0x7FFFFFFF);
    }
    const uint32_t total = cov_setup<kAll>(s, j < n, px0, py0, cam.W, cam.H, s_cov, s_own);
    float4 iz;   // (the line's segment)
    int vis = 0;
    wave_coverage(s_cov, s_own, total, [&](int p, int tnum, int tden, int, int cr) {
        bool stored = true;
        if constexpr (TRIM) stored = abs(cr) <= vis;
        if constexpr (ZC) {
            if (hides && stored) stored = depth_key_iz(iz.x, iz.y, tnum, tden, iz.z) <= s_hide[0].z[p];
        }
        atomicAdd(&s_cnt[p], stored ? 1u : 0x10000u);
    }, [&](int o, int p, int n, bool steep) {
        // a line hidden as a whole: its pixels are only counted, as differences along the line (+1
        // where it begins, -1 behind its end) that two row sums add up below
        if constexpr (TRIM) vis = s_vis[o];
        if (!hides) return false;
        if constexpr (ZC) iz = s_iz[o];
        if (!line_hidden(s_hide[0], nearest_key(iz), p, n, steep)) return false;
        uint32_t* d = steep ? s_dr : s_dc;
        const int i = steep ? p : ((p & 15) << 4 | p >> 4);   // (columns are kept transposed)
        atomicAdd(&d[ZC ? i : 0], 1u);
        if ((i & 15) + n < kTile) atomicSub(&d[ZC ? i + n : 0], 1u);
        return true;
    });
    __syncthreads();
    if (hides) {
        const uint32_t r = row_inclusive_sum(s_dr[t]), v = row_inclusive_sum(s_dc[t]);
        if (r) atomicAdd(&s_cnt[t], r << 16);
        if (v) atomicAdd(&s_cnt[(t & 15) << 4 | t >> 4], v << 16);
        __syncthreads();
    }
    uint32_t c = s_cnt[t];
    uint32_t base = 0;
    if (TRIM || ZC) {
        if (c >> 16) atomicAdd(&f.pix_off[q], c >> 16);
        c &= 0xFFFFu;
    }
    if (c) base = atomicAdd(&f.pix_cnt[q], c);
    f.item_base[(size_t)item * kTilePix + t] = base;
    PHASE_END(f.ctr, 0);
}

// The fragments a batch of a tile may take (a multiple of kNT, up to kCap).  A large frame fills
// the chip with full batches, which share their fixed cost (prologue, scans) over the most
// fragments; a small one, or a tile whose fragments fit one batch, is bound by a batch's length
// (each thread shades its run one fragment after the other), so its batches are cut short: down to
// one fragment per thread, and about 2048 batches a frame as estimated from its list entries (4
// fragments each).  Shading of 1k strands at 256 x 256: 17.8 -> 8.4 us; 10k at 720p 32 -> 26.5 us; the
// combed groom's far view 51 -> 23 us (47 k, 0.66 M and 0.16 M fragments).
__device__ inline uint32_t batch_cap(uint32_t tile_total, uint32_t pairs) {
    if (tile_total <= (uint32_t)kCap) return kNT;
    const uint32_t c = (pairs / (512u * kNT) + 1u) * kNT;
    return min(c, (uint32_t)kCap);
}

// Greedy batch packing of whole pixels: from p0 skip empty pixels, then take the longest run
// [p0, p1) whose fragments fit the tile's batch size (batch_cap); a pixel deeper than that forms a
// batch of its own (deeper than an LDS batch, kCap, it is "oversized").  Every lane finds, in parallel, the next non-empty pixel at or
// after it and the end of a batch that would start at it; the chain of batch starts is then
// followed (by one lane when it is short, by pointer doubling over all lanes when it is long)
// and marked in a 256-bit mask of the tile.  batch_records turns the mask
// into the batch table in parallel (a batch runs to the next start, or to the tile's end: the
// pixels in between are empty).
__global__ __launch_bounds__(kNT) void k_tile_prep(FrameBufs f) {
    __shared__ uint32_t s_off[kTilePix + 1], s_tmp[kNT];
    __shared__ uint16_t s_nxt[kTilePix + 1], s_end[kTilePix], s_jump[kTilePix + 1];
    __shared__ uint8_t s_on[kTilePix + 1];
    __shared__ uint32_t s_mask[kTilePix / 32];
    const int tile = blockIdx.x, t = threadIdx.x;
    if (f.item_start[tile] == f.item_start[tile + 1]) {   // (no segments: most tiles of most views)
        if (t < kTilePix / 32) f.batch_mask[(size_t)tile * (kTilePix / 32) + t] = 0u;
        if (t == 0) f.tile_all[tile] = f.tile_tot[tile] = f.tile_nb[tile] = 0u;
        return;
    }
    const size_t q = (size_t)tile * kTilePix + t;
    const uint32_t c = f.pix_cnt[q];
    // the pixels' offsets and, with those the count pass left out (its numbers in pix_off), all
    // fragments of the tile and its pixels deeper than a batch
    const uint32_t left = f.pix_off[q];
    const unsigned long long deep = __ballot(c + left > (uint32_t)kCap);
    const uint32_t cx = wave_inclusive_sum(c), lx = wave_inclusive_sum(left);
    if ((t & 63) == 63) {
        s_tmp[t >> 6] = cx;
        s_tmp[kNT / 64 + (t >> 6)] = lx;
    }
    __syncthreads();
    uint32_t ex = cx - c, total = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kNT / 64; ++w) {
        const uint32_t a = s_tmp[w];
        if (w < (t >> 6)) ex += a;
        total += a;
        all += s_tmp[kNT / 64 + w];
    }
    if (t == 0) f.tile_all[tile] = total + all;
    if ((t & 63) == 0 && deep) atomicAdd(&f.ctr->deep_pixels, (uint32_t)__popcll(deep));
    if (f.opaque && f.pix_kmax[q] == 0xFFFFFFFFu) f.pix_kmax[q] = 0u;
    s_off[t] = ex;
    f.pix_off[q] = ex;
    if (t == 0) s_off[kTilePix] = total;
    if (t < kTilePix / 32) s_mask[t] = 0u;
    __syncthreads();
    {   // next non-empty pixel q >= t: the smallest q with s_off[q + 1] > s_off[t]
        int lo = t, hi = kTilePix;
        const uint32_t o = s_off[t];
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (s_off[mid + 1] > o) hi = mid; else lo = mid + 1;
        }
        s_nxt[t] = (uint16_t)lo;
    }
    const uint32_t cap = f.full_batches ? (uint32_t)kCap : batch_cap(total, f.ctr->sizes[0]);
    if (c > cap) {
        s_end[t] = (uint16_t)(t + 1);
    } else {   // the largest p1 with s_off[p1] - s_off[t] <= cap
        int lo = t + 1, hi = kTilePix;
        const uint32_t o0 = s_off[t];
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_off[mid] - o0 <= cap) lo = mid; else hi = mid - 1;
        }
        s_end[t] = (uint16_t)lo;
    }
    if (t == 0) s_nxt[kTilePix] = (uint16_t)kTilePix;
    __syncthreads();
    if (total <= 16u * cap) {   // a short chain (at most ~32 batches): one lane follows it
        if (t == 0) {
            uint32_t nb = 0;
            for (int p = s_nxt[0]; p < kTilePix; p = s_nxt[s_end[p]]) {
                s_mask[p >> 5] |= 1u << (p & 31);
                ++nb;
            }
            f.tile_tot[tile] = total;
            f.tile_nb[tile] = nb;
        }
    } else {
        // a long chain: every pixel marks where its batch's successor starts, and the marks
        // spread from the first start by pointer doubling (after step k, every start within
        // 2^(k+1) batches of the first; a tile has at most kTilePix = 2^8 batches).  A mark
        // seen early only spreads further along the same chain.
        s_jump[t] = s_nxt[s_end[t]];
        s_on[t] = 0;
        if (t == 0) {
            s_jump[kTilePix] = (uint16_t)kTilePix;
            s_on[kTilePix] = 0;
        }
        __syncthreads();
        if (t == 0) s_on[s_nxt[0]] = 1;
        __syncthreads();
#pragma unroll 1
        for (int k = 0; k < 8; ++k) {
            const int j = s_jump[t];
            if (s_on[t]) s_on[j] = 1;
            const uint16_t jj = s_jump[j];
            __syncthreads();
            s_jump[t] = jj;
            __syncthreads();
        }
        const bool on = s_on[t] != 0;
        const unsigned long long bm = __ballot(on);
        if ((t & 63) == 0) {
            s_mask[t >> 5] = (uint32_t)bm;
            s_mask[(t >> 5) + 1] = (uint32_t)(bm >> 32);
            s_tmp[t >> 6] = (uint32_t)__popcll(bm);
        }
        __syncthreads();
        if (t == 0) {
            uint32_t nb = 0;
            for (int w2 = 0; w2 < kNT / 64; ++w2) nb += s_tmp[w2];
            f.tile_tot[tile] = total;
            f.tile_nb[tile] = nb;
        }
    }
    __syncthreads();
    if (t < kTilePix / 32) f.batch_mask[(size_t)tile * (kTilePix / 32) + t] = s_mask[t];
}

// The batch table: one record (tile, first pixel, end pixel, oversized) per marked start, in
// pixel order, at the tile's batch offset.
// By a block of kNT threads; s_mask and s_thk: kTilePix / 32 words each.
__device__ inline void batch_records(const FrameBufs& f, int tile, uint32_t* s_mask, uint32_t* s_thk) {
    const int t = threadIdx.x;
    if (t < kTilePix / 32) s_mask[t] = f.batch_mask[(size_t)tile * (kTilePix / 32) + t];
    // (mixed frames: which pixels hold a thick-hair fragment, as bits)
    const unsigned long long tb = __ballot(f.pix_thick && f.pix_thick[(size_t)tile * kTilePix + t] != 0);
    if ((t & 63) == 0) {
        s_thk[t >> 5] = (uint32_t)tb;
        s_thk[(t >> 5) + 1] = (uint32_t)(tb >> 32);
    }
    __syncthreads();
    const int w = t >> 5, b = t & 31;
    if (!((s_mask[w] >> b) & 1u)) return;
    uint32_t idx = __popc(s_mask[w] & ((1u << b) - 1u));
    for (int k = 0; k < w; ++k) idx += __popc(s_mask[k]);
    int end = kTilePix;
    const uint32_t above = b == 31 ? 0u : (s_mask[w] >> (b + 1));
    if (above) {
        end = t + 1 + __ffs(above) - 1;
    } else {
        for (int k = w + 1; k < kTilePix / 32; ++k)
            if (s_mask[k]) {
                end = 32 * k + __ffs(s_mask[k]) - 1;
                break;
            }
    }
    const size_t tq = (size_t)tile * kTilePix;
    const bool oversized = f.pix_cnt[tq + t] > (uint32_t)kCap;
    const uint32_t off0 = f.pix_off[tq + t];
    const uint32_t off1 = end < kTilePix ? f.pix_off[tq + end] : f.tile_tot[tile];
    bool thick = false;   // a thick-hair fragment in pixels [t, end)
    for (int k = w; k <= (end - 1) >> 5; ++k) {
        uint32_t m = s_thk[k];
        if (k == w) m &= ~((1u << b) - 1u);
        if (k == (end - 1) >> 5 && ((end - 1) & 31) != 31) m &= (2u << ((end - 1) & 31)) - 1u;
        thick |= m != 0u;
    }
    const uint32_t pos = xcd_block_of(f.batch_start[tile] + idx, f.batch_start[f.T]);
    f.batches[pos] = pack_batch(tile, t, end, oversized, f.frag_base[tile] + off0, off1 - off0, thick);
    if (thick) f.thick_list[atomicAdd(&f.ctr->thick_batches, 1u)] = pos;
}

// Mixed frames, after the emit pass (which marks the thick-hair pixels); in other frames the emit
// pass writes the records itself.
__global__ __launch_bounds__(kNT) void k_batch_records(FrameBufs f) {
    __shared__ uint32_t s_mask[kTilePix / 32], s_thk[kTilePix / 32];
    if (f.ctr->cap_overflow || f.tile_nb[blockIdx.x] == 0) return;
    batch_records(f, blockIdx.x, s_mask, s_thk);
}

// Emit pass: every fragment into the frame's fragment buffer at
// frag_base[tile] + pix_off[pixel] + (the item's slice of the pixel) + local slot, and each
// pixel's depth-key range (LDS-aggregated per item).
// MIXED: a mixed-level frame, whose thick-hair pixels are marked in f.pix_thick.  ZC: the frame
// has an opaque pass, or may have one (f.opaque == 2, where ctr->hides says: one kernel, its LDS has
// room for both); the fragments stored are exactly those that the count pass counted.
template <bool MIXED, bool ZC>
__global__ __launch_bounds__(kNT) void k_emit(FrameBufs f, CamConst cam) {
    __shared__ uint32_t s_cur[kTilePix], s_pos[kTilePix], s_kmin[kTilePix], s_kmax[kTilePix];
    __shared__ uint8_t s_thk[kTilePix];   // mixed frames: the pixel holds a thick-hair fragment
    __shared__ CovSetup s_cov[kNT];
    __shared__ uint8_t s_own[kNT / 64 * kCovLinesPerWave];
    __shared__ float4 s_iz[kNT];
    __shared__ HideOf<ZC> s_hide[1];
    PHASE_BEGIN();
    const uint32_t n_items = f.item_start[f.T];
    if (blockIdx.x >= n_items || f.ctr->cap_overflow) return;
    const bool hides = ZC && (!MIXED || f.opaque != 2 || f.ctr->hides != 0);
    const uint32_t item = xcd_contiguous(blockIdx.x, n_items);
    const int t = threadIdx.x;
    const uint2 it = f.item_tab[item];
    const int tile = (int)it.x;
    const size_t q = (size_t)tile * kTilePix + t;
    s_cur[t] = 0;
    s_kmin[t] = 0xFFFFFFFFu;
    s_kmax[t] = 0;
    s_thk[t] = 0;
    s_pos[t] = f.frag_base[tile] + f.pix_off[q] + f.item_base[(size_t)item * kTilePix + t];
    __syncthreads();
    const int px0 = (tile % f.ntx) * kTile, py0 = (tile / f.ntx) * kTile;
    const uint32_t lstart = f.tile_start[tile];
    const uint32_t n = f.tile_start[tile + 1] - lstart;
    const uint32_t j = it.y * kNT + t;
    SegRec s{};
    uint32_t gseg = 0;
    if (j < n) {
        gseg = f.list[lstart + j];
        s = f.seg[gseg];
    }
    // (w: each owner's record word, the global segment id or list index; bit 31: a thick hair of a
    // mixed frame)
    s_iz[t] = key_inputs(s);
    s_iz[t].w = __uint_as_float((f.gid ? gseg : j) | (MIXED && (s.hwfx & kFlagThick) ? 0x80000000u : 0u));
    const bool valid = j < n;
    if constexpr (ZC) {
        const uint32_t km = f.pix_kmax[q], z0 = kmax_hides(km) ? km : 0xFFFFFFFFu;
        const int gx = px0 + (t % kTile), gy = py0 + (t / kTile);
        if (hides) hide_setup(s_hide[0], gx < cam.W && gy < cam.H ? z0 : 0u);
    }
    auto drop = [&](int i0, int i1, int j0, int j1) {
        return hides && box_hidden(s_hide[0], nearest_key(s), i0, i1, j0, j1);
    };
    const uint32_t total = f.trim ? cov_setup<kVisible>(s, valid, px0, py0, cam.W, cam.H, s_cov, s_own, drop)
                                  : cov_setup<kAll>(s, valid, px0, py0, cam.W, cam.H, s_cov, s_own, drop);
    float4 iz;   // (the line's segment)
    wave_coverage(s_cov, s_own, total, [&](int p, int tnum, int tden, int, int) {
        const uint32_t key = depth_key_iz(iz.x, iz.y, tnum, tden, iz.z);
        if (hides && key > s_hide[0].z[ZC ? p : 0]) return;
        const uint32_t slot = atomicAdd(&s_cur[p], 1u);
        atomicMin(&s_kmin[p], key);
        atomicMax(&s_kmax[p], key);
        const uint32_t id = __float_as_uint(iz.w);
        if (MIXED && (id >> 31)) s_thk[p] = 1;
        f.frags[s_pos[p] + slot] = make_uint2(key, (id & 0xFFFFFFu) | ((uint32_t)p << 24));
    }, [&](int o, int p, int n, bool steep) {
        iz = s_iz[o];
        return hides && line_hidden(s_hide[0], nearest_key(iz), p, n, steep);
    });
    __syncthreads();
    if (s_cur[t]) {
        atomicMin(&f.pix_kmin[q], s_kmin[t]);
        atomicMax(&f.pix_kmax[q], kmax_seen(s_kmax[t]));
        if (MIXED && s_thk[t]) f.pix_thick[q] = 1;
    }
    // the tile's batch records, by the block of its first chunk (s_pos is free once the waves pass the
    // barrier above)
    if (!MIXED && it.y == 0) batch_records(f, tile, s_pos, s_pos + kTilePix / 32);
    PHASE_END(f.ctr, 1);
}

// The bucket map's scale of a pixel of cnt records with keys in [kmin, kmax].
__device__ inline float bucket_scale(uint32_t cnt, uint32_t kmin, uint32_t kmax) {
    return (float)cnt * __builtin_amdgcn_rcpf((float)(kmax - kmin) + 1.0f);
}

// Exact per-pixel order of the Fb records rec (records i = t + qq kNT; entries beyond Fb are
// ignored) of whole pixels with counts, key minima, bucket scales and offsets in s_cnt /
// s_kmin / s_scale / s_off, into s_B.  Bucket sort with one bucket per record, bucket = the
// record's place in its pixel's linear key range (s_scale[p] = count / (key range + 1): a
// monotone map, so sorted buckets give a sorted pixel); the records are scattered to bucket
// order in s_A, and each record's place inside its bucket is its rank there by (key, segment
// id), which is unique within a pixel.  A thread's LDS reads of one step are issued together,
// and a bucket of up to four records is ranked from one set of reads (larger ones loop).
// s_bk must hold Fb zeros on entry.  Ends with a barrier.
__device__ inline void order_batch(uint32_t Fb, const uint2 (&rec)[kPerThread], const uint32_t* s_cnt,
                                   const uint32_t* s_kmin, const float* s_scale, const uint32_t* s_off,
                                   uint32_t* s_tmp, uint2* s_A, uint2* s_B, uint32_t* s_bk, const uint32_t* list,
                                   bool gid) {
    const int t = threadIdx.x;
    uint32_t my_b[kPerThread], my_r[kPerThread];
    {
        uint32_t kmn[kPerThread], cnt[kPerThread], off[kPerThread];
        float sc[kPerThread];
#pragma unroll
        for (int qq = 0; qq < kPerThread; ++qq) {
            const uint32_t p = rec[qq].y >> 24;   // (< 256 for any record)
            kmn[qq] = s_kmin[p];
            sc[qq] = s_scale[p];
            off[qq] = s_off[p];
            cnt[qq] = s_cnt[p];
        }
#pragma unroll
        for (int qq = 0; qq < kPerThread; ++qq)
            my_b[qq] = off[qq] + min(cnt[qq] - 1u, (uint32_t)((float)(rec[qq].x - kmn[qq]) * sc[qq]));
#pragma unroll
        for (int qq = 0; qq < kPerThread; ++qq)
            if (t + qq * kNT < Fb) my_r[qq] = atomicAdd(&s_bk[my_b[qq]], 1u);
    }
    __syncthreads();
    {   // exclusive scan of the bucket counters, kOwn consecutive per thread (odd, so the
        // lanes' strided reads fall in distinct LDS banks)
        constexpr int kOwn = kPerThread + 1;
        uint32_t loc[kOwn];
        uint32_t sum = 0;
#pragma unroll
        for (int qq = 0; qq < kOwn; ++qq) {
            const uint32_t i = t * kOwn + qq;
            loc[qq] = i < Fb ? s_bk[i] : 0u;
            sum += loc[qq];
        }
        uint32_t ex;
        block_exscan_u32(sum, s_tmp, ex);
#pragma unroll
        for (int qq = 0; qq < kOwn; ++qq) {
            const uint32_t i = t * kOwn + qq;
            if (i < Fb) s_bk[i] = ex;
            ex += loc[qq];
        }
    }
    __syncthreads();
    uint32_t b0[kPerThread], b1[kPerThread];
#pragma unroll
    for (int qq = 0; qq < kPerThread; ++qq) {
        const bool ok = t + qq * kNT < Fb;
        b0[qq] = ok ? s_bk[my_b[qq]] : 0u;
        b1[qq] = ok && my_b[qq] + 1 < Fb ? s_bk[my_b[qq] + 1] : Fb;
    }
#pragma unroll
    for (int qq = 0; qq < kPerThread; ++qq)
        if (t + qq * kNT < Fb) s_A[b0[qq] + my_r[qq]] = rec[qq];
    __syncthreads();
    // ranks, two records at a time (each one's bucket read with independent loads)
    constexpr uint32_t kSmall = 4;
    static_assert(kPerThread % 2 == 0, "records are ranked in pairs");
#pragma unroll
    for (int q0 = 0; q0 < kPerThread; q0 += 2) {
        uint2 u[2][kSmall];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int qq = q0 + h;
            const uint32_t n = t + qq * kNT < Fb ? b1[qq] - b0[qq] : 1u;
#pragma unroll
            for (uint32_t k = 0; k < kSmall; ++k) u[h][k] = n > 1 ? s_A[b0[qq] + min(k, n - 1)] : make_uint2(0u, 0u);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int qq = q0 + h;
            if (t + qq * kNT >= Fb) continue;
            const uint2 me = rec[qq];
            const uint32_t n = b1[qq] - b0[qq];
            uint32_t rank = 0;
            auto before = [&](const uint2& v) {   // (key, segment id) of v below me's
                bool less = v.x < me.x;
                if (v.x == me.x) less = seg_of(v.y, list, gid) < seg_of(me.y, list, gid);
                return less;
            };
#pragma unroll
            for (uint32_t k = 0; k < kSmall; ++k)
                if (k < n && k != my_r[qq]) rank += before(u[h][k]);
            for (uint32_t k = kSmall; k < n; ++k)
                if (k != my_r[qq]) rank += before(s_A[b0[qq] + k]);
            s_B[b0[qq] + rank] = me;
        }
    }
    __syncthreads();
}

// The backward pass's ordering: the same buckets, records staged in s_A and sorted in place in
// s_B by insertion inside each bucket.  (The rank-based routine above gives the same order, but
// inside k_batch_bwd, whose registers are at the 256 + AGPR limit, its use changes that
// kernel's gradients; this variant is the one validated there.)  s_bk must hold Fb zeros.
__device__ inline void order_batch_insertion(uint32_t Fb, const uint32_t* s_cnt, const uint32_t* s_kmin,
                                             const uint32_t* s_kmax, const uint32_t* s_off, uint32_t* s_tmp,
                                             const uint2* s_A, uint2* s_B, uint32_t* s_bk, const uint32_t* list) {
    const int t = threadIdx.x;
    uint32_t my_b[kPerThread], my_r[kPerThread];
#pragma unroll
    for (int qq = 0; qq < kPerThread; ++qq) {
        const uint32_t i = t + qq * kNT;
        if (i < Fb) {
            const uint2 rec = s_A[i];
            const uint32_t p = rec.y >> 24;
            const uint32_t kmn = s_kmin[p], cnt = s_cnt[p];
            const float scale = (float)cnt * __builtin_amdgcn_rcpf((float)(s_kmax[p] - kmn) + 1.0f);
            const uint32_t bucket = min(cnt - 1u, (uint32_t)((float)(rec.x - kmn) * scale));
            my_b[qq] = s_off[p] + bucket;
            my_r[qq] = atomicAdd(&s_bk[my_b[qq]], 1u);
        }
    }
    __syncthreads();
    {
        uint32_t loc[kPerThread];
        uint32_t sum = 0;
#pragma unroll
        for (int qq = 0; qq < kPerThread; ++qq) {
            const uint32_t i = t * kPerThread + qq;
            loc[qq] = i < Fb ? s_bk[i] : 0u;
            sum += loc[qq];
        }
        uint32_t ex;
        block_exscan_u32(sum, s_tmp, ex);
#pragma unroll
        for (int qq = 0; qq < kPerThread; ++qq) {
            const uint32_t i = t * kPerThread + qq;
            if (i < Fb) s_bk[i] = ex;
            ex += loc[qq];
        }
    }
    __syncthreads();
#pragma unroll
    for (int qq = 0; qq < kPerThread; ++qq) {
        const uint32_t i = t + qq * kNT;
        if (i < Fb) s_B[s_bk[my_b[qq]] + my_r[qq]] = s_A[i];
    }
    __syncthreads();
    for (uint32_t bi = t; bi < Fb; bi += kNT) {
        const uint32_t b0 = s_bk[bi];
        const uint32_t b1 = bi + 1 < Fb ? s_bk[bi + 1] : Fb;
        for (uint32_t i = b0 + 1; i < b1; ++i) {
            const uint2 v = s_B[i];
            const uint32_t vseg = list[v.y & 0xFFFFFFu];
            uint32_t jx = i;
            while (jx > b0) {
                const uint2 u2 = s_B[jx - 1];
                bool greater = u2.x > v.x;
                if (u2.x == v.x) greater = list[u2.y & 0xFFFFFFu] > vseg;
                if (!greater) break;
                s_B[jx] = u2;
                --jx;
            }
            s_B[jx] = v;
        }
    }
    __syncthreads();
}

// LDS working set of one batch.
struct BatchLds {
    uint32_t* s_cnt;
    uint32_t* s_kmin;
    float* s_scale;
    uint32_t* s_off;
    uint32_t* s_tmp;
    uint2* s_B;
    uint2* s_A;
    uint32_t* s_bk;
    float* s_agg;
    uint32_t* s_aggh;
};

// Exact order, shading and blending of the Fb records staged in s_A (whole pixels whose
// counts, key minima, bucket scales and offsets are in s_cnt / s_kmin / s_scale / s_off).  Finished pixels are
// written to rgba, or (slice_out != nullptr, a single pixel's key slice) their (C, T) goes to
// slice_out.  rank0 / cnt_total place a slice inside its pixel for the debug dump; by_seg: the
// records carry segment ids in place of keys (a slice inside one key, key_of_slice).
template <int KIND, int MODEL, bool SHADOW>
__device__ inline void sort_shade_blend(const FrameBufs& f, const ShadeArgs& a, float* __restrict__ rgba,
                                        const DebugDump& dbg, int has_dbg, const BatchLds& L_, const uint32_t* list,
                                        const uint2 (&rec)[kPerThread], int px0, int py0, uint32_t Fb, float* slice_out,
                                        uint32_t rank0, uint32_t cnt_total, bool by_seg = false,
                                        uint32_t key_of_slice = 0u) {
    uint32_t* s_cnt = L_.s_cnt;
    uint32_t* s_kmin = L_.s_kmin;
    const float* s_scale = L_.s_scale;
    uint32_t* s_off = L_.s_off;
    uint32_t* s_tmp = L_.s_tmp;
    uint2* s_B = L_.s_B;
    uint2* s_A = L_.s_A;
    uint32_t* s_bk = L_.s_bk;
    float* s_agg = L_.s_agg;
    uint32_t* s_aggh = L_.s_aggh;
    const int t = threadIdx.x;
    const int W = a.cam.W, H = a.cam.H;
    PHASE_BEGIN();
    const bool gid = f.gid != 0;
    order_batch(Fb, rec, s_cnt, s_kmin, s_scale, s_off, s_tmp, s_A, s_B, s_bk, list, gid);
    PHASE_END(f.ctr, 2);
    // ---- shade and blend: thread t takes the run [rb, re) of consecutive fragments of the
    // ordered batch, shades them in order and composites them front to back ("over") as it
    // goes, restarting at each pixel's first fragment.  A pixel that begins and ends inside
    // the run is finished there; the run's first pixel, when it began in an earlier run, is
    // finished after a segmented scan of the runs' open composites gives what lies in front.
    // The segment ids of a thread's fragments are gathered up front (independent loads) and
    // each fragment's segment inputs are fetched one fragment ahead, so that the gathers
    // overlap the shading arithmetic.  (Not for the R / TT / TRT thick-hair shading: its
    // registers would then exceed the budget of three waves per SIMD.)
    constexpr bool kAhead = KIND == 0 || KIND == 3 || (KIND == 1 && MODEL == 1);
    const uint32_t run = (Fb + kNT - 1) / kNT;   // at most kPerThread
    const uint32_t rb = min(Fb, t * run), re = min(Fb, rb + run);
    // Mixed frames shade before they blend: a wave whose lanes held both strand and thick-hair
    // fragments would run both shading paths in turn, so the batch's fragments are listed
    // strands first, thick hairs after, shaded kNT at a time down that list (only the wave at
    // the boundary holds both kinds), and each one's (alpha, L) is staged in LDS for the blend.
    // (Not with the debug dump, which also records h, nor in a batch of strands alone.)
    bool staged = false;
    float4* s_res = reinterpret_cast<float4*>(s_A);   // free once the batch is ordered
    if (KIND == 2 && !has_dbg) {
        uint16_t* s_lst = reinterpret_cast<uint16_t*>(reinterpret_cast<uint32_t*>(s_A) + 4 * kCap);
        uint32_t thick = 0, ns = 0;
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const uint32_t i = t + k * kNT;
            if (i < Fb) {
                if (a.seg[seg_of(s_B[i].y, list, gid)].hwfx & kFlagThick) thick |= 1u << k;
                else ++ns;
            }
        }
        uint32_t ex;
        const uint32_t tot = block_exscan_u32(ns | (uint32_t)__popc(thick) << 16, s_tmp, ex);
        const uint32_t n_s = tot & 0xFFFFu;
        staged = (tot >> 16) > 0;   // uniform across the block
        if (staged) {
            uint32_t ps = ex & 0xFFFFu, pt = n_s + (ex >> 16);
#pragma unroll
            for (int k = 0; k < kPerThread; ++k) {
                const uint32_t i = t + k * kNT;
                if (i < Fb) s_lst[((thick >> k) & 1u) ? pt++ : ps++] = (uint16_t)i;
            }
            __syncthreads();
            for (uint32_t jj = t; jj < Fb; jj += kNT) {
                const uint32_t i = s_lst[jj];
                const uint2 rec = s_B[i];
                const uint32_t p = rec.y >> 24;
                float al, hh, L[3];
                shade_inputs<KIND, MODEL, SHADOW>(a, fetch_segment<KIND>(a, seg_of(rec.y, list, gid)),
                                                  px0 + (int)(p % kTile), py0 + (int)(p / kTile), al, hh, L);
                s_res[i] = make_float4(al, L[0], L[1], L[2]);
            }
            __syncthreads();
        }
    }
    uint32_t gs[kAhead ? kPerThread : 1];
    SegInputs nxt{};
    if (kAhead) {
#pragma unroll
        for (int j = 0; j < kPerThread; ++j) {
            const uint32_t i = rb + j;
            gs[j] = i < re ? seg_of(s_B[i].y, list, gid) : 0u;
        }
        if (rb < re) nxt = fetch_segment<KIND>(a, gs[0]);
    }
    float C0 = 0.f, C1 = 0.f, C2 = 0.f, T = 1.f;   // the open pixel's composite so far
    uint32_t head = 0;                             // the open pixel began in this run
    float H0 = 0.f, H1 = 0.f, H2 = 0.f, HT = 1.f;  // the run's first pixel, begun earlier, ended here
    int hp = -1;
    auto finish = [&](int p, float c0, float c1, float c2, float tt) {
        if (slice_out) {
            slice_out[0] = c0; slice_out[1] = c1; slice_out[2] = c2; slice_out[3] = tt;
        } else {
            const int gx = px0 + (p % kTile), gy = py0 + (p / kTile);
            if (gx < W && gy < H) reinterpret_cast<float4*>(rgba)[(size_t)gy * W + gx] = make_float4(c0, c1, c2, 1.0f - tt);
        }
    };
    for (uint32_t i = rb; i < re; ++i) {
        SegInputs cur{};
        uint32_t gseg = 0;
        if (!(KIND == 2 && staged)) {   // (the next fragment's inputs are requested first)
            if (!kAhead) gs[0] = seg_of(s_B[i].y, list, gid);
            cur = kAhead ? nxt : fetch_segment<KIND>(a, gs[0]);
            gseg = gs[0];
            if (kAhead) {
#pragma unroll
                for (int j = 0; j + 1 < (kAhead ? kPerThread : 1); ++j) gs[j] = gs[j + 1];
                if (i + 1 < re) nxt = fetch_segment<KIND>(a, gs[0]);
            }
        }
        const uint2 rec = s_B[i];
        const uint32_t p = rec.y >> 24;
        const uint32_t p_beg = s_off[p], p_end = s_off[p + 1];
        if (i == p_beg) { C0 = C1 = C2 = 0.f; T = 1.f; head = 1; }
        const int gx = px0 + (int)(p % kTile), gy = py0 + (int)(p / kTile);
        float al, hh, L[3];
        if (KIND == 2 && staged) {
            const float4 r = s_res[i];
            al = r.x; L[0] = r.y; L[1] = r.z; L[2] = r.w;
            hh = 0.f;
        } else {
            shade_inputs<KIND, MODEL, SHADOW>(a, cur, gx, gy, al, hh, L);
        }
        C0 += T * (al * L[0]);
        C1 += T * (al * L[1]);
        C2 += T * (al * L[2]);
        T *= 1.0f - al;
        if (i + 1 == p_end) {
            if (head) finish((int)p, C0, C1, C2, T);
            else { H0 = C0; H1 = C1; H2 = C2; HT = T; hp = (int)p; }
        }
        if (has_dbg) {
            const int dx = gx - dbg.x0, dy = gy - dbg.y0;
            if (dx >= 0 && dy >= 0 && dx < dbg.w && dy < dbg.h) {
                const uint32_t rank = i - p_beg + rank0;
                const int q2 = dy * dbg.w + dx;
                if (rank == 0) dbg.counts[q2] = cnt_total ? cnt_total : s_cnt[p];
                if ((int)rank < dbg.stride) {
                    const size_t o = (size_t)q2 * dbg.stride + rank;
                    dbg.keys[o] = by_seg ? key_of_slice : rec.x;
                    dbg.segs[o] = gseg;
                    dbg.alpha[o] = al;
                    dbg.hoff[o] = hh;
                }
            }
        }
    }
    PHASE_END(f.ctr, 3);
    // inclusive scan of the runs' open composites, (l) then (r) = r.head ? r : (l.C + l.T r.C,
    // l.T r.T): within the wave by shuffles, then across the block's waves through LDS; a thread
    // with no fragments passes its left neighbour's composite through
    const int lane = t & 63, wv = t >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const float c0 = __shfl_up(C0, off), c1 = __shfl_up(C1, off), c2 = __shfl_up(C2, off);
        const float tt = __shfl_up(T, off);
        const uint32_t hh2 = __shfl_up(head, off);
        if (lane >= off && !head) {
            C0 = c0 + tt * C0;
            C1 = c1 + tt * C1;
            C2 = c2 + tt * C2;
            T = tt * T;
            head = hh2;
        }
    }
    const float l0 = __shfl_up(C0, 1), l1 = __shfl_up(C1, 1), l2 = __shfl_up(C2, 1), lT = __shfl_up(T, 1);
    const uint32_t lh = __shfl_up(head, 1);
    if (lane == 63) {
        s_agg[4 * wv + 0] = C0; s_agg[4 * wv + 1] = C1; s_agg[4 * wv + 2] = C2; s_agg[4 * wv + 3] = T;
        s_aggh[wv] = head;
    }
    __syncthreads();
    if (hp >= 0) {   // what lies in front of this run: earlier waves, then earlier lanes of this wave
        float e0 = 0.f, e1 = 0.f, e2 = 0.f, eT = 1.f;
        for (int w2 = 0; w2 < wv; ++w2) {
            if (s_aggh[w2]) { e0 = s_agg[4 * w2 + 0]; e1 = s_agg[4 * w2 + 1]; e2 = s_agg[4 * w2 + 2]; eT = s_agg[4 * w2 + 3]; }
            else {
                e0 = e0 + eT * s_agg[4 * w2 + 0];
                e1 = e1 + eT * s_agg[4 * w2 + 1];
                e2 = e2 + eT * s_agg[4 * w2 + 2];
                eT = eT * s_agg[4 * w2 + 3];
            }
        }
        if (lane > 0) {
            if (lh) { e0 = l0; e1 = l1; e2 = l2; eT = lT; }
            else {
                e0 = e0 + eT * l0;
                e1 = e1 + eT * l1;
                e2 = e2 + eT * l2;
                eT = eT * lT;
            }
        }
        finish(hp, e0 + eT * H0, e1 + eT * H1, e2 + eT * H2, eT * HT);
    }
    PHASE_END(f.ctr, 4);
}

// Slice of a deep pixel's k records at src: among the records that val(r, v) admits, with
// value v in [lo, end), the longest run of leading histogram bins holding at most kCap of them
// (bins refined until one fits).  Returns 0 with [lo, *hi) and its record count *Fb, or 2 when
// more than kCap admitted records share the single value lo.  Values are 32-bit, so lo < 2^32,
// the bin width stays below 2^22 and bins are exact 32-bit quotients.  s_bk holds the
// histogram (kCap bins); all threads call it; ends with a barrier.
template <class Val>
__device__ inline uint32_t refine_slice(uint32_t k, const uint2* __restrict__ src, unsigned long long lo,
                                        unsigned long long end, Val&& val, uint32_t* s_bk, uint32_t* s_tmp,
                                        unsigned long long* s_range, uint32_t& s_slot, uint32_t& s_flag,
                                        unsigned long long& hi_out, uint32_t& Fb) {
    constexpr uint32_t kBins = kCap;
    const int t = threadIdx.x;
    unsigned long long range_hi = end;
    while (true) {
        const unsigned long long width = (range_hi - lo + kBins - 1) / kBins;
        const uint32_t lo32 = (uint32_t)lo, w32 = (uint32_t)width;
        for (uint32_t i = t; i < kBins; i += kNT) s_bk[i] = 0;
        __syncthreads();
        // histogram of the admitted values in [lo, range_hi); each lane's loads issued together
        for (uint32_t i0 = 0; i0 < k; i0 += kNT * kPerThread) {
            uint2 rr[kPerThread];
#pragma unroll
            for (int qq = 0; qq < kPerThread; ++qq) {
                const uint32_t i = i0 + t + qq * kNT;
                rr[qq] = i < k ? src[i] : make_uint2(0u, 0u);
            }
#pragma unroll
            for (int qq = 0; qq < kPerThread; ++qq) {
                const uint32_t i = i0 + t + qq * kNT;
                uint32_t v;
                if (i < k && val(rr[qq], v) && v >= lo32 && (unsigned long long)v < range_hi)
                    atomicAdd(&s_bk[(v - lo32) / w32], 1u);
            }
        }
        __syncthreads();
        // the longest run of leading bins holding at most kCap records, from a block scan of the
        // bin counts (lane t owns bins t * kPerThread ...): the one lane that owns the run's last
        // bin writes the slice; lane 0 flags a first bin that alone exceeds kCap
        {
            const uint32_t used = (uint32_t)((range_hi - lo + width - 1) / width);
            uint32_t loc[kPerThread], sum = 0;
#pragma unroll
            for (int qq = 0; qq < kPerThread; ++qq) {
                const uint32_t i = t * kPerThread + qq;
                loc[qq] = i < used ? s_bk[i] : 0u;
                sum += loc[qq];
            }
            uint32_t incl;
            block_exscan_u32(sum, s_tmp, incl);
#pragma unroll
            for (int qq = 0; qq < kPerThread; ++qq) {
                const uint32_t i = t * kPerThread + qq;
                incl += loc[qq];
                if (i < used && incl <= (uint32_t)kCap) {
                    const uint32_t nxt = i + 1 >= used ? 0u : (qq + 1 < kPerThread ? loc[qq + 1] : s_bk[i + 1]);
                    if (i + 1 >= used || incl + nxt > (uint32_t)kCap) {
                        s_flag = 0;
                        s_range[1] = min(range_hi, lo + (unsigned long long)(i + 1) * width);
                        s_slot = incl;
                    }
                }
            }
            if (t == 0 && loc[0] > (uint32_t)kCap) {
                s_flag = width == 1 ? 2u : 1u;     // 1: refine inside the first bin; 2: one value overflows
                s_range[1] = lo + width;
            }
        }
        __syncthreads();
        const uint32_t flag = s_flag;
        range_hi = s_range[1];
        Fb = s_slot;
        __syncthreads();
        if (flag != 1) {
            hi_out = range_hi;
            return flag;
        }
    }
}

// One LDS batch of whole pixels: exact per-pixel order, shading, front-to-back blending.  A
// pixel deeper than one batch (its own "oversized" batch) is processed in depth-key slices:
// a histogram over the pixel's key range picks the longest run of bins that fits LDS, those
// records are gathered and processed exactly, and the slice composites chain front to back.
// (LDS holds four blocks per CU; strand instances keep their registers within four waves per SIMD,
// thick hairs' heavier shading within three.  Shadowed strands wait for their map texels at three
// waves, and spill little at four: 100k at 1080p 1365 -> 1235 us.)
template <int KIND, int MODEL, bool SHADOW>
__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu((KIND == 0 || KIND == 3) ? 4 : 3))) void k_batch(
    FrameBufs f, ShadeArgs a, float* __restrict__ rgba, DebugDump dbg, int has_dbg) {
    __shared__ uint32_t s_cnt[kTilePix], s_kmin[kTilePix], s_off[kTilePix + 1];
    __shared__ float s_scale[kTilePix];   // count / (key range + 1): the bucket map of the ordering
    __shared__ uint32_t s_tmp[kNT];
    __shared__ __align__(16) uint2 s_B[kCap];
    // staged records (2 words) + bucket counters; in mixed frames also, after the ordering, each
    // fragment's (alpha, L) and the batch's fragments listed strands first (kCap 16-bit entries)
    __shared__ __align__(16) uint32_t s_work[KIND == 2 ? 4 * kCap + kCap / 2 : 3 * kCap];
    __shared__ float s_agg[kNT / 64 * 4];     // wave aggregates of the blend scan (C rgb, T)
    __shared__ uint32_t s_aggh[kNT / 64];
    __shared__ float s_slice[4];
    __shared__ unsigned long long s_range[2];
    __shared__ uint32_t s_slot, s_flag;
    BatchLds L_{s_cnt, s_kmin, s_scale, s_off, s_tmp, s_B, reinterpret_cast<uint2*>(s_work), s_work + 2 * kCap, s_agg,
                s_aggh};
    PHASE_BEGIN();

    const uint32_t n_batches = f.batch_start[f.T];
    // Mixed frames take two launches.  When at most an eighth of the batches hold thick-hair
    // fragments, the strand-only kernel (KIND 3, four waves per SIMD) takes the batches of
    // strands alone and this one (KIND 2) those holding thick hairs, block b the b-th of their
    // list (spread over the grid, and so over the XCDs, wherever on screen the thick hairs lie).
    // Otherwise KIND 2 takes every batch, so that its long thick-hair batches interleave with
    // the rest, and KIND 3 does nothing.
    uint32_t bi = blockIdx.x;
    if (KIND == 2 || KIND == 3) {
        const bool one = f.thick_list == nullptr || 8u * f.ctr->thick_batches > n_batches;
        if (KIND == 3 && one) return;
        if (KIND == 2 && !one) {
            if (blockIdx.x >= f.ctr->thick_batches) return;
            bi = f.thick_list[blockIdx.x];
        }
    }
    const uint4 br = f.batches[bi];   // in the table's capacity; used only below n_batches
    if (bi >= n_batches || f.ctr->cap_overflow) return;
    const BatchRec b = unpack_batch(br);
    if (KIND == 3 && b.thick) return;
    const int tile = b.tile, p0 = b.p0, p1 = b.p1;
    const int t = threadIdx.x;
    const int px0 = (tile % f.ntx) * kTile, py0 = (tile / f.ntx) * kTile;
    const int W = a.cam.W, H = a.cam.H;
    const uint32_t* list = f.list + f.tile_start[tile];
    const size_t q = (size_t)tile * kTilePix + t;
    const uint2* src = f.frags + b.frag0;
    if (!b.over) {
        // the batch's records, its pixels' counts, key ranges and offsets: all loads in flight
        // together before the first barrier
        const uint32_t Fb = b.nfrag;
        uint2 rec[kPerThread];
#pragma unroll
        for (int qq = 0; qq < kPerThread; ++qq) {
            const uint32_t i = t + qq * kNT;
            rec[qq] = i < Fb ? src[i] : make_uint2(0u, 0u);
        }
        const uint32_t tile_off0 = f.pix_off[(size_t)tile * kTilePix + p0];
        if (t >= p0 && t < p1) {
            const uint32_t cnt = f.pix_cnt[q], kmn = f.pix_kmin[q];
            s_cnt[t] = cnt;
            s_kmin[t] = kmn;
            s_scale[t] = bucket_scale(cnt, kmn, kmax_key(f.pix_kmax[q]));
            s_off[t] = f.pix_off[q] - tile_off0;
        }
        if (t == 0) s_off[p1] = Fb;
        for (uint32_t i = t; i < Fb; i += kNT) L_.s_bk[i] = 0;
        __syncthreads();
        PHASE_END(f.ctr, 5);
        sort_shade_blend<KIND, MODEL, SHADOW>(f, a, rgba, dbg, has_dbg, L_, list, rec, px0, py0, Fb, nullptr, 0, 0);
        return;
    }
    // ---- a pixel deeper than one batch: exact slices in (key, segment id) order
    const int p = p0;
    const size_t qp = (size_t)tile * kTilePix + p;
    const uint32_t k = b.nfrag;
    const unsigned long long key_end = (unsigned long long)kmax_key(f.pix_kmax[qp]) + 1ull;
    unsigned long long lo = f.pix_kmin[qp];
    float C0 = 0.f, C1 = 0.f, C2 = 0.f, T = 1.f;   // carried composite (thread 0)
    uint32_t done = 0;
    PHASE_ADD(f.ctr, 7, k);
    PHASE_END(f.ctr, 5);
    // one slice: the records whose value (their key, or inside one key their segment id) lies
    // in [v_lo, v_hi), staged as (value, local index | pixel), ordered, shaded and blended
    auto run_slice = [&](uint32_t Fb, unsigned long long v_lo, unsigned long long v_hi, auto&& val, bool by_seg,
                         uint32_t key) {
        if (t == 0) s_slot = 0;
        __syncthreads();
        for (uint32_t i0 = 0; i0 < k; i0 += kNT * kPerThread) {
            uint2 rr[kPerThread];
#pragma unroll
            for (int qq = 0; qq < kPerThread; ++qq) {
                const uint32_t i = i0 + t + qq * kNT;
                rr[qq] = i < k ? src[i] : make_uint2(0u, 0u);
            }
#pragma unroll
            for (int qq = 0; qq < kPerThread; ++qq) {
                const uint32_t i = i0 + t + qq * kNT;
                uint32_t v;
                if (i < k && val(rr[qq], v) && (unsigned long long)v >= v_lo && (unsigned long long)v < v_hi)
                    L_.s_A[atomicAdd(&s_slot, 1u)] = make_uint2(v, rr[qq].y);
            }
        }
        __syncthreads();
        for (uint32_t i = t; i < Fb; i += kNT) L_.s_bk[i] = 0;
        if (t == 0) {
            s_cnt[p] = Fb;
            s_kmin[p] = (uint32_t)v_lo;
            s_scale[p] = bucket_scale(Fb, (uint32_t)v_lo, (uint32_t)(v_hi - 1));
            s_off[p] = 0;
            s_off[p + 1] = Fb;
        }
        __syncthreads();
        PHASE_END(f.ctr, 6);
        uint2 rec[kPerThread];
#pragma unroll
        for (int qq = 0; qq < kPerThread; ++qq) {
            const uint32_t i = t + qq * kNT;
            rec[qq] = i < Fb ? L_.s_A[i] : make_uint2(0u, 0u);
        }
        sort_shade_blend<KIND, MODEL, SHADOW>(f, a, rgba, dbg, has_dbg, L_, list, rec, px0, py0, Fb, s_slice, done, k,
                                              by_seg, key);
        PHASE_RESET();
        __syncthreads();
        if (t == 0) {
            C0 += T * s_slice[0];
            C1 += T * s_slice[1];
            C2 += T * s_slice[2];
            T *= s_slice[3];
        }
        done += Fb;
        __syncthreads();
    };
    auto by_key = [&](const uint2& r, uint32_t& v) { v = r.x; return true; };
    while (lo < key_end) {
        unsigned long long hi;
        uint32_t Fb;
        const uint32_t flag = refine_slice(k, src, lo, key_end, by_key, L_.s_bk, s_tmp, s_range, s_slot, s_flag, hi, Fb);
        if (flag == 0) {
            // (a slice of leading empty bins holds no record and changes nothing)
            if (Fb) run_slice(Fb, lo, hi, by_key, false, 0u);
            lo = hi;
            continue;
        }
        // more than one batch of fragments at one key K0: slices by segment id inside it (a
        // segment meets a pixel once, so every id range refines down to a slice that fits)
        const uint32_t K0 = (uint32_t)lo;
        auto by_seg = [&](const uint2& r, uint32_t& v) {
            if (r.x != K0) return false;
            v = seg_of(r.y, list, f.gid != 0);
            return true;
        };
        unsigned long long slo = 0;
        const unsigned long long send = 1ull << 32;
        while (slo < send) {
            unsigned long long shi;
            if (refine_slice(k, src, slo, send, by_seg, L_.s_bk, s_tmp, s_range, s_slot, s_flag, shi, Fb) != 0) {
                if (t == 0) atomicAdd(&f.ctr->overflow_pixels, 1u);   // (not reachable: ids are unique)
                return;
            }
            if (Fb) run_slice(Fb, slo, shi, by_seg, true, K0);
            slo = shi;
        }
        lo = (unsigned long long)K0 + 1ull;
    }
    if (t == 0) {
        const int gx = px0 + (p % kTile), gy = py0 + (p / kTile);
        if (gx < W && gy < H) reinterpret_cast<float4*>(rgba)[(size_t)gy * W + gx] = make_float4(C0, C1, C2, 1.0f - T);
    }
}

// ---------------------------------------------------------------------------------------
// Backward pass (thick-hair levels): vector-Jacobian product of the frame with respect to
// each cluster segment's |a|, |b| and its cluster's r and sigma_a.  Per batch:
//   1. the forward's exact per-pixel order (same bucket sort);
//   2. alpha_k and L_k per fragment (float);
//   3. front-to-back prefix T_k and back-to-front suffix (C_k+, S_k+) by two segmented scans;
//      with dC, dA the pixel's output adjoint:
//        dLoss/dalpha_k = T_k [dC . (L_k - C_k+) + dA S_k+],   dLoss/dL_k = dC T_k alpha_k;
//   4. alpha_k and L_k again as Dual<6> (forward-mode partials in |a|, |b|, r, sigma_a rgb)
//      contracted with the step-3 adjoints; partials summed per list entry in LDS, then one
//      global atomic per (batch, list entry, parameter).
constexpr int kNAcc = 1024;          // list entries with LDS accumulators (others go straight to global)
using Dual6 = Dual<6>;

// d hw / d|a|, d hw / d|b| of the float32 half-width (support of the ellipse across the view at
// the segment midpoint, times fy / z_mid).
__device__ inline void halfwidth_partials(const CamConst& c, const SegRec& s, const float4& q0, const float4& q1,
                                          const float4& q2, float a_len, float b_len, float& da, float& db) {
    const float tx = q1.x - q0.x, ty = q1.y - q0.y, tz = q1.z - q0.z;
    const float tl = norm3f(tx, ty, tz);
    const float ux = tx / tl, uy = ty / tl, uz = tz / tl;
    const float mx = (q0.x + q1.x) * 0.5f, my = (q0.y + q1.y) * 0.5f, mz = (q0.z + q1.z) * 0.5f;
    float wx = c.pos[0] - mx, wy = c.pos[1] - my, wz = c.pos[2] - mz;
    const float wl = norm3f(wx, wy, wz);
    wx /= wl; wy /= wl; wz /= wl;
    const float dwu = (wx * ux + wy * uy) + wz * uz;
    const float px = wx - dwu * ux, py = wy - dwu * uy, pz = wz - dwu * uz;
    const float pl = norm3f(px, py, pz);
    const float zm = (1.0f / s.iza + 1.0f / s.izb) * 0.5f;
    const float k = c.fy / zm;
    if (!(pl > 1e-7f)) {
        da = a_len >= b_len ? k : 0.0f;
        db = a_len >= b_len ? 0.0f : k;
        return;
    }
    const float xx = px / pl, xy = py / pl, xz = pz / pl;
    const float yx = uy * xz - uz * xy, yy = uz * xx - ux * xz, yz = ux * xy - uy * xx;
    const float hx = q2.x, hy = q2.y, hz = q2.z;
    const float bhx = uy * hz - uz * hy, bhy = uz * hx - ux * hz, bhz = ux * hy - uy * hx;
    const float ca = (hx * yx + hy * yy) + hz * yz;
    const float cb = (bhx * yx + bhy * yy) + bhz * yz;
    const float W = sqrtf(a_len * a_len * ca * ca + b_len * b_len * cb * cb);
    da = W > 0.0f ? k * a_len * ca * ca / W : 0.0f;
    db = W > 0.0f ? k * b_len * cb * cb / W : 0.0f;
}

constexpr int kMaxBwdSlices = 64;    // slices of one pixel deeper than a batch (more: HAIR_ERANGE)

template <int MODEL>
__global__ __launch_bounds__(kNT) void k_batch_bwd(FrameBufs f, ShadeArgs a, GradOut g, int S, int K) {
    __shared__ uint32_t s_cnt[kTilePix], s_kmin[kTilePix], s_kmax[kTilePix], s_off[kTilePix + 1];
    __shared__ uint32_t s_tmp[kNT];
    __shared__ __align__(16) uint2 s_B[kCap];
    __shared__ __align__(16) float s_work[4 * kCap];     // sort staging, then (alpha, L) -> adjoints
    __shared__ float s_T[kCap];                          // front-to-back transmittance before each fragment
    __shared__ float s_acc[6 * kNAcc];                   // per list entry partial sums
    __shared__ float s_dpix[4 * kTilePix];               // output adjoint of the batch's pixels
    __shared__ float s_agg[kNT * 4];
    __shared__ uint32_t s_aggh[kNT];
    // a pixel deeper than one batch: its slices (value range, by segment id inside key), their
    // composites (C rgb, T) and the boundary values each slice's adjoints need
    __shared__ unsigned long long s_range[2];
    __shared__ uint32_t s_slot, s_flag;
    __shared__ unsigned long long s_sl_lo[kMaxBwdSlices], s_sl_hi[kMaxBwdSlices];
    __shared__ uint32_t s_sl_key[kMaxBwdSlices], s_sl_n[kMaxBwdSlices];
    __shared__ float4 s_sl_agg[kMaxBwdSlices];
    __shared__ float4 s_sl_after[kMaxBwdSlices];        // (C rgb, S) of the slices behind
    __shared__ float s_sl_before[kMaxBwdSlices];         // T of the slices in front
    uint2* s_A = reinterpret_cast<uint2*>(s_work);
    uint32_t* s_bk = reinterpret_cast<uint32_t*>(s_work) + 2 * kCap;
    float4* s_p4 = reinterpret_cast<float4*>(s_work);

    const uint32_t n_batches = f.batch_start[f.T];
    const uint4 br = f.batches[blockIdx.x];
    if (blockIdx.x >= n_batches || f.ctr->cap_overflow) return;
    const BatchRec b = unpack_batch(br);
    const int tile = b.tile, p0 = b.p0, p1 = b.p1;
    const int t = threadIdx.x;
    const int px0 = (tile % f.ntx) * kTile, py0 = (tile / f.ntx) * kTile;
    const int W = a.cam.W, H = a.cam.H;
    const uint32_t lstart = f.tile_start[tile];
    const uint32_t n = f.tile_start[tile + 1] - lstart;
    const uint32_t* list = f.list + lstart;
    const size_t q = (size_t)tile * kTilePix + t;
    const uint32_t tile_off0 = f.pix_off[(size_t)tile * kTilePix + p0];
    if (t >= p0 && t < p1) {
        s_cnt[t] = f.pix_cnt[q];
        s_kmin[t] = f.pix_kmin[q];
        s_kmax[t] = kmax_key(f.pix_kmax[q]);
        s_off[t] = f.pix_off[q] - tile_off0;
        const int gx = px0 + (t % kTile), gy = py0 + (t / kTile);
        const bool in = gx < W && gy < H;
        const float4 dp = in ? reinterpret_cast<const float4*>(g.d_rgba)[(size_t)gy * W + gx] : make_float4(0, 0, 0, 0);
        s_dpix[4 * t + 0] = dp.x; s_dpix[4 * t + 1] = dp.y; s_dpix[4 * t + 2] = dp.z; s_dpix[4 * t + 3] = dp.w;
    }
    if (t == 0) s_off[p1] = b.nfrag;
    for (int i = t; i < 6 * kNAcc; i += kNT) s_acc[i] = 0.0f;
    __syncthreads();
    const uint2* src = f.frags + b.frag0;

    // Steps 2-4 on the Fb records ordered in s_B (whole pixels, or one slice of one pixel).  A
    // slice's pixel starts with transmittance T_in (the slices in front) and ends over the
    // composite (C_out rgb, S_out) of the slices behind it; whole pixels start at 1 and end over
    // (0, 1).  grads = false: only the slice's own composite, into agg (C rgb, T).
    auto slice_core = [&](uint32_t Fb, float T_in, float4 out_c, bool grads, float4* agg) __attribute__((always_inline)) {
        // ---- 2. alpha and L per fragment (float)
        for (uint32_t i = t; i < Fb; i += kNT) {
            const uint2 rec = s_B[i];
            const uint32_t p = rec.y >> 24;
            const uint32_t gseg = list[rec.y & 0xFFFFFFu];
            float al, hh, L[3];
            shade_fragment<1, MODEL>(a, gseg, px0 + (int)(p % kTile), py0 + (int)(p / kTile), al, hh, L);
            s_p4[i] = make_float4(al, L[0], L[1], L[2]);
        }
        __syncthreads();
        // ---- 3a. forward: T before each fragment (segmented exclusive product over runs)
        const uint32_t run = (Fb + kNT - 1) / kNT;
        const uint32_t rb = min(Fb, t * run), re = min(Fb, rb + run);
        {
            float T = 1.f;
            uint32_t head = 0;
            for (uint32_t i = rb; i < re; ++i) {
                const uint32_t p = s_B[i].y >> 24;
                if (i == s_off[p]) { T = 1.f; head = 1; }
                T *= 1.0f - s_p4[i].x;
            }
            s_agg[4 * t + 3] = T;
            s_aggh[t] = head;
            __syncthreads();
            for (int off = 1; off < kNT; off <<= 1) {
                float tt = 1;
                uint32_t hh2 = 0;
                const bool has = t >= off;
                if (has) { tt = s_agg[4 * (t - off) + 3]; hh2 = s_aggh[t - off]; }
                __syncthreads();
                if (has && !s_aggh[t]) { s_agg[4 * t + 3] = tt * s_agg[4 * t + 3]; s_aggh[t] = hh2; }
                __syncthreads();
            }
            T = t > 0 ? s_agg[4 * (t - 1) + 3] : 1.f;
            for (uint32_t i = rb; i < re; ++i) {
                const uint32_t p = s_B[i].y >> 24;
                if (i == s_off[p]) T = 1.f;
                s_T[i] = T_in * T;
                T *= 1.0f - s_p4[i].x;
            }
            __syncthreads();
        }
        if (!grads) {   // the slice's own composite: C = sum T_k alpha_k L_k, T = prod (1 - alpha_k)
            float c0 = 0.f, c1 = 0.f, c2 = 0.f;
            for (uint32_t i = t; i < Fb; i += kNT) {
                const float4 v = s_p4[i];
                const float w = s_T[i] * v.x;
                c0 += w * v.y;
                c1 += w * v.z;
                c2 += w * v.w;
            }
            s_agg[4 * t + 0] = c0; s_agg[4 * t + 1] = c1; s_agg[4 * t + 2] = c2;
            __syncthreads();
            if (t == 0) {
                float4 r = make_float4(0.f, 0.f, 0.f, 1.f);
                for (int i = 0; i < kNT; ++i) { r.x += s_agg[4 * i]; r.y += s_agg[4 * i + 1]; r.z += s_agg[4 * i + 2]; }
                if (Fb) r.w = s_T[Fb - 1] * (1.0f - s_p4[Fb - 1].x);
                *agg = r;
            }
            __syncthreads();
            return;
        }
        // ---- 3b. backward: suffix composite (C+, S+) after each fragment, then the adjoints
        {
            // run aggregate from the run start through its first pixel end (or the whole run)
            float C0 = 0.f, C1 = 0.f, C2 = 0.f, Sx = 1.f;
            uint32_t tail = 0;
            for (uint32_t i = re; i > rb; --i) {
                const uint32_t k = i - 1;
                const uint32_t p = s_B[k].y >> 24;
                if (k + 1 == s_off[p] + s_cnt[p]) { C0 = C1 = C2 = 0.f; Sx = 1.f; tail = 1; }
                const float4 v = s_p4[k];
                C0 = v.x * v.y + (1.0f - v.x) * C0;
                C1 = v.x * v.z + (1.0f - v.x) * C1;
                C2 = v.x * v.w + (1.0f - v.x) * C2;
                Sx = (1.0f - v.x) * Sx;
            }
            s_agg[4 * t + 0] = C0; s_agg[4 * t + 1] = C1; s_agg[4 * t + 2] = C2; s_agg[4 * t + 3] = Sx;
            s_aggh[t] = tail;
            __syncthreads();
            // right-to-left inclusive scan: R_t = agg_t.tail ? agg_t : agg_t over R_{t+1}
            for (int off = 1; off < kNT; off <<= 1) {
                float c0 = 0, c1 = 0, c2 = 0, ss = 1;
                const bool has = t + off < kNT;
                if (has) {
                    c0 = s_agg[4 * (t + off) + 0]; c1 = s_agg[4 * (t + off) + 1];
                    c2 = s_agg[4 * (t + off) + 2]; ss = s_agg[4 * (t + off) + 3];
                }
                const uint32_t my_tail = s_aggh[t];
                const uint32_t r_tail = has ? s_aggh[t + off] : 0u;
                __syncthreads();
                if (has && !my_tail) {
                    const float mS = s_agg[4 * t + 3];
                    s_agg[4 * t + 0] = s_agg[4 * t + 0] + mS * c0;
                    s_agg[4 * t + 1] = s_agg[4 * t + 1] + mS * c1;
                    s_agg[4 * t + 2] = s_agg[4 * t + 2] + mS * c2;
                    s_agg[4 * t + 3] = mS * ss;
                    s_aggh[t] = r_tail;
                }
                __syncthreads();
            }
            if (t + 1 < kNT) { C0 = s_agg[4 * (t + 1) + 0]; C1 = s_agg[4 * (t + 1) + 1]; C2 = s_agg[4 * (t + 1) + 2]; Sx = s_agg[4 * (t + 1) + 3]; }
            else { C0 = C1 = C2 = 0.f; Sx = 1.f; }
            __syncthreads();
            for (uint32_t i = re; i > rb; --i) {
                const uint32_t k = i - 1;
                const uint32_t p = s_B[k].y >> 24;
                if (k + 1 == s_off[p] + s_cnt[p]) { C0 = C1 = C2 = 0.f; Sx = 1.f; }
                const float4 v = s_p4[k];
                const float Tk = s_T[k];
                const float dR = s_dpix[4 * p + 0], dG = s_dpix[4 * p + 1], dB = s_dpix[4 * p + 2], dA = s_dpix[4 * p + 3];
                // behind fragment k: the rest of its pixel's records here, then what lies behind
                const float Ca0 = C0 + Sx * out_c.x, Ca1 = C1 + Sx * out_c.y, Ca2 = C2 + Sx * out_c.z;
                const float Sa = Sx * out_c.w;
                const float g_alpha = Tk * (dR * (v.y - Ca0) + dG * (v.z - Ca1) + dB * (v.w - Ca2) + dA * Sa);
                const float ta = Tk * v.x;
                C0 = v.x * v.y + (1.0f - v.x) * C0;
                C1 = v.x * v.z + (1.0f - v.x) * C1;
                C2 = v.x * v.w + (1.0f - v.x) * C2;
                Sx = (1.0f - v.x) * Sx;
                s_p4[k] = make_float4(g_alpha, dR * ta, dG * ta, dB * ta);
            }
        }
        __syncthreads();
        // ---- 4. partials: alpha and L as Dual6, contracted with the adjoints.  A fragment whose
        // four adjoints are all zero (behind an opaque fragment of its pixel, T_k = 0, or in a
        // pixel without output adjoint) contributes exactly nothing; the others are listed first
        // (in s_T, free after step 3) so that every lane's Dual6 work is a fragment that counts.
        uint32_t* s_idx = reinterpret_cast<uint32_t*>(s_T);
        uint32_t n_live;
        {
            uint32_t mine = 0;
            for (uint32_t i = t; i < Fb; i += kNT) {
                const float4 v = s_p4[i];
                mine += (v.x != 0.0f || v.y != 0.0f || v.z != 0.0f || v.w != 0.0f) ? 1u : 0u;
            }
            uint32_t pos;
            n_live = block_exscan_u32(mine, s_tmp, pos);
            for (uint32_t i = t; i < Fb; i += kNT) {
                const float4 v = s_p4[i];
                if (v.x != 0.0f || v.y != 0.0f || v.z != 0.0f || v.w != 0.0f) s_idx[pos++] = i;
            }
            __syncthreads();
        }
        for (uint32_t kk = t; kk < n_live; kk += kNT) {
            const uint32_t i = s_idx[kk];
            const uint2 rec = s_B[i];
            const uint32_t p = rec.y >> 24;
            const uint32_t j = rec.y & 0xFFFFFFu;
            const uint32_t gseg = list[j];
            const float4 adj = s_p4[i];
            const SegRec s = a.seg[gseg];
            const ShadeRec& srec = a.shade[gseg];
            const float4 q0 = srec.q0, q1 = srec.q1, q2 = srec.q2, q3 = srec.q3;
            float dha, dhb;
            halfwidth_partials(a.cam, s, q0, q1, q2, q3.x, q3.y, dha, dhb);
            Dual6 hw(s.hw);
            hw.d[0] = dha;
            hw.d[1] = dhb;
            const Dual6 al = Dual6::seed(q3.x, 0), bl = Dual6::seed(q3.y, 1), rr = Dual6::seed(q3.w, 2);
            const Dual6 sig[3] = {Dual6::seed(q0.w, 3), Dual6::seed(q1.w, 4), Dual6::seed(q2.w, 5)};
            Dual6 alpha, hoff, L[3];
            shade_core<1, MODEL, Dual6>(a, s, q0, q1, q2, q3.z, px0 + (int)(p % kTile), py0 + (int)(p / kTile), hw, al,
                                        bl, rr, sig, alpha, hoff, L);
            float gp[6];
#pragma unroll
            for (int m = 0; m < 6; ++m)
                gp[m] = adj.x * alpha.d[m] + adj.y * L[0].d[m] + adj.z * L[1].d[m] + adj.w * L[2].d[m];
            if (j < (uint32_t)kNAcc) {
#pragma unroll
                for (int m = 0; m < 6; ++m) atomicAdd(&s_acc[m * kNAcc + j], gp[m]);
            } else {
                const uint32_t par = g.rows ? g.rows[gseg] >> 6 : gseg;   // a piece's segment
                const int owner = (int)par / S;
                atomicAdd(&g.d_axes[2 * par], gp[0]);
                atomicAdd(&g.d_axes[2 * par + 1], gp[1]);
                atomicAdd(&g.d_r[owner], gp[2]);
                atomicAdd(&g.d_sig[owner], gp[3]);
                atomicAdd(&g.d_sig[K + owner], gp[4]);
                atomicAdd(&g.d_sig[2 * K + owner], gp[5]);
            }
        }
        __syncthreads();
    };

    if (!b.over) {
        const uint32_t Fb = b.nfrag;
        for (uint32_t i = t; i < Fb; i += kNT) {
            s_A[i] = src[i];
            s_bk[i] = 0;
        }
        __syncthreads();
        order_batch_insertion(Fb, s_cnt, s_kmin, s_kmax, s_off, s_tmp, s_A, s_B, s_bk, list);
        slice_core(Fb, 1.0f, make_float4(0.f, 0.f, 0.f, 1.f), true, nullptr);
    } else {
        // ---- a pixel deeper than one batch: the forward's slices in (key, segment id) order,
        // each differentiated with the transmittance of the slices in front of it and the
        // composite of the slices behind it (two sweeps: composites, then adjoints)
        const int p = p0;
        const uint32_t k = b.nfrag;
        const unsigned long long key_end = (unsigned long long)s_kmax[p] + 1ull;
        auto by_key = [&](const uint2& r, uint32_t& v) { v = r.x; return true; };
        // stage the records of slice [v_lo, v_hi) (by key, or inside key K0 by segment id) in
        // s_B, ordered, as a one-pixel batch
        auto stage = [&](uint32_t Fb, unsigned long long v_lo, unsigned long long v_hi, bool by_seg, uint32_t K0)
            __attribute__((always_inline)) {
            if (t == 0) s_slot = 0;
            __syncthreads();
            for (uint32_t i = t; i < k; i += kNT) {
                const uint2 r = src[i];
                uint32_t v = r.x;
                bool in = true;
                if (by_seg) {
                    in = r.x == K0;
                    if (in) v = list[r.y & 0xFFFFFFu];
                }
                if (in && (unsigned long long)v >= v_lo && (unsigned long long)v < v_hi)
                    s_A[atomicAdd(&s_slot, 1u)] = make_uint2(v, r.y);
            }
            __syncthreads();
            for (uint32_t i = t; i < Fb; i += kNT) s_bk[i] = 0;
            if (t == 0) {
                s_cnt[p] = Fb;
                s_kmin[p] = (uint32_t)v_lo;
                s_kmax[p] = (uint32_t)(v_hi - 1);
                s_off[p] = 0;
                s_off[p + 1] = Fb;
            }
            __syncthreads();
            order_batch_insertion(Fb, s_cnt, s_kmin, s_kmax, s_off, s_tmp, s_A, s_B, s_bk, list);
        };
        uint32_t nsl = 0;
        bool ok = true;
        auto add_slice = [&](uint32_t Fb, unsigned long long v_lo, unsigned long long v_hi, bool by_seg, uint32_t K0)
            __attribute__((always_inline)) {
            if (nsl >= (uint32_t)kMaxBwdSlices) { ok = false; return; }
            stage(Fb, v_lo, v_hi, by_seg, K0);
            slice_core(Fb, 1.0f, make_float4(0.f, 0.f, 0.f, 1.f), false, &s_sl_agg[nsl]);
            if (t == 0) {
                s_sl_lo[nsl] = v_lo;
                s_sl_hi[nsl] = v_hi;
                s_sl_key[nsl] = by_seg ? K0 : 0xFFFFFFFFu;
                s_sl_n[nsl] = Fb | (by_seg ? 0x80000000u : 0u);
            }
            ++nsl;
        };
        unsigned long long lo = s_kmin[p];
        while (ok && lo < key_end) {
            unsigned long long hi;
            uint32_t Fb;
            const uint32_t flag = refine_slice(k, src, lo, key_end, by_key, s_bk, s_tmp, s_range, s_slot, s_flag, hi, Fb);
            if (flag == 0) {
                if (Fb) add_slice(Fb, lo, hi, false, 0u);
                lo = hi;
                continue;
            }
            const uint32_t K0 = (uint32_t)lo;
            auto by_seg = [&](const uint2& r, uint32_t& v) {
                if (r.x != K0) return false;
                v = list[r.y & 0xFFFFFFu];
                return true;
            };
            unsigned long long slo = 0;
            const unsigned long long send = 1ull << 32;
            while (ok && slo < send) {
                unsigned long long shi;
                if (refine_slice(k, src, slo, send, by_seg, s_bk, s_tmp, s_range, s_slot, s_flag, shi, Fb) != 0) {
                    ok = false;
                    break;
                }
                if (Fb) add_slice(Fb, slo, shi, true, K0);
                slo = shi;
            }
            lo = (unsigned long long)K0 + 1ull;
        }
        if (!ok) {   // more slices than the kernel keeps: reported, not differentiated
            if (t == 0) atomicAdd(&f.ctr->overflow_pixels, 1u);
            return;
        }
        if (t == 0) {   // transmittance in front of each slice and the composite behind it
            float T = 1.f;
            for (uint32_t i = 0; i < nsl; ++i) {
                s_sl_before[i] = T;
                T *= s_sl_agg[i].w;
            }
            float4 behind = make_float4(0.f, 0.f, 0.f, 1.f);
            for (uint32_t i = nsl; i > 0; --i) {
                s_sl_after[i - 1] = behind;
                const float4 c = s_sl_agg[i - 1];
                behind = make_float4(c.x + c.w * behind.x, c.y + c.w * behind.y, c.z + c.w * behind.z, c.w * behind.w);
            }
        }
        __syncthreads();
        for (uint32_t i = 0; i < nsl; ++i) {
            const uint32_t Fb = s_sl_n[i] & 0x7FFFFFFFu;
            const bool by_seg = (s_sl_n[i] >> 31) != 0;
            stage(Fb, s_sl_lo[i], s_sl_hi[i], by_seg, s_sl_key[i]);
            slice_core(Fb, s_sl_before[i], s_sl_after[i], true, nullptr);
        }
    }
    const uint32_t nacc = min(n, (uint32_t)kNAcc);
    for (uint32_t j = t; j < nacc; j += kNT) {
        float v[6];
        bool any = false;
#pragma unroll
        for (int m = 0; m < 6; ++m) {
            v[m] = s_acc[m * kNAcc + j];
            any |= v[m] != 0.0f;
        }
        if (!any) continue;
        const uint32_t gseg = list[j];
        const uint32_t par = g.rows ? g.rows[gseg] >> 6 : gseg;
        const int owner = (int)par / S;
        atomicAdd(&g.d_axes[2 * par], v[0]);
        atomicAdd(&g.d_axes[2 * par + 1], v[1]);
        atomicAdd(&g.d_r[owner], v[2]);
        atomicAdd(&g.d_sig[owner], v[3]);
        atomicAdd(&g.d_sig[K + owner], v[4]);
        atomicAdd(&g.d_sig[2 * K + owner], v[5]);
    }
}

// ---------------------------------------------------------------------------------------
// Thick-hair construction (Sec. 5.1 step 3), float64 sums in member order.
__global__ void k_build_centers(const float* __restrict__ vx, const float* __restrict__ vy,
                                const float* __restrict__ vz, const float* __restrict__ width,
                                const float* __restrict__ sig, int n_strands, int V,
                                const int32_t* __restrict__ members, const int32_t* __restrict__ mstart, int K,
                                float* cx, float* cy, float* cz, float* r, float* csig, int32_t* n_total) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= K * V) return;
    const int c = g / V, k = g - c * V;
    const int b = mstart[c], e = mstart[c + 1];
    double sx = 0, sy = 0, sz = 0;
    for (int m = b; m < e; ++m) {
        const int v = members[m] * V + k;
        sx += (double)vx[v];
        sy += (double)vy[v];
        sz += (double)vz[v];
    }
    const double N = (double)(e - b);
    cx[g] = (float)(sx / N);
    cy[g] = (float)(sy / N);
    cz[g] = (float)(sz / N);
    if (k == 0) {
        double sw = 0, s0 = 0, s1 = 0, s2 = 0;
        for (int m = b; m < e; ++m) {
            const int s = members[m];
            sw += (double)width[s];
            s0 += (double)sig[s];
            s1 += (double)sig[n_strands + s];
            s2 += (double)sig[2 * n_strands + s];
        }
        r[c] = (float)((sw / N) * 0.5);
        csig[c] = (float)(s0 / N);
        csig[K + c] = (float)(s1 / N);
        csig[2 * K + c] = (float)(s2 / N);
        n_total[c] = e - b;
    }
}

__global__ void k_build_ellipses(const float* __restrict__ vx, const float* __restrict__ vy,
                                 const float* __restrict__ vz, int V, const int32_t* __restrict__ members,
                                 const int32_t* __restrict__ mstart, int K, const float* __restrict__ cx,
                                 const float* __restrict__ cy, const float* __restrict__ cz,
                                 const float* __restrict__ r, float* ahat, float* axes) {
    const int S = V - 1;
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= K * S) return;
    const int c = g / S, k = g - c * S;
    const int ia = c * V + k;
    const double ax = cx[ia], ay = cy[ia], az = cz[ia];
    const double bx = cx[ia + 1], by = cy[ia + 1], bz = cz[ia + 1];
    double ux = bx - ax, uy = by - ay, uz = bz - az;
    const double ul = sqrt(ux * ux + uy * uy + uz * uz);
    ux /= ul; uy /= ul; uz /= ul;
    // basis of the plane orthogonal to u: start from the axis of smallest |u_j| (lowest index on ties)
    const double fx = fabs(ux), fy = fabs(uy), fz = fabs(uz);
    int j = 0;
    if (fy < fx) j = 1;
    if (fz < (j == 0 ? fx : fy)) j = 2;
    double ex = j == 0, ey = j == 1, ez = j == 2;
    const double eu = ex * ux + ey * uy + ez * uz;
    ex -= eu * ux; ey -= eu * uy; ez -= eu * uz;
    const double el = sqrt(ex * ex + ey * ey + ez * ez);
    ex /= el; ey /= el; ez /= el;
    const double fx2 = uy * ez - uz * ey, fy2 = uz * ex - ux * ez, fz2 = ux * ey - uy * ex;
    const double mx = 0.5 * (ax + bx), my = 0.5 * (ay + by), mz = 0.5 * (az + bz);
    const int b0 = mstart[c], b1 = mstart[c + 1];
    double c11 = 0, c12 = 0, c22 = 0;
    for (int m = b0; m < b1; ++m) {
        const int v = members[m] * V + k;
        const double qx = 0.5 * ((double)vx[v] + (double)vx[v + 1]) - mx;
        const double qy = 0.5 * ((double)vy[v] + (double)vy[v + 1]) - my;
        const double qz = 0.5 * ((double)vz[v] + (double)vz[v + 1]) - mz;
        const double q1 = qx * ex + qy * ey + qz * ez;
        const double q2 = qx * fx2 + qy * fy2 + qz * fz2;
        c11 += q1 * q1;
        c12 += q1 * q2;
        c22 += q2 * q2;
    }
    const double N = (double)(b1 - b0);
    c11 /= N; c12 /= N; c22 /= N;
    const double hm = 0.5 * (c11 + c22), hd = 0.5 * (c11 - c22);
    const double rad = sqrt(hd * hd + c12 * c12);
    const double l1 = fmax(hm + rad, 0.0), l2 = fmax(hm - rad, 0.0);
    double v1 = 1.0, v2 = 0.0;
    if (!((l1 - l2) <= 1e-12 * (l1 + l2))) {
        // eigenvector of l1: (l1 - c22, c12) or (c12, l1 - c11), the better conditioned
        const double a1 = l1 - c22, a2 = c12, b1v = c12, b2 = l1 - c11;
        if (a1 * a1 + a2 * a2 >= b1v * b1v + b2 * b2) { v1 = a1; v2 = a2; } else { v1 = b1v; v2 = b2; }
        const double vl = sqrt(v1 * v1 + v2 * v2);
        v1 /= vl; v2 /= vl;
    }
    const int nseg = K * S;
    ahat[g] = (float)(v1 * ex + v2 * fx2);
    ahat[nseg + g] = (float)(v1 * ey + v2 * fy2);
    ahat[2 * nseg + g] = (float)(v1 * ez + v2 * fz2);
    const double rr = (double)r[c];
    axes[2 * g] = (float)(rr + 2.0 * sqrt(l1));
    axes[2 * g + 1] = (float)(rr + 2.0 * sqrt(l2));
}

inline int blocks_for(size_t n, int per) { return (int)((n + per - 1) / per); }


// ---------------------------------------------------------------------------------------
// Curved thick hairs: the centre line is the uniform Catmull-Rom spline through the level's
// centre vertices (ends clamped), each segment split into m equal parameter steps by its
// screen length (Sec. 5.2, tessellation by distance; Sec. 6, spline centre lines).  The
// points decide integers (snapped endpoints), so the basis is evaluated with one rounding
// per operation in a fixed order; u = 0 and u = 1 return the vertices themselves.

__device__ inline void spline_point(const LevelDev& lv, int owner, int k, float u, float& x, float& y, float& z) {
    const int base = owner * (lv.S + 1);
    if (u == 0.0f || u == 1.0f) {
        const int i = base + k + (u == 1.0f ? 1 : 0);
        x = lv.vx[i];
        y = lv.vy[i];
        z = lv.vz[i];
        return;
    }
    const int i0 = base + max(k - 1, 0), i1 = base + k, i2 = base + k + 1, i3 = base + min(k + 2, lv.S);
    const float u2 = u * u, u3 = u2 * u;
    const float w0 = 0.5f * ((2.0f * u2 - u3) - u);
    const float w1 = 0.5f * ((3.0f * u3 - 5.0f * u2) + 2.0f);
    const float w2 = 0.5f * ((4.0f * u2 - 3.0f * u3) + u);
    const float w3 = 0.5f * (u3 - u2);
    x = ((w0 * lv.vx[i0] + w1 * lv.vx[i1]) + w2 * lv.vx[i2]) + w3 * lv.vx[i3];
    y = ((w0 * lv.vy[i0] + w1 * lv.vy[i1]) + w2 * lv.vy[i2]) + w3 * lv.vy[i3];
    z = ((w0 * lv.vz[i0] + w1 * lv.vz[i1]) + w2 * lv.vz[i2]) + w3 * lv.vz[i3];
}

// Steps of segment g: the smallest m in [1, max_sub] with (m T16)^2 >= dX^2 + dY^2 (snapped
// screen extent of the straight segment); 1 when an endpoint is not on screen.
__global__ __launch_bounds__(256) void k_tess_count(LevelDev lv, CamConst cam, int T16, int max_sub,
                                                    uint32_t* __restrict__ cnt) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= lv.nseg) return;
    const int owner = g / lv.S, k = g - owner * lv.S;
    const int va = owner * (lv.S + 1) + k;
    const PPoint A = project_point(cam, lv.vx[va], lv.vy[va], lv.vz[va]);
    const PPoint B = project_point(cam, lv.vx[va + 1], lv.vy[va + 1], lv.vz[va + 1]);
    int m = 1;
    if (A.ok && B.ok) {
        const long long dx = (long long)rintf(B.X16) - (long long)rintf(A.X16);
        const long long dy = (long long)rintf(B.Y16) - (long long)rintf(A.Y16);
        const long long d2 = dx * dx + dy * dy;
        while (m < max_sub && (long long)(m * T16) * (long long)(m * T16) < d2) ++m;
    }
    cnt[g] = (uint32_t)m;
}

// Row list: g << 4 | j for the m steps j of every segment g, at start[g].
__global__ __launch_bounds__(256) void k_tess_fill(const uint32_t* __restrict__ cnt, const uint32_t* __restrict__ start,
                                                   int nseg, uint32_t* __restrict__ rows) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= nseg) return;
    const uint32_t m = cnt[g], o = start[g];
    for (uint32_t j = 0; j < m; ++j) rows[o + j] = ((uint32_t)g << 4) | j;
}

// Row r: step j of segment g, from P(j / m) to P((j + 1) / m), with segment g's cross-section.
__global__ __launch_bounds__(256) void k_project_tess(LevelDev lv, const uint32_t* __restrict__ rows, int nrows,
                                                      const uint32_t* __restrict__ cnt, CamConst cam,
                                                      SegRec* __restrict__ seg, ShadeRec* __restrict__ shade) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nrows) return;
    const uint32_t e = rows[r];
    const int g = (int)(e >> 4), j = (int)(e & 15u);
    const int m = (int)cnt[g];
    const int owner = g / lv.S, k = g - owner * lv.S;
    float ax, ay, az, bx, by, bz;
    spline_point(lv, owner, k, (float)j / (float)m, ax, ay, az);
    spline_point(lv, owner, k, (float)(j + 1) / (float)m, bx, by, bz);
    seg[r] = project_segment_at(lv, g, ax, ay, az, bx, by, bz, cam, shade + r);
}

// ---------------------------------------------------------------------------------------
// Long segments (an axis extent above kMaxAxis sub-pixels, both endpoints on the guard band)
// are drawn as m = min(ceil(extent / kSplitLen), kMaxPieces) pieces of equal screen parameter:
// piece j runs between the world points of screen parameters j / m and (j + 1) / m, found
// with the perspective-correct parameter t_w = s izB / (izA + s (izB - izA)) in float32 (one
// rounding per operation) and exact at s = 0 and 1.  A piece keeps its segment's attributes.
__device__ inline uint32_t split_pieces(const LevelDev& lv, int g, const CamConst& cam) {
    const int owner = g / lv.S, k = g - owner * lv.S;
    const int va = owner * (lv.S + 1) + k;
    const PPoint A = project_point(cam, lv.vx[va], lv.vy[va], lv.vz[va]);
    const PPoint B = project_point(cam, lv.vx[va + 1], lv.vy[va + 1], lv.vz[va + 1]);
    int m = 1;
    if (A.ok && B.ok) {
        const int dx = abs((int)rintf(B.X16) - (int)rintf(A.X16)), dy = abs((int)rintf(B.Y16) - (int)rintf(A.Y16));
        const int ext = max(dx, dy);
        if (ext > kMaxAxis) m = min((ext + kSplitLen - 1) / kSplitLen, kMaxPieces);
    }
    return (uint32_t)m;
}

__global__ __launch_bounds__(256) void k_split_count(LevelDev lv, CamConst cam, uint32_t* __restrict__ cnt) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= lv.nseg) return;
    cnt[g] = split_pieces(lv, g, cam);
}

// The same over the rows of a mixed frame (sel[i] = level << 28 | segment of that level).
__global__ __launch_bounds__(256) void k_split_count_mixed(HierDev h, const uint32_t* __restrict__ sel, int nsel,
                                                           CamConst cam, uint32_t* __restrict__ cnt) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nsel) return;
    const uint32_t e = sel[i];
    cnt[i] = split_pieces(h.lv[e >> 28], (int)(e & 0x0FFFFFFFu), cam);
}

// Row list: g << 6 | j for the m pieces j of every segment g, at start[g].
__global__ __launch_bounds__(256) void k_split_fill(const uint32_t* __restrict__ cnt, const uint32_t* __restrict__ start,
                                                    int nseg, uint32_t* __restrict__ rows) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= nseg) return;
    const uint32_t m = cnt[g], o = start[g];
    for (uint32_t j = 0; j < m; ++j) rows[o + j] = ((uint32_t)g << 6) | j;
}

__device__ inline void split_point(float ax, float ay, float az, float bx, float by, float bz, float izA, float izB,
                                   int j, int m, float& x, float& y, float& z) {
    if (j == 0) { x = ax; y = ay; z = az; return; }
    if (j == m) { x = bx; y = by; z = bz; return; }
    const float s = (float)j / (float)m;
    const float iz = izA + s * (izB - izA);
    const float tw = (s * izB) / iz;
    x = ax + tw * (bx - ax);
    y = ay + tw * (by - ay);
    z = az + tw * (bz - az);
}

// Piece j of m of segment g of lv (the whole segment when m = 1).
__device__ inline SegRec project_piece(const LevelDev& lv, int g, int j, int m, const CamConst& cam, ShadeRec* sr,
                                       bool packed) {
    if (m == 1) return project_segment(lv, g, cam, sr, packed);
    const int owner = g / lv.S, k = g - owner * lv.S;
    const int va = owner * (lv.S + 1) + k;
    const float ax = lv.vx[va], ay = lv.vy[va], az = lv.vz[va];
    const float bx = lv.vx[va + 1], by = lv.vy[va + 1], bz = lv.vz[va + 1];
    const PPoint A = project_point(cam, ax, ay, az), B = project_point(cam, bx, by, bz);
    float p0x, p0y, p0z, p1x, p1y, p1z;
    split_point(ax, ay, az, bx, by, bz, A.iz, B.iz, j, m, p0x, p0y, p0z);
    split_point(ax, ay, az, bx, by, bz, A.iz, B.iz, j + 1, m, p1x, p1y, p1z);
    return project_segment_at(lv, g, p0x, p0y, p0z, p1x, p1y, p1z, cam, sr, packed);
}

// Row r: piece j of segment g (a whole segment when it has one piece), with segment g's
// attributes; strand levels write the packed strand shading record.
__global__ __launch_bounds__(256) void k_project_split(LevelDev lv, const uint32_t* __restrict__ rows, int nrows,
                                                       const uint32_t* __restrict__ cnt, CamConst cam,
                                                       SegRec* __restrict__ seg, ShadeRec* __restrict__ shade) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nrows) return;
    const uint32_t e = rows[r];
    const int g = (int)(e >> 6), j = (int)(e & 63u);
    ShadeRec sr;
    sr.q3 = make_float4(0.f, 0.f, 0.f, 0.f);
    seg[r] = project_piece(lv, g, j, (int)cnt[g], cam, &sr, lv.kind == 0);
    shade[r] = sr;
}

// Row r of a mixed frame drawn in pieces: piece j of selection row i (rows[r] = i << 6 | j),
// with the record layout of k_project_mixed.
__global__ __launch_bounds__(256) void k_project_split_mixed(HierDev h, const uint32_t* __restrict__ sel,
                                                             const uint32_t* __restrict__ rows, int nrows,
                                                             const uint32_t* __restrict__ cnt, CamConst cam,
                                                             SegRec* __restrict__ seg, ShadeRec* __restrict__ shade) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nrows) return;
    const uint32_t e = rows[r];
    const int i = (int)(e >> 6), j = (int)(e & 63u);
    const uint32_t s = sel[i];
    const int L = (int)(s >> 28), g = (int)(s & 0x0FFFFFFFu);
    SegRec rec = project_piece(h.lv[L], g, j, (int)cnt[i], cam, shade + r, false);
    if (h.lv[L].kind == 1) rec.hwfx |= kFlagThick;
    else shade[r].q3 = make_float4(0.5f * h.lv[L].width[g / h.lv[L].S], 0.0f, 0.0f, -1.0f);
    seg[r] = rec;
}

// ---------------------------------------------------------------------------------------
// Shadow pass: deep opacity map toward a directional light (Sec. 5.2 shadow pass; its count
// feeds the forward lobes of Sec. 4).  The light view is an orthographic raster with the
// camera pass's integer coverage rule, so binning and the coverage arithmetic are the camera
// kernels'; the projection and the two map passes are the light's own.  Every float
// step that decides an integer (bounds, grid, snapping, depth) is a single rounding per
// operation in a fixed order (this file is compiled without contraction).


// World half-width padding the grid: a strand's radius, a thick hair's larger semi-axis.
__device__ inline float pad_halfwidth(const LevelDev& lv, int g) {
    return lv.kind == 0 ? 0.5f * lv.width[g / lv.S] : fmaxf(lv.axes[2 * g], lv.axes[2 * g + 1]);
}

// A mixed frame's shadow pass reads its rows from the camera pass's shading records instead
// of a level: q0.xyz, q1.xyz the world endpoints, q2.xyz a^, and q3 = (|a|, |b|, n_total, r)
// for a thick hair or (radius, 0, 0, -1) for a strand.
__device__ inline bool row_is_strand(const ShadeRec& r) { return r.q3.w < 0.0f; }

// Endpoints of segment (or row) g.
__device__ inline void dom_endpoints(const LevelDev& lv, const ShadeRec* rows, int g, float& ax, float& ay, float& az,
                                     float& bx, float& by, float& bz) {
    if (rows) {
        const float4 q0 = rows[g].q0, q1 = rows[g].q1;
        ax = q0.x; ay = q0.y; az = q0.z;
        bx = q1.x; by = q1.y; bz = q1.z;
        return;
    }
    const int owner = g / lv.S, k = g - owner * lv.S;
    const int va = owner * (lv.S + 1) + k;
    ax = lv.vx[va]; ay = lv.vy[va]; az = lv.vz[va];
    bx = lv.vx[va + 1]; by = lv.vy[va + 1]; bz = lv.vz[va + 1];
}

constexpr int kDomBoundThreads = 256;
constexpr int kDomBoundMaxBlocks = 1024;

// Per block: (min u - w, max u + w, min v - w, max v + w, max z) over its segments' endpoints.
__global__ __launch_bounds__(kDomBoundThreads) void k_dom_bounds(LevelDev lv, const ShadeRec* __restrict__ rows,
                                                                DomBasis b, float* __restrict__ part) {
    __shared__ float s_red[5][kDomBoundThreads];
    float umin = INFINITY, umax = -INFINITY, vmin = INFINITY, vmax = -INFINITY, zmax = -INFINITY;
    for (int g = blockIdx.x * kDomBoundThreads + threadIdx.x; g < lv.nseg; g += gridDim.x * kDomBoundThreads) {
        float pe[2][3];
        dom_endpoints(lv, rows, g, pe[0][0], pe[0][1], pe[0][2], pe[1][0], pe[1][1], pe[1][2]);
        const float w = !rows ? pad_halfwidth(lv, g)
                              : (row_is_strand(rows[g]) ? rows[g].q3.x : fmaxf(rows[g].q3.x, rows[g].q3.y));
        for (int e = 0; e < 2; ++e) {
            const float x = pe[e][0], y = pe[e][1], z = pe[e][2];
            const float u = dot_e(b.e1, x, y, z), v = dot_e(b.e2, x, y, z), d = dot_e(b.d, x, y, z);
            umin = fminf(umin, u - w);
            umax = fmaxf(umax, u + w);
            vmin = fminf(vmin, v - w);
            vmax = fmaxf(vmax, v + w);
            zmax = fmaxf(zmax, d);
        }
    }
    const int t = threadIdx.x;
    s_red[0][t] = umin; s_red[1][t] = -umax; s_red[2][t] = vmin; s_red[3][t] = -vmax; s_red[4][t] = -zmax;
    __syncthreads();
    for (int h = kDomBoundThreads / 2; h > 0; h >>= 1) {
        if (t < h)
            for (int c = 0; c < 5; ++c) s_red[c][t] = fminf(s_red[c][t], s_red[c][t + h]);
        __syncthreads();
    }
    if (t < 5) part[5 * blockIdx.x + t] = s_red[t][0];
}

// One block: reduce the partial bounds and set the grid (texel size = extent / (R - 2), one
// texel of margin; z_ref = z_max + 1 so that iz = z_ref - z >= 1 orders like inverse depth).
__global__ __launch_bounds__(kDomBoundThreads) void k_dom_grid(const float* __restrict__ part, int nb, DomBasis b,
                                                             int R, DomGrid* __restrict__ grid) {
    __shared__ float s_red[5][kDomBoundThreads];
    const int t = threadIdx.x;
    float m[5] = {INFINITY, INFINITY, INFINITY, INFINITY, INFINITY};
    for (int i = t; i < nb; i += kDomBoundThreads)
        for (int c = 0; c < 5; ++c) m[c] = fminf(m[c], part[5 * i + c]);
    for (int c = 0; c < 5; ++c) s_red[c][t] = m[c];
    __syncthreads();
    for (int h = kDomBoundThreads / 2; h > 0; h >>= 1) {
        if (t < h)
            for (int c = 0; c < 5; ++c) s_red[c][t] = fminf(s_red[c][t], s_red[c][t + h]);
        __syncthreads();
    }
    if (t == 0) {
        const float umin = s_red[0][0], umax = -s_red[1][0], vmin = s_red[2][0], vmax = -s_red[3][0];
        const float zmax = -s_red[4][0];
        const float ext = fmaxf(fmaxf(umax - umin, vmax - vmin), 1e-6f);
        DomGrid gr;
        gr.b = b;
        gr.s = ext / (float)(R - 2);
        gr.u0 = umin - gr.s;
        gr.v0 = vmin - gr.s;
        gr.rs = rcp_of(gr.s);
        gr.k16 = 16.0f / gr.s;
        gr.z_ref = zmax + 1.0f;
        gr.R = R;
        *grid = gr;
    }
}

// Light-view record of segment g: snapped texel coordinates (1/16 texel), iz = z_ref - z, and
// the half-width in texels (a strand's radius; a thick hair's support across the light).
__global__ __launch_bounds__(256) void k_project_light(LevelDev lv, const ShadeRec* __restrict__ rows,
                                                       const DomGrid* __restrict__ grid, SegRec* __restrict__ seg) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= lv.nseg) return;
    const DomGrid gr = *grid;
    const int owner = g / lv.S;
    float ax, ay, az, bx, by, bz;
    dom_endpoints(lv, rows, g, ax, ay, az, bx, by, bz);
    const bool strand = rows ? row_is_strand(rows[g]) : lv.kind == 0;
    float hw;
    if (strand) {
        hw = (rows ? rows[g].q3.x : 0.5f * lv.width[owner]) / gr.s;
    } else {
        const float tx = bx - ax, ty = by - ay, tz = bz - az;
        const float tl = norm3f(tx, ty, tz);
        const float ux = tx / tl, uy = ty / tl, uz = tz / tl;
        const float wx = gr.b.omega[0], wy = gr.b.omega[1], wz = gr.b.omega[2];
        const float dwu = (wx * ux + wy * uy) + wz * uz;
        const float px = wx - dwu * ux, py = wy - dwu * uy, pz = wz - dwu * uz;
        const float pl = norm3f(px, py, pz);
        const float xx = px / pl, xy = py / pl, xz = pz / pl;
        const float yx = uy * xz - uz * xy, yy = uz * xx - ux * xz, yz = ux * xy - uy * xx;
        const float hx = rows ? rows[g].q2.x : lv.ahat[g];
        const float hy = rows ? rows[g].q2.y : lv.ahat[lv.nseg + g];
        const float hz = rows ? rows[g].q2.z : lv.ahat[2 * lv.nseg + g];
        const float bhx = uy * hz - uz * hy, bhy = uz * hx - ux * hz, bhz = ux * hy - uy * hx;
        const float a_len = rows ? rows[g].q3.x : lv.axes[2 * g], b_len = rows ? rows[g].q3.y : lv.axes[2 * g + 1];
        const float pa = a_len * ((hx * yx + hy * yy) + hz * yz);
        const float pb = b_len * ((bhx * yx + bhy * yy) + bhz * yz);
        float W = sqrtf(pa * pa + pb * pb);
        if (!(pl > 1e-7f)) W = fmaxf(a_len, b_len);
        hw = W / gr.s;
    }
    SegRec r;
    r.xa = (int)rintf((dot_e(gr.b.e1, ax, ay, az) - gr.u0) * gr.k16);
    r.ya = (int)rintf((dot_e(gr.b.e2, ax, ay, az) - gr.v0) * gr.k16);
    r.xb = (int)rintf((dot_e(gr.b.e1, bx, by, bz) - gr.u0) * gr.k16);
    r.yb = (int)rintf((dot_e(gr.b.e2, bx, by, bz) - gr.v0) * gr.k16);
    r.iza = gr.z_ref - dot_e(gr.b.d, ax, ay, az);
    r.izb = gr.z_ref - dot_e(gr.b.d, bx, by, bz);
    r.hw = hw;
    const float hw16 = 16.0f * hw;
    r.hwfx = 0;
    if (isfinite(hw16) && hw16 >= 0.0f) {
        const float c16 = ceilf(hw16);
        if (abs(r.xb - r.xa) > kMaxAxis || abs(r.yb - r.ya) > kMaxAxis || c16 > (float)kMaxHwFx)
            r.hwfx = kFlagCulledLong;
        else
            r.hwfx = (int)c16 | kFlagVisible;
    }
    seg[g] = r;
}

// A block of the map passes takes four chunks of a tile's list, which saves three of four rounds of
// global atomics, where the light view has the items to keep the chip's 2048 block slots filled that
// way (a warm frame's grid may be larger: the view's own count decides.  20k strands, map 256, on a
// workspace that has drawn a large frame: 0.285 ms a frame by the grid, 0.254 by the count).
__device__ inline uint32_t dom_group(uint32_t n_items) { return n_items >= 8192 ? 4u : 1u; }

// The shadow map of a light view is two passes over the tiles' lists, with no fragment stored:
// k_dom_first finds per texel the first hit iz0 (the smallest depth key), k_dom_layers adds every
// fragment's expected hair count to its layer floor((iz0 - iz) / delta) (clamped to K - 1): a strand
// its box coverage alpha, a thick hair alpha rho kappa l_max sqrt(1 - h^2) (Sec. 4, hair number; the
// chord along the light at the texel's offset h = delta / hw).  The counts are 32.32 fixed-point
// sums (they commute, so the atomics give the same sums in any order; counts are far below 2^31
// hairs), in LDS for dom_group chunks of a tile's list and added to the texels' sums in acc
// ([tile][layer][texel]) once.  k_dom_texels writes (iz0, C_0 .. C_6) with C the cumulative counts;
// iz0 = 0 marks a texel without hair.  Bound by the coverage arithmetic (VALU), done twice; storing
// the fragments in between cost more (100k strands, 1024^2 map, 34 M fragments: count + emit +
// resolve 145 + 280 + 305 us -> 230 + 356).  A pass over a sample of each list, so that the first one
// could skip what lies behind, gained nothing.
__global__ __launch_bounds__(kNT) void k_dom_first(FrameBufs f, CamConst cam) {
    __shared__ uint32_t s_z[kTilePix];
    __shared__ float4 s_iz[kNT];
    __shared__ CovSetup s_cov[kNT];
    __shared__ uint8_t s_own[kNT / 64 * kCovLinesPerWave];
    const uint32_t n_items = f.item_start[f.T];
    if (blockIdx.x >= n_items || f.ctr->cap_overflow) return;
    const uint2 it = f.item_tab[xcd_contiguous(blockIdx.x, n_items)];
    const uint32_t group = dom_group(n_items);
    if (it.y % group) return;
    const int t = threadIdx.x, tile = (int)it.x;
    const int px0 = (tile % f.ntx) * kTile, py0 = (tile / f.ntx) * kTile;
    const uint32_t lstart = f.tile_start[tile], n = f.tile_start[tile + 1] - lstart;
    const size_t q = (size_t)tile * kTilePix + t;
    const uint32_t z0 = f.pix_kmin[q];
    s_z[t] = z0;
    for (uint32_t k = it.y; k < it.y + group && k * kNT < n; ++k) {
        const uint32_t j = k * kNT + t;
        SegRec s{};
        if (j < n) s = f.seg[f.list[lstart + j]];
        s_iz[t] = key_inputs(s);
        const uint32_t total = cov_setup<kAll>(s, j < n, px0, py0, cam.W, cam.H, s_cov, s_own);
        float4 iz;   // (the line's segment)
        wave_coverage(s_cov, s_own, total, [&](int p, int tnum, int tden, int, int) {
            const uint32_t z = s_z[p];
            if (iz_bound(iz, tnum) < iz_of_key(z)) return;
            const uint32_t key = depth_key_iz(iz.x, iz.y, tnum, tden, iz.z);
            if (key < z) atomicMin(&s_z[p], key);
        }, [&](int o, int, int, bool) {
            iz = s_iz[o];
            return false;
        });
        __syncthreads();
    }
    if (s_z[t] < z0) atomicMin(&f.pix_kmin[q], s_z[t]);
}

// THICK: the level can hold thick hairs.  The launch adds the layers [l0, l0 + nl) of K (ALL: l0 = 0, nl = K),
// with acc as [tile][nl][texel] (see launch_dom_map).  Dynamic LDS: nl x kTilePix sums.
template <bool THICK, bool ALL>
__global__ __launch_bounds__(kNT) void k_dom_layers(FrameBufs f, CamConst cam, LevelDev lv,
                                                    const ShadeRec* __restrict__ rows,
                                                    const DomGrid* __restrict__ grid, int K, int l0, int nl, float delta,
                                                    float rdelta, unsigned long long* __restrict__ acc) {
    extern __shared__ unsigned long long s_acc[];
    __shared__ float s_iz0[kTilePix];
    __shared__ float4 s_seg[kNT];                  // (iza, izb, hw, sqrt(t_den))
    __shared__ float2 s_rcp[kNT];                  // (1 / sqrt(t_den), 1 / t_den)
    __shared__ float4 s_thk[THICK ? kNT : 1];      // (rho, kappa, 2 |a| |b| / (hw s), 0: strand, 1: thick hair)
    __shared__ CovSetup s_cov[kNT];
    __shared__ uint8_t s_own[kNT / 64 * kCovLinesPerWave];
    const uint32_t n_items = f.item_start[f.T];
    if (blockIdx.x >= n_items || f.ctr->cap_overflow) return;
    const uint2 it = f.item_tab[xcd_contiguous(blockIdx.x, n_items)];
    const uint32_t group = dom_group(n_items);
    if (it.y % group) return;
    const int t = threadIdx.x, tile = (int)it.x;
    const int px0 = (tile % f.ntx) * kTile, py0 = (tile / f.ntx) * kTile;
    const uint32_t lstart = f.tile_start[tile], n = f.tile_start[tile + 1] - lstart;
    s_iz0[t] = iz_of_key(f.pix_kmin[(size_t)tile * kTilePix + t]);
    for (int k = 0; k < nl; ++k) s_acc[k * kTilePix + t] = 0ull;
    for (uint32_t k = it.y; k < it.y + group && k * kNT < n; ++k) {
        const uint32_t j = k * kNT + t;
        SegRec s{};
        if (j < n) {
            const uint32_t g = f.list[lstart + j];
            s = f.seg[g];
            if constexpr (THICK) {
                float4 th = make_float4(0.f, 0.f, 0.f, 0.f);
                if (rows ? !row_is_strand(rows[g]) : lv.kind != 0) {
                    const int owner = g / lv.S;
                    const float a = rows ? rows[g].q3.x : lv.axes[2 * g], b = rows ? rows[g].q3.y : lv.axes[2 * g + 1];
                    const float m = rows ? rows[g].q3.z : (float)lv.n_total[owner], r = rows ? rows[g].q3.w : lv.r[owner];
                    th.x = fminf(fmaxf(m * r * r / (a * b), 0.0f), 1.0f);
                    th.y = sqrtf(m / (3.14159265358979f * a * b));
                    th.z = 2.0f * a * b / (s.hw * grid->s);
                    th.w = 1.0f;
                }
                s_thk[t] = th;
            }
        }
        const int dx = s.xb - s.xa, dy = s.yb - s.ya;
        const float td = (float)(dx * dx + dy * dy), sq = sqrtf(td);
        s_seg[t] = make_float4(s.iza, s.izb, s.hw, sq);
        s_rcp[t] = make_float2(1.0f / sq, 1.0f / td);
        const uint32_t total = cov_setup<kAll>(s, j < n, px0, py0, cam.W, cam.H, s_cov, s_own);
        float4 e, th;   // (the line's segment)
        float2 rc;
        wave_coverage(s_cov, s_own, total, [&](int p, int tnum, int tden, int, int cr) {
            // (rounded like the keys of k_dom_first, so that the first hit itself lies in layer 0)
            const float tt = div_rcp((float)tnum, (float)tden, rc.y);
            const float iz = e.x + tt * (e.y - e.x);
            int layer = min(K - 1, (int)floorf(div_by(s_iz0[p] - iz, delta, rdelta)));
            if (!ALL) {
                layer -= l0;
                if ((unsigned)layer >= (unsigned)nl) return;
            }
            const float dl = div_rcp(fabsf((float)cr), e.w, rc.x) * (1.0f / 16.0f);
            const float hw = e.z;
            float c = fminf(fmaxf(fminf(dl + hw, 0.5f) - fmaxf(dl - hw, -0.5f), 0.0f), 1.0f);
            if constexpr (THICK) {
                if (th.w > 0.0f) {
                    const float h = fminf(dl / hw, 1.0f);
                    // (a degenerate, zero-width thick hair holds no hairs across the light)
                    c = hw > 0.0f ? c * th.x * th.y * th.z * sqrtf((1.0f - h) * (1.0f + h)) : 0.0f;
                }
            }
            // 32.32 fixed point, rounded: whole part, then the exact rest in 2^-32
            const uint32_t hi = (uint32_t)c;
            const uint32_t lo = (uint32_t)((double)(c - (float)hi) * 4294967296.0 + 0.5);
            const unsigned long long fx = (unsigned long long)hi << 32 | lo;
            if (fx) atomicAdd(&s_acc[layer * kTilePix + p], fx);
        }, [&](int o, int, int, bool) {
            e = s_seg[o];
            rc = s_rcp[o];
            if constexpr (THICK) th = s_thk[o];
            return false;
        });
        __syncthreads();
    }
    for (int k = 0; k < nl; ++k) {
        const unsigned long long v = s_acc[k * kTilePix + t];
        if (v) atomicAdd(&acc[((size_t)tile * nl + k) * kTilePix + t], v);
    }
}

// (nl == K: whole texels; nl == 1: acc holds the sum of the layers 0 .. l0)
__global__ __launch_bounds__(kNT) void k_dom_texels(FrameBufs f, int R, int K, int l0, int nl,
                                                    const unsigned long long* __restrict__ acc, float4* __restrict__ tex) {
    if (f.ctr->cap_overflow) return;
    const int tile = blockIdx.x, t = threadIdx.x;
    const int px = (tile % f.ntx) * kTile + t % kTile, py = (tile / f.ntx) * kTile + t / kTile;
    float C[kDomMaxLayers] = {};
    float iz0 = 0.0f;
    if (f.tile_start[tile + 1] > f.tile_start[tile]) {
        iz0 = iz_of_key(f.pix_kmin[(size_t)tile * kTilePix + t]);
        unsigned long long run = 0;
#pragma unroll
        for (int k = 0; k < kDomMaxLayers; ++k) {
            if (k < nl) run += acc[((size_t)tile * nl + k) * kTilePix + t];
            C[k] = (float)((double)run * (1.0 / 4294967296.0));
        }
    }
    if (px >= R || py >= R) return;
    const size_t o = 2 * ((size_t)py * R + px);
    if (nl < K) {
        float* texel = reinterpret_cast<float*>(tex + o);
        if (l0 == 0) texel[0] = iz0;
        for (int k = l0; k < (l0 + 1 < K ? l0 + 1 : kDomMaxLayers); ++k) texel[1 + k] = C[0];
        return;
    }
    tex[o] = make_float4(iz0, C[0], C[1], C[2]);
    tex[o + 1] = make_float4(C[3], C[4], C[5], C[6]);
}
}  // namespace

// ---------------------------------------------------------------------------------------
hipError_t launch_project(const LevelDev& lv, const CamConst& cam, SegRec* seg, ShadeRec* shade, hipStream_t st) {
    if (lv.nseg == 0) return hipSuccess;
    hipLaunchKernelGGL(k_project, dim3(blocks_for(lv.nseg, 256)), dim3(256), 0, st, lv, cam, seg, shade);
    return hipGetLastError();
}

hipError_t launch_tess(const LevelDev& lv, const CamConst& cam, int32_t max_px, int32_t max_sub, uint32_t* cnt,
                       uint32_t* start, uint32_t* scan_tmp, hipStream_t st) {
    if (lv.nseg == 0) return hipSuccess;
    hipLaunchKernelGGL(k_tess_count, dim3(blocks_for(lv.nseg, 256)), dim3(256), 0, st, lv, cam, 16 * max_px, max_sub,
                       cnt);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_exscan(cnt, start, lv.nseg, scan_tmp, st);
}

hipError_t launch_tess_fill(const uint32_t* cnt, const uint32_t* start, int32_t nseg, uint32_t* rows, hipStream_t st) {
    if (nseg == 0) return hipSuccess;
    hipLaunchKernelGGL(k_tess_fill, dim3(blocks_for(nseg, 256)), dim3(256), 0, st, cnt, start, nseg, rows);
    return hipGetLastError();
}

hipError_t launch_split(const LevelDev& lv, const CamConst& cam, uint32_t* cnt, uint32_t* start, uint32_t* scan_tmp,
                        hipStream_t st) {
    if (lv.nseg == 0) return hipSuccess;
    hipLaunchKernelGGL(k_split_count, dim3(blocks_for(lv.nseg, 256)), dim3(256), 0, st, lv, cam, cnt);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_exscan(cnt, start, lv.nseg, scan_tmp, st);
}

hipError_t launch_split_mixed(const HierDev& h, const uint32_t* sel, int32_t nsel, const CamConst& cam, uint32_t* cnt,
                              uint32_t* start, uint32_t* scan_tmp, hipStream_t st) {
    if (nsel == 0) return hipSuccess;
    hipLaunchKernelGGL(k_split_count_mixed, dim3(blocks_for(nsel, 256)), dim3(256), 0, st, h, sel, nsel, cam, cnt);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_exscan(cnt, start, nsel, scan_tmp, st);
}

hipError_t launch_project_split_mixed(const HierDev& h, const uint32_t* sel, const uint32_t* rows, int32_t nrows,
                                      const uint32_t* cnt, const CamConst& cam, SegRec* seg, ShadeRec* shade,
                                      hipStream_t st) {
    if (nrows == 0) return hipSuccess;
    hipLaunchKernelGGL(k_project_split_mixed, dim3(blocks_for(nrows, 256)), dim3(256), 0, st, h, sel, rows, nrows, cnt,
                       cam, seg, shade);
    return hipGetLastError();
}

hipError_t launch_split_fill(const uint32_t* cnt, const uint32_t* start, int32_t nseg, uint32_t* rows, hipStream_t st) {
    if (nseg == 0) return hipSuccess;
    hipLaunchKernelGGL(k_split_fill, dim3(blocks_for(nseg, 256)), dim3(256), 0, st, cnt, start, nseg, rows);
    return hipGetLastError();
}

hipError_t launch_project_split(const LevelDev& lv, const uint32_t* rows, int32_t nrows, const uint32_t* cnt,
                                const CamConst& cam, SegRec* seg, ShadeRec* shade, hipStream_t st) {
    if (nrows == 0) return hipSuccess;
    hipLaunchKernelGGL(k_project_split, dim3(blocks_for(nrows, 256)), dim3(256), 0, st, lv, rows, nrows, cnt, cam, seg,
                       shade);
    return hipGetLastError();
}

hipError_t launch_project_tess(const LevelDev& lv, const uint32_t* rows, int32_t nrows, const uint32_t* cnt,
                               const CamConst& cam, SegRec* seg, ShadeRec* shade, hipStream_t st) {
    if (nrows == 0) return hipSuccess;
    hipLaunchKernelGGL(k_project_tess, dim3(blocks_for(nrows, 256)), dim3(256), 0, st, lv, rows, nrows, cnt, cam, seg,
                       shade);
    return hipGetLastError();
}

int dom_bound_blocks(int32_t nseg) {
    return std::max(1, std::min(kDomBoundMaxBlocks, (int)((nseg + kDomBoundThreads - 1) / kDomBoundThreads)));
}

hipError_t launch_dom_grid(const LevelDev& lv, const ShadeRec* rows, const DomBasis& b, int32_t R, float* part,
                           DomGrid* grid, hipStream_t st) {
    const int nb = dom_bound_blocks(lv.nseg);
    hipLaunchKernelGGL(k_dom_bounds, dim3(nb), dim3(kDomBoundThreads), 0, st, lv, rows, b, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_dom_grid, dim3(1), dim3(kDomBoundThreads), 0, st, part, nb, b, R, grid);
    return hipGetLastError();
}

hipError_t launch_project_light(const LevelDev& lv, const ShadeRec* rows, const DomGrid* grid, SegRec* seg,
                                hipStream_t st) {
    if (lv.nseg == 0) return hipSuccess;
    hipLaunchKernelGGL(k_project_light, dim3(blocks_for(lv.nseg, 256)), dim3(256), 0, st, lv, rows, grid, seg);
    return hipGetLastError();
}

hipError_t launch_dom_map(const FrameBufs& f, const CamConst& cam, const LevelDev& lv, const ShadeRec* rows,
                          const DomGrid* grid, int32_t K, int32_t nl, float delta, float rdelta, uint32_t n_items,
                          unsigned long long* acc, float4* tex, hipStream_t st) {
    // n_items: the grid (at least the view's items, which the kernels read)
    const bool thick = rows || lv.kind != 0;
    auto layers = nl == K ? (thick ? &k_dom_layers<true, true> : &k_dom_layers<false, true>)
                          : (thick ? &k_dom_layers<true, false> : &k_dom_layers<false, false>);
    if (n_items) hipLaunchKernelGGL(k_dom_first, dim3(n_items), dim3(kNT), 0, st, f, cam);
    // all layers in one pass, or one after the other into the same sums (which then run on)
    for (int l0 = 0; l0 < K; l0 += nl) {
        if (n_items)
            hipLaunchKernelGGL(layers, dim3(n_items), dim3(kNT), 8 * kTilePix * nl, st, f, cam, lv, rows, grid, K, l0, nl,
                               delta, rdelta, acc);
        hipLaunchKernelGGL(k_dom_texels, dim3(f.T), dim3(kNT), 0, st, f, cam.W, K, l0, nl, acc, tex);
    }
    return hipGetLastError();
}

BinPlan bin_plan(int32_t nseg, int32_t T, bool wide) {
    BinPlan p;
    p.lanes = wide ? kBinLanes : 1;
    p.range = std::min(T, kMaxLdsTiles);
    const int bytes = 4 * p.range;
    const int per_cu = std::max(1, std::min(2, (160 * 1024) / (bytes + 2048)));
    long nb = 256L * per_cu;
    nb = std::min(nb, std::max(32L, (long)((1 << 24) / std::max(T, 1))));
    nb = std::min(nb, std::max(1L, ((long)nseg * p.lanes + kBinThreads - 1) / kBinThreads));
    p.nb = (int)std::max(1L, nb);
    p.per_block = (nseg + p.nb - 1) / p.nb;
    return p;
}

// Dynamic LDS above 64 KiB is declared to the runtime first (gfx950 has 160 KiB per CU); a
// runtime that needs no declaration may refuse the call, and the launch itself then decides.
static hipError_t allow_lds(const void* fn, int bytes) {
    if (bytes > 64 * 1024 && hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess)
        (void)hipGetLastError();
    return hipSuccess;
}

hipError_t launch_bins(const SegRec* seg, int32_t nseg, const CamConst& cam, const BinPlan& p, bool areas, uint32_t* M,
                       BlockStats* blk, uint32_t* tot, Counters* ctr, hipStream_t st) {
    const int ntx = (cam.W + kTile - 1) / kTile, nty = (cam.H + kTile - 1) / kTile, T = ntx * nty;
    auto kernel = p.lanes > 1 ? &k_bin_count<kBinLanes, false> : areas ? &k_bin_count<1, true> : &k_bin_count<1, false>;
    hipError_t e = allow_lds(reinterpret_cast<const void*>(kernel), 4 * p.range);
    if (e != hipSuccess) return e;
    for (int t0 = 0; t0 < T; t0 += p.range) {
        const int nt = std::min(p.range, T - t0);
        hipLaunchKernelGGL(kernel, dim3(p.nb), dim3(kBinThreads), 4 * nt, st, seg, nseg, p.per_block, ntx, nty,
                           t0, nt, M, blk);
    }
    hipLaunchKernelGGL(k_bin_offsets, dim3(blocks_for(T, 64)), dim3(1024), 0, st, M, p.nb, T, tot, blk, ctr, areas);
    return hipGetLastError();
}

// One block scans 4096 counts in about 2.3 us, so above some 16 k the three launches of the chunked scan
// (about 12 us) are faster (65,536 tessellated segments: 36 -> 12 us).
constexpr int kScanOneLaunch = 1 << 14;
hipError_t launch_exscan(const uint32_t* cnt, uint32_t* start, int32_t n, uint32_t* scratch, hipStream_t st) {
    if (n <= kScanOneLaunch) {
        hipLaunchKernelGGL(k_scan1, dim3(1), dim3(1024), 0, st, cnt, start, n);
        return hipGetLastError();
    }
    const int nb = (n + kScanChunk - 1) / kScanChunk;
    uint32_t* part = scratch;            // [nb]
    uint32_t* base = scratch + nb + 1;   // [nb + 1]
    hipLaunchKernelGGL(k_scan_local, dim3(nb), dim3(1024), 0, st, cnt, start, part, n);
    hipLaunchKernelGGL(k_scan1, dim3(1), dim3(1024), 0, st, part, base, nb);
    hipLaunchKernelGGL(k_scan_add, dim3(nb), dim3(1024), 0, st, start, base, n, nb);
    return hipGetLastError();
}

hipError_t launch_scatter(const FrameBufs& f, int32_t nseg, const CamConst& cam, const BinPlan& p, const uint32_t* M,
                          uint32_t* list, float* rgba, unsigned long long* acc, size_t n_acc, uint2* item_tab,
                          uint32_t cap_items, hipStream_t st) {
    const int ntx = (cam.W + kTile - 1) / kTile, nty = (cam.H + kTile - 1) / kTile, T = ntx * nty;
    auto kernel = p.lanes > 1 ? &k_scatter<kBinLanes> : &k_scatter<1>;
    hipError_t e = allow_lds(reinterpret_cast<const void*>(kernel), 4 * p.range);
    if (e != hipSuccess) return e;
    const FillArgs fill{f.pix_cnt, f.pix_off, f.pix_kmin, f.pix_kmax, f.opaque ? 0xFFFFFFFFu : 0u, f.pix_thick,
                        reinterpret_cast<float4*>(rgba), rgba ? (size_t)cam.W * cam.H : 0,
                        reinterpret_cast<uint4*>(acc), n_acc / 2, f.item_start, item_tab, cap_items};
    // (a block per 8 tiles keeps the clearing spread over the chip whatever the segment count)
    for (int t0 = 0; t0 < T; t0 += p.range) {
        const int nt = std::min(p.range, T - t0);
        const int grid = t0 == 0 ? std::max(p.nb, std::min(256, blocks_for(T, 8))) : p.nb;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kBinThreads), 4 * nt, st, f.seg, nseg, p.per_block, p.nb, ntx, nty,
                           t0, nt, f.tile_start, M, list, f.ctr, fill);
    }
    return hipGetLastError();
}

hipError_t launch_lists_scan(const uint32_t* tot, int T, uint32_t* tile_start, uint32_t* item_start, Counters* ctr,
                             uint32_t cap_pairs, uint32_t cap_items, hipStream_t st) {
    hipLaunchKernelGGL(k_lists_scan, dim3(2), dim3(1024), 0, st, tot, T, tile_start, item_start, ctr, cap_pairs,
                       cap_items);
    return hipGetLastError();
}

hipError_t launch_tile_scans(const FrameBufs& f, uint32_t* frag_base, uint32_t* batch_start, uint32_t cap_frags,
                             uint32_t cap_batches, hipStream_t st) {
    hipLaunchKernelGGL(k_tile_scans, dim3(3), dim3(1024), 0, st, f.tile_tot, frag_base, f.tile_nb, batch_start, f.T,
                       f.ctr, cap_frags, cap_batches, f.tile_all);
    return hipGetLastError();
}

hipError_t launch_sum_tiles(const FrameBufs& f, hipStream_t st) {
    hipLaunchKernelGGL(k_sum_tiles, dim3(1), dim3(1024), 0, st, f);
    return hipGetLastError();
}

hipError_t launch_tile_items(const uint32_t* tile_start, int T, uint32_t* items, Counters* ctr, hipStream_t st) {
    hipLaunchKernelGGL(k_tile_items, dim3(blocks_for(T, 256)), dim3(256), 0, st, tile_start, T, items, ctr);
    return hipGetLastError();
}

template <bool TRIM>
static void launch_count_trim(const FrameBufs& f, const CamConst& cam, uint32_t grid, uint32_t most, hipStream_t st) {
    const dim3 b(kNT);
    if (f.opaque == 0) {
        hipLaunchKernelGGL((k_count<TRIM, false, false>), dim3(grid), b, 0, st, f, cam);
    } else if (f.opaque == 1) {
        hipLaunchKernelGGL(k_opaque<false>, dim3(grid), b, 0, st, f, cam, 1);
        hipLaunchKernelGGL(k_opaque<false>, dim3(grid), b, 0, st, f, cam, 0);
        hipLaunchKernelGGL((k_count<TRIM, true, false>), dim3(grid), b, 0, st, f, cam);
    } else {
        const dim3 few(std::min(grid, std::min(most, 12288u)));
        hipLaunchKernelGGL(k_opaque<true>, few, b, 0, st, f, cam, 1);
        hipLaunchKernelGGL(k_opaque<true>, few, b, 0, st, f, cam, 0);
        hipLaunchKernelGGL((k_count<TRIM, true, true>), dim3(grid), b, 0, st, f, cam);
    }
}
// Mixed frames (f.opaque == 2) launch the opaque pass, and the device chooses whether it only leaves.  Its
// blocks then take items in turn, so that there are few to leave (a warm grid has the size of the largest
// frame so far: 20 k blocks that leave took 8 us, 12288 take 4.6), and enough for items of very different
// cost (both launches of a frame of 14 k items: 4608 blocks 57 us, 12288 50, a block each without a choice
// 45).  The count pass is one kernel for both, with the LDS of frames that hide: a frame of 18 M fragments
// that does not takes 10 us more than with a kernel of its own (six blocks per CU instead of eight), one
// that does is spared that kernel's launch, 5 us.
hipError_t launch_count(const FrameBufs& f, const CamConst& cam, uint32_t grid, int32_t rows, hipStream_t st) {
    if (grid == 0) return hipSuccess;
    const uint32_t most = std::max(1024u, (uint32_t)rows / 16);
    if (f.trim) launch_count_trim<true>(f, cam, grid, most, st);
    else launch_count_trim<false>(f, cam, grid, most, st);
    return hipGetLastError();
}

hipError_t launch_tile_prep(const FrameBufs& f, hipStream_t st) {
    hipLaunchKernelGGL(k_tile_prep, dim3(f.T), dim3(kNT), 0, st, f);
    return hipGetLastError();
}

hipError_t launch_batch_records(const FrameBufs& f, hipStream_t st) {
    if (!f.pix_thick) return hipSuccess;   // (k_emit wrote them)
    hipLaunchKernelGGL(k_batch_records, dim3(f.T), dim3(kNT), 0, st, f);
    return hipGetLastError();
}

hipError_t launch_emit(const FrameBufs& f, const CamConst& cam, uint32_t grid, hipStream_t st) {
    if (grid == 0) return hipSuccess;
    const dim3 g(grid), b(kNT);
    if (f.pix_thick && f.opaque) hipLaunchKernelGGL((k_emit<true, true>), g, b, 0, st, f, cam);
    else if (f.pix_thick) hipLaunchKernelGGL((k_emit<true, false>), g, b, 0, st, f, cam);
    else if (f.opaque) hipLaunchKernelGGL((k_emit<false, true>), g, b, 0, st, f, cam);
    else hipLaunchKernelGGL((k_emit<false, false>), g, b, 0, st, f, cam);
    return hipGetLastError();
}

hipError_t launch_batches(const FrameBufs& f, const LevelDev& lv, const CamConst& cam, const LightsConst& lights,
                          const MatConst& mat, uint32_t n_batches, float* rgba, const DebugDump* dbg, hipStream_t st) {
    // n_batches: the grid (at least the frame's batch count, which the kernels read)
    if (n_batches == 0) return hipSuccess;
    ShadeArgs a;
    a.cam = cam;
    a.lights = lights;
    a.mat = mat;
    a.seg = f.seg;
    a.shade = f.shade;
    DebugDump d = dbg ? *dbg : DebugDump{};
    const int hd = dbg ? 1 : 0;
    const dim3 g(n_batches), b(kNT);
    bool shadow = false;
    for (int i = 0; i < lights.n; ++i) shadow |= lights.dom[i].grid != nullptr;
    if (lv.kind != 2) {
        if (shadow) {
            if (mat.model == 0) {
                if (lv.kind == 0) hipLaunchKernelGGL((k_batch<0, 0, true>), g, b, 0, st, f, a, rgba, d, hd);
                else hipLaunchKernelGGL((k_batch<1, 0, true>), g, b, 0, st, f, a, rgba, d, hd);
            } else {
                if (lv.kind == 0) hipLaunchKernelGGL((k_batch<0, 1, true>), g, b, 0, st, f, a, rgba, d, hd);
                else hipLaunchKernelGGL((k_batch<1, 1, true>), g, b, 0, st, f, a, rgba, d, hd);
            }
        } else if (mat.model == 0) {
            if (lv.kind == 0) hipLaunchKernelGGL((k_batch<0, 0, false>), g, b, 0, st, f, a, rgba, d, hd);
            else hipLaunchKernelGGL((k_batch<1, 0, false>), g, b, 0, st, f, a, rgba, d, hd);
        } else {
            if (lv.kind == 0) hipLaunchKernelGGL((k_batch<0, 1, false>), g, b, 0, st, f, a, rgba, d, hd);
            else hipLaunchKernelGGL((k_batch<1, 1, false>), g, b, 0, st, f, a, rgba, d, hd);
        }
        return hipGetLastError();
    }
    // A mixed frame: the strand-only batches (KIND 3), then those holding thick-hair fragments
    // (KIND 2); the kernels choose between them on the device (see k_batch).
    if (shadow) {
        if (mat.model == 0) {
            hipLaunchKernelGGL((k_batch<3, 0, true>), g, b, 0, st, f, a, rgba, d, hd);
            hipLaunchKernelGGL((k_batch<2, 0, true>), g, b, 0, st, f, a, rgba, d, hd);
        } else {
            hipLaunchKernelGGL((k_batch<3, 1, true>), g, b, 0, st, f, a, rgba, d, hd);
            hipLaunchKernelGGL((k_batch<2, 1, true>), g, b, 0, st, f, a, rgba, d, hd);
        }
    } else if (mat.model == 0) {
        hipLaunchKernelGGL((k_batch<3, 0, false>), g, b, 0, st, f, a, rgba, d, hd);
        hipLaunchKernelGGL((k_batch<2, 0, false>), g, b, 0, st, f, a, rgba, d, hd);
    } else {
        hipLaunchKernelGGL((k_batch<3, 1, false>), g, b, 0, st, f, a, rgba, d, hd);
        hipLaunchKernelGGL((k_batch<2, 1, false>), g, b, 0, st, f, a, rgba, d, hd);
    }
    return hipGetLastError();
}

hipError_t launch_lod_init(const HierDev& h, const CamConst& cam, float eps_w, int32_t* levels, hipStream_t st) {
    const int gk = h.G * h.S;
    if (gk == 0) return hipSuccess;
    hipLaunchKernelGGL(k_lod_init, dim3((gk + 3) / 4), dim3(256), 0, st, h, cam, eps_w, levels);
    return hipGetLastError();
}

hipError_t launch_lod_update(const HierDev& h, const CamConst& cam, float eps_w, int32_t* levels, hipStream_t st) {
    const int gk = h.G * h.S;
    if (gk == 0) return hipSuccess;
    hipLaunchKernelGGL(k_lod_update, dim3((gk + 3) / 4), dim3(256), 0, st, h, cam, eps_w, levels);
    return hipGetLastError();
}

hipError_t launch_select(const HierDev& h, const int32_t* levels, uint32_t* cnt, uint32_t* sel_start,
                         uint32_t* scan_tmp, hipStream_t st) {
    const int gk = h.G * h.S;
    if (gk <= kScanOneBlock) {
        hipLaunchKernelGGL(k_select, dim3(1), dim3(1024), 0, st, h, levels, sel_start);
        return hipGetLastError();
    }
    hipError_t e = launch_fill_u32(sel_start + gk + 1, 0u, 2, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sel_count, dim3(blocks_for(gk, 256)), dim3(256), 0, st, h, levels, cnt, sel_start + gk + 1);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return launch_exscan(cnt, sel_start, gk, scan_tmp, st);
}

hipError_t launch_select_fill(const HierDev& h, const int32_t* levels, const uint32_t* sel_start, uint32_t* sel,
                              hipStream_t st) {
    const int gk = h.G * h.S;
    hipLaunchKernelGGL(k_sel_fill, dim3((gk + 3) / 4), dim3(256), 0, st, h, levels, sel_start, sel);
    return hipGetLastError();
}

hipError_t launch_project_mixed(const HierDev& h, const uint32_t* sel, int32_t nsel, const CamConst& cam, SegRec* seg,
                                ShadeRec* shade, hipStream_t st) {
    if (nsel == 0) return hipSuccess;
    hipLaunchKernelGGL(k_project_mixed, dim3(blocks_for(nsel, 256)), dim3(256), 0, st, h, sel, nsel, cam, seg, shade);
    return hipGetLastError();
}

hipError_t launch_batches_bwd(const FrameBufs& f, const LevelDev& lv, const CamConst& cam, const LightsConst& lights,
                              const MatConst& mat, uint32_t n_batches, const GradOut& grad, hipStream_t st) {
    if (n_batches == 0) return hipSuccess;
    ShadeArgs a;
    a.cam = cam;
    a.lights = lights;
    a.mat = mat;
    a.seg = f.seg;
    a.shade = f.shade;
    if (mat.model == 0)
        hipLaunchKernelGGL(k_batch_bwd<0>, dim3(n_batches), dim3(kNT), 0, st, f, a, grad, lv.S, lv.n_owner);
    else
        hipLaunchKernelGGL(k_batch_bwd<1>, dim3(n_batches), dim3(kNT), 0, st, f, a, grad, lv.S, lv.n_owner);
    return hipGetLastError();
}

hipError_t launch_build_centers(const float* vx, const float* vy, const float* vz, const float* width, const float* sig,
                                int32_t n_strands, int32_t V, const int32_t* members, const int32_t* member_start,
                                int32_t K, float* cx, float* cy, float* cz, float* r, float* csig, int32_t* n_total,
                                hipStream_t st) {
    hipLaunchKernelGGL(k_build_centers, dim3(blocks_for((size_t)K * V, 128)), dim3(128), 0, st, vx, vy, vz, width, sig,
                       n_strands, V, members, member_start, K, cx, cy, cz, r, csig, n_total);
    return hipGetLastError();
}

hipError_t launch_build_ellipses(const float* vx, const float* vy, const float* vz, int32_t V, const int32_t* members,
                                 const int32_t* member_start, int32_t K, const float* cx, const float* cy,
                                 const float* cz, const float* r, float* ahat, float* axes, hipStream_t st) {
    hipLaunchKernelGGL(k_build_ellipses, dim3(blocks_for((size_t)K * (V - 1), 128)), dim3(128), 0, st, vx, vy, vz, V,
                       members, member_start, K, cx, cy, cz, r, ahat, axes);
    return hipGetLastError();
}

hipError_t launch_check_caps(const FrameBufs& f, const FrameCaps& caps, int stage, hipStream_t st) {
    hipLaunchKernelGGL(k_check_caps, dim3(1), dim3(64), 0, st, f, caps, stage);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t v, size_t n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u32, dim3(min(blocks_for(n, 256), 4096)), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

// Issue-rate probe: every lane runs `iters` rounds of 8 independent chains of one instruction
// (0: v_fma_f32, 1: v_exp_f32, 2: v_rcp_f32, 3: v_sqrt_f32, 4: v_mul_lo_u32, 5: v_mul_u32_u24),
// so that the rate, not the latency, bounds the kernel.  The chains stay finite and bounded
// (exp2 of a value in [-1, 0], rcp alternating, sqrt toward 1, integer products wrapping);
// their sum is stored only if it equals an impossible value, which keeps them live.
template <int KIND>
__global__ __launch_bounds__(256) void k_probe_rate(float* __restrict__ out, int iters) {
    float a[8];
    uint32_t u[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        a[i] = 0.5f + 1e-3f * (float)(threadIdx.x & 63) + 0.01f * (float)i;
        u[i] = threadIdx.x * 8u + (uint32_t)i + 1u;
    }
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (KIND == 0) a[i] = __builtin_fmaf(a[i], 0.999f, 1e-4f);
            if (KIND == 1) a[i] = __builtin_amdgcn_exp2f(-a[i]);
            if (KIND == 2) a[i] = __builtin_amdgcn_rcpf(a[i]);
            if (KIND == 3) a[i] = __builtin_amdgcn_sqrtf(a[i]);
            if (KIND == 4) u[i] = u[i] * 0x9E3779B1u;
            if (KIND == 5) u[i] = __umul24(u[i], 0x3779B1u);
        }
    }
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) sum += a[i] + (float)u[i];
    if (sum == -1.0f) out[0] = sum;
}

hipError_t launch_probe_rate(int kind, int blocks, int iters, float* out, hipStream_t st) {
    switch (kind) {
        case 0: hipLaunchKernelGGL(k_probe_rate<0>, dim3(blocks), dim3(256), 0, st, out, iters); break;
        case 1: hipLaunchKernelGGL(k_probe_rate<1>, dim3(blocks), dim3(256), 0, st, out, iters); break;
        case 2: hipLaunchKernelGGL(k_probe_rate<2>, dim3(blocks), dim3(256), 0, st, out, iters); break;
        case 3: hipLaunchKernelGGL(k_probe_rate<3>, dim3(blocks), dim3(256), 0, st, out, iters); break;
        case 4: hipLaunchKernelGGL(k_probe_rate<4>, dim3(blocks), dim3(256), 0, st, out, iters); break;
        default: hipLaunchKernelGGL(k_probe_rate<5>, dim3(blocks), dim3(256), 0, st, out, iters); break;
    }
    return hipGetLastError();
}

hipError_t launch_set3(const Arrays3& a, hipStream_t st) {
    const size_t n = std::max(a.n[0], std::max(a.n[1], a.n[2]));
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_set3, dim3(min(blocks_for(n, 256), 4096)), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_fill_f32(float* p, float v, size_t n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_f32, dim3(min(blocks_for(n, 256), 4096)), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

}  // namespace hair
