// Per-fragment scattering on the device: single fibre (R / TT / TRT) and the aggregated
// thick-hair model.  Written once as templates over the scalar type so the forward pass
// (float) and the backward pass (forward-mode dual numbers) share the definition.
//
//   f_single = sum_p A_p M_p N_p                      (Sec. 3.1, eq. bcsdf; Marschner lobes)
//   f_ours   = S (sum_p A_p M_p N_p + A_B M_B N_B)     (Sec. 4, eq. our_bcsdf)
//
// Lobe definitions (the readings the library fixes where the paper prints none):
//   M_p = 1/2 G(beta_p, theta_h - alpha_p), G a Gaussian with standard deviation beta;
//   N_p = logistic of standard deviation beta_n about Phi(p, h) = 2 p gamma_t - 2 gamma_o + p pi,
//         trimmed to [-pi, pi] and renormalised;
//   A_R = F, A_TT = (1 - F)^2 T, A_TRT = (1 - F)^2 F T^2 with Fresnel F at cos(x_d) cos(gamma_o),
//         Bravais index eta' = sqrt(eta^2 - sin^2 x_d) / cos x_d, T = exp(-sigma_a 2 cos gamma_t / cos theta_t),
//         x_d = |theta_i - theta_o| / 2.
// Thick hairs (Sec. 4): A_p = a_F^{n-1} a_p, variances add (beta^2 + (n-1) sigma_f^2), a_F / a_B
// are 8-node Gauss-Legendre h-averages of the single-fibre albedos toward |phi| > pi/2 /
// |phi| < pi/2, A_B = A_1+ + A_1 + A_3 with d_1+ = 0.6, N_B = [|phi| < pi/2] / pi,
// S = P_s a_F + max(0, 1 - P_m - P_s) for |phi| < pi/2 with c_m = 0.2, and n = 1 for
// |phi| < pi/2 or a single-hair cluster.
//
// R / TT / D model (Sec. 3.1 eq. bcsdf with constant RGB attenuations A_R, A_TT, A_D; Sec. 4
// modified lobes): M_R = 1/2 G(beta_R, theta_h), N_R = 1 / (2 pi); M_TT = 1/2 G(beta_TT,
// theta_h), N_TT = G(gamma_TT, phi - pi); M_D = 1 / pi, N_D = 1 / (2 pi).  For thick hairs the
// three lobes take a_F^{n-1} and variances widened by (n-1) sigma_f^2; a_F, a_B, sigma_f^2 and
// sigma_b^2 do not depend on the view and are folded on the host.  The B lobe and S are shared
// with the Marschner variant.
//
// Float arithmetic: the scattering terms use the hardware exp2 / reciprocal / square-root
// instructions and fitted polynomials for arcsine and arctangent (coefficients and error
// bounds in hair_fastmath_coef.h); every such step is within a few float32 ulps, far inside the
// renderer's radiance tolerance.  The view angles enter through sin / cos products (x_d from
// cos(theta_i - theta_o) by the half-angle identities), so no trigonometric call remains.
//
// Azimuths are kept in turns (angle / 2 pi): the wrap to half a turn is one subtraction of the
// nearest whole number, and the multiples of pi in the exit azimuths are exact.
#pragma once

#include <type_traits>

#include "hair_internal.h"
#include "hair_fastmath_coef.h"

// Multiply-adds in the scattering terms may fuse (one rounding instead of two); nothing here
// decides an integer.  The library's other code is compiled without contraction.
#pragma clang fp contract(fast)

namespace hair {

constexpr float kPi = 3.14159265358979323846f;
constexpr float kHalfPi = 1.57079632679489661923f;
constexpr float kTwoPi = 6.28318530717958647692f;
constexpr float kInvTwoPi = 0.15915494309189533577f;
constexpr float kInvPi = 0.31830988618379067154f;
constexpr float kInvTwoPi2 = 0.05066059182116888572f;   // 1 / (2 pi^2) = M_D N_D
constexpr float kInvSqrt2Pi = 0.39894228040143267794f;
constexpr float kLog2e = 1.44269504088896340736f;
constexpr float kSqrt3 = 1.73205080756887729353f;
constexpr float kD1Plus = 0.6f;     // Sec. 4, A_1+ path-series constant
constexpr float kCm = 0.2f;         // Sec. 4, multiple-hair shadowing constant

// ---- float function set; the dual-number type provides the same names ----
__device__ inline float m_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ inline float m_exp_half(float x) { return __builtin_amdgcn_exp2f((-0.5f * kLog2e) * x); }   // exp(-x / 2)
__device__ inline float m_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ inline float m_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline float m_div(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }
__device__ inline float m_rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }

// arcsine on [-1, 1]: polynomial on [0, 1/2], asin(x) = pi/2 - 2 asin(sqrt((1 - x) / 2)) above
__device__ inline float m_asin(float x) {
    const float ax = fabsf(x);
    const bool big = ax > 0.5f;
    const float t = big ? 0.5f * (1.0f - ax) : ax * ax;
    const float z = big ? __builtin_amdgcn_sqrtf(t) : ax;
    float p = kAsinP[4];
    p = p * t + kAsinP[3];
    p = p * t + kAsinP[2];
    p = p * t + kAsinP[1];
    p = p * t + kAsinP[0];
    float r = z + (z * t) * p;
    r = big ? kHalfPi - 2.0f * r : r;
    return copysignf(r, x);
}

// asin of an offset refracted into the fibre, |x| <= 1 / eta: from eta = 1.4706 on one polynomial
// covers it without the half-angle step (8 terms instead of 5, a square root and four selects).
__device__ inline float m_asin_refracted(float x, const MatConst& m) {
    if (m.eta < 1.4706f) return m_asin(x);
    const float t = x * x;
    float p = kAsinW[7];
#pragma unroll
    for (int i = 6; i >= 0; --i) p = p * t + kAsinW[i];
    return x + (x * t) * p;
}

// atan2 by octant reduction to atan(a), a in [0, 1]: the angle of (|x|, |y|) in the first quadrant,
// in the unit of Q's polynomial, with quarter a quarter of a turn.
__device__ inline float atan_quadrant(float ax, float ay, const float (&Q)[9], float quarter) {
    const float mx = fmaxf(ax, ay), mn = fminf(ax, ay);
    const float a = mx > 0.0f ? mn * __builtin_amdgcn_rcpf(mx) : 0.0f;
    const float t = a * a;
    float q = Q[8];
#pragma unroll
    for (int i = 7; i >= 0; --i) q = q * t + Q[i];
    const float r = a * q;
    return ay > ax ? quarter - r : r;
}

// half of atan2
__device__ inline float m_half_atan2(float y, float x) {
    const float r = atan_quadrant(fabsf(x), fabsf(y), kAtanHalfQ, 0.5f * kHalfPi);
    return copysignf(x < 0.0f ? kHalfPi - r : r, y);
}

// tanh on x >= 0: polynomial up to 5/8, 1 - 2 / (e^2x + 1) above
__device__ inline float m_tanh(float x) {
    const float t = x * x;
    float p = kTanhH[4];
#pragma unroll
    for (int i = 3; i >= 0; --i) p = p * t + kTanhH[i];
    const float big = 1.0f - 2.0f * __builtin_amdgcn_rcpf(__builtin_amdgcn_exp2f(x * (2.0f * kLog2e)) + 1.0f);
    return x > 0.625f ? big : x + (x * t) * p;
}
__device__ inline float m_abs(float x) { return fabsf(x); }
// x^y for x >= 0 (0^0 = 1)
__device__ inline float m_pow(float x, float y) {
    if (y == 0.0f) return 1.0f;
    if (x == 0.0f) return 0.0f;
    return __builtin_amdgcn_exp2f(y * __builtin_amdgcn_logf(x));
}
__device__ inline float m_min(float a, float b) { return fminf(a, b); }
__device__ inline float m_max(float a, float b) { return fmaxf(a, b); }
__device__ inline float m_val(float x) { return x; }

template <class T> struct V3 { T x, y, z; };
template <class T> __device__ inline V3<T> v3(T x, T y, T z) { return {x, y, z}; }
template <class T> __device__ inline T dot(const V3<T>& a, const V3<T>& b) { return (a.x * b.x + a.y * b.y) + a.z * b.z; }
template <class T> __device__ inline V3<T> cross(const V3<T>& a, const V3<T>& b) {
    return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
template <class T> __device__ inline V3<T> sub(const V3<T>& a, const V3<T>& b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
template <class T, class S> __device__ inline V3<T> scale(const V3<T>& a, S s) { return {a.x * s, a.y * s, a.z * s}; }

template <class T> __device__ inline T clampv(T x, float lo, float hi) { return m_min(m_max(x, T(lo)), T(hi)); }

// Gaussian of variance v at x
template <class T> __device__ inline T gaussian(T v, T x) {
    const T ib = m_rsqrt(v);
    return m_exp_half((x * x) * (ib * ib)) * (kInvSqrt2Pi * ib);
}

// the azimuth x (turns) wrapped to [-1/2, 1/2]
__device__ inline float wrap_turn(float x) { return x - rintf(x); }
template <class T> __device__ inline T wrap_turn(T x) { return x - rintf(m_val(x)); }

// logistic density of scale s trimmed to half a turn each way, at x turns; k = 2 pi log2(e) / s,
// norm = 1 / (s tanh(pi / 2s))
template <class T> __device__ inline T trimmed_logistic(T x, T k, T norm) {
    T e = m_exp2(-m_abs(x) * k);
    T one_e = 1.0f + e;
    return e * norm * m_rcp(one_e * one_e);
}

// A lobe's masses toward |phi| < pi/2 (back) and |phi| > pi/2 (front), its exit azimuth at y turns:
// the 2 pi-periodic trimmed logistic of the material's scale s over the half turn about the light.
// With r = |wrap(y)| the half turn that holds the lobe's centre reaches a = 2 pi |r - 1/4| beyond it
// on one side and pi - a on the other, and the logistic's difference over it, renormalised by
// tanh(pi / 2s), is (1 + K) / (1 + K + e^(-a/s) + e^(-(pi-a)/s)), K = e^(-pi/s): one reciprocal for
// both masses, and no difference of numbers near 1.
__device__ inline void hemisphere_masses(float y, const MatConst& m, float& back, float& front) {
    const float a = m.n_k2 * fabsf(wrap_turn(y)) - 0.25f * m.n_k2;    // log2(e) a / s, negative: centre behind
    const float outer = m_exp2(-fabsf(a)) + m_exp2(fabsf(a) - 0.5f * m.n_k2);
    const float r = m_rcp(m.one_k + outer);
    const float in = m.one_k * r, out = outer * r;
    back = a <= 0.0f ? in : out;
    front = a <= 0.0f ? out : in;
}

// (one reciprocal of the product of the two denominators, both at least cos theta_t > 0)
template <class T> __device__ inline T fresnel(T cos_i, const MatConst& m) {
    T sin2_t = (1.0f - cos_i * cos_i) * m.inv_eta2;
    T cos_t = m_sqrt(1.0f - sin2_t);
    T ec = m.eta * cos_t, ei = m.eta * cos_i;
    T ds = cos_i + ec, dp = ei + cos_t;
    T inv = m_rcp(ds * dp);
    T rs = (cos_i - ec) * dp * inv;
    T rp = (ei - cos_t) * ds * inv;
    return 0.5f * (rs * rs + rp * rp);
}

// View/light geometry of one fragment and light (independent of the fitted parameters).
struct LightView {
    float theta_h;     // (theta_i + theta_o) / 2
    float cos_ti;      // cos theta_i (irradiance foreshortening)
    float phi;         // relative azimuth, in turns
    float phi_opp;     // the azimuth about the opposite direction, phi - 1/2 wrapped
    float cos_phi;
    float sxd2, cxd;   // sin^2 x_d, cos x_d
    float inv_eta_p;   // 1 / eta' (Bravais index at x_d)
    float inv_ctt;     // 1 / cos theta_t, sin theta_t = sin x_d / eta
};

// sin_ti / sin_to: sines of the longitudinal angles (cos_to = cos theta_o >= 0); wx, wy: light
// direction in the normal plane, so that cos theta_i = |(wx, wy)| (taken from the components,
// not from 1 - sin^2).  theta_h = (theta_i + theta_o) / 2 is half the angle whose sine and
// cosine the sum formulas give (one arctangent per light; theta_o itself is not needed; the halving
// is in its coefficients).
// 1 / eta' = cos x_d / sqrt(eta^2 - sin^2 x_d) and 1 / cos theta_t = eta / sqrt(eta^2 - sin^2 x_d)
// share their square root.
__device__ inline LightView light_view(float sin_ti, float sin_to, float cos_to, float wx, float wy, bool degen,
                                       const MatConst& m) {
    LightView v;
    const float si = fminf(fmaxf(sin_ti, -1.0f), 1.0f);
    const float r2 = wx * wx + wy * wy;
    const float r_w = m_rsqrt(r2);
    const float ci = r2 > 0.0f ? r2 * r_w : 0.0f;
    v.cos_ti = ci;
    v.theta_h = m_half_atan2(si * cos_to + ci * sin_to, ci * cos_to - si * sin_to);
    const float c = fminf(fmaxf(ci * cos_to + si * sin_to, -1.0f), 1.0f);   // cos(theta_i - theta_o)
    v.sxd2 = 0.5f * (1.0f - c);
    v.cxd = m_sqrt(0.5f * (1.0f + c));
    const float r_e = m_rsqrt(m.eta * m.eta - v.sxd2);
    v.inv_eta_p = v.cxd * r_e;
    v.inv_ctt = m.eta * r_e;
    if (degen || !(r2 > 0.0f)) {
        v.phi = 0.0f;
        v.phi_opp = 0.5f;
        v.cos_phi = 1.0f;
    } else {
        // (both from the quadrant's angle: near the opposite direction, where the transmitted lobe
        // lies, phi_opp keeps the digits that phi rounds off)
        const float r = atan_quadrant(fabsf(wx), fabsf(wy), kAtanTurnsQ, 0.25f), o = 0.5f - r;
        v.phi = copysignf(wx < 0.0f ? o : r, -wy);
        v.phi_opp = copysignf(wx < 0.0f ? r : o, wy);
        v.cos_phi = wx * r_w;
    }
    return v;
}

// Refraction at offset h (incidence angle gamma_o = asin h, cos gamma_o given).  With the
// absorption transmittance T_c = exp2(-sigl_c path) of channel c (sigl: absorption times log2(e)),
// A_R = F, A_TT = (1 - F)^2 T_c and A_TRT = (1 - F)^2 F T_c^2: a sum over the three lobes is
// g_R x_R + T_c (g_TT x_TT + T_c g_TRT x_TRT) per channel, with g the channel-independent factors.
template <class T> struct Refraction {
    T g[3];         // F, (1 - F)^2, (1 - F)^2 F
    T path;
};

template <class T>
__device__ inline Refraction<T> refraction(const LightView& v, T sgt, T cgo, const MatConst& m) {
    Refraction<T> o;
    const T cgt = m_sqrt(1.0f - sgt * sgt);
    const T F = fresnel(v.cxd * cgo, m);
    const T one_f = 1.0f - F;
    o.path = (2.0f * v.inv_ctt) * cgt;
    o.g[0] = F;
    o.g[1] = one_f * one_f;
    o.g[2] = o.g[1] * F;
    return o;
}

// phi minus the exit azimuth Phi(p) = 2 p gamma_t - 2 gamma_o + p pi of the three lobes, wrapped
template <class T>
__device__ inline void lobe_azimuths(const LightView& v, const T& gamma_o, const T& gamma_t, T w[3]) {
    w[0] = wrap_turn(T(kInvPi * gamma_o + v.phi));
    w[1] = wrap_turn(T(kInvPi * (gamma_o - gamma_t) + v.phi_opp));
    w[2] = wrap_turn(T(kInvPi * (gamma_o - 2.0f * gamma_t) + v.phi));
}

// Single-fibre BCSDF, RGB (gamma_o = asin h, cgo = cos gamma_o).  M_p N_p's two amplitudes are one
// host constant.  About 200 instructions a light; the azimuths in turns and the single arcsine
// polynomial took 40 away (k_batch of 300k strands at 3840 x 2160: -3%) and halve the transmitted
// lobe's error.
template <class T>
__device__ inline void f_single(const LightView& v, T h, T gamma_o, T cgo, const T sigl[3], const MatConst& m,
                                T out[3]) {
    const T sgt = h * v.inv_eta_p;
    const Refraction<T> rf = refraction(v, sgt, cgo, m);
    T w[3], q[3];
    lobe_azimuths(v, gamma_o, m_asin_refracted(sgt, m), w);
    for (int p = 0; p < 3; ++p) {
        const float x = v.theta_h - m.alpha_p[p];
        const float M = m_exp2(-m.g_k2[p] * (x * x));
        const T e = m_exp2(-m_abs(w[p]) * m.n_k2);
        const T one_e = 1.0f + e;
        q[p] = rf.g[p] * ((m.mn_amp[p] * M) * (e * m_rcp(one_e * one_e)));
    }
    for (int c = 0; c < 3; ++c) {
        const T Tc = m_exp2(-sigl[c] * rf.path);
        out[c] = q[0] + Tc * (q[1] + Tc * q[2]);
    }
}

// Hemisphere albedos a_F, a_B (RGB) and variances sigma_f^2, sigma_b^2 at the light's x_d.
// The 8-node rule is symmetric in h and so is each node's contribution (h -> -h flips the
// sign of gamma_o, gamma_t and of every exit azimuth, which leaves the attenuations and the
// hemispheres' masses unchanged): the four nodes h > 0 are evaluated with doubled weights.  Only the
// transmittances depend on the fibre; everything else of a node is plain float in both directions,
// and the R lobe's masses, which no light changes, are host constants.  Bound by VALU issue: per node
// two lobes' masses, one Fresnel term and three exponentials instead of three lobes' differences of
// CDFs and nine products of attenuation and mass.  100k shadowed strands at 1080p: k_batch 1543 ->
// 1375 us, and with the nodes in a loop (no spills in the thick-hair kernels, 88 bytes instead of 124
// here) 1235 -> 1209; the fitting step's backward pass (500 thick hairs at 512 x 512) 124 -> 109 us.
__constant__ static const float kGLgof[4] = {(float)kGLgo[0], (float)kGLgo[1], (float)kGLgo[2], (float)kGLgo[3]};
template <class T>
__device__ inline void hemisphere_stats(const LightView& v, const T sigl[3], const MatConst& m, T aF[3], T aB[3],
                                        T& var_f, T& var_b) {
    float f0 = 0.0f, b0 = 0.0f;                          // the R lobe's sums, equal in all channels
    T f1(0.0f), f2(0.0f), b1(0.0f), b2(0.0f);            // TT and TRT, summed over the channels
    for (int c = 0; c < 3; ++c) aF[c] = aB[c] = T(0.0f);
    constexpr int kUnroll = std::is_same<T, float>::value ? 1 : 4;   // (unrolled, the float path spills)
#pragma unroll kUnroll
    for (int k = 0; k < 4; ++k) {
        const float sgt = kGLx[k] * v.inv_eta_p;
        const Refraction<float> rf = refraction(v, sgt, kGLcgo[k], m);
        const float go = kGLgof[k], gt = m_asin_refracted(sgt, m);
        float B1, F1, B2, F2;
        hemisphere_masses(0.5f - kInvPi * (go - gt), m, B1, F1);
        hemisphere_masses(kInvPi * (2.0f * gt - go), m, B2, F2);
        // (weights: 2 x (1/2 of the node weight on [-1, 1]))
        const float g0 = kGLw[k] * rf.g[0], g1 = kGLw[k] * rf.g[1], g2 = kGLw[k] * rf.g[2];
        const float uF1 = g1 * F1, uB1 = g1 * B1, uF2 = g2 * F2, uB2 = g2 * B2;
        f0 = f0 + g0 * m.r_front[k];
        b0 = b0 + g0 * m.r_back[k];
        T s1(0.0f), s2(0.0f);
        for (int c = 0; c < 3; ++c) {
            const T Tc = m_exp2(-sigl[c] * rf.path);
            const T Tc2 = Tc * Tc;
            aF[c] = aF[c] + Tc * uF1 + Tc2 * uF2;
            aB[c] = aB[c] + Tc * uB1 + Tc2 * uB2;
            s1 = s1 + Tc;
            s2 = s2 + Tc2;
        }
        f1 = f1 + s1 * uF1;
        f2 = f2 + s2 * uF2;
        b1 = b1 + s1 * uB1;
        b2 = b2 + s2 * uB2;
    }
    for (int c = 0; c < 3; ++c) {
        aF[c] = aF[c] + f0;
        aB[c] = aB[c] + b0;
    }
    const float v0 = m.beta_p[0] * m.beta_p[0], v1 = m.beta_p[1] * m.beta_p[1], v2 = m.beta_p[2] * m.beta_p[2];
    var_f = m_div(3.0f * f0 * v0 + f1 * v1 + f2 * v2, 3.0f * f0 + f1 + f2);
    var_b = m_div(3.0f * b0 * v0 + b1 * v1 + b2 * v2, 3.0f * b0 + b1 + b2);
}

// Thick-hair inputs of one fragment and light.
template <class T> struct ClusterFrag {
    T n_total;     // members
    T rho;         // hair density
    T n_F, n_B;    // hair counts toward / away from the light
};

// B lobe (A_1+ + A_1 + A_3 toward the back hemisphere) added to out, then the
// shadowing-masking factor S applied (Sec. 4; both only for clusters of two or more hairs).
template <class T>
__device__ inline void back_lobe_shadow(const LightView& v, const T aF[3], const T aB[3], const T& var_f,
                                        const T& var_b, const ClusterFrag<T>& cf, bool back_hemi, bool multi,
                                        T out[3]) {
    if (multi) {
        T A1[3], A3[3], A1p[3];
        T m1 = T(0.0f), m3 = T(0.0f), m1p = T(0.0f);
        for (int c = 0; c < 3; ++c) {
            T aF2 = aF[c] * aF[c];
            T iom = m_rcp(1.0f - aF2);
            A1[c] = aB[c] * aF2 * iom;
            A3[c] = aB[c] * aB[c] * aB[c] * aF2 * (iom * iom * iom);
            A1p[c] = kD1Plus * aB[c] * aF[c] * (1.0f - m_pow(aF[c], 2.0f * cf.n_B)) * iom;
            m1 = m1 + A1[c] * (1.0f / 3.0f);
            m3 = m3 + A3[c] * (1.0f / 3.0f);
            m1p = m1p + A1p[c] * (1.0f / 3.0f);
        }
        T varB = m_div(m1 * (var_b + 2.0f * var_f) + m3 * (3.0f * var_b + 2.0f * var_f) +
                           m1p * (var_b + (2.0f * cf.n_B - 1.0f) * var_f),
                       m1 + m3 + m1p);
        if (back_hemi) {
            T MB = 0.5f * gaussian(varB, T(v.theta_h)) * (1.0f / kPi);
            for (int c = 0; c < 3; ++c) out[c] = out[c] + (A1p[c] + A1[c] + A3[c]) * MB;
        }
    }
    if (back_hemi && multi) {
        T one_rho = 1.0f - cf.rho;
        T Ps = one_rho * (1.0f - v.cos_phi);
        T Pn = m_max(1.0f - kCm * one_rho - Ps, T(0.0f));
        for (int c = 0; c < 3; ++c) out[c] = (Ps * aF[c] + Pn) * out[c];
    }
}

// Aggregated BCSDF, RGB.
template <class T>
__device__ inline void f_ours(const LightView& v, T h, T gamma_o, T cgo, const T sigl[3], const MatConst& m,
                              const ClusterFrag<T>& cf, T out[3]) {
    const bool back_hemi = fabsf(v.phi) < 0.25f;
    const bool multi = m_val(cf.n_total) >= 2.0f;
    T aF[3], aB[3], var_f, var_b;
    hemisphere_stats(v, sigl, m, aF, aB, var_f, var_b);
    const T sgt = h * v.inv_eta_p;
    const Refraction<T> rf = refraction(v, sgt, cgo, m);
    T nm1 = cf.n_F - 1.0f;
    T extra = nm1 * var_f;
    T s_bar = (kSqrt3 * kInvPi) * m_sqrt(T(m.beta_n * m.beta_n) + extra);
    T inv_sb = m_rcp(s_bar);
    T norm = m_rcp(s_bar * m_tanh(kPi * 0.5f * inv_sb));
    T w[3], q[3];
    lobe_azimuths(v, gamma_o, m_asin_refracted(sgt, m), w);
    for (int p = 0; p < 3; ++p) {
        T M = 0.5f * gaussian(T(m.beta_p[p] * m.beta_p[p]) + extra, T(v.theta_h - m.alpha_p[p]));
        q[p] = rf.g[p] * (M * trimmed_logistic(w[p], inv_sb * (kTwoPi * kLog2e), norm));
    }
    for (int c = 0; c < 3; ++c) {
        const T Tc = m_exp2(-sigl[c] * rf.path);
        out[c] = m_pow(aF[c], nm1) * (q[0] + Tc * (q[1] + Tc * q[2]));
    }
    back_lobe_shadow(v, aF, aB, var_f, var_b, cf, back_hemi, multi, out);
}

// R / TT / D single fibre, RGB.  psi is the azimuth about the opposite direction.
template <class T>
__device__ inline void f_single_rttd(const LightView& v, const MatConst& m, T out[3]) {
    const float th2 = v.theta_h * v.theta_h;
    const float psi = kTwoPi * v.phi_opp;
    const float MNR = m.d_amp[0] * m_exp2(-m.d_k2[0] * th2) * kInvTwoPi;
    const float MNT = m.d_amp[1] * m_exp2(-(m.d_k2[1] * th2 + m.tt_k2 * (psi * psi))) * m.tt_amp;
    for (int c = 0; c < 3; ++c) out[c] = T(m.A[0][c] * MNR + m.A[1][c] * MNT + m.A[2][c] * kInvTwoPi2);
}

// Aggregated R^ / TT^ / D^ / B^ model, RGB.
template <class T>
__device__ inline void f_ours_rttd(const LightView& v, const MatConst& m, const ClusterFrag<T>& cf, T out[3]) {
    const bool back_hemi = fabsf(v.phi) < 0.25f;
    const bool multi = m_val(cf.n_total) >= 2.0f;
    const float psi = kTwoPi * v.phi_opp;
    T nm1 = cf.n_F - 1.0f;
    T extra = nm1 * m.var_f;
    T MNR = 0.5f * gaussian(T(m.d_beta2[0]) + extra, T(v.theta_h)) * kInvTwoPi;
    T MNT = 0.5f * gaussian(T(m.d_beta2[1]) + extra, T(v.theta_h)) *
            gaussian(T(m.gamma2) + extra, T(psi));
    T aF[3], aB[3];
    for (int c = 0; c < 3; ++c) {
        aF[c] = T(m.aF[c]);
        aB[c] = T(m.aB[c]);
        out[c] = m_pow(aF[c], nm1) * (m.A[0][c] * MNR + m.A[1][c] * MNT + m.A[2][c] * kInvTwoPi2);
    }
    back_lobe_shadow(v, aF, aB, T(m.var_f), T(m.var_b), cf, back_hemi, multi, out);
}

}  // namespace hair

#pragma clang fp contract(off)
