// qs_adjoint.hip -- derivatives of the energy histogram with respect to the
// eight shot parameters: the tangent kernel (adjoint, or forward pass with a
// derivative tape), the tape contraction and the per-shot reduction.
#include "qs_device.h"

namespace qs {

// ===========================================================================
// Adjoint: derivatives of a weighted sum of the energy histogram,
//   L = sum_k w_k H_k   (w = dL/dH from the caller),
// with respect to the eight shot parameters (a0, W0, x and y offsets, delay,
// gamma0, sigma_gamma, divergence).  Every sample's trajectory is integrated
// again together with its tangents: forward-mode derivatives of the discrete
// RK4 map itself, so no trajectory is stored.  The final tangents are
// contracted with the sample's sensitivities dL/dmu_f and dL/dsig2_f, taken
// from its deposited law; the sums over samples are reduced per work item and
// per shot in a fixed order.
//
// Tangent directions.  The sample state depends on the parameters through
// the amplitude a(psi) = a0 S(x_e, y_e, z_e) f(psi) cos psi along the path
// (Sec. 2, eq. a0eff) and through the initial energy.  gamma0 and
// sigma_gamma only enter the initial energy (mu_0 = gamma0 + sigma_gamma n3),
// so the sigma_gamma tangent is n3 times the gamma0 tangent.  With the
// amplitude frozen at a0,eff every amplitude direction forces the system
// with a multiple of S0 f cos psi, so one tangent serves a0 and the four
// geometric parameters.
// ===========================================================================
// Radiation functions in the combinations the Jacobian uses:
//   g,  E1 = 2g + G1,  E2 = 2g + 4 G1 + G2,  E3 = 6 G1 + 6 G2 + G3,  h,  H1
// (G1 = chi g', G2 = chi^2 g'', G3 = chi^3 g''', H1 = chi h').  The FP32
// derivative table stores these combinations; the FP64 one the plain
// functions.
template <class T>
struct RadJ {
    T g, E1, E2, E3, h, H1;
};

// One FP32 derivative-table cell in registers (see RadCell32).
struct RadCell6 {
    float4 q[kDerivFuncs];
    float tw, ts;
};

// Index from chi clamped to the octave cells, as rad_lookup32 (the first
// octave cell extrapolates linearly down to chi = 0).
__device__ __forceinline__ void rad6_lookup32(const float *__restrict__ tab, float chi,
                                              RadCell6 &cell) {
    const float xc = fminf(fmaxf(chi, 0x1p-20f), 0x1.fffffep7f);
    const uint32_t b = __float_as_uint(xc);
    const uint32_t c = ((b - ((uint32_t)(127 + kEMin) << 23)) >> (23 - kSB32)) + 1u;
    const float tw = __uint_as_float((uint32_t)(254 + kSB32 - (int)(b >> 23)) << 23);
    const float ts = -__uint_as_float(b & ~((1u << (23 - kSB32)) - 1)) * tw;
    const float4 *T = reinterpret_cast<const float4 *>(tab);
#pragma unroll
    for (int f = 0; f < kDerivFuncs; ++f) cell.q[f] = T[f * kCells32 + c];
    cell.tw = tw;
    cell.ts = ts;
}

__device__ __forceinline__ RadJ<float> rad6_cell_eval(const RadCell6 &cell, float chi) {
    const float t = fmaf(chi, cell.tw, cell.ts);
    float v[kDerivFuncs];
#pragma unroll
    for (int f = 0; f < kDerivFuncs; ++f) {
        const float4 &q = cell.q[f];
        v[f] = fmaf(t, fmaf(t, fmaf(t, q.w, q.z), q.y), q.x);
    }
    return RadJ<float>{v[0], v[1], v[2], v[3], v[4], v[5]};
}

// FP64 table, cell-major [cell][g, G1, G2, h, G3, H1][power]: the plain
// functions, combined here.
__device__ __forceinline__ void rad6_cell_eval64(const double *q, double t,
                                                 double v[kDerivFuncs]) {
#pragma unroll
    for (int f = 0; f < kDerivFuncs; ++f)
        v[f] = fma(t, fma(t, fma(t, q[4 * f + 3], q[4 * f + 2]), q[4 * f + 1]), q[4 * f]);
}

__device__ __forceinline__ void rad6_plain64(const double *__restrict__ tab, double chi,
                                             double v[kDerivFuncs]) {
    double t;
    const uint32_t c = min(rad_index64(chi, t), (uint32_t)kCells64 - 1);
    rad6_cell_eval64(tab + (size_t)c * (4 * kDerivFuncs), t, v);
}

__device__ __forceinline__ RadJ<double> radj_combine(const double v[kDerivFuncs]) {
    const double g = v[0], G1 = v[1], G2 = v[2], h = v[3], G3 = v[4], H1 = v[5];
    return RadJ<double>{g, fma(2.0, g, G1), fma(4.0, G1, fma(2.0, g, G2)), fma(6.0, G1 + G2, G3),
                        h, H1};
}

// Where a stage takes its radiation functions from.  FP32: the LDS table,
// read at stages 2 and 4 only -- stage 3 reuses stage 2's cell and the next
// step's stage 1 reuses stage 4's (as in the forward phase loop).  FP64: the
// table's window in LDS at every stage.
template <class T>
struct RadSrc;
template <>
struct RadSrc<float> {
    const float *tab;
    RadCell6 carry, mid;
    __device__ __forceinline__ void init(float chi) { rad6_lookup32(tab, chi, carry); }
    __device__ __forceinline__ RadJ<float> s1(float chi) { return rad6_cell_eval(carry, chi); }
    __device__ __forceinline__ RadJ<float> s2(float chi) {
        rad6_lookup32(tab, chi, mid);
        return rad6_cell_eval(mid, chi);
    }
    __device__ __forceinline__ RadJ<float> s3(float chi) { return rad6_cell_eval(mid, chi); }
    __device__ __forceinline__ RadJ<float> s4(float chi) {
        rad6_lookup32(tab, chi, carry);
        return rad6_cell_eval(carry, chi);
    }
};
template <>
struct RadSrc<double> {
    const TabWindow<kWinDeriv64, kDerivFuncs> *win;
    __device__ __forceinline__ void init(double) {}
    __device__ __forceinline__ RadJ<double> ev(double chi) {
        double v[kDerivFuncs];
        win->eval(chi, v);
        return radj_combine(v);
    }
    __device__ __forceinline__ RadJ<double> s1(double chi) { return ev(chi); }
    __device__ __forceinline__ RadJ<double> s2(double chi) { return ev(chi); }
    __device__ __forceinline__ RadJ<double> s3(double chi) { return ev(chi); }
    __device__ __forceinline__ RadJ<double> s4(double chi) { return ev(chi); }
};

__device__ __forceinline__ float recip(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double recip(double x) { return 1.0 / x; }

// Right-hand side f = (dmu/dpsi, dsig2/dpsi) of the moment system and its
// partial derivatives with respect to mu, sig2 and the amplitude a.  With
// chi d/dchi written D (D g = G1, D G1 = G1 + G2, D G2 = 2 G2 + G3,
// D h = H1) and u = K a^2:
//   f_mu  = -u (mu^2 g + sig2 E2 / 2),      f_s2 = -2 u mu sig2 E1 + C_D |a|^3 mu^4 h,
//   d f_mu / d mu   = -u (mu E1 + sig2 E3 / (2 mu)),
//   d f_mu / d sig2 = -u E2 / 2,
//   d f_s2 / d mu   = -2 u sig2 E2 + C_D |a|^3 mu^3 (4 h + H1),
//   d f_s2 / d sig2 = -2 u mu E1,
//   d f_mu / d a    = -K a (mu^2 E1 + sig2 (E2 + E3 / 2)),
//   d f_s2 / d a    = -2 K a mu sig2 (E1 + E2) + C_D a |a| mu^4 (3 h + H1).
// Classical model (g = 1, no diffusion; sig2 stays 0): f_mu = -u mu^2.
template <class T>
struct Jac {
    T fm, fs;  // f
    T mm, ms, sm, ss;  // d f / d (mu, sig2)
    T ma, sa;  // d f / d a
};

// Per-stage amplitude constants: a, K a, C_D a |a|, 2 |a| / a_S.
template <class T>
struct StageAmp {
    T a, Ka, cda, chi_per_mu;
    __device__ __forceinline__ StageAmp(T a_, const Phys<T> &ph)
        : a(a_), Ka(ph.K * a_), cda(ph.CD * a_ * fabs(a_)), chi_per_mu(ph.two_over_aS * fabs(a_)) {}
};

template <class T>
__device__ __forceinline__ Jac<T> jac_quantum(T mu, T s2, const StageAmp<T> &A, const RadJ<T> &r) {
    Jac<T> J;
    const T u = A.Ka * A.a;
    const T mu2 = mu * mu;
    const T hs = T(0.5) * s2;
    const T c3 = A.cda * mu2;        // C_D a |a| mu^2
    const T c3a = c3 * mu * A.a;     // C_D |a|^3 mu^3
    const T u2 = T(-2) * u;
    J.fm = -u * fma(mu2, r.g, hs * r.E2);
    J.fs = fma(u2 * mu * s2, r.E1, c3a * mu * r.h);
    J.mm = -u * fma(mu, r.E1, hs * r.E3 * recip(mu));
    J.ms = T(-0.5) * u * r.E2;
    J.sm = fma(u2 * s2, r.E2, c3a * fma(T(4), r.h, r.H1));
    J.ss = u2 * mu * r.E1;
    J.ma = -A.Ka * fma(mu2, r.E1, s2 * fma(T(0.5), r.E3, r.E2));
    J.sa = fma(T(-2) * A.Ka * mu * s2, r.E1 + r.E2, c3 * mu2 * fma(T(3), r.h, r.H1));
    return J;
}

template <class T>
__device__ __forceinline__ Jac<T> jac_classical(T mu, const StageAmp<T> &A) {
    Jac<T> J;
    const T u = A.Ka * A.a;
    J.fm = -u * mu * mu;
    J.mm = T(-2) * u * mu;
    J.ma = T(-2) * A.Ka * mu * mu;
    J.fs = J.ms = J.sm = J.ss = J.sa = T(0);
    return J;
}

// 2x2 matrices [[a, b], [c, d]] and 2-vectors acting on (mu, sig2); in the
// classical model only the mu entries are used.
template <class T>
struct Mat2 {
    T a, b, c, d;
};
template <class T>
struct Vec2 {
    T x, y;
};

// K (I + s M) = K + s K M
template <class T, bool Q>
__device__ __forceinline__ Mat2<T> kism(const Jac<T> &K, T s, const Mat2<T> &M) {
    Mat2<T> R;
    if (Q) {
        R.a = fma(s, fma(K.mm, M.a, K.ms * M.c), K.mm);
        R.b = fma(s, fma(K.mm, M.b, K.ms * M.d), K.ms);
        R.c = fma(s, fma(K.sm, M.a, K.ss * M.c), K.sm);
        R.d = fma(s, fma(K.sm, M.b, K.ss * M.d), K.ss);
    } else {
        R.a = fma(s, K.mm * M.a, K.mm);
        R.b = R.c = R.d = T(0);
    }
    return R;
}

// s K v
template <class T, bool Q>
__device__ __forceinline__ Vec2<T> skv(const Jac<T> &K, T s, const Vec2<T> &v) {
    Vec2<T> r;
    if (Q) {
        r.x = s * fma(K.mm, v.x, K.ms * v.y);
        r.y = s * fma(K.sm, v.x, K.ss * v.y);
    } else {
        r.x = s * K.mm * v.x;
        r.y = T(0);
    }
    return r;
}

// One RK4 step of (mu, sig2), linearised.  The tangent of any direction obeys
//   dk1 = K1 V + g1 d1,            dk2 = K2 (V + h/2 dk1) + g2 dh,
//   dk3 = K3 (V + h/2 dk2) + g3 dh, dk4 = K4 (V + h dk3) + g4 d4,
//   V' = V + h/6 (dk1 + 2 dk2 + 2 dk3 + dk4),
// with K_s = d f / d(mu, sig2) and g_s = d f / d a at stage s, and d1, dh, d4
// the direction's amplitude derivatives at psi_j, psi_j + h/2, psi_j + h.
// That map is linear, V' = A V + P1 d1 + Ph dh + P4 d4, and A, P1, Ph, P4 are
// shared by all directions, so they are formed once per step.
template <class T, bool Q>
struct StepLin {
    Mat2<T> A;
    Vec2<T> P1, Ph, P4;
    T dmu, ds2;  // the state increment
};

template <class T, bool Q, class Src = RadSrc<T>>
__device__ __forceinline__ StepLin<T, Q> rk4_linear(T mu, T s2, const StageAmp<T> &A1,
                                                    const StageAmp<T> &Ah, const StageAmp<T> &A4,
                                                    T h, Src &rad, T &chi_hi) {
    // The stage matrices M_s = K_s (I + c_s M_{s-1}) and the forcing chains
    // e_s1 = c_s K_s e_{s-1,1}, e_sh = c_s K_s e_{s-1,h} (+ g_s) are summed
    // with the RK4 weights as they are formed, so only the running sums and
    // the latest stage stay live.
    const T hh = T(0.5) * h, h6 = h * T(1.0 / 6.0);
    StepLin<T, Q> L;
    // stage 1
    Jac<T> K1;
    if (Q) {
        const T chi = A1.chi_per_mu * mu;
        chi_hi = fmax(chi_hi, chi);
        K1 = jac_quantum(mu, s2, A1, rad.s1(chi));
    } else {
        K1 = jac_classical(mu, A1);
    }
    Mat2<T> M{K1.mm, K1.ms, K1.sm, K1.ss};
    Mat2<T> SA = M;                  // M1 + 2 M2 + 2 M3 + M4
    Vec2<T> e1{K1.ma, K1.sa};        // g1, e21, e31, e41
    Vec2<T> S1 = e1;                 // g1 + 2 e21 + 2 e31 + e41
    T Sm = K1.fm, Ss = K1.fs;        // k1 + 2 k2 + 2 k3 + k4
    // stage 2
    const T m2 = fma(hh, K1.fm, mu), s22 = fma(hh, K1.fs, s2);
    Jac<T> K2;
    if (Q) {
        const T chi = Ah.chi_per_mu * m2;
        chi_hi = fmax(chi_hi, chi);
        K2 = jac_quantum(m2, s22, Ah, rad.s2(chi));
    } else {
        K2 = jac_classical(m2, Ah);
    }
    M = kism<T, Q>(K2, hh, M);
    SA = Mat2<T>{fma(T(2), M.a, SA.a), fma(T(2), M.b, SA.b), fma(T(2), M.c, SA.c),
                 fma(T(2), M.d, SA.d)};
    e1 = skv<T, Q>(K2, hh, e1);
    S1 = Vec2<T>{fma(T(2), e1.x, S1.x), fma(T(2), e1.y, S1.y)};
    Vec2<T> eh{K2.ma, K2.sa};                        // g2, e3h, e4h
    Vec2<T> Sh{T(2) * eh.x, T(2) * eh.y};           // 2 g2 + 2 e3h + e4h
    Sm = fma(T(2), K2.fm, Sm);
    Ss = fma(T(2), K2.fs, Ss);
    // stage 3
    const T m3 = fma(hh, K2.fm, mu), s23 = fma(hh, K2.fs, s2);
    Jac<T> K3;
    if (Q) {
        const T chi = Ah.chi_per_mu * m3;
        chi_hi = fmax(chi_hi, chi);
        K3 = jac_quantum(m3, s23, Ah, rad.s3(chi));
    } else {
        K3 = jac_classical(m3, Ah);
    }
    M = kism<T, Q>(K3, hh, M);
    SA = Mat2<T>{fma(T(2), M.a, SA.a), fma(T(2), M.b, SA.b), fma(T(2), M.c, SA.c),
                 fma(T(2), M.d, SA.d)};
    e1 = skv<T, Q>(K3, hh, e1);
    S1 = Vec2<T>{fma(T(2), e1.x, S1.x), fma(T(2), e1.y, S1.y)};
    eh = skv<T, Q>(K3, hh, eh);
    eh.x += K3.ma;
    eh.y += K3.sa;
    Sh = Vec2<T>{fma(T(2), eh.x, Sh.x), fma(T(2), eh.y, Sh.y)};
    Sm = fma(T(2), K3.fm, Sm);
    Ss = fma(T(2), K3.fs, Ss);
    // stage 4
    const T m4 = fma(h, K3.fm, mu), s24 = fma(h, K3.fs, s2);
    Jac<T> K4;
    if (Q) {
        const T chi = A4.chi_per_mu * m4;
        chi_hi = fmax(chi_hi, chi);
        K4 = jac_quantum(m4, s24, A4, rad.s4(chi));
    } else {
        K4 = jac_classical(m4, A4);
    }
    M = kism<T, Q>(K4, h, M);
    e1 = skv<T, Q>(K4, h, e1);
    eh = skv<T, Q>(K4, h, eh);
    // assemble
    L.A.a = fma(h6, SA.a + M.a, T(1));
    L.A.b = h6 * (SA.b + M.b);
    L.A.c = h6 * (SA.c + M.c);
    L.A.d = fma(h6, SA.d + M.d, T(1));
    L.P1.x = h6 * (S1.x + e1.x);
    L.P1.y = h6 * (S1.y + e1.y);
    L.Ph.x = h6 * (Sh.x + eh.x);
    L.Ph.y = h6 * (Sh.y + eh.y);
    L.P4.x = h6 * K4.ma;
    L.P4.y = h6 * K4.sa;
    L.dmu = h6 * (Sm + K4.fm);
    L.ds2 = h6 * (Ss + K4.fs);
    return L;
}

// Spatial factor of eq. a0eff and its logarithmic derivatives with respect to
// the sample position (x, y, z) and the spot size W0:
//   ln S = -p - ln(q)/2,  p = (x^2 + y^2) / (W0^2 q),  q = 1 + (z / zR)^2,
//   d/dx = -2 x / (W0^2 q),  d/dz = 2 (z / zR^2) (p - 1/2) / q,
//   d/dW0 = (2 / W0) (p - 2 (z/zR)^2 (p - 1/2) / q)   (zR = pi W0^2 / lambda).
template <class T>
struct SpD {
    T S, Lx, Ly, Lz, Lw;
};

__device__ __forceinline__ SpD<float> spatial_d(float x, float y, float z, float inv_w0sq,
                                                float inv_zR, float inv_w0) {
    const float zz = z * inv_zR;
    const float q = fmaf(zz, zz, 1.0f);
    const float rq = __builtin_amdgcn_rsqf(q);
    const float iq = rq * rq;
    const float p = fmaf(x, x, y * y) * inv_w0sq * iq;
    SpD<float> r;
    r.S = __builtin_amdgcn_exp2f(-1.4426950408889634f * p) * rq;
    const float m = -2.0f * inv_w0sq * iq;
    r.Lx = m * x;
    r.Ly = m * y;
    const float B = iq * (p - 0.5f);
    r.Lz = 2.0f * zz * inv_zR * B;
    r.Lw = 2.0f * inv_w0 * fmaf(-2.0f * zz * zz, B, p);
    return r;
}

__device__ __forceinline__ SpD<double> spatial_d(double x, double y, double z, double inv_w0sq,
                                                 double inv_zR, double inv_w0) {
    const double zz = z * inv_zR;
    double iq;
    const double rq = inv_sqrt64(fma(zz, zz, 1.0), iq);
    const double p = fma(x, x, y * y) * inv_w0sq * iq;
    SpD<double> r;
    r.S = exp64(-p) * rq;
    const double m = -2.0 * inv_w0sq * iq;
    r.Lx = m * x;
    r.Ly = m * y;
    const double B = iq * (p - 0.5);
    r.Lz = 2.0 * zz * inv_zR * B;
    r.Lw = 2.0 * inv_w0 * fma(-2.0 * zz * zz, B, p);
    return r;
}

// Directions of the local-amplitude tangents: a0, W0, x offset, y offset,
// delay, gamma0, divergence.
constexpr int kDirLocal = 7;
constexpr int kDirA0eff = 2;  // a0 (all amplitude directions), gamma0

// Geometry of one sample in the adjoint's precision.
template <class T>
struct AdjPath {
    T xc, yc, thx, thy, zstar, hz;     // hz = z / 2
    T dthx, dthy;                      // d theta / d div_mrad = 1e-3 n4, 1e-3 n5
    T inv_w0sq, inv_zR, inv_w0, a0, zfac;  // zfac = d z* / d delay = c / 2
    // amplitude without the carrier and its derivative in each direction
    __device__ __forceinline__ void amp(T ell, T fc, T &a, T *da) const {
        const SpD<T> d = spatial_d(fma(thx, ell, xc), fma(thy, ell, yc), zstar - ell, inv_w0sq,
                                   inv_zR, inv_w0);
        const T Sf = d.S * fc;
        a = a0 * Sf;
        da[0] = Sf;
        da[1] = a * d.Lw;
        da[2] = a * d.Lx;
        da[3] = a * d.Ly;
        da[4] = a * zfac * d.Lz;
        da[5] = T(0);
        da[6] = a * (hz + ell) * fma(dthx, d.Lx, dthy * d.Ly);
    }
};

// A sample's draw, its path in FP64 and the spatial factor at its collision
// point with the log-derivatives.  The tangent loop recomputes this where it
// needs it (FP64 steps, the chain to the parameters at the end) instead of
// carrying it through the phase steps: the draw is a few hundred operations
// against the thousands a step costs, and the registers go to the loop.
struct AdjSample {
    SampleCoords sc;
    AdjPath<double> p;
    SpD<double> d0;
};

// The sample index hidden from the optimiser, so that a recomputation is not
// merged with an earlier one into values kept live in between.
__device__ __forceinline__ int64_t opaque_index(int64_t i) {
    asm volatile("" : "+v"(i));
    return i;
}

__device__ __forceinline__ void adj_sample(const BatchParams &P, const ShotParams &sp, int64_t i,
                                           AdjSample &s) {
    constexpr double kHalfC = 0.5 * 0.299792458;  // d z* / d delay [um/fs]
    sample_coords(sp, P.key0, P.key1, i, s.sc);
    const double z = s.sc.z;
    s.p.xc = fma(s.sc.thx, 0.5 * z, s.sc.x);
    s.p.yc = fma(s.sc.thy, 0.5 * z, s.sc.y);
    s.p.thx = s.sc.thx;
    s.p.thy = s.sc.thy;
    s.p.zstar = fma(0.5, z, sp.z_delay);
    s.p.hz = 0.5 * z;
    s.p.dthx = 1e-3 * s.sc.n[4];
    s.p.dthy = 1e-3 * s.sc.n[5];
    s.p.inv_w0sq = sp.inv_w0sq;
    s.p.inv_zR = sp.inv_zR;
    s.p.inv_w0 = sqrt(sp.inv_w0sq);
    s.p.a0 = sp.a0;
    s.p.zfac = kHalfC;
    s.d0 = spatial_d(s.p.xc, s.p.yc, s.p.zstar, sp.inv_w0sq, sp.inv_zR, s.p.inv_w0);
}

template <class T>
__device__ __forceinline__ AdjPath<T> adj_path_cast(const AdjPath<double> &p) {
    AdjPath<T> r;
    r.xc = (T)p.xc;
    r.yc = (T)p.yc;
    r.thx = (T)p.thx;
    r.thy = (T)p.thy;
    r.zstar = (T)p.zstar;
    r.hz = (T)p.hz;
    r.dthx = (T)p.dthx;
    r.dthy = (T)p.dthy;
    r.inv_w0sq = (T)p.inv_w0sq;
    r.inv_zR = (T)p.inv_zR;
    r.inv_w0 = (T)p.inv_w0;
    r.a0 = (T)p.a0;
    r.zfac = (T)p.zfac;
    return r;
}

// Sensitivities of one sample's share of L = sum_k w_k H_k to the centre v
// and the variance sig2 of its energy law.  Writing F for the law's CDF and
// e_j = lo + j width (j = 0..n) for the bin edges, the sample adds F(e_0) to
// the underflow, F(e_{k+1}) - F(e_k) to bin k and 1 - F(e_n) to the overflow,
// so its share is sum_j c_j F(e_j) + w_over with c_j = w_{j-1} - w_j
// (w_{-1} = w_under, w_n = w_over).  For the three laws (with t = e_j - v):
//   Gaussian N(v, s^2):  dF/dv = -phi(t/s)/s,          dF/ds = -(t/s) phi(t/s)/s;
//   box of width b:      dF/dv = -1/b for |t| < b/2,   no s;
//   box (x) N(0, s^2):   dF/dv = -(Phi((t + b/2)/s) - Phi((t - b/2)/s)) / b,
//                        dF/ds = (phi((t + b/2)/s) - phi((t - b/2)/s)) / b.
// Edges beyond 9 standard deviations add nothing at FP64 precision.
__device__ __forceinline__ double phi_pdf(double z) {
    return 0.39894228040143267794 * exp64(-0.5 * z * z);
}

// The edge weights c_j from the upstream weights W (n bins, underflow, overflow).
struct EdgeWeights {
    const double *W;
    int n;
    __device__ __forceinline__ double operator()(int j) const {
        return (j == 0 ? W[n] : W[j - 1]) - (j == n ? W[n + 1] : W[j]);
    }
};

// Edges evenly spaced (dz = b/s) let the densities follow by multiplications,
//   phi(z + dz) = phi(z) r,  r = exp(-z dz - dz^2/2),  r -> r exp(-dz^2),
// anew from their exponentials every kChunk edges (the products' roundings grow
// with the square of the edges).  Where the box spans at most a quarter standard
// deviation its mass is the density at its centre times a polynomial in z^2,
//   Phi(z + d) - Phi(z - d) = phi(z) Int_(-d)^d e^(-z u - u^2/2) du
//                           = phi(z) P(z^2),  P(x) = sum_k x^k m_2k / (2k)!,
//   d = dz/2, m_2k = Int_(-d)^d u^2k e^(-u^2/2) du
// (eight terms: the ninth is below 3e-17 of the sum at six standard deviations),
// and the derivative along s is that of the mass by z,
//   phi(z + d) - phi(z - d) = -z phi(z) (P(z^2) - 2 P'(z^2)),
// without the difference of the densities, which cancels in small boxes; wider
// boxes take erfc at their ends, shared by neighbouring edges.
// Over random laws with edges 0.003 to 1 standard deviations apart the sums of
// normal laws are 3e-16 to 2.0e-15 of the sum of magnitudes off (rms; an exponential
// an edge 2e-16 to 1.8e-15, sixteen edges a chunk 4e-16 to 3.9e-15), those of boxes
// 3e-16 to 8e-16 (two erfc and two exponentials an edge 3e-16 to 1.8e-15, sixteen
// edges a chunk and the difference of the densities 4e-16 to 7.3e-15).
// Bound by FP64 issue, by the widest law of each wavefront.  With two erfc and
// two exponentials a box edge and one exponential a normal edge the contraction
// of tapes took 466 us for 50,001 samples (boxes), 367 us for 2^20 (normal
// laws of both histograms) and 580 us for 2^21 (normal); so 110, 322 and
// 386 us (four edges a chunk: 114, 408, 498).
constexpr int kChunk = 8;

template <class Weights>
__device__ __forceinline__ void law_sensitivity(double v, double s2, int dep, double ksig,
                                                double lo, double wb, int n, Weights c, double &lv,
                                                double &ls2) {
    lv = 0.0;
    ls2 = 0.0;
    const double s = sqrt(fmax(s2, 0.0));
    const double half = 0.5 * wb;
    int mode;
    double se = s, dse = 0.0;  // law width and d se / d sig2
    if (dep == 2) {            // GAUSS
        const double ks = ksig * wb;
        se = sqrt(s * s + ks * ks);
        mode = se > 0.0 ? 2 : 0;
        if (s2 > 0.0) dse = 0.5 / se;
    } else if (dep == 1) {  // CIC
        mode = s > 0.0 ? 3 : 1;
        if (s > 0.0) dse = 0.5 / s;
    } else {
        mode = s > 0.0 ? 2 : 0;
        if (s > 0.0) dse = 0.5 / s;
    }
    if (mode == 0) return;
    const double reach = mode == 1 ? half : (mode == 2 ? 9.0 * se : 9.0 * se + half);
    const int ja = (int)fmin(fmax(ceil((v - reach - lo) / wb), 0.0), (double)n + 1.0);
    const int jb = (int)fmin(fmax(floor((v + reach - lo) / wb), -1.0), (double)n);
    const double inv_se = mode >= 2 ? 1.0 / se : 0.0;
    const double dz = wb * inv_se, d = 0.5 * dz;
    const double q = exp64(-dz * dz);
    auto z_at = [&](int j) { return (fma((double)j, wb, lo) - v) * inv_se; };
    double sv = 0.0, ss = 0.0;
    if (mode == 1) {
        for (int j = ja; j <= jb; ++j)
            if (fabs(fma((double)j, wb, lo) - v) < half) sv += c(j);
        lv = -sv / wb;
        return;
    }
    if (mode == 2) {
        // sv = sum c phi / se, ss = sum c (-z) phi / se
        for (int j0 = ja; j0 <= jb; j0 += kChunk) {
            double z = z_at(j0), f = phi_pdf(z), r = exp64(-z * dz - d * dz);
            const int j1 = min(j0 + kChunk - 1, jb);
            for (int j = j0; j <= j1; ++j) {
                const double cf = c(j) * f;
                sv += cf;
                ss = fma(-z, cf, ss);
                f *= r;
                r *= q;
                z += dz;
            }
        }
        lv = -sv * inv_se;
        ls2 = ss * inv_se * dse;
        return;
    }
    if (dz <= 0.25) {
        // coefficients m_2k / (2k)! of the box mass, m_2k = 2 sum_i (-1)^i
        // d^(2k+2i+1) / (2^i i! (2k+2i+1)); d <= 1/8
        constexpr int kTerms = 8;
        double C[kTerms], D[kTerms];  // of P and P - 2 P'
        {
            const double d2 = d * d;
            double lead = 2.0 * d;  // 2 d^(2k+1) / (2k)!
#pragma unroll
            for (int k = 0; k < kTerms; ++k) {
                double m = 0.0, w = 1.0;
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    m = fma(w, 1.0 / (2 * k + 2 * i + 1), m);
                    w *= d2 * (-0.5 / (i + 1));
                }
                C[k] = lead * m;
                lead *= d2 * (1.0 / ((2 * k + 1) * (2 * k + 2)));
            }
#pragma unroll
            for (int k = 0; k < kTerms; ++k)
                D[k] = k + 1 < kTerms ? fma(-2.0 * (k + 1), C[k + 1], C[k]) : C[k];
        }
        for (int j0 = ja; j0 <= jb; j0 += kChunk) {
            double z = z_at(j0), f = phi_pdf(z), r = exp64(-z * dz - d * dz);
            const int j1 = min(j0 + kChunk - 1, jb);
            for (int j = j0; j <= j1; ++j) {
                const double z2 = z * z, cf = c(j) * f;
                double p = C[kTerms - 1], dp = D[kTerms - 1];
#pragma unroll
                for (int k = kTerms - 2; k >= 0; --k) {
                    p = fma(p, z2, C[k]);
                    dp = fma(dp, z2, D[k]);
                }
                sv = fma(cf, p, sv);
                ss = fma(-z * cf, dp, ss);
                f *= r;
                r *= q;
                z += dz;
            }
        }
    } else if (ja <= jb) {
        const double rt = 0.70710678118654752440;
        double zm = 0.0, em = 0.0, gm = 0.0;
        for (int j = ja - 1; j <= jb; ++j) {  // (the first: the lower end of box ja only)
            const double zp = z_at(j) + d, ep = erfc(fabs(zp) * rt), gp = phi_pdf(zp);
            // Phi(zp) - Phi(zm) from the tails on either side of the centre
            const double p = zm > 0.0 ? 0.5 * (em - ep)
                                      : (zp < 0.0 ? 0.5 * (ep - em) : 1.0 - 0.5 * (ep + em));
            const double cj = j < ja ? 0.0 : c(j);
            sv = fma(cj, p, sv);
            ss = fma(cj, gp - gm, ss);
            zm = zp;
            em = ep;
            gm = gp;
        }
    }
    lv = -sv / wb;
    ls2 = ss / wb * dse;
}

// Edge weights formed once, in LDS.
struct EdgesLds {
    const double *c;
    __device__ __forceinline__ double operator()(int j) const { return c[j]; }
};

// One sample's gradient terms g along the eight parameters, from its energy
// state (mu, sig2), its derivatives (derivs(p, dmu, dsig2), asked for at the
// end: nothing of them is held over the laws' edges) and the edge weights of
// the energy (we) and angle (wa) histograms.  OBS: also the angle-histogram
// and moment terms.  The draw gives the rest of these: theta = div n
// (derivative n in mrad per mrad), gamma0,i = gamma0 + sigma_gamma n3, and
// a0,eff = a0 S0 with S0 at the collision point
// (ln S0 derivatives of spatial_d; the divergence moves the collision point
// by theta z / 2).  The angle law is N(theta_x, sig_th^2) with sig_th^2 =
// C^2 a0,eff^2 max(sig2, 0) / mu^4 (Sec. 5.2), deposited like the energy law;
// the moments are those of the finalize kernel:
//   mean gamma = sum mu / W,   std^2 = sum (mu^2 + sig2^+) / W - mean^2,
//   mean and rms of theta_x (rms with sig_th^2) and theta_y, mean a0,eff,
//   mean 1 - mu / gamma0,i, mean sqrt(sig2^+);
// the weight, the largest chi and the FP64-shadow fields carry no derivative.
template <bool OBS, class Weights, class Derivs>
__device__ __forceinline__ void sample_gradient(const BatchParams &P, const ShotParams &sp,
                                                const ShotGrad &go, int64_t i, double mu,
                                                double s2, Weights we, Weights wa, Derivs derivs,
                                                double *g) {
    const bool obs = OBS && (go.d_angle || go.d_moments);
    SampleCoords sc{};
    SpD<double> d0{};
    double aeff = 0.0, thx = 0.0, q = 0.0, sig_th = 0.0;
    const double s2p = fmax(s2, 0.0);
    if (obs) {
        sample_coords(sp, P.key0, P.key1, i, sc);
        const double z = sc.z;
        const double xc = fma(sc.thx, 0.5 * z, sc.x), yc = fma(sc.thy, 0.5 * z, sc.y);
        const double zstar = fma(0.5, z, sp.z_delay);
        d0 = spatial_d(xc, yc, zstar, sp.inv_w0sq, sp.inv_zR, sqrt(sp.inv_w0sq));
        aeff = sp.a0 * d0.S;
        thx = 1e3 * sc.thx;
        const double C = 1e3 * P.c_theta * 0.79788456080286535588;
        q = C * C / (mu * mu * mu * mu);
        sig_th = sqrt(q * aeff * aeff * s2p);
    }
    // dL = Lmu dmu + Ls2 dsig2 + Ls2p dsig2^+ + Lx dtheta_x + Ly dtheta_y
    //      + Lq dsig_th^2 + La da0eff + Lg dgamma0,i
    double Lv = 0.0, Ls = 0.0, Lx = 0.0, Lq = 0.0;
#pragma unroll 1
    for (int law = 0; law < (OBS ? 2 : 1); ++law) {  // (one copy of the code)
        if (law ? !go.d_angle : !go.d_energy) continue;
        double lv, ls;
        law_sensitivity(law ? thx : mu, law ? sig_th * sig_th : s2, P.deposit, P.ksig_bins,
                        law ? sp.th_lo : sp.e_lo, law ? sp.th_w : sp.e_w, law ? sp.n_th : sp.n_e,
                        law ? wa : we, lv, ls);
        if (law) {
            Lx = lv;
            Lq = ls;
        } else {
            Lv = lv;
            Ls = ls;
        }
    }
    double Lmu = 0.0, Ls2 = 0.0, Ly = 0.0, La = 0.0, Lg = 0.0;
    if (OBS && go.d_moments) {
        const double thy = 1e3 * sc.thy, sigf = sqrt(s2p);
        const double *u = go.d_moments, *M = go.moments;
        const double iW = 1.0 / (double)sp.n_samples;
        Lmu += u[1] * iW;
        if (M[2] > 0.0) {
            Lmu += u[2] * (mu - M[1]) * iW / M[2];
            Ls2 += u[2] * 0.5 * iW / M[2];
        }
        Lx += u[3] * iW;
        if (M[4] > 0.0) {
            Lx += u[4] * thx * iW / M[4];
            Lq += u[4] * 0.5 * iW / M[4];
        }
        Ly += u[5] * iW;
        if (M[6] > 0.0) Ly += u[6] * thy * iW / M[6];
        La += u[7] * iW;
        Lmu -= u[9] * iW / sc.g0;
        Lg += u[9] * iW * mu / (sc.g0 * sc.g0);
        if (sigf > 0.0) Ls2 += u[10] * iW * 0.5 / sigf;
    }
    constexpr double kHalfC = 0.5 * 0.299792458;  // d z* / d delay [um/fs]
    const double a2 = aeff * aeff;
#pragma unroll
    for (int p = 0; p < kGradParams; ++p) {
        double dm, ds;
        derivs(p, dm, ds);
        g[p] = go.d_energy ? fma(Lv, dm, Ls * ds) : 0.0;
        if (obs) {
            double da = 0.0;
            if (p == 0) da = d0.S;
            if (p == 1) da = aeff * d0.Lw;
            if (p == 2) da = aeff * d0.Lx;
            if (p == 3) da = aeff * d0.Ly;
            if (p == 4) da = aeff * kHalfC * d0.Lz;
            if (p == 7)
                da = aeff * (0.5 * sc.z) * fma(1e-3 * sc.n[4], d0.Lx, 1e-3 * sc.n[5] * d0.Ly);
            const double ds2p = s2 > 0.0 ? ds : 0.0;
            const double dq = q * fma(2.0 * aeff * s2p, da, fma(a2, ds2p, -4.0 * a2 * s2p * dm / mu));
            const double dth_x = p == 7 ? sc.n[4] : 0.0, dth_y = p == 7 ? sc.n[5] : 0.0;
            const double dg = p == 5 ? 1.0 : (p == 6 ? sc.n[3] : 0.0);
            g[p] += Lmu * dm + Ls2 * ds2p + Lx * dth_x + Ly * dth_y + Lq * dq + La * da + Lg * dg;
        }
    }
}

// One step of the tangents of every direction: V' = A V + P1 d1 + Ph dh + P4 d4
// (d1, dh, d4: the direction's amplitude derivatives at the three stage
// points; the gamma0 direction GD has none).
template <class T, bool QUANTUM, int ND, int GD>
__device__ __forceinline__ void tangent_update(const StepLin<T, QUANTUM> &L, const T *da1,
                                               const T *dah, const T *da4, T *vm, T *vs) {
#pragma unroll
    for (int d = 0; d < ND; ++d) {
        T fm = T(0), fs = T(0);
        if (d != GD) {
            fm = fma(L.P1.x, da1[d], fma(L.Ph.x, dah[d], L.P4.x * da4[d]));
            fs = fma(L.P1.y, da1[d], fma(L.Ph.y, dah[d], L.P4.y * da4[d]));
        }
        const T m0 = vm[d];
        if (QUANTUM) {
            const T s0 = vs[d];
            vm[d] = fma(L.A.a, m0, fma(L.A.b, s0, fm));
            vs[d] = fma(L.A.c, m0, fma(L.A.d, s0, fs));
        } else {
            vm[d] = fma(L.A.a, m0, fm);
        }
    }
}

// FP64 steps of the mixed-precision tangent loop, from step j on for as long
// as some lane of the wavefront has chi above the threshold at a step start
// (the rule of the forward pass).  The state advances by the forward pass's
// FP64 step (FP64 amplitudes, the FP64 table's window in LDS);
// the tangents by the FP32 step linearisation at the state rounded to FP32,
// with the FP32 amplitude derivatives and derivative table as in the FP32
// steps (the linearisation is rounded to FP32 either way), with the FP32
// loop's table cells carried from stage to stage as there.  A1, da1 and those
// cells carry over to the step the segment returns, the first not taken.
template <bool LOCAL, int ND, int GD, class Tab>
__device__ __forceinline__ int tangent_fp64_segment(
    const BatchParams &P, const AdjPath<double> &pd, double S0d, const AdjPath<float> &pf,
    float S0f, const float *__restrict__ env32, const double *__restrict__ env64, const Tab &tabd,
    RadSrc<float> &rad, const Phys<float> &phf, int j, double &mu, double &s2, float *vm,
    float *vs, float *da1, StageAmp<float> &A1, float &cmx, float &chi_hi, double &chd) {
    const Phys<double> phd{P.K, P.CD, P.two_over_aS};
    const int N = P.n_steps;
    const double h = P.h, psi0 = -P.psi_max, ell = P.ell_per_psi;
    const float hf = (float)P.h, psi0f = (float)(-P.psi_max), ellf = (float)P.ell_per_psi;
    auto amp64 = [&](double psi, double fc) {
        if (LOCAL) {
            const double e = psi * ell;
            return pd.a0 * spatial(fma(pd.thx, e, pd.xc), fma(pd.thy, e, pd.yc), pd.zstar - e,
                                   pd.inv_w0sq, pd.inv_zR) * fc;
        }
        return pd.a0 * S0d * fc;
    };
    auto amp32 = [&](float psi, float fc, float &a, float *da) {
        if (LOCAL) {
            pf.amp(psi * ellf, fc, a, da);
        } else {
            const float Sf = S0f * fc;
            a = pf.a0 * Sf;
            da[0] = Sf;
            da[1] = 0.0f;
        }
    };
    AmpFactors<double> F1(amp64(fma((double)j, h, psi0), env64[2 * j]), phd);
    for (;;) {
        // tangents: FP32 linearisation at the rounded state
        const float psif = fmaf((float)j, hf, psi0f);
        float ahf, a4f, dah[ND], da4[ND];
        amp32(fmaf(0.5f, hf, psif), env32[2 * j + 1], ahf, dah);
        amp32(psif + hf, env32[2 * j + 2], a4f, da4);
        const StageAmp<float> Ah(ahf, phf), A4(a4f, phf);
        const StepLin<float, true> L =
            rk4_linear<float, true>((float)mu, (float)s2, A1, Ah, A4, hf, rad, chi_hi);
        tangent_update<float, true, ND, GD>(L, da1, dah, da4, vm, vs);
        A1 = A4;
#pragma unroll
        for (int d = 0; d < ND; ++d) da1[d] = da4[d];
        // state: the forward pass's FP64 step
        const double psi = fma((double)j, h, psi0);
        const double ah = amp64(fma(0.5, h, psi), env64[2 * j + 1]);
        const double a4 = amp64(psi + h, env64[2 * j + 2]);
        double dm, ds;
        rk4_q64(mu, s2, F1, ah, a4, h, phd, tabd, dm, ds, chd);
        mu += dm;
        s2 += ds;
        ++j;
        if (j >= N) break;
        const double chi = F1.cpm * mu;
        cmx = fmaxf(cmx, (float)chi);
        if (!__any(chi > (double)P.chi_fp64)) break;
    }
    return j;
}

// Final state of one sample and its derivatives along the eight parameters
// (order of the grad outputs: a0, W0, x offset, y offset, delay, gamma0,
// sigma_gamma, divergence).
struct SampleTangent {
    double mu, s2;
    double dmu[kGradParams], ds2[kGradParams];
    double S0, g0, thx, thy;
    float cmx;
};

// The final derivatives along the eight parameters from the tangents (vm, vs) and
// the sample's draw.
template <class T, bool QUANTUM, bool LOCAL>
__device__ __forceinline__ void chain_params(const ShotParams &sp, const AdjSample &se,
                                             const T *vm, const T *vs, double *dmu, double *ds2) {
    const double *nrm = se.sc.n;
    const SpD<double> &d0 = se.d0;
    const double z = se.sc.z;
    constexpr double kHalfC = 0.5 * 0.299792458;  // d z* / d delay [um/fs]
    const double dthx_dd = 1e-3 * nrm[4], dthy_dd = 1e-3 * nrm[5];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const T *v = c == 0 ? vm : vs;
        double *d = c == 0 ? dmu : ds2;
        if (c == 1 && !QUANTUM) {
#pragma unroll
            for (int p = 0; p < kGradParams; ++p) d[p] = 0.0;
            continue;
        }
        if (LOCAL) {
            d[0] = v[0];
            d[1] = v[1];
            d[2] = v[2];
            d[3] = v[3];
            d[4] = v[4];
            d[5] = v[5];
            d[6] = nrm[3] * (double)v[5];
            d[7] = v[6];
        } else {
            // every amplitude direction is a multiple of the a0 tangent
            const double b = sp.a0 * (double)v[0];
            d[0] = v[0];
            d[1] = b * d0.Lw;
            d[2] = b * d0.Lx;
            d[3] = b * d0.Ly;
            d[4] = b * kHalfC * d0.Lz;
            d[5] = v[1];
            d[6] = nrm[3] * (double)v[1];
            d[7] = b * (0.5 * z) * fma(dthx_dd, d0.Lx, dthy_dd * d0.Ly);
        }
    }
}

// One sample: trajectory, tangents, and the chain to the eight parameters.
// rad: the radiation functions of the linearisation; tabd: those of the FP64
// steps of a mixed-precision pass.
template <int PREC, bool QUANTUM, bool LOCAL, class Src, class Tab>
__device__ __forceinline__ void tangent_sample(const BatchParams &P, const ShotParams &sp,
                                               int64_t i, const float *__restrict__ env32,
                                               const double *__restrict__ env64, Src rad,
                                               const Tab &tabd, SampleTangent &o, int &flags) {
    using T = typename std::conditional<PREC == PREC_F64, double, float>::type;
    // FP32 with FP64 steps where chi is above the threshold (quantum only)
    constexpr bool MIX = PREC == PREC_F32MIX;
    static_assert(!MIX || QUANTUM, "FP64 steps are a quantum-model option");
    constexpr int ND = LOCAL ? kDirLocal : kDirA0eff;
    constexpr int GD = LOCAL ? 5 : 1;  // the gamma0 direction: no amplitude forcing
    const int N = P.n_steps;
    const T *env;
    if constexpr (PREC == PREC_F64)
        env = env64;
    else
        env = env32;
    Phys<T> ph;
    ph.K = (T)P.K;
    ph.CD = (T)P.CD;
    ph.two_over_aS = (T)P.two_over_aS;
    const float chi_top = (float)(1 << (kEMax + 1));

    // ---- sample and geometry (FP64) ----
    AdjSample smp;
    adj_sample(P, sp, i, smp);
    const double g0 = smp.sc.g0;
    AdjPath<T> pth = adj_path_cast<T>(smp.p);
    const T S0 = (T)smp.d0.S;
    const T ell_per_psi = (T)P.ell_per_psi;
    const T h = (T)P.h;
    const T psi0 = (T)(-P.psi_max);

    T vm[ND], vs[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) vm[d] = vs[d] = T(0);
    vm[GD] = T(1);  // d mu_0 / d gamma0

    T mu = (T)g0, mu_lo = T(0), s2 = T(0), s2_lo = T(0);
    double g0_rest = 0.0;
    if constexpr (PREC != PREC_F64) {
        mu_lo = (T)(g0 - (double)mu);
        g0_rest = (g0 - (double)mu) - (double)mu_lo;
    }
    T chi_hi = T(0);
    float cmx = 0.0f;  // largest chi at a step start
    T a1, da1[ND];
    if (LOCAL) {
        pth.amp(psi0 * ell_per_psi, env[0], a1, da1);
    } else {
        const T Sf = S0 * env[0];
        a1 = pth.a0 * Sf;
        da1[0] = Sf;
        da1[1] = T(0);
    }
    StageAmp<T> A1(a1, ph);
    if (QUANTUM) rad.init(A1.chi_per_mu * mu);
    double chd = 0.0;  // largest chi of the FP64 steps
    for (int j = 0; j < N;) {
        const T chi1 = A1.chi_per_mu * mu;
        cmx = fmaxf(cmx, (float)chi1);
        if constexpr (MIX) {
            if (__any(chi1 > P.chi_fp64)) {
                // FP64 steps while some lane of the wavefront has chi above
                // the threshold; the FP32 pair takes the state back at the
                // exit step (amplitude, derivatives and cells carry over)
                double mud = ((double)mu + (double)mu_lo) + g0_rest;
                double s2d = (double)s2 + (double)s2_lo;
                g0_rest = 0.0;  // now held by the state
                AdjSample sd;
                adj_sample(P, sp, opaque_index(i), sd);
                j = tangent_fp64_segment<LOCAL, ND, GD>(P, sd.p, sd.d0.S, pth, S0, env32, env64,
                                                        tabd, rad, ph, j, mud, s2d, vm, vs, da1,
                                                        A1, cmx, chi_hi, chd);
                mu = (float)mud;
                mu_lo = (float)(mud - (double)mu);
                s2 = (float)s2d;
                s2_lo = (float)(s2d - (double)s2);
                continue;
            }
        }
        const T psi = fma((T)j, h, psi0);
        T ah, a4, dah[ND], da4[ND];
        if (LOCAL) {
            pth.amp(fma(T(0.5), h, psi) * ell_per_psi, env[2 * j + 1], ah, dah);
            pth.amp((psi + h) * ell_per_psi, env[2 * j + 2], a4, da4);
        } else {
            const T Sh = S0 * env[2 * j + 1], S4 = S0 * env[2 * j + 2];
            ah = pth.a0 * Sh;
            a4 = pth.a0 * S4;
            dah[0] = Sh;
            da4[0] = S4;
            dah[1] = da4[1] = T(0);
        }
        const StageAmp<T> Ah(ah, ph), A4(a4, ph);
        const StepLin<T, QUANTUM> L = rk4_linear<T, QUANTUM>(mu, s2, A1, Ah, A4, h, rad, chi_hi);
        tangent_update<T, QUANTUM, ND, GD>(L, da1, dah, da4, vm, vs);
        if constexpr (PREC == PREC_F64) {
            mu += L.dmu;
            s2 += L.ds2;
        } else {
            comp_add(mu, mu_lo, L.dmu);
            comp_add(s2, s2_lo, L.ds2);
        }
        A1 = A4;
#pragma unroll
        for (int d = 0; d < ND; ++d) da1[d] = da4[d];
        ++j;
    }
    if constexpr (MIX) chi_hi = fmax(chi_hi, (T)chd);
    o.mu = ((double)mu + (double)mu_lo) + g0_rest;
    o.s2 = (double)s2 + (double)s2_lo;
    o.cmx = fmaxf(cmx, (float)(A1.chi_per_mu * mu));  // the end of the last step
    // the draw again for the chain (not carried through the loop)
    AdjSample se;
    adj_sample(P, sp, opaque_index(i), se);
    o.S0 = se.d0.S;
    o.g0 = se.sc.g0;
    o.thx = se.sc.thx;
    o.thy = se.sc.thy;
    if (QUANTUM && !((float)chi_hi < chi_top)) flags |= kFlagRange;
    if (!(o.mu > 0.0) || !isfinite(o.mu) || !isfinite(o.s2)) flags |= kFlagNonFinite;

    chain_params<T, QUANTUM, LOCAL>(sp, se, vm, vs, o.dmu, o.ds2);
}

// The sums of a wavefront's eight values into a row of the gradient partials
// (stored column after column).
__device__ __forceinline__ void grad_row(const BatchParams &P, int64_t row, const double *g) {
#pragma unroll
    for (int p = 0; p < kGradParams; ++p) {
        const double v = wave_sum_last(g[p]);
        if ((threadIdx.x & 63) == 63) P.partials[(size_t)p * kGradRows * P.n_items + row] = v;
    }
}

// The final state of sample i, for the deposit and in the tape, and its derivatives.
__device__ __forceinline__ void tape_state(const BatchParams &P, const ShotParams &sp, int64_t i,
                                           const SampleTangent &o) {
    const int64_t k = sp.state_off + i;
    P.st.mu[k] = o.mu;
    P.st.s2[k] = o.s2;
    P.st.S0[k] = o.S0;
    P.st.g0[k] = o.g0;
    P.st.thx[k] = o.thx;
    P.st.thy[k] = o.thy;
    P.st.cmx[k] = o.cmx;
    P.tape[k] = o.mu;
    P.tape[P.tape_n + k] = o.s2;
}
__device__ __forceinline__ void tape_derivs(const BatchParams &P, const ShotParams &sp, int64_t i,
                                            const double *dmu, const double *ds2) {
    double *tp = P.tape + sp.state_off + i;
#pragma unroll
    for (int p = 0; p < kGradParams; ++p) {
        tp[(2 + p) * P.tape_n] = dmu[p];
        tp[(2 + kGradParams + p) * P.tape_n] = ds2[p];
    }
}

// One sample of the tangent kernels.  TAPE = true: the forward pass that also
// records the derivatives: the final state for the deposit kernel and the tape
// entries (mu, sig2 and their eight derivatives, structure of arrays).  TAPE =
// false: the adjoint: its derivatives contracted at once with its law
// sensitivities, into g.
template <int PREC, bool QUANTUM, bool LOCAL, bool TAPE, class Src, class Tab>
__device__ __forceinline__ void tangent_one(const BatchParams &P, const ShotParams &sp, int s,
                                            int64_t i, const float *__restrict__ env32,
                                            const double *__restrict__ env64, const Src &rad,
                                            const Tab &tabd, double *g) {
    int flags = 0;
    SampleTangent o;
    tangent_sample<PREC, QUANTUM, LOCAL>(P, sp, i, env32, env64, rad, tabd, o, flags);
    if (TAPE) {
        tape_state(P, sp, i, o);
        tape_derivs(P, sp, i, o.dmu, o.ds2);
    } else if (!(flags & kFlagNonFinite)) {
        const ShotGrad &go = P.gouts[s];
        sample_gradient<true>(
            P, sp, go, i, o.mu, o.s2, EdgeWeights{go.d_energy, sp.n_e},
            EdgeWeights{go.d_angle, sp.n_th},
            [&](int p, double &dm, double &ds) {
                dm = o.dmu[p];
                ds = o.ds2[p];
            },
            g);
    }
    if (flags) atomicOr(&P.flags[s], flags);
}

// FP32 passes and classical FP64 passes: blocks take items of kPhaseBlock
// samples.  Occupancy: the FP32 tape pass is latency-bound and fits 168 VGPRs,
// three waves per SIMD; every other pass is held to 256 (two waves).
template <int PREC, bool QUANTUM, bool LOCAL, bool TAPE>
__global__ __launch_bounds__(kPhaseBlock)
__attribute__((amdgpu_waves_per_eu((TAPE && PREC == PREC_F32) ? 3 : 2))) void tangent_kernel(
    BatchParams P, const float *__restrict__ env32, const double *__restrict__ env64) {
    static_assert(PREC == PREC_F32 || !QUANTUM, "tangent64_kernel");
    __shared__ __align__(16) float tab32[QUANTUM ? kCells32 * 4 * kDerivFuncs : 4];
    __shared__ int64_t slot;
    if (QUANTUM) {
        const float4 *src = reinterpret_cast<const float4 *>(P.rad32d);
        float4 *dst = reinterpret_cast<float4 *>(tab32);
        for (int k = threadIdx.x; k < kCells32 * kDerivFuncs; k += blockDim.x) dst[k] = src[k];
        __syncthreads();
    }
    using T = typename std::conditional<PREC == PREC_F64, double, float>::type;
    RadSrc<T> rad{};  // (classical: not read)
    if constexpr (PREC == PREC_F32) rad.tab = tab32;
    for (;;) {
        const int64_t item = next_item(&P.queue[0], &slot);
        if (item >= P.n_items) break;
        const int s = __builtin_amdgcn_readfirstlane(find_shot(P.shots, P.n_shots, item, false));
        const ShotParams &sp = P.shots[s];
        double g[kGradParams];
#pragma unroll
        for (int p = 0; p < kGradParams; ++p) g[p] = 0.0;
        const int64_t i = (item - sp.item0) * kPhaseBlock + threadIdx.x;
        if (i < sp.n_samples)
            tangent_one<PREC, QUANTUM, LOCAL, TAPE>(P, sp, s, i, env32, env64, rad, 0, g);
        if (!TAPE) grad_row(P, item * kGradRows + (threadIdx.x >> 6), g);
    }
}

// Small FP32 quantum tape passes with the local amplitude (at most an item a CU):
// as phase_pair_kernel, the steps of a wavefront of samples are divided over
// wavefronts that would otherwise leave their SIMDs to one each.  Three roles, kTrioSteps
// steps apart, with LDS buffers and a barrier of the block between them: the
// amplitudes at the steps' middles and ends; the trajectory and its step
// linearisation (ten values a step); the amplitudes' derivatives and the seven
// tangents.  The same operations as tangent_sample, the same bits.  50,001 samples x
// 512 steps 591 -> 514 us, 5003 a step of 1.15 -> 0.98 us (the second role keeps 390 of
// the 560 instructions a step); beyond an item a CU tangent_kernel, whose wavefronts
// then share SIMDs.
constexpr int kTrioSteps = 4;
constexpr int kTrioBlock = 3 * kPhaseBlock;

struct TrioLds {
    float2 a[2][kPhaseBlock / 64][kTrioSteps][64];    // amplitudes at the middle, the end
    float4 A[2][kPhaseBlock / 64][kTrioSteps][64];    // StepLin: A
    float4 P1h[2][kPhaseBlock / 64][kTrioSteps][64];  // P1, Ph
    float2 P4[2][kPhaseBlock / 64][kTrioSteps][64];   // P4
};

__global__ __launch_bounds__(kTrioBlock) void tangent_trio_kernel(
    BatchParams P, const float *__restrict__ env32, const double *__restrict__ env64) {
    __shared__ __align__(16) float tab32[kCells32 * 4 * kDerivFuncs];
    __shared__ int64_t slot;
    extern __shared__ __align__(16) unsigned char trio_lds[];
    TrioLds &B = *reinterpret_cast<TrioLds *>(trio_lds);
    {
        const float4 *src = reinterpret_cast<const float4 *>(P.rad32d);
        float4 *dst = reinterpret_cast<float4 *>(tab32);
        for (int k = threadIdx.x; k < kCells32 * kDerivFuncs; k += blockDim.x) dst[k] = src[k];
        __syncthreads();
    }
    constexpr int kTrios = kPhaseBlock / 64, ND = kDirLocal, GD = 5;
    const int N = P.n_steps, nbuf = (N + kTrioSteps - 1) / kTrioSteps;
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int role = wid / kTrios, w = wid % kTrios;
    const Phys<float> ph{(float)P.K, (float)P.CD, (float)P.two_over_aS};
    const float h = (float)P.h, psi0 = (float)(-P.psi_max), ell = (float)P.ell_per_psi;
    for (;;) {
        const int64_t item = next_item(&P.queue[0], &slot);
        if (item >= P.n_items) break;
        const int s = __builtin_amdgcn_readfirstlane(find_shot(P.shots, P.n_shots, item, false));
        const ShotParams &sp = P.shots[s];
        // (lanes past the samples take the last one: every wavefront meets the
        // same barriers)
        const int64_t k = (item - sp.item0) * kPhaseBlock + 64 * w + lane;
        const bool live = k < sp.n_samples;
        const int64_t i = live ? k : sp.n_samples - 1;
        AdjSample smp;
        adj_sample(P, sp, i, smp);
        const AdjPath<float> pth = adj_path_cast<float>(smp.p);
        auto middle = [&](int j, float &ah, float *dah) {
            const float psi = fma((float)j, h, psi0);
            pth.amp(fma(0.5f, h, psi) * ell, env32[2 * j + 1], ah, dah);
        };
        auto end = [&](int j, float &a4, float *da4) {
            const float psi = fma((float)j, h, psi0);
            pth.amp((psi + h) * ell, env32[2 * j + 2], a4, da4);
        };
        // interval t: amplitudes of buffer t, trajectory of t - 1, tangents of t - 2
        if (role == 0) {
            for (int t = 0; t < nbuf + 2; ++t) {
                const int j1 = t < nbuf ? min(N, (t + 1) * kTrioSteps) : 0;
                for (int j = t * kTrioSteps; j < j1; ++j) {
                    float ah, a4, da[ND];
                    middle(j, ah, da);
                    end(j, a4, da);
                    B.a[t & 1][w][j - t * kTrioSteps][lane] = make_float2(ah, a4);
                }
                __syncthreads();
            }
        } else if (role == 1) {
            const double g0 = smp.sc.g0;
            float mu = (float)g0, mu_lo = (float)(g0 - (double)mu), s2 = 0.0f, s2_lo = 0.0f;
            const double g0_rest = (g0 - (double)mu) - (double)mu_lo;
            float chi_hi = 0.0f, cmx = 0.0f, a1, da1[ND];
            pth.amp(psi0 * ell, env32[0], a1, da1);
            StageAmp<float> A1(a1, ph);
            RadSrc<float> rad{};
            rad.tab = tab32;
            rad.init(A1.chi_per_mu * mu);
            __syncthreads();
            for (int t = 1; t < nbuf + 2; ++t) {
                const int c = t - 1, j1 = c < nbuf ? min(N, (c + 1) * kTrioSteps) : 0;
                for (int j = c * kTrioSteps; j < j1; ++j) {
                    const int q = j - c * kTrioSteps;
                    const float2 a = B.a[c & 1][w][q][lane];
                    cmx = fmaxf(cmx, A1.chi_per_mu * mu);
                    const StageAmp<float> Ah(a.x, ph), A4(a.y, ph);
                    const StepLin<float, true> L =
                        rk4_linear<float, true>(mu, s2, A1, Ah, A4, h, rad, chi_hi);
                    B.A[c & 1][w][q][lane] = make_float4(L.A.a, L.A.b, L.A.c, L.A.d);
                    B.P1h[c & 1][w][q][lane] = make_float4(L.P1.x, L.P1.y, L.Ph.x, L.Ph.y);
                    B.P4[c & 1][w][q][lane] = make_float2(L.P4.x, L.P4.y);
                    comp_add(mu, mu_lo, L.dmu);
                    comp_add(s2, s2_lo, L.ds2);
                    A1 = A4;
                }
                __syncthreads();
            }
            if (live) {
                SampleTangent o;
                o.mu = ((double)mu + (double)mu_lo) + g0_rest;
                o.s2 = (double)s2 + (double)s2_lo;
                o.cmx = fmaxf(cmx, A1.chi_per_mu * mu);  // the end of the last step
                o.S0 = smp.d0.S;
                o.g0 = g0;
                o.thx = smp.sc.thx;
                o.thy = smp.sc.thy;
                int flags = 0;
                if (!(chi_hi < (float)(1 << (kEMax + 1)))) flags |= kFlagRange;
                if (!(o.mu > 0.0) || !isfinite(o.mu) || !isfinite(o.s2)) flags |= kFlagNonFinite;
                tape_state(P, sp, i, o);
                if (flags) atomicOr(&P.flags[s], flags);
            }
        } else {
            float vm[ND], vs[ND], a1, da1[ND];
#pragma unroll
            for (int d = 0; d < ND; ++d) vm[d] = vs[d] = 0.0f;
            vm[GD] = 1.0f;  // d mu_0 / d gamma0
            pth.amp(psi0 * ell, env32[0], a1, da1);
            __syncthreads();
            __syncthreads();
            for (int t = 2; t < nbuf + 2; ++t) {
                const int c = t - 2, j1 = min(N, (c + 1) * kTrioSteps);
                for (int j = c * kTrioSteps; j < j1; ++j) {
                    const int q = j - c * kTrioSteps;
                    float ah, a4, dah[ND], da4[ND];
                    middle(j, ah, dah);
                    end(j, a4, da4);
                    const float4 A = B.A[c & 1][w][q][lane], p = B.P1h[c & 1][w][q][lane];
                    const float2 p4 = B.P4[c & 1][w][q][lane];
                    StepLin<float, true> L;
                    L.A = Mat2<float>{A.x, A.y, A.z, A.w};
                    L.P1 = Vec2<float>{p.x, p.y};
                    L.Ph = Vec2<float>{p.z, p.w};
                    L.P4 = Vec2<float>{p4.x, p4.y};
                    tangent_update<float, true, ND, GD>(L, da1, dah, da4, vm, vs);
#pragma unroll
                    for (int d = 0; d < ND; ++d) da1[d] = da4[d];
                }
                __syncthreads();
            }
            if (live) {
                double dmu[kGradParams], ds2[kGradParams];
                chain_params<float, true, true>(sp, smp, vm, vs, dmu, ds2);
                tape_derivs(P, sp, i, dmu, ds2);
            }
        }
    }
}

// Quantum passes with FP64 steps (all of them, or where chi is high): as
// phase64_kernel, one block a CU with a window of the FP64 table in LDS (FP64
// passes: of the derivative table; with FP32 steps: of the forward table,
// beside the FP32 derivative table), its wavefronts taking items of 64 samples
// on their own, with FP32 steps in order of the group's chi scale.  Two
// wavefronts a SIMD (256 registers; the passes with FP32 steps spill about 100
// accesses, most of them where FP64 steps begin and end).  Bound by VALU issue:
// eight quantum shots of 2^18 x 512 with the tape 26.9 -> 18.4 ms, 100,001 FP64
// samples x 512 3.74 -> 2.09 ms, 5000 2.02 -> 1.28 ms, against the tables read from
// L2 (with FP32 steps a wavefront at a time through LDS staging rows).
constexpr int kTangent64Block = 512;

template <int PREC, bool LOCAL, bool TAPE>
__global__ __launch_bounds__(kTangent64Block) void tangent64_kernel(
    BatchParams P, const float *__restrict__ env32, const double *__restrict__ env64) {
    constexpr bool kMix = PREC == PREC_F32MIX;
    extern __shared__ double2 win[];
    __shared__ __align__(16) float tab32[kMix ? kCells32 * 4 * kDerivFuncs : 4];
    using Win = typename std::conditional<kMix, TabWindow<kWinDerivMix, 4>,
                                          TabWindow<kWinDeriv64, kDerivFuncs>>::type;
    const Win tabd(win, kMix ? P.rad64 : P.rad64d);
    using T = typename std::conditional<kMix, float, double>::type;
    RadSrc<T> rad{};
    if constexpr (kMix) {
        const float4 *src = reinterpret_cast<const float4 *>(P.rad32d);
        float4 *dst = reinterpret_cast<float4 *>(tab32);
        for (int k = threadIdx.x; k < kCells32 * kDerivFuncs; k += blockDim.x) dst[k] = src[k];
        rad.tab = tab32;
    } else {
        rad.win = &tabd;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    int s_prev = 0;  // the shot of the wavefront's previous item
    for (;;) {
        unsigned int taken = 0;
        if (lane == 0) taken = atomicAdd(&P.queue[0], 1u);
        const int64_t item = __builtin_amdgcn_readfirstlane(taken);
        if (item >= kGradRows * P.n_items) break;
        const int s = __builtin_amdgcn_readfirstlane(
            find_shot_from(P.shots, P.n_shots, item / kGradRows, false, s_prev));
        s_prev = s;
        const ShotParams &sp = P.shots[s];
        const int64_t k = item - kGradRows * sp.item0;
        if (64 * k >= sp.n_samples) continue;
        int64_t first = 64 * k, i = first + lane;
        bool live = i < sp.n_samples;
        if constexpr (kMix) {
            first = ordered_round<64>(sp.n_samples, k);
            const int64_t base = first & ~(kChiGroup - 1ll);
            const int cnt = (int)min((int64_t)kChiGroup, sp.n_samples - base);
            const int rank = (int)(first - base) + lane;
            live = rank < cnt;
            i = ordered_sample(P, sp, base, cnt, rank);
        }
        double g[kGradParams];
#pragma unroll
        for (int p = 0; p < kGradParams; ++p) g[p] = 0.0;
        if (live) tangent_one<PREC, true, LOCAL, TAPE>(P, sp, s, i, env32, env64, rad, tabd, g);
        if (!TAPE) grad_row(P, kGradRows * sp.item0 + first / 64, g);
    }
}

// The adjoint from a tape: contraction of the recorded derivatives with the
// law sensitivities (144 bytes read a sample).
// OBS: some shot also has angle-histogram or moment weights (the contraction
// of the energy terms alone keeps its small register budget).
// The gradient terms g of sample i from its tape entries.  False if the sample's
// state is not finite.
template <bool OBS, class Weights>
__device__ __forceinline__ bool contract_sample(const BatchParams &P, const ShotParams &sp, int s,
                                                int64_t i, Weights we, Weights wa, double *g) {
    const int64_t n = P.tape_n;
    const double *t = P.tape + sp.state_off + i;
    const double mu = t[0], s2 = t[n];
    if (!(mu > 0.0 && isfinite(mu) && isfinite(s2))) {
#pragma unroll
        for (int p = 0; p < kGradParams; ++p) g[p] = 0.0;
        return false;
    }
    sample_gradient<OBS>(
        P, sp, P.gouts[s], i, mu, s2, we, wa,
        [&](int p, double &dm, double &ds) {
            dm = t[(2 + p) * n];
            ds = t[(2 + kGradParams + p) * n];
        },
        g);
    return true;
}

// The edge weights of shot s to LDS: n_e + 1 words of the energy histogram,
// (OBS) then n_th + 1 of the angle histogram.
template <bool OBS>
__device__ __forceinline__ void edges_to_lds(const BatchParams &P, const ShotParams &sp, int s,
                                             double *wsh) {
    const EdgeWeights we{P.gouts[s].d_energy, sp.n_e}, wa{P.gouts[s].d_angle, sp.n_th};
    if (we.W)
        for (int k = threadIdx.x; k <= sp.n_e; k += blockDim.x) wsh[k] = we(k);
    if (OBS && wa.W)
        for (int k = threadIdx.x; k <= sp.n_th; k += blockDim.x) wsh[sp.n_e + 1 + k] = wa(k);
}

template <bool OBS>
__global__ __launch_bounds__(kPhaseBlock) void contract_kernel(BatchParams P) {
    extern __shared__ double wsh[];  // the edge weights of the block's current shot
    __shared__ int64_t slot;
    int s_w = -1;  // the shot whose weights wsh holds (block-uniform)
    for (;;) {
        const int64_t item = next_item(&P.queue[0], &slot);
        if (item >= P.n_items) break;
        const int s = __builtin_amdgcn_readfirstlane(find_shot(P.shots, P.n_shots, item, false));
        const ShotParams &sp = P.shots[s];
        if (s != s_w) {
            // (the previous item's reads ended at next_item's barriers)
            edges_to_lds<OBS>(P, sp, s, wsh);
            __syncthreads();
            s_w = s;
        }
        double g[kGradParams];
#pragma unroll
        for (int p = 0; p < kGradParams; ++p) g[p] = 0.0;
        const int64_t i = (item - sp.item0) * kPhaseBlock + threadIdx.x;
        if (i < sp.n_samples &&
            !contract_sample<OBS>(P, sp, s, i, EdgesLds{wsh}, EdgesLds{wsh + sp.n_e + 1}, g))
            atomicOr(&P.flags[s], kFlagNonFinite);
        grad_row(P, item * kGradRows + (threadIdx.x >> 6), g);
    }
}

// The same for the tape of a pass with FP64 steps, a group of kChiGroup samples
// at a time.  The tangent pass sums a group's terms a wavefront of 64 chi ranks
// at a time; the tape is in sample order.  The terms are formed in sample
// order (every tape line read once, whole) and go through LDS, from where
// they are summed as the tangent pass sums them, so that the result equals
// the recomputing adjoint's bit for bit.  (Reading the tape in chi order fetched
// every line about eight times: 2^21 samples 1283 -> 580 us with the order in a
// kernel of its own.)
constexpr int kContractBlock = 512;

template <bool OBS, bool LDSW>
__global__ __launch_bounds__(kContractBlock) void contract_group_kernel(BatchParams P) {
    // [kGradParams][kChiGroup], then (LDSW) the shot's edge weights
    extern __shared__ double terms[];
    double *wsh = terms + kGradParams * kChiGroup;
    __shared__ int64_t slot;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int s_w = -1;  // the shot whose weights wsh holds (block-uniform)
    for (;;) {
        const int64_t group = next_item(&P.queue[0], &slot);
        if (group >= P.n_gitems) break;
        const int s = __builtin_amdgcn_readfirstlane(find_group_shot(P.shots, P.n_shots, group));
        const ShotParams &sp = P.shots[s];
        const int64_t base = (group - sp.gitem0) * kChiGroup;
        const int cnt = (int)min((int64_t)kChiGroup, sp.n_samples - base);
        if (LDSW && s != s_w) edges_to_lds<OBS>(P, sp, s, wsh);
        s_w = s;
        __syncthreads();  // (also: the previous group's terms have been summed)
        for (int q = threadIdx.x; q < cnt; q += kContractBlock) {
            double g[kGradParams];
            bool ok;
            if constexpr (LDSW)
                ok = contract_sample<OBS>(P, sp, s, base + q, EdgesLds{wsh},
                                          EdgesLds{wsh + sp.n_e + 1}, g);
            else
                ok = contract_sample<OBS>(P, sp, s, base + q,
                                          EdgeWeights{P.gouts[s].d_energy, sp.n_e},
                                          EdgeWeights{P.gouts[s].d_angle, sp.n_th}, g);
            if (!ok) atomicOr(&P.flags[s], kFlagNonFinite);
#pragma unroll
            for (int p = 0; p < kGradParams; ++p) terms[p * kChiGroup + q] = g[p];
        }
        __syncthreads();
        for (int k = wid; 64 * k < cnt; k += kContractBlock / 64) {  // wavefronts of chi ranks
            const int r = 64 * k + lane;
            const int q = r < cnt ? P.order[sp.state_off + base + r] : 0;
            double g[kGradParams];
#pragma unroll
            for (int p = 0; p < kGradParams; ++p) g[p] = r < cnt ? terms[p * kChiGroup + q] : 0.0;
            grad_row(P, kGradRows * sp.item0 + base / 64 + k, g);
        }
    }
}

// One block per shot: fixed-order sum of the shot's rows, two wavefronts a
// column (rows l, l + 128, ... and l + 64, l + 192, ... for lane l).
constexpr int kGradFinBlock = 64 * 2 * kGradParams;

__global__ __launch_bounds__(kGradFinBlock) void grad_finalize_kernel(BatchParams P) {
    const int s = blockIdx.x;
    const ShotParams &sp = P.shots[s];
    const ShotGrad &so = P.gouts[s];
    const int64_t rows = (sp.n_samples + 63) / 64;
    __shared__ double half[2][kGradParams];
    const int lane = threadIdx.x & 63, p = (threadIdx.x >> 6) >> 1, h = (threadIdx.x >> 6) & 1;
    const double *col = P.partials + (size_t)p * kGradRows * P.n_items + kGradRows * sp.item0;
    double acc = 0.0;
#pragma unroll 8
    for (int64_t b = 64 * h + lane; b < rows; b += 128) acc += col[b];
    acc = wave_sum(acc);
    if (lane == 0) half[h][p] = acc;
    __syncthreads();
    if (threadIdx.x < kGradParams) so.grad[threadIdx.x] = half[0][threadIdx.x] + half[1][threadIdx.x];
    if (threadIdx.x == 0 && so.status) {
        const int fl = P.flags[s];
        *so.status = (fl & kFlagNonFinite) ? 4 : ((fl & kFlagRange) ? 6 : 0);
    }
}

// FP64-shadow report of each shot: the batch is the FP64 view pass, the FP32
// view pass's gradients sit span doubles before its own (span 0: zeros).
__global__ __launch_bounds__(256) void grad_shadow_kernel(BatchParams P, int64_t span) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= P.n_shots) return;
    const ShotGrad &so = P.gouts[s];
    double *o = so.errors;
    if (!o) return;
    if (span == 0) {
        for (int q = 0; q < 1 + 2 * kGradParams; ++q) o[q] = 0.0;
        return;
    }
    o[0] = (double)P.shots[s].n_samples;
    for (int p = 0; p < kGradParams; ++p) {
        const double g64 = so.grad[p], g32 = so.grad[p - span];
        o[1 + p] = g32 - g64;
        o[1 + kGradParams + p] = g64;
    }
}

__global__ void rad_derivs_kernel(const float *rad32d, const double *rad64d, int prec, int64_t n,
                                  const double *chi, double *out, int *flags) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const int fl = (chi[k] < (double)(1 << (kEMax + 1))) ? 0 : kFlagRange;
    double v[kDerivFuncs];
    if (prec == 0) {
        // the FP32 table holds combinations: undo them
        RadCell6 cell;
        rad6_lookup32(rad32d, (float)chi[k], cell);
        const RadJ<float> r = rad6_cell_eval(cell, (float)chi[k]);
        const double g = r.g, G1 = (double)r.E1 - 2.0 * g;
        const double G2 = (double)r.E2 - 2.0 * g - 4.0 * G1;
        v[0] = g;
        v[1] = G1;
        v[2] = G2;
        v[3] = r.h;
        v[4] = (double)r.E3 - 6.0 * (G1 + G2);
        v[5] = r.H1;
    } else {
        rad6_plain64(rad64d, chi[k], v);
    }
    for (int f = 0; f < kDerivFuncs; ++f) out[kDerivFuncs * k + f] = v[f];
    if (fl) atomicOr(flags, fl);
}

// ===========================================================================
// Launchers
// ===========================================================================
template <int PREC, bool QUANTUM, bool LOCAL, bool TAPE>
static PassKernel tangent_of() {
    if constexpr (QUANTUM && PREC != PREC_F32)
        return {reinterpret_cast<const void *>(&tangent64_kernel<PREC, LOCAL, TAPE>),
                kTangent64Block,
                PREC == PREC_F32MIX ? sizeof(double2) * kCellVals / 2 * kWinDerivMix
                                    : sizeof(double2) * 2 * kDerivFuncs * kWinDeriv64,
                true};
    else
        return {reinterpret_cast<const void *>(&tangent_kernel<PREC, QUANTUM, LOCAL, TAPE>),
                kPhaseBlock, 0, false};
}

template <bool TAPE>
static PassKernel select_tangent(int prec, int rr, int amp) {
    const bool q = rr == 1, l = amp == 1;
    if (prec == PREC_F64)
        return q ? (l ? tangent_of<PREC_F64, true, true, TAPE>()
                      : tangent_of<PREC_F64, true, false, TAPE>())
                 : (l ? tangent_of<PREC_F64, false, true, TAPE>()
                      : tangent_of<PREC_F64, false, false, TAPE>());
    if (prec == PREC_F32MIX && q)  // FP64 steps are a quantum-model option
        return l ? tangent_of<PREC_F32MIX, true, true, TAPE>()
                 : tangent_of<PREC_F32MIX, true, false, TAPE>();
    return q ? (l ? tangent_of<PREC_F32, true, true, TAPE>()
                  : tangent_of<PREC_F32, true, false, TAPE>())
             : (l ? tangent_of<PREC_F32, false, true, TAPE>()
                  : tangent_of<PREC_F32, false, false, TAPE>());
}

hipError_t launch_tangent(const BatchParams &p, const float *env32, const double *env64, int prec,
                          int rr, int amp, bool tape, hipStream_t s) {
    if (tape && prec == PREC_F32 && rr == 1 && amp == 1) {
        int device = 0, ncu = 0;
        hipError_t e = hipGetDevice(&device);
        if (e == hipSuccess)
            e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device);
        if (e != hipSuccess) return e;
        if (p.n_items <= ncu) {
            const PassKernel k{reinterpret_cast<const void *>(&tangent_trio_kernel), kTrioBlock,
                               sizeof(TrioLds), false};
            e = hipFuncSetAttribute(k.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.lds);
            if (e != hipSuccess) return e;
            return run_pass(k, p, env32, env64, 0, s);
        }
    }
    return run_pass(tape ? select_tangent<true>(prec, rr, amp) : select_tangent<false>(prec, rr, amp),
                    p, env32, env64, 0, s);
}

hipError_t launch_contract(const BatchParams &p, bool obs, int max_edges, hipStream_t s) {
    // a tape of a pass with FP64 steps is summed over that pass's rounds
    const bool grouped = p.prec == PREC_F32MIX;
    // the edge weights in LDS: at most 64 KB (4096 bins each); beside a
    // group's terms (128 KB) those that fit, else they are read from memory
    const size_t wb = (size_t)max_edges * sizeof(double);
    const bool ldsw = !grouped || wb <= 24 * 1024;
    const void *fn =
        !grouped ? (obs ? reinterpret_cast<const void *>(&contract_kernel<true>)
                        : reinterpret_cast<const void *>(&contract_kernel<false>))
        : ldsw   ? (obs ? reinterpret_cast<const void *>(&contract_group_kernel<true, true>)
                        : reinterpret_cast<const void *>(&contract_group_kernel<false, true>))
                 : (obs ? reinterpret_cast<const void *>(&contract_group_kernel<true, false>)
                        : reinterpret_cast<const void *>(&contract_group_kernel<false, false>));
    const int block = grouped ? kContractBlock : kPhaseBlock;
    const size_t lds = (grouped ? (size_t)kGradParams * kChiGroup * sizeof(double) : 0) +
                       (ldsw ? wb : 0);
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    int grid = 0;
    if (e == hipSuccess)
        e = resident_grid(fn, block, lds, grouped ? p.n_gitems : p.n_items, &grid);
    if (e != hipSuccess) return e;
    BatchParams pc = p;
    void *args[] = {&pc};
    return hipLaunchKernel(fn, dim3((unsigned)grid), dim3(block), args, lds, s);
}

hipError_t launch_grad_finalize(const BatchParams &p, hipStream_t s) {
    grad_finalize_kernel<<<p.n_shots, kGradFinBlock, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_grad_shadow(const BatchParams &p, int64_t span, hipStream_t s) {
    grad_shadow_kernel<<<(p.n_shots + 255) / 256, 256, 0, s>>>(p, span);
    return hipGetLastError();
}

hipError_t launch_radiation_derivs(const float *rad32d, const double *rad64d, int prec, int64_t n,
                                   const double *chi, double *out, int *flags, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int64_t blocks = (n + 255) / 256;
    rad_derivs_kernel<<<(unsigned)blocks, 256, 0, s>>>(rad32d, rad64d, prec, n, chi, out, flags);
    return hipGetLastError();
}

}  // namespace qs
