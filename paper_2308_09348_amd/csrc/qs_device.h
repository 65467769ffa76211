// qs_device.h -- device helpers shared by the kernels of the library: the
// sample generator, the radiation-function table lookups, the moment system,
// the spatial factor and ballistic path, RK4 steps, compensated sums, work
// items and wavefront reductions.
#pragma once

#include <hip/hip_runtime.h>
#include <climits>
#include <math.h>

#include <type_traits>

#include "qs_internal.h"

namespace qs {

// ===========================================================================
// Philox4x32-10 (Salmon et al., SC'11) and Box-Muller normals
// ===========================================================================
__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        const uint32_t lo0 = 0xD2511F53u * c[0], hi0 = __umulhi(0xD2511F53u, c[0]);
        const uint32_t lo1 = 0xCD9E8D57u * c[2], hi1 = __umulhi(0xCD9E8D57u, c[2]);
        const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
        c[0] = n0;
        c[1] = lo1;
        c[2] = n2;
        c[3] = lo0;
    }
}

// The beam coordinates of sample i of a shot (a volume element of Sec. 2):
// counter (i, shot, k, 0) for k = 0, 1 gives eight words, the first six make
// 24-bit uniforms u = ((r >> 8) + 1/2) 2^-24, and Box-Muller on the pairs
// (u0, u1), (u2, u3), (u4, u5) gives six standard normals n.  Transverse
// position: x_off + sigma_r (n0, n1), or for a flat-top beam the uniform disk
// x_off + sigma_r sqrt(u0) (cos 2 pi u1, sin 2 pi u1); longitudinal offset
// sigma_z n2, or sigma_z (u2 - 1/2) for a flat-top beam of length sigma_z;
// gamma0 + sigma_gamma n3; angles div (n4, n5).
struct SampleCoords {
    double x, y, z, g0, thx, thy;
    double n[6];
};

// Sample i of a shot table entry: sample i draw_stride of the shot (a view
// with draw_stride > 1 holds every draw_stride-th sample).
__device__ __forceinline__ void sample_coords(const ShotParams &sp, uint32_t k0, uint32_t k1,
                                              int64_t i, SampleCoords &sc) {
    uint32_t r[8];
    const uint32_t ctr0 = (uint32_t)(i * (int64_t)sp.draw_stride);
#pragma unroll
    for (uint32_t k = 0; k < 2; ++k) {
        uint32_t c[4] = {ctr0, (uint32_t)sp.shot_word, k, 0u};
        philox4x32_10(c, k0, k1);
        r[4 * k + 0] = c[0];
        r[4 * k + 1] = c[1];
        r[4 * k + 2] = c[2];
        r[4 * k + 3] = c[3];
    }
    double u[6], cs0 = 0.0, sn0 = 0.0;
#pragma unroll
    for (int m = 0; m < 6; ++m) u[m] = ((double)(r[m] >> 8) + 0.5) * 0x1p-24;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const double R = sqrt(-2.0 * log(u[2 * m]));
        double s, c;
        sincospi(2.0 * u[2 * m + 1], &s, &c);
        sc.n[2 * m] = R * c;
        sc.n[2 * m + 1] = R * s;
        if (m == 0) {
            cs0 = c;
            sn0 = s;
        }
    }
    // selects rather than branches: the hot loops that follow keep their
    // register budget
    const bool flat_r = (sp.profile & kFlatR) != 0;
    const double rad = sp.sigma_r * sqrt(u[0]);
    sc.x = fma(flat_r ? rad : sp.sigma_r, flat_r ? cs0 : sc.n[0], sp.x_off);
    sc.y = fma(flat_r ? rad : sp.sigma_r, flat_r ? sn0 : sc.n[1], sp.y_off);
    sc.z = sp.sigma_z * ((sp.profile & kFlatZ) ? u[2] - 0.5 : sc.n[2]);
    sc.g0 = fma(sp.sigma_gamma, sc.n[3], sp.gamma0);
    sc.thx = sp.div_rad * sc.n[4];
    sc.thy = sp.div_rad * sc.n[5];
}

// ===========================================================================
// Radiation functions: the combinations T1 = g, T2 = 2g + chi g', T3 = g + 2 chi g' +
// chi^2 g''/2 and T4 = h from per-cell cubics
// ===========================================================================
__device__ __forceinline__ void rad_eval32(const float *__restrict__ tab, float chi, float &g,
                                           float &G1, float &G2, float &hq) {
    // exponent and the top kSB32 mantissa bits give the cell directly
    const uint32_t b = __float_as_uint(chi);
    int c = (int)(b >> (23 - kSB32)) - ((127 + kEMin) << kSB32) + 1;
    float t = __uint_as_float(((b & ((1u << (23 - kSB32)) - 1)) << kSB32) | 0x3f800000u) - 1.0f;
    if (c < 1) {  // chi < 2^kEMin: the first cell, linear in chi
        c = 0;
        t = chi * 0x1p20f;
    }
    c = min(c, kCells32 - 1);  // chi >= 2^(kEMax+1) is reported by the caller
    // function-major layout: four arrays of 16-byte cubics, so that the cells
    // read by one wavefront start on eight different 4-bank groups of LDS
    const float4 *T = reinterpret_cast<const float4 *>(tab);
    const float4 q0 = T[c], q1 = T[kCells32 + c], q2 = T[2 * kCells32 + c],
                 q3 = T[3 * kCells32 + c];
    g = fmaf(t, fmaf(t, fmaf(t, q0.w, q0.z), q0.y), q0.x);
    G1 = fmaf(t, fmaf(t, fmaf(t, q1.w, q1.z), q1.y), q1.x);
    G2 = fmaf(t, fmaf(t, fmaf(t, q2.w, q2.z), q2.y), q2.x);
    hq = fmaf(t, fmaf(t, fmaf(t, q3.w, q3.z), q3.y), q3.x);
}

// One FP32 table cell held in registers.  Any chi near the cell maps to
// its local coordinate by t = chi * tw + ts; the RK4 stages that share a
// phase with the previous lookup (stage 3 after stage 2, the next step's
// stage 1 after stage 4) evaluate the same cubics a hair outside [0, 1]
// instead of reading LDS again.
struct RadCell32 {
    float4 q0, q1, q2, q3;
    float tw, ts;
};

// The index comes from chi clamped to the octave cells [2^kEMin, 2^(kEMax+1)).
// Below 2^kEMin the first octave cell's cubic is extrapolated down to chi = 0
// (t >= -2^kSB32): there g, chi g', chi^2 g'' and h are linear in chi to
// 1e-12, and so is the cell's cubic.  Above the table the result is not used
// (the caller reports the range error).
// With ncell, *nq also receives that cell's entry of ncell (a per-cell cubic
// of another function on the same cells).
__device__ __forceinline__ void rad_lookup32(const float *__restrict__ tab, float chi,
                                             RadCell32 &cell,
                                             const float4 *__restrict__ ncell = nullptr,
                                             float4 *nq = nullptr) {
    const float xc = fminf(fmaxf(chi, 0x1p-20f), 0x1.fffffep7f);
    const uint32_t b = __float_as_uint(xc);
    // cell 1 + (b - bits(2^kEMin)) >> (23 - SB): non-negative by the clamp
    const uint32_t c = ((b - ((uint32_t)(127 + kEMin) << 23)) >> (23 - kSB32)) + 1u;
    // cell start 2^e (1 + sub/2^SB) and inverse width 2^(SB - e)
    const float tw = __uint_as_float((uint32_t)(254 + kSB32 - (int)(b >> 23)) << 23);
    const float ts = -__uint_as_float(b & ~((1u << (23 - kSB32)) - 1)) * tw;
    const float4 *T = reinterpret_cast<const float4 *>(tab);
    cell.q0 = T[c];
    cell.q1 = T[kCells32 + c];
    cell.q2 = T[2 * kCells32 + c];
    cell.q3 = T[3 * kCells32 + c];
    cell.tw = tw;
    cell.ts = ts;
    if (ncell) *nq = ncell[c];
}

__device__ __forceinline__ void rad_cell_eval(const RadCell32 &cell, float chi, float &g,
                                              float &G1, float &G2, float &hq) {
    // returns the four table functions of the cell (see rhs_q32)
    const float t = fmaf(chi, cell.tw, cell.ts);
    g = fmaf(t, fmaf(t, fmaf(t, cell.q0.w, cell.q0.z), cell.q0.y), cell.q0.x);
    G1 = fmaf(t, fmaf(t, fmaf(t, cell.q1.w, cell.q1.z), cell.q1.y), cell.q1.x);
    G2 = fmaf(t, fmaf(t, fmaf(t, cell.q2.w, cell.q2.z), cell.q2.y), cell.q2.x);
    hq = fmaf(t, fmaf(t, fmaf(t, cell.q3.w, cell.q3.z), cell.q3.y), cell.q3.x);
}

// FP64 cell of chi and the coordinate t in the cell.  Chi outside the table (also any
// negative chi that does not round to 0, and NaN) gives a number past the last cell, to be
// clamped to that; it is reported by the caller.
// All in the upper word: the cell from its top bits, t = (chi - cell start)
// 2^(SB - e), both operations exact.  Below 2^kEMin64 the same of y = chi / 8 +
// (7/8) 2^kEMin64, which runs evenly through the last 16 cells of the octave below
// (above, y is less than chi): two operations on every chi, no branch and no
// selects (an even cell index by selects of its own cost FP64 passes 10%).
__device__ __forceinline__ uint32_t rad_index64(double chi, double &t) {
    constexpr int kLow = 20 - kSB64;  // bits of the upper word below the cell index
    constexpr double kMin = 1.0 / (1 << -kEMin64);
    static_assert(kLow64 == 16 && kSB64 == 6, "an eighth of an octave");
    const double y = fmax(chi, fma(chi, 0.125, 0.875 * kMin));
    const uint32_t hi = (uint32_t)__double2hiint(y);
    const double start = __hiloint2double((int)(hi >> kLow << kLow), 0);
    const double inv = __hiloint2double((int)((uint32_t)(2046 + kSB64) - (hi >> 20)) << 20, 0);
    t = (y - start) * inv;
    // (unsigned: the small y of a negative chi wraps)
    return (hi >> kLow) - (((1023 + kEMin64) << kSB64) - kLow64);
}

__device__ __forceinline__ void rad_cell_eval64(const double *q, double t, double &g, double &G1,
                                                double &G2, double &hq) {
    g = fma(t, fma(t, fma(t, q[3], q[2]), q[1]), q[0]);
    G1 = fma(t, fma(t, fma(t, q[7], q[6]), q[5]), q[4]);
    G2 = fma(t, fma(t, fma(t, q[11], q[10]), q[9]), q[8]);
    hq = fma(t, fma(t, fma(t, q[15], q[14]), q[13]), q[12]);
}

__device__ __forceinline__ void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Chi at coordinate t in [0, 1) of a table cell (sb: sub-cells per octave, emin:
// the lowest octave; the `low` cells before it, a power of two of them, are even
// in chi below 2^emin), the four Chebyshev nodes of a cell
// and the monomial coefficients l[0..3] of the Lagrange polynomial of node m
// (a cubic through the node values v_m is sum_m v_m l_m(t)).
__device__ __forceinline__ double cell_chi(int cell, double t, int sb, int emin, int low) {
    if (cell < low) return ldexp(((double)cell + t) / (double)low, emin);
    const int c = cell - low;
    const int e = emin + (c >> sb);
    const int sub = c & ((1 << sb) - 1);
    return ldexp(1.0 + ((double)sub + t) / (double)(1 << sb), e);
}

__device__ __forceinline__ double cheb_node(int m) {
    return 0.5 * (1.0 - cospi((2.0 * m + 1.0) / 8.0));
}

__device__ __forceinline__ void cheb_basis(int m, double l[4]) {
    double r[3];
    int k = 0;
    double den = 1.0;
    for (int n = 0; n < 4; ++n)
        if (n != m) {
            r[k++] = cheb_node(n);
            den *= cheb_node(m) - cheb_node(n);
        }
    // (t - r0)(t - r1)(t - r2) / den
    l[3] = 1.0 / den;
    l[2] = -(r[0] + r[1] + r[2]) / den;
    l[1] = (r[0] * r[1] + r[0] * r[2] + r[1] * r[2]) / den;
    l[0] = -(r[0] * r[1] * r[2]) / den;
}

// The drift's combinations of the forward functions (any linear one of them:
// values or coefficients).
__device__ __forceinline__ double drift_mix2(double g, double G1) { return fma(2.0, g, G1); }
__device__ __forceinline__ double drift_mix3(double g, double G1, double G2) {
    return fma(0.5, G2, fma(2.0, G1, g));
}

// The table of a pass without FP64 steps of the quantum model.
struct NoTable {
    __device__ __forceinline__ void eval(double, double *) const {}
};
// An FP64 table of F functions (cells of F cubics) with N of its cells in LDS, its
// first or (BASED) those from c0 on, each 16-byte word of the cells in an array
// of its own, so that lanes on neighbouring cells read neighbouring 16-byte
// words.  Where some lane's cell lies outside them the wavefront reads the
// global table.  The two branches meet in the functions' values: meeting in the
// coefficients took 4 F more registers, and reads of the same width in both are
// merged by the compiler into flat loads, which wait for both memories.  The
// values are those of the global table; the forward table's (F = 4) are combined
// for the drift (T1 .. T4), coefficient by coefficient, as the cells are staged.
template <int N, int F, bool BASED = false>
struct TabWindow {
    const double2 *win;  // [2 F][N]
    const double *p;     // the whole table, cell-major
    int c0;
    __device__ __forceinline__ void eval(double chi, double v[F]) const {
        double t;
        const uint32_t c = rad_index64(chi, t), k = BASED ? c - (uint32_t)c0 : c;
        if (__all(k < (uint32_t)N)) {
            const double2 *w = win + k;
            double2 q[2 * F];
#pragma unroll
            for (int e = 0; e < 2 * F; ++e) q[e] = w[e * N];
#pragma unroll
            for (int f = 0; f < F; ++f)
                v[f] = fma(t, fma(t, fma(t, q[2 * f + 1].y, q[2 * f + 1].x), q[2 * f].y), q[2 * f].x);
        } else {
            // (two powers at a time: with a whole cell's 4 F coefficients at once in
            // registers the mixed tape pass spilled more: eight shots of 2^18 x 2048
            // steps 68.1 ms, 65.6 so)
            const double *cell = p + (size_t)min(c, (uint32_t)kCells64 - 1) * (4 * F);
#pragma unroll
            for (int e = 2; e >= 0; e -= 2) {
                double q[2][F];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
#pragma unroll
                    for (int f = 0; f < F; ++f) q[k][f] = cell[4 * f + e + k];
                    if constexpr (F == 4) {
                        q[k][2] = drift_mix3(q[k][0], q[k][1], q[k][2]);
                        q[k][1] = drift_mix2(q[k][0], q[k][1]);
                    }
                }
#pragma unroll
                for (int f = 0; f < F; ++f)
                    v[f] = e == 2 ? fma(t, q[1][f], q[0][f])
                                  : fma(t, fma(t, v[f], q[1][f]), q[0][f]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // filled by all threads of the block; a barrier must follow
    __device__ __forceinline__ TabWindow(double2 *w, const double *tab, int first = 0)
        : win(w), p(tab), c0(first) {
        static_assert(N <= kCells64, "a part of the table");
        const double2 *src = reinterpret_cast<const double2 *>(tab) + 2 * F * (size_t)first;
        if constexpr (F == 4) {
            for (int k = threadIdx.x; k < 2 * N; k += blockDim.x) {  // half a cell
                const int cell = k >> 1, half = k & 1;
                const double2 *q = src + 8 * cell + half;
                const double2 g = q[0], G1 = q[2], G2 = q[4], h = q[6];
                double2 *o = w + half * N + cell;
                o[0] = g;
                o[2 * N] = make_double2(drift_mix2(g.x, G1.x), drift_mix2(g.y, G1.y));
                o[4 * N] = make_double2(drift_mix3(g.x, G1.x, G2.x), drift_mix3(g.y, G1.y, G2.y));
                o[6 * N] = h;
            }
        } else {
            for (int k = threadIdx.x; k < 2 * F * N; k += blockDim.x) {
                const int cell = k / (2 * F);
                w[(k - cell * (2 * F)) * N + cell] = src[k];
            }
        }
    }
};

// ===========================================================================
// The moment system (second-order closure of the drift-diffusion process
// whose drift is eq. dpdtRR in phase units):
//   dmu/dpsi   = A + A'' sig2 / 2,   dsig2/dpsi = 2 A' sig2 + D,
//   A = -K a^2 mu^2 g,  A' = -K a^2 mu (2g + G1),  A'' = -K a^2 (2g + 4G1 + G2),
//   D = C_D |a|^3 mu^4 h,  chi = 2 mu |a| / a_S.
// ===========================================================================
template <class T>
struct Phys {
    T K, CD, two_over_aS;
};

// 1/sqrt(q) and iq = 1/q for q >= 1, from the hardware's estimate y of the root
// (about 2^-24): with e = 1 - q y^2, q^-1/2 = y (1 + e/2 + 3 e^2/8 + ..) and 1/q =
// y^2 (1 + e + e^2 + ..), each within an ulp (the square of the rounded root has
// two).  q beyond 1e300 counts as 1e300, the factor it gives as 0.
__device__ __forceinline__ double inv_sqrt64(double q, double &iq) {
    q = fmin(q, 1e300);
    const double y = __builtin_amdgcn_rsq(q), y2 = y * y;
    const double e = fma(-q, y2, 1.0);
    iq = fma(y2, fma(e, e, e), y2);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// e^x for x < 700 (0 below -800): x = k ln 2 + r, |r| <= ln 2 / 2, ln 2 in two parts
// of which the upper has 33 bits, so that k times it is exact (Cody and Waite's
// reduction, with the parts of fdlibm's e_exp.c), then the Taylor polynomial of
// degree 12, scaled by 2^k.  Of the remainder, r^13 / 13!, the share 0.955 (ln 2 / 2)^2
// r^11 / 13! goes into the eleventh coefficient, which leaves 8e-18 of it (1.7e-16
// at the ends without): over [-20, 0] within 1.45e-16 of e^x, rms 4.9e-17 (3.5e-16,
// 6.1e-17).
__device__ __forceinline__ double exp64(double x) {
    x = fmax(x, -800.0);
    const double k = rint(x * 1.44269504088896340736);
    const double r = fma(-k, 1.9082149292705877e-10, fma(-k, 0.693147180369123816490, x));
    double p = 1.0 / 479001600.0;
    p = fma(p, r, 1.0 / 39916800.0 + 0.955 * 0.120113253 / 6227020800.0);
    p = fma(p, r, 1.0 / 3628800.0);
    p = fma(p, r, 1.0 / 362880.0);
    p = fma(p, r, 1.0 / 40320.0);
    p = fma(p, r, 1.0 / 5040.0);
    p = fma(p, r, 1.0 / 720.0);
    p = fma(p, r, 1.0 / 120.0);
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return ldexp(p, (int)k);
}

// Spatial factor a/a0 of eq. a0eff at (x, y, z) [um].  The FP32 version uses
// the hardware reciprocal, reciprocal square root and base-2 exponential
// (about one ulp each; the exponent's argument rounding adds |r2/q| ulps,
// which matters only where the factor itself is small).
__device__ __forceinline__ float spatial(float x, float y, float z, float inv_w0sq, float inv_zR) {
    const float zz = z * inv_zR;
    const float q = fmaf(zz, zz, 1.0f);
    const float rq = __builtin_amdgcn_rsqf(q);  // 1/sqrt(q); 1/q = rq^2
    const float r2 = fmaf(x, x, y * y) * inv_w0sq;
    return __builtin_amdgcn_exp2f(-1.4426950408889634f * r2 * (rq * rq)) * rq;
}
__device__ __forceinline__ double spatial(double x, double y, double z, double inv_w0sq,
                                          double inv_zR) {
    const double zz = z * inv_zR;
    double iq;
    const double rq = inv_sqrt64(fma(zz, zz, 1.0), iq);
    const double r2 = fma(x, x, y * y) * inv_w0sq;
    return exp64(-r2 * iq) * rq;
}

// Higher transverse modes (amplitude only, peak 1 in the focal plane): with
// u = x/W, v = y/W, W = W0 sqrt(q), q = 1 + z^2/zR^2,
//   Hermite-Gauss m, n:  |H_m(sqrt2 u) H_n(sqrt2 v)| exp(-(u^2 + v^2)) / sqrt(q),
//   Laguerre-Gauss p, l: t^(|l|/2) |L_p^|l|(t)| exp(-t/2) / sqrt(q), t = 2(u^2 + v^2),
// divided by the mode's focal-plane peak; H and L by their three-term
// recurrences (H_(k+1) = 2s H_k - 2k H_(k-1); (k+1) L_(k+1) =
// (2k + 1 + l - t) L_k - (k + l) L_(k-1)).
template <class T>
__device__ __forceinline__ T hermite(int m, T s) {
    T h0 = T(1), h1 = T(2) * s;
    if (m == 0) return h0;
    for (int k = 1; k < m; ++k) {
        const T h2 = fma(T(2) * s, h1, T(-2 * k) * h0);
        h0 = h1;
        h1 = h2;
    }
    return h1;
}
template <class T>
__device__ __forceinline__ T spatial_mode(T x, T y, T z, T inv_w0sq, T inv_zR, int mode, int mm,
                                          int mn, T inv_norm) {
    const T zz = z * inv_zR;
    const T q = fma(zz, zz, T(1));
    const T iq = T(1) / q;
    const T u2 = x * x * inv_w0sq * iq, v2 = y * y * inv_w0sq * iq;
    const T g = exp(-(u2 + v2)) * sqrt(iq) * inv_norm;
    if (mode == 1) {  // Hermite-Gauss
        const T r2 = sqrt(T(2) * inv_w0sq * iq);
        return fabs(hermite<T>(mm, x * r2) * hermite<T>(mn, y * r2)) * g;
    }
    const int l = abs(mn);  // Laguerre-Gauss, p = mm
    const T t = T(2) * (u2 + v2);
    T L0 = T(1), L1 = T(1 + l) - t, Lp = L0;
    if (mm >= 1) Lp = L1;
    for (int k = 1; k < mm; ++k) {
        const T L2 = (fma(T(2 * k + 1 + l) - t, L1, T(-(k + l)) * L0)) / T(k + 1);
        L0 = L1;
        L1 = L2;
        Lp = L2;
    }
    T tp = T(1);
    for (int k = 0; k < l / 2; ++k) tp *= t;
    if (l & 1) tp *= sqrt(t);
    return tp * fabs(Lp) * g;
}

// Geometry of one sample along its ballistic path: at phase psi it has
// travelled l = psi lambda / (4 pi) past its collision point.  mode != 0
// selects a higher transverse mode (QS_MODE_HG 1, QS_MODE_LG 2).
// MODES = false compiles the Gaussian focus alone (the hot loop's register
// budget does not carry the mode recurrences).
template <class T, bool MODES = true>
struct Path {
    T xc, yc, thx, thy, zstar, inv_w0sq, inv_zR;
    int mode, mm, mn;
    T inv_norm;
    __device__ __forceinline__ T S(T ell) const {
        if constexpr (MODES) {
            if (mode != 0)
                return spatial_mode<T>(fma(thx, ell, xc), fma(thy, ell, yc), zstar - ell,
                                       inv_w0sq, inv_zR, mode, mm, mn, inv_norm);
        }
        return spatial(fma(thx, ell, xc), fma(thy, ell, yc), zstar - ell, inv_w0sq, inv_zR);
    }
};

// Sample i of a shot (Sec. 2 volume element): its initial Lorentz factor and
// angles, its ballistic path and the spatial factor at its collision point.
template <bool MODES = true>
__device__ __forceinline__ void draw_sample(const ShotParams &sp, uint32_t key0, uint32_t key1,
                                            int64_t i, double &g0, double &thx, double &thy,
                                            Path<double, MODES> &pd, double &S0) {
    SampleCoords sc;
    sample_coords(sp, key0, key1, i, sc);
    const double x = sc.x, y = sc.y, z = sc.z;
    g0 = sc.g0;
    thx = sc.thx;
    thy = sc.thy;
    pd.xc = fma(thx, 0.5 * z, x);
    pd.yc = fma(thy, 0.5 * z, y);
    pd.thx = thx;
    pd.thy = thy;
    pd.zstar = fma(0.5, z, sp.z_delay);
    pd.inv_w0sq = sp.inv_w0sq;
    pd.inv_zR = sp.inv_zR;
    pd.mode = sp.mode;
    pd.mm = sp.mode_m;
    pd.mn = sp.mode_n;
    pd.inv_norm = sp.mode_inv_norm;
    S0 = sp.plane_wave ? 1.0 : pd.S(0.0);
}

// Order in which the lanes of a block take the samples of an FP32 pass: by an
// FP32 estimate of the chi scale S0 gamma0 of a sample at its collision point
// (the first counter block's normals by Box-Muller in FP32, the collision
// point without the divergence's shift, below 1e-2 um).  The results of these
// passes do not depend on the order.
__device__ __forceinline__ float chi_key32(const ShotParams &sp, uint32_t k0, uint32_t k1,
                                           int64_t i) {
    uint32_t c[4] = {(uint32_t)(i * (int64_t)sp.draw_stride), (uint32_t)sp.shot_word, 0u, 0u};
    philox4x32_10(c, k0, k1);
    float u[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) u[m] = ((float)(c[m] >> 8) + 0.5f) * 0x1p-24f;
    const float R0 = __builtin_sqrtf(-2.0f * __logf(u[0])), R1 = __builtin_sqrtf(-2.0f * __logf(u[2]));
    float s0, c0, s1, c1;
    __sincosf(6.28318530717958648f * u[1], &s0, &c0);
    __sincosf(6.28318530717958648f * u[3], &s1, &c1);
    const bool flat_r = (sp.profile & kFlatR) != 0;
    const float sr = (float)sp.sigma_r, rad = flat_r ? sr * __builtin_sqrtf(u[0]) : sr * R0;
    const float x = fmaf(rad, c0, (float)sp.x_off), y = fmaf(rad, s0, (float)sp.y_off);
    const float z = (float)sp.sigma_z * ((sp.profile & kFlatZ) ? u[2] - 0.5f : R1 * c1);
    const float g0 = fmaf((float)sp.sigma_gamma, R1 * s1, (float)sp.gamma0);
    if (sp.plane_wave) return g0;
    return g0 * spatial(x, y, fmaf(0.5f, z, (float)sp.z_delay), sp.inv_w0sqf, sp.inv_zRf);
}

// Order of the G samples from `base` on by chi_key32 (stable: ties by index);
// s_idx[r] receives the offset of rank r; offsets at or past `end` (no sample)
// rank last.  B threads take part.
template <int G, int B>
__device__ __forceinline__ void chi_order32(const ShotParams &sp, uint32_t key0, uint32_t key1,
                                            int64_t base, int64_t end, float *s_key,
                                            unsigned short *s_idx) {
    static_assert(G % B == 0 && G <= 65536, "group of whole rounds, 16-bit offsets");
    __syncthreads();  // the previous group's order is no longer read
    for (int q = threadIdx.x; q < G; q += B) {
        const int64_t i = base + q;
        // (a key that is no number, where 1/w0^2 overflows FP32, has no rank: lowest)
        s_key[q] = i < end ? fmaxf(chi_key32(sp, key0, key1, i), -0x1.fffffep127f)
                           : __builtin_inff();
    }
    __syncthreads();
    for (int q = threadIdx.x; q < G; q += B) {
        const float k = s_key[q];
        int rank = 0;
        for (int j = 0; j < G; ++j) {
            const float kj = s_key[j];
            rank += (kj < k || (kj == k && j < q)) ? 1 : 0;
        }
        s_idx[rank] = (unsigned short)q;
    }
    __syncthreads();
}

// Work item k of a shot in a pass with FP64 steps, as the first sample of its
// round of SIZE samples: the rounds of highest chi of all groups come first (a
// round costs up to several times as much in FP64 steps), so that the last
// items of a launch are short ones: one quantum shot of 2^18 x 2048 steps, two
// items a resident block, 6.44 -> 5.05 ms; eight with the tape 98.5 -> 95.2 ms.
template <int SIZE>
__device__ __forceinline__ int64_t ordered_round(int64_t n_samples, int64_t k) {
    constexpr int kPer = kChiGroup / SIZE;  // rounds of a full group
    const int64_t nr = (n_samples + SIZE - 1) / SIZE, full = nr / kPer;
    const int last = (int)(nr - full * kPer);  // rounds of a group short of kPer
    const int64_t top = (kPer - last) * full;  // items above the short group's rounds
    int64_t group, round;
    if (k < top) {
        group = k % full;
        round = kPer - 1 - k / full;
    } else {
        group = (k - top) % (full + 1);
        round = last - 1 - (k - top) / (full + 1);
    }
    return group * kChiGroup + round * SIZE;
}

// Sample of lane rank `rank` of a group of cnt samples from `base` on of a shot
// in a pass with FP64 steps (order_kernel); ranks at or past cnt (no sample)
// take the last rank's.
__device__ __forceinline__ int64_t ordered_sample(const BatchParams &P, const ShotParams &sp,
                                                  int64_t base, int cnt, int rank) {
    return base + P.order[sp.state_off + base + min(rank, cnt - 1)];
}

// One RK4 step of the classical model (g = 1, sig2 stays 0) from psi_j with
// amplitudes a1 = a(psi_j), ah = a(psi_j + h/2), a4 = a(psi_j + h).
template <class T>
__device__ __forceinline__ T rk4_classical(T mu, T a1, T ah, T a4, T h, const Phys<T> &ph) {
    const T hh = T(0.5) * h;
    auto f = [&](T m, T a) { return -(ph.K * (a * a)) * m * m; };
    const T k1 = f(mu, a1);
    const T k2 = f(fma(hh, k1, mu), ah);
    const T k3 = f(fma(hh, k2, mu), ah);
    const T k4 = f(fma(h, k3, mu), a4);
    const T h6 = h * T(1.0 / 6.0);
    return h6 * (k1 + T(2) * (k2 + k3) + k4);
}

// Moment right-hand side (quantum model) from the table's combined functions
// at chi = two_over_aS mu |a|:
//   dmu/dpsi   = -K a^2 (mu^2 T1 + sig2 T3),
//   dsig2/dpsi = -2 K a^2 mu sig2 T2 + C_D a^2 |a| mu^4 T4.
// The factors that depend on the amplitude only are formed once per phase
// point (stages 2 and 3 share one, stage 4 hands its to the next stage 1).
template <class T>
struct AmpFactors {
    T nu;   // -K a^2
    T nu2;  // -2 K a^2
    T cd;   // C_D a^2 |a|
    T cpm;  // chi per unit mu: 2 |a| / a_S
    __device__ __forceinline__ AmpFactors() {}
    __device__ __forceinline__ AmpFactors(T a, const Phys<T> &ph) {
        const T aa = fabs(a), a2 = a * a;
        nu = -ph.K * a2;
        nu2 = T(2) * nu;
        cd = ph.CD * aa * a2;
        cpm = ph.two_over_aS * aa;
    }
};
using AmpQ = AmpFactors<float>;

// x: dmu/dpsi over nu.
template <class T>
__device__ __forceinline__ void rhs_quantum(T mu, T s2, const AmpFactors<T> &A, T T1, T T2, T T3,
                                            T T4, T &x, T &ds2) {
    const T mu2 = mu * mu;
    x = fma(mu2, T1, s2 * T3);
    ds2 = fma(A.nu2 * mu * s2, T2, A.cd * (mu2 * mu2) * T4);
}

// One FP64 RK4 step of the quantum moment system; A1 (the factors at psi_j) is
// replaced by those at psi_j + h.
template <class Tab>
__device__ __forceinline__ void rk4_q64(double mu, double s2, AmpFactors<double> &A1, double ah,
                                        double a4, double h, const Phys<double> &ph,
                                        const Tab &tab, double &dmu, double &ds2,
                                        double &chi_hi) {
    const double hh = 0.5 * h;
    double k1m, k1s, k2m, k2s, k3m, k3s, k4m, k4s;
    auto stage = [&](double m, double s, const AmpFactors<double> &A, double &km, double &ks) {
        const double chi = A.cpm * m;
        chi_hi = fmax(chi_hi, chi);
        double T[4];
        tab.eval(chi, T);
        double x;
        rhs_quantum(m, s, A, T[0], T[1], T[2], T[3], x, ks);
        km = A.nu * x;
    };
    stage(mu, s2, A1, k1m, k1s);
    const AmpFactors<double> Ah(ah, ph);
    stage(fma(hh, k1m, mu), fma(hh, k1s, s2), Ah, k2m, k2s);
    stage(fma(hh, k2m, mu), fma(hh, k2s, s2), Ah, k3m, k3s);
    A1 = AmpFactors<double>(a4, ph);
    stage(fma(h, k3m, mu), fma(h, k3s, s2), A1, k4m, k4s);
    const double h6 = h * (1.0 / 6.0);
    dmu = h6 * (k1m + 2.0 * (k2m + k3m) + k4m);
    ds2 = h6 * (k1s + 2.0 * (k2s + k3s) + k4s);
}

// One FP32 RK4 step of the quantum moment system with two table reads:
// stage 2 and stage 4 read LDS, stage 3 reuses stage 2's cell, and stage 4's
// cell is handed to the next step's stage 1 (with its amplitude factors).
// Ah, A4: the factors at psi_j + h/2 and psi_j + h (A1 is replaced by A4).
// The increments are h6 dm and h6 ds, h6 = h/6.  Products that are added to
// something are fused here by name, not as the compiler finds them: it does so
// within a block of code, and the kernels that share this step divide it
// differently.  ROUND: the sum k2 + k3 of the energy takes both rounded, else the
// product of k2 unrounded (see q32_steps).
template <bool ROUND>
__device__ __forceinline__ void rk4_q32(float mu, float s2, AmpQ &A1, const AmpQ &Ah,
                                        const AmpQ &A4, float h, const float *__restrict__ tab,
                                        RadCell32 &carry, float &dm, float &ds, float &chi_hi) {
#pragma clang fp contract(off)
    const float hh = 0.5f * h;
    float g, G1, G2, hq;
    // stage 1 (cell and amplitude factors carried from the previous stage 4)
    const float c1 = A1.cpm * mu;
    rad_cell_eval(carry, c1, g, G1, G2, hq);
    float x1, k1s;
    rhs_quantum(mu, s2, A1, g, G1, G2, hq, x1, k1s);
    const float k1m = A1.nu * x1;
    // stage 2 (table read)
    const float m2 = fmaf(hh, k1m, mu), s22 = fmaf(hh, k1s, s2);
    const float c2 = Ah.cpm * m2;
    RadCell32 mid;
    rad_lookup32(tab, c2, mid);
    rad_cell_eval(mid, c2, g, G1, G2, hq);
    float x2, k2s;
    rhs_quantum(m2, s22, Ah, g, G1, G2, hq, x2, k2s);
    // stage 3 (same phase as stage 2: reuse its cell)
    const float k2m = Ah.nu * x2;
    const float m3 = fmaf(hh, k2m, mu), s23 = fmaf(hh, k2s, s2);
    const float c3 = Ah.cpm * m3;
    rad_cell_eval(mid, c3, g, G1, G2, hq);
    float x3, k3s;
    rhs_quantum(m3, s23, Ah, g, G1, G2, hq, x3, k3s);
    const float k3m = Ah.nu * x3;
    const float k23 = ROUND ? k2m + k3m : fmaf(Ah.nu, x2, k3m);
    // stage 4 (table read; its cell serves the next step's stage 1)
    A1 = A4;
    const float m4 = fmaf(h, k3m, mu), s24 = fmaf(h, k3s, s2);
    const float c4 = A1.cpm * m4;
    rad_lookup32(tab, c4, carry);
    rad_cell_eval(carry, c4, g, G1, G2, hq);
    float x4, k4s;
    rhs_quantum(m4, s24, A1, g, G1, G2, hq, x4, k4s);
    // the range check takes the chi of the table reads: stages 1 and 3
    // evaluate the cells of stages 4 and 2 at a chi a hair away (the state
    // moved by less than one step's increment)
    chi_hi = fmaxf(chi_hi, fmaxf(c2, c4));
    dm = fmaf(A1.nu, x4, fmaf(2.0f, k23, k1m));
    ds = fmaf(2.0f, k2s + k3s, k1s) + k4s;
}

// Steps j0 .. j1 - 1 (j0 even) of the FP32 quantum model with the local amplitude by
// step(j, round): of two steps the first rounds k2 (rk4_q32), a last one does not.
// Every kernel that takes such steps has this rule, so that a shot gives the same
// bits in all of them; which of the two a step takes is of no account (a last bit of
// its increment), and these are what the passes have always given.
template <class Step>
__device__ __forceinline__ void q32_steps(int j0, int j1, Step step) {
    int j = j0;
    for (; j + 1 < j1; j += 2) {
        step(j, std::true_type{});
        step(j + 1, std::false_type{});
    }
    if (j < j1) step(j, std::false_type{});
}

// Compensated accumulation: (hi, lo) += d or c d, renormalised (Fast2Sum, |hi| >= |d|).
__device__ __forceinline__ void comp_add(float &hi, float &lo, float d) {
    const float dd = d + lo;
    const float s = hi + dd;
    lo = dd - (s - hi);
    hi = s;
}
__device__ __forceinline__ void comp_add(float &hi, float &lo, float c, float d) {
    const float dd = fmaf(c, d, lo);
    const float s = hi + dd;
    lo = dd - (s - hi);
    hi = s;
}

// ===========================================================================
// Work items.  A launch covers n_shots shots; phase items are tiles of
// kPhaseBlock consecutive samples of one shot (one sample per lane), deposit
// items tiles of dep_tile samples (a multiple of kMomTile, the tile of the
// moment partial sums).  Blocks take items from a counter; an item's result
// does not depend on which block runs it, nor on dep_tile, so the output is
// deterministic, and a shot gives the same bits alone or in a batch.
// ===========================================================================
__device__ __forceinline__ int find_shot(const ShotParams *shots, int n_shots, int64_t item,
                                         bool deposit) {
    int lo = 0, hi = n_shots - 1;  // largest s whose first item is <= item
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        const int64_t first = deposit ? shots[mid].ditem0 : shots[mid].item0;
        if (first <= item)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// The same from shot s0 on, for a block that took an item of shot s0 before
// (a block takes items in increasing order, so the shot is s0 or a later one,
// mostly within a few): a doubling search forward from s0, then bisection.
__device__ __forceinline__ int find_shot_from(const ShotParams *shots, int n_shots, int64_t item,
                                              bool deposit, int s0) {
    auto first = [&](int s) { return deposit ? shots[s].ditem0 : shots[s].item0; };
    int lo = s0, step = 1;  // first(lo) <= item throughout
    while (lo + step < n_shots && first(lo + step) <= item) {
        lo += step;
        step <<= 1;
    }
    int hi = min(lo + step, n_shots) - 1;  // first(hi + 1) > item, or hi the last shot
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first(mid) <= item)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// The shot of a group of the mixed-precision derivative passes.
__device__ __forceinline__ int find_group_shot(const ShotParams *shots, int n_shots, int64_t grp) {
    int lo = 0, hi = n_shots - 1;  // largest s whose first group is <= grp
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (shots[mid].gitem0 <= grp)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ int64_t next_item(unsigned int *counter, int64_t *slot) {
    if (threadIdx.x == 0) *slot = (int64_t)atomicAdd(counter, 1u);
    __syncthreads();
    const int64_t item = *slot;
    __syncthreads();
    return item;
}

// Bilinear weights of a sample on its shot's node grid (a0,eff / a0 = S0 in
// [0, 1]; with one gamma0 node the last two weights are zero) and the nodes' states.
struct NodeCell {
    double w[4];
    int n[4];
    __device__ __forceinline__ NodeCell(const ShotParams &sp, double S0, double g0) {
        const int K = sp.n_anode, M = sp.n_gnode;
        const double ta = S0 * (double)(K - 1);
        const int k = min((int)ta, K - 2);
        const double fa = ta - (double)k;
        int m = 0;
        double fg = 0.0;
        if (M > 1) {
            const double tg =
                fmin(fmax((g0 - sp.g_node_lo) / sp.g_node_step, 0.0), (double)(M - 1));
            m = min((int)tg, M - 2);
            fg = tg - (double)m;
        }
        w[0] = (1.0 - fa) * (1.0 - fg);
        w[1] = fa * (1.0 - fg);
        w[2] = (1.0 - fa) * fg;
        w[3] = fa * fg;
        n[0] = k * M + m;
        n[1] = n[0] + M;
        n[2] = M > 1 ? n[0] + 1 : n[0];
        n[3] = M > 1 ? n[1] + 1 : n[1];
    }
};

// Coordinates of the samples of a plane-wave reconstruction (S0, gamma0, the
// angles), a wavefront a tile of kPhaseBlock samples.
__device__ __forceinline__ void draw_samples(const BatchParams &P) {
    const int lane = threadIdx.x & 63;
    int s_prev = 0;  // the shot of the wavefront's previous tile
    for (;;) {
        unsigned int taken = 0;
        if (lane == 0) taken = atomicAdd(&P.queue[2], 1u);
        const int64_t item = __builtin_amdgcn_readfirstlane(taken);
        if (item >= P.n_draws) break;
        const int s = __builtin_amdgcn_readfirstlane(
            find_shot_from(P.draw_shots, P.n_shots, item, false, s_prev));
        s_prev = s;
        const ShotParams &sp = P.draw_shots[s];
        const int64_t i0 = (item - sp.item0) * kPhaseBlock;
        const int64_t i1 = i0 + kPhaseBlock < sp.n_samples ? i0 + kPhaseBlock : sp.n_samples;
        for (int64_t i = i0 + lane; i < i1; i += 64) {
            double g0, thx, thy, S0;
            Path<double> pd;
            draw_sample(sp, P.key0, P.key1, i, g0, thx, thy, pd, S0);
            const int64_t o = sp.state_off + i;
            P.draw_st.S0[o] = S0;
            P.draw_st.g0[o] = g0;
            P.draw_st.thx[o] = thx;
            P.draw_st.thy[o] = thy;
        }
    }
}

// ===========================================================================
// Deposit of sample laws into fixed-point histograms
// ===========================================================================
// The deposited law of a sample is its own law (a point at v if s = 0, else
// N(v, s^2)) convolved with the deposit kernel (POINT: none; CIC: a box one
// bin wide; GAUSS: N(0, (ksig bins)^2)).  Bin masses are differences of the
// law's CDF at the bin edges, quantised to 2^-32 so that every sample adds
// exactly 2^32; beyond 6 standard deviations the CDF is taken as 0 or 1 (the
// neglected mass, 2e-9 a sample, goes to the edge bins of the window).  The
// CDF is evaluated in FP32 on whichever side of v keeps it small (the tail),
// so its error is a few ulps of the smaller tail mass.  For the box (x)
// Gaussian law the CDF is a difference of Psi(x) = Int_-inf^x Phi(u/s) du at
// the two box ends, and consecutive edges share one end.  Psi is of order s
// while the difference is of order one bin, so for laws wider than 4 bins
// that difference would lose log2(s / bin) bits in FP32; there the CDF is
// the box average of Phi as a series in beta = bin / s instead,
//   F = Phi(z) + beta^2/24 Phi''(z) + beta^4/1920 Phi''''(z),  z = t / s,
// whose next term is below 2e-9 for beta <= 1/4.
constexpr unsigned long long kOne = 1ull << 32;

// erfc(a) for a >= 0 without branches, given ea2 = exp(-a^2): the
// Chebyshev-fitted form erfc(a) = t exp(-a^2 + P(t)), t = 1 / (1 + a/2), of
// Press, Teukolsky, Vetterling and Flannery, Numerical Recipes (2nd ed.,
// Sec. 6.2), fractional error below 1.2e-7 for every a >= 0.  The library
// erfcf branches on the argument range, which costs a wavefront every branch
// its lanes take.
__device__ __forceinline__ float erfc_pos(float a, float ea2) {
    const float t = __builtin_amdgcn_rcpf(fmaf(0.5f, a, 1.0f));
    float p = 0.17087277f;
    p = fmaf(p, t, -0.82215223f);
    p = fmaf(p, t, 1.48851587f);
    p = fmaf(p, t, -1.13520398f);
    p = fmaf(p, t, 0.27886807f);
    p = fmaf(p, t, -0.18628806f);
    p = fmaf(p, t, 0.09678418f);
    p = fmaf(p, t, 0.37409196f);
    p = fmaf(p, t, 1.00002368f);
    p = fmaf(p, t, -1.26551223f);
    return t * ea2 * __expf(p);
}

// One law of a lane, ready for the wavefront deposit: kind 1 box, 2 Gaussian,
// 3 box (x) Gaussian, 4 box (x) Gaussian wider than 4 bins (the series), over
// edges ka .. kb (t0 = edge ka - v; sf the width, for kind 4 beta^2 instead);
// kind 0 when the sample deposits as a point (NGP bin in `ngp`: 0 underflow,
// k + 1 for bin k, n + 1 overflow), -1 when the lane has no sample.
struct LawLane {
    int kind, ka, kb, ngp;
    float t0, sf, inv_s;
};

// (inv_w: 1 / w; the window and bin decisions take the product, which
// differs from the quotient by an ulp at most: a value within 1e-16 of an
// edge may fall on either side)
__device__ __forceinline__ LawLane law_setup(double v, double s, int dep, double ksig, double lo,
                                             double w, double inv_w, int n) {
    LawLane L{0, 0, -1, 0, 0.0f, 0.0f, 0.0f};
    const double half = 0.5 * w;
    double se = s;
    if (dep == 2) {  // GAUSS
        const double ks = ksig * w;
        se = sqrt(s * s + ks * ks);
        L.kind = se > 0.0 ? 2 : 0;
    } else if (dep == 1) {  // CIC
        L.kind = s > 0.0 ? 3 : 1;
    } else {
        L.kind = s > 0.0 ? 2 : 0;
    }
    if (L.kind != 0) {
        const double reach =
            L.kind == 1 ? half : (L.kind == 2 ? 6.0 * se : 6.0 * se + half);
        const int ka =
            max((int)fmin(fmax(ceil((v - reach - lo) * inv_w), -1.0), (double)n + 1.0), 0);
        const int kb =
            min((int)fmin(fmax(floor((v + reach - lo) * inv_w), -1.0), (double)n + 1.0), n);
        if (ka > kb) {
            L.kind = 0;  // the whole law lies inside one bin (or outside)
        } else {
            L.ka = ka;
            L.kb = kb;
            L.t0 = (float)(fma((double)ka, w, lo) - v);
            L.sf = (float)se;
            L.inv_s = L.kind >= 2 ? __builtin_amdgcn_rcpf((float)se) : 0.0f;  // about one ulp
            if (L.kind == 3 && se >= 4.0 * w) {
                L.kind = 4;
                const float beta = (float)w * L.inv_s;
                L.sf = beta * beta;
            }
        }
    }
    if (L.kind == 0) {
        const double x = (v - lo) * inv_w;  // bin floor(x); v on an edge goes up
        L.ngp = !(x >= 0.0) ? 0 : (x >= (double)n ? n + 1 : (int)x + 1);
    }
    return L;
}

// Inclusive prefix maximum over the 64 lanes of a wavefront (DPP: shifts
// within rows of 16 lanes, then the row ends broadcast to the rows after).
__device__ __forceinline__ int wave_incl_max(int v) {
    v = max(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x111, 0xf, 0xf, false));  // row_shr:1
    v = max(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x112, 0xf, 0xf, false));  // row_shr:2
    v = max(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x114, 0xf, 0xf, false));  // row_shr:4
    v = max(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x118, 0xf, 0xf, false));  // row_shr:8
    v = max(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x142, 0xa, 0xf, false));  // row_bcast:15
    v = max(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x143, 0xc, 0xf, false));  // row_bcast:31
    return v;
}

// The laws of the 64 lanes of a wavefront, deposited together.  A law spans
// anywhere from one bin to the whole window, so one lane per law would leave
// most lanes idle behind the widest: instead the work of all 64 laws is laid
// end to end and the lanes take 64 consecutive pieces at a time; a lane finds
// its law from the marked starts of the block through a prefix maximum, and
// reads the law from the wavefront's LDS rows.  Two passes:
//  - positions (the box, the narrow box (x) Gaussian, Gaussians whose edges
//    lie more than a quarter standard deviation apart): one piece per edge,
//    law s taking edges ka - 1 .. kb (the first only to supply the lower box
//    end of edge ka), each edge's CDF evaluated on its own;
//  - runs (the wide box (x) Gaussian series and Gaussians with edges at most a
//    quarter standard deviation apart): one piece per run of up to kRunLen
//    consecutive edges on one side of the law's centre, starting at the run's
//    edge farthest from the centre.  The tail there is evaluated as in the
//    position pass; towards the centre the run adds the integral of the
//    Gaussian density phi over each edge interval by Boole's rule on four
//    subintervals of h = dz / 4 (dz: edge spacing in standard deviations, at
//    most 1/4), or by Simpson's on two of h = dz / 2 when every run of the
//    wavefront has dz <= 1/10, phi following the lattice by
//    phi(a - h) = phi(a) e^(a h - h^2/2) (one exponential a run: the ratio
//    itself shrinks by e^(-h^2) from one subinterval to the next).  Boole's
//    rule errs by 8/945 h^7 phi^(6), below 1e-5 of an interval's mass out to
//    6.4 standard deviations (its sixth derivative is He6(a) phi); Simpson's
//    by h^5/90 phi^(4), below 1e-5 of it out to 4 and below 4e-5 out to 6
//    standard deviations at dz <= 1/10, where the masses are below 1e-9 of a
//    sample; the products' roundings grow with the square of the edges
//    walked.  An FP32 emulation of thirteen-edge runs starting out to 6.2
//    standard deviations finds at most 2.0e-5 relative error in an
//    interval's mass with Boole's rule (dz in [0.02, 0.25]), and 1.2e-5 with
//    Simpson's (dz in [0.02, 0.125]) for runs starting within 4, against the
//    1e-4 a bin may err.
// Q[e] (u64) accumulates the quantised weight at or below edge e of the laws
// that cover e; cnt[c] (u32) counts the samples whose weight is all at or
// below edge c - 1 (a point in bin c - 1, or a law ending at edge c - 1), so
// that edge e carries Q[e] + 2^32 sum_(c <= e) cnt[c] in total.
//
// Per-wavefront LDS rows of wave_deposit: the 64 laws (kind | ka << 3, t0,
// sf, inv_s), their run shape (edges, edges below the centre), the piece
// offsets, and the start marks of a block of 64 pieces (-1 between uses; set
// to -1 once before the first use).
struct WaveLaws {
    int4 *rec;
    int2 *ext;
    int *off;
    int *mark;
};

// Edges a run.  Consecutive lanes of one law walk runs whose edges lie kRunLen
// words of 8 bytes apart: with eight, every second lane's atomic falls on the
// same 4-byte LDS bank (16 banks on); with an odd length they spread over the
// banks (the deposit's bank-conflict cycles drop by three quarters).  Thirteen
// rather than nine spreads a run's set-up over more edges (4% less time); the
// products' roundings grow with the square of the length.
constexpr int kRunLen = 13;

// Owner of piece p of a block (base .. base + 63): the last lane whose first
// piece is <= p.  Lanes with pieces mark their start if it falls in the block
// (starts are distinct); a prefix maximum carries each start to the pieces
// after it, the previous block's last owner (carry) to those before the first.
__device__ __forceinline__ int piece_owner(bool has, int off, int base, int carry,
                                           const WaveLaws &WL) {
    const int lane = threadIdx.x & 63;
    if (has && off >= base && off < base + 64) WL.mark[off - base] = lane;
    wave_sync_lds();
    const int m = WL.mark[lane];
    WL.mark[lane] = -1;
    return max(wave_incl_max(m), carry);
}

// Exclusive scan of n over the wavefront; *total receives the sum.
__device__ __forceinline__ int wave_excl_scan(int n, int *total) {
    const int lane = threadIdx.x & 63;
    int incl = n;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    *total = __builtin_amdgcn_readlane(incl, 63);
    return incl - n;
}

// Quantised weight of a CDF value at edge e (F: the tail mass on the side of
// the edge away from the law's centre), added to Q[e].
__device__ __forceinline__ void add_edge(unsigned long long *Q, int e, float F, bool upper) {
    F = fminf(fmaxf(F, 0.0f), 1.0f);
    // below 1, 2^32 F rounds to at most 2^32 - 256: 32 bits
    const unsigned long long qf =
        F >= 1.0f ? kOne : (unsigned long long)(uint32_t)rintf(F * 4294967296.0f);
    const unsigned long long q = upper ? kOne - qf : qf;
    if (q) atomicAdd(&Q[e], q);
}

// The same for an edge of a run, from 2^32 F: the tail mass F lies between 0 and
// about one half, so 2^32 F fits 32 bits, and the weight on the upper side,
// 2^32 - 2^32 F, has its high word set only when 2^32 F rounds to zero.  SPLIT:
// the upper side's tails go to an array of their own (Qe points into it) as they
// are, the 2^32 of each upper edge counted once a law at its first upper edge.
template <bool SPLIT>
__device__ __forceinline__ void add_run_edge(unsigned long long *Qe, float F32, bool upper) {
    const uint32_t qf = (uint32_t)rintf(F32);
    if constexpr (SPLIT) {
        atomicAdd(Qe, (unsigned long long)qf);
    } else {
        const uint32_t lo = upper ? 0u - qf : qf;
        const uint32_t hi = upper && qf == 0u ? 1u : 0u;
        atomicAdd(Qe, ((unsigned long long)hi << 32) | lo);
    }
}

// The edges of one run from the tail inwards (see wave_deposit): a0, ph0 and
// T0 are the distance from the centre, the density and the tail mass at the
// run's first edge; each step adds the density's integral over one edge
// interval, by Simpson's rule on two subintervals (SIMP) or Boole's on four,
// the density following the lattice by phi(a - h) = phi(a) e^(a h - h^2/2): the
// ratio itself shrinks by e^(-h^2) from one subinterval to the next.  The density
// and the tail are carried in units of 2^-32 (exact scalings of the same
// values), WIDE is the wide box (x) Gaussian with its series term, and `step` is
// the constant 1 with SPLIT (the upper side's array runs backwards): an edge
// takes 18 vector instructions with the series and 12 without, where it took 22
// (focused laws, 2^22 samples: 776 -> 706 us of deposit).
template <bool SIMP, bool SPLIT, bool WIDE>
__device__ __forceinline__ void walk_run(unsigned long long *qe, int step, int len, float sf,
                                         float da, float a0, float ph0, float T0, bool upper) {
    constexpr int kSub = SIMP ? 2 : 4;
    const float hs = da * (1.0f / kSub);
    const float q = __expf(-hs * hs), qn = __expf(-(float)kSub * hs * hs);
    const float cb = hs * (SIMP ? 1.0f / 3.0f : 2.0f / 45.0f);
    float a = a0, ph = ph0 * 0x1p32f, T = T0 * 0x1p32f;
    float rho = __expf(fmaf(a, hs, -0.5f * hs * hs));  // phi(a - hs) / phi(a)
    for (int k = 0; k < kRunLen; ++k) {
        if (k < len) {
            if (k > 0) {
                // from the previous edge (a) one edge towards the centre
                float r = rho;
                const float p1 = ph * r;
                r *= q;
                const float p2 = p1 * r;
                if constexpr (SIMP) {
                    T = fmaf(cb, fmaf(4.0f, p1, ph + p2), T);
                    ph = p2;
                } else {
                    r *= q;
                    const float p3 = p2 * r;
                    r *= q;
                    const float p4 = p3 * r;
                    T = fmaf(cb, fmaf(7.0f, ph + p4, fmaf(32.0f, p1 + p3, 12.0f * p2)), T);
                    ph = p4;
                }
                rho *= qn;
                a -= da;
            }
            float F = T;
            if constexpr (WIDE) {
                // the series' even terms beside the tail (sf holds beta^2), with
                // the sign of the tail on either side
                const float c =
                    sf * fmaf(sf * (1.0f / 1920.0f), fmaf(a, a, -3.0f), 1.0f / 24.0f);
                F = fmaf(a * ph, c, T);
            }
            add_run_edge<SPLIT>(SPLIT ? qe + k : qe + step * k, F, upper);
        }
    }
}

// SPLIT: the runs' upper-side tails go to QU (see add_run_edge; edge e at QU[-e],
// so that runs on either side walk upwards in memory), and a law
// walked in runs counts its sample at its first upper edge instead of past
// its last edge: edge e carries Q[e] - QU[-e] + 2^32 sum_(c <= e) cnt[c].
// dep: the launch's deposit kind (runs are of kind 4 in CIC, else of kind 2).
template <bool SPLIT>
__device__ __forceinline__ void wave_deposit(const LawLane &L, int dep, double w, float hf,
                                             unsigned long long *Q, unsigned long long *QU,
                                             unsigned int *cnt, const WaveLaws &WL) {
    const int lane = threadIdx.x & 63;
    const float wf = (float)w, inv_w = (float)(1.0 / w);
    // runs: the wide box (x) Gaussian, and Gaussians with dz <= 1/4
    const bool run = L.kind == 4 || (L.kind == 2 && wf * L.inv_s <= 0.25f);
    const int ne = L.kind > 0 ? L.kb - L.ka + 1 : 0;  // edges of the law
    // edges at or below the centre (t <= 0, as the position pass decides it)
    int nl = 0;
    if (run) {
        nl = min(max((int)floorf(-L.t0 * inv_w) + 1, 0), ne);
        if (nl > 0 && fmaf((float)(nl - 1), wf, L.t0) > 0.0f) --nl;
        if (nl < ne && fmaf((float)nl, wf, L.t0) <= 0.0f) ++nl;
    }
    if (L.kind == 0) atomicAdd(&cnt[L.ngp], 1u);
    if (L.kind > 0) atomicAdd(&cnt[SPLIT && run ? L.ka + nl : L.kb + 1], 1u);
    WL.rec[lane] = make_int4(L.kind | (L.ka << 3), __float_as_int(L.t0), __float_as_int(L.sf),
                             __float_as_int(L.inv_s));
    WL.ext[lane] = make_int2(ne, nl);

    // ---- position pass ----
    const int np = L.kind > 0 && !run ? ne + 1 : 0;
    int total;
    int off = wave_excl_scan(np, &total);
    WL.off[lane] = off;
    float cP = 0.0f, cPc = 0.0f;  // box ends of the previous block's last position
    int carry = 0;                // owner of the previous block's last position
    for (int base = 0; base < total; base += 64) {
        const int p = base + lane;
        const int own = piece_owner(np > 0, off, base, carry, WL);
        carry = __builtin_amdgcn_readlane(own, 63);
        const int4 r = WL.rec[own];
        const int kind = r.x & 7, ka = r.x >> 3;
        const int rel = p - WL.off[own] - 1;  // edge - ka
        const float t0 = __int_as_float(r.y), sf = __int_as_float(r.z);
        const float inv_s = __int_as_float(r.w);
        wave_sync_lds();  // the marks and rows are rewritten after this block
        const bool live = p < total && rel >= 0;
        const float t = fmaf((float)rel, wf, t0);
        const bool upper = t > 0.0f;
        // One Gaussian tail a position, without branches (one exponential
        // serves phi and the tail): at the edge for the Gaussian law, at the
        // upper box end x = t + b/2 for the narrow box (x) Gaussian, whose CDF
        // is a difference of Psi(x) = x Phi(x/s) + s phi(x/s) at the two box
        // ends; Psi(x) and Psi(x) - x = -x Phi(-x/s) + s phi(x/s) are formed
        // from the tail on the side of x (no cancellation) and consecutive
        // edges share one end.  All positions of a law are alike, so the box
        // ends passed between lanes are those of narrow laws only.
        const float x = kind == 3 ? t + hf : t;
        const float zz = x * inv_s;
        const float e2 = __expf(-0.5f * zz * zz);  // relative error below 2e-6 out to 6 sigma
        const float phz = 0.39894228040143267794f * e2;
        const float tail = 0.5f * erfc_pos(fabsf(zz) * 0.70710678118654752440f, e2);
        float P = 0.0f, Pc = 0.0f;
        if (__any(kind == 3)) {
            const float ph = sf * phz;
            const float lo = fmaf(x, tail, ph);   // Psi(x) when x <= 0
            const float hi = fmaf(-x, tail, ph);  // Psi(x) - x when x > 0
            P = zz <= 0.0f ? lo : hi + x;
            Pc = zz <= 0.0f ? lo - x : hi;
        }
        float lP = __shfl_up(P, 1, 64), lPc = __shfl_up(Pc, 1, 64);
        if (lane == 0) {
            lP = cP;
            lPc = cPc;
        }
        cP = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(P), 63));
        cPc = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(Pc), 63));
        if (live) {
            const float Fbox = upper ? 0.5f - t * inv_w : fmaf(t, inv_w, 0.5f);
            const float Fpsi = upper ? (lPc - Pc) * inv_w : (P - lP) * inv_w;
            const float F = kind == 3 ? Fpsi : (kind == 2 ? tail : Fbox);
            add_edge(Q, ka + rel, F, upper);
        }
    }
    wave_sync_lds();  // the offsets are rewritten below

    // ---- run pass ----
    const int rl = run ? (nl + kRunLen - 1) / kRunLen : 0;
    const int nr = run ? rl + (ne - nl + kRunLen - 1) / kRunLen : 0;
    off = wave_excl_scan(nr, &total);
    WL.off[lane] = off;
    carry = 0;
    for (int base = 0; base < total; base += 64) {
        const int p = base + lane;
        const int own = piece_owner(nr > 0, off, base, carry, WL);
        carry = __builtin_amdgcn_readlane(own, 63);
        const int4 r = WL.rec[own];
        const int2 x2 = WL.ext[own];
        const int j = p - WL.off[own];  // run of the law
        wave_sync_lds();
        const int ka = r.x >> 3;
        const float t0 = __int_as_float(r.y), sf = __int_as_float(r.z);
        const float inv_s = __int_as_float(r.w);
        const int n_e = x2.x, n_l = x2.y, r_l = (n_l + kRunLen - 1) / kRunLen;
        const bool upper = j >= r_l;
        // first edge (farthest from the centre) and length of the run
        const int rel0 = upper ? n_e - 1 - (j - r_l) * kRunLen : j * kRunLen;
        const int len = p < total ? (upper ? min(kRunLen, n_e - n_l - (j - r_l) * kRunLen)
                                           : min(kRunLen, n_l - j * kRunLen))
                                  : 0;
        const int step = upper ? -1 : 1;
        const float da = wf * inv_s;  // edge spacing in standard deviations
        // the tail at the run's first edge
        const float a0 = fabsf(fmaf((float)rel0, wf, t0) * inv_s);
        const float e2 = __expf(-0.5f * a0 * a0);
        const float ph0 = 0.39894228040143267794f * e2;
        const float T0 = 0.5f * erfc_pos(a0 * 0.70710678118654752440f, e2);
        unsigned long long *qe = SPLIT && upper ? QU - (ka + rel0) : Q + (ka + rel0);
        // Simpson's rule on half edges where the laws of all the wavefront's
        // runs have edges at most a tenth of a standard deviation apart (its
        // error then stays within 1e-5 of an interval's mass out to four
        // standard deviations), Boole's on quarter edges otherwise
        if (__all(!(p < total) || da <= 0.1f)) {
            if (dep == 1)
                walk_run<true, SPLIT, true>(qe, step, len, sf, da, a0, ph0, T0, upper);
            else
                walk_run<true, SPLIT, false>(qe, step, len, sf, da, a0, ph0, T0, upper);
        } else {
            if (dep == 1)
                walk_run<false, SPLIT, true>(qe, step, len, sf, da, a0, ph0, T0, upper);
            else
                walk_run<false, SPLIT, false>(qe, step, len, sf, da, a0, ph0, T0, upper);
        }
    }
    wave_sync_lds();  // the next call rewrites the rows
}

// ===========================================================================
// Wavefront reductions
// ===========================================================================
// The sum over the wavefront in lane 63, by DPP moves (no LDS traffic): within
// rows of 16 lanes, then the row ends to the rows after.
__device__ __forceinline__ double wave_sum_last(double v) {
    auto step = [](double x, auto ctrl, auto rows) {
        const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), decltype(ctrl)::value,
                                                   decltype(rows)::value, 0xf, false);
        const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), decltype(ctrl)::value,
                                                   decltype(rows)::value, 0xf, false);
        return x + __hiloint2double(hi, lo);
    };
    using std::integral_constant;
    v = step(v, integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});  // row_shr:1
    v = step(v, integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});  // row_shr:2
    v = step(v, integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});  // row_shr:4
    v = step(v, integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});  // row_shr:8
    v = step(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});  // row_bcast:15
    v = step(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});  // row_bcast:31
    return v;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// Grid of resident blocks for a persistent work-queue kernel (never more
// blocks than items; at most cap blocks a CU when cap > 0).
inline hipError_t resident_grid(const void *fn, int block, size_t lds, int64_t items, int *grid,
                                int cap = 0) {
    int device = 0, ncu = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&device);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, block, lds);
    if (e != hipSuccess) return e;
    if (cap > 0 && per_cu > cap) per_cu = cap;
    int64_t g = (int64_t)(per_cu < 1 ? 1 : per_cu) * ncu;
    if (g > items) g = items;
    *grid = (int)(g < 1 ? 1 : g);
    return hipSuccess;
}

// A kernel over the phase items of a launch.  wide: one block a CU (its LDS holds
// a window of the FP64 table), whose wavefronts take items of 64 samples; block
// is then the most threads.
struct PassKernel {
    const void *fn;
    int block;
    size_t lds;
    bool wide;
};

// cap: resident blocks of kPhaseBlock threads a CU at most (0: all that fit).
inline hipError_t run_pass(const PassKernel &k, const BatchParams &p, const float *env32,
                           const double *env64, int cap, hipStream_t s) {
    int grid = 0, block = k.block;
    hipError_t e;
    if (k.wide) {
        // as many wavefronts a CU as the launch has work for
        int device = 0, ncu = 0;
        e = hipGetDevice(&device);
        if (e == hipSuccess)
            e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(k.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.lds);
        if (e != hipSuccess) return e;
        constexpr int kPer = kPhaseBlock / 64;
        const int64_t waves = p.n_items * kPer;
        int64_t per = (waves + ncu - 1) / ncu;
        const int64_t most = cap > 0 && cap * kPer < block / 64 ? cap * kPer : block / 64;
        if (per > most) per = most;
        if (per < 1) per = 1;
        block = 64 * (int)per;
        const int64_t blocks = (waves + per - 1) / per;
        grid = (int)(blocks < ncu ? (blocks < 1 ? 1 : blocks) : ncu);
    } else {
        // (a block draws a tile a wavefront)
        constexpr int kPer = kPhaseBlock / 64;
        e = resident_grid(k.fn, block, k.lds, p.n_items + (p.n_draws + kPer - 1) / kPer, &grid,
                          cap);
        if (e != hipSuccess) return e;
    }
    BatchParams pc = p;
    const float *e32 = env32;
    const double *e64 = env64;
    void *args[] = {&pc, &e32, &e64};
    return hipLaunchKernel(k.fn, dim3((unsigned)grid), dim3(block), args, k.lds, s);
}

}  // namespace qs
