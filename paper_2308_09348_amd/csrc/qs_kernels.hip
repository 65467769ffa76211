// qs_kernels.hip -- gfx950 kernels of the beam-phase-space integrator.
//
// Hot path (Amaro & Vranic, arXiv 2308.09348).  The phase kernel gives one
// lane one beam sample at a time: it draws the sample (Philox4x32-10 +
// Box-Muller), places it on its ballistic path through the focused pulse
// (Sec. 2, eq. a0eff, Table 1 offsets) and integrates its mean energy and
// energy variance along the phase with RK4 under the radiation-reaction drift
// of eq. dpdtRR (classical limit: eq. PWCRR), with the state in registers and
// the radiation-function table in LDS.  It writes the final state (56 bytes a
// sample).  The deposit kernel turns final states into energy and angle laws
// (eq. dNda2dNdgf as a push-forward; Sec. 5.2 divergence) deposited into
// block-private LDS histograms in 32.32 fixed point, merged into global
// integer histograms (order-independent), plus FP64 moment partials that a
// finalize kernel reduces in a fixed order.  The split keeps the FP64
// deposit arithmetic from setting the register budget of the phase loop.
// Nothing here is a dense contraction, so no MFMA: the bound is the vector
// ALU of the phase loop.
#include "qs_device.h"

namespace qs {

// ===========================================================================
// Phase kernel: sample -> ballistic path -> RK4 phase loop -> final state
// ===========================================================================
// The envelope tables come as separate restrict-qualified arguments: the
// kernel never writes them, so the compiler reads them with scalar loads
// (every lane of a wavefront is at the same phase step).
// NODES: the lane runs node i = k n_gnode + m of the shot's plane-wave
// reconstruction grid (a0,eff = a0 k / (n_anode - 1), gamma0 of node m, no
// angles) instead of drawing sample i; the caller passes the node view of the
// shot table (its node count and node offset as samples and state offset).
// FP64 steps of the mixed-precision loop from step j on, for as long as some
// lane of the wavefront has chi above the threshold at the step start: the
// amplitude's spatial factor is carried from one step's end to the next
// step's start, as in the FP64 loop.  Returns the first step not taken.
template <bool MODES, class Tab>
__device__ __forceinline__ int fp64_segment(const BatchParams &P, const ShotParams &sp,
                                            const Path<double, MODES> &pd, bool local,
                                            double a0S0, const double *__restrict__ env64, int j,
                                            const Tab &tabd, double &mu, double &s2, float &cmx,
                                            double &chd) {
    const Phys<double> phd{P.K, P.CD, P.two_over_aS};
    const int N = P.n_steps;
    AmpFactors<double> A1(
        (local ? sp.a0 * pd.S(fma((double)j, P.h, -P.psi_max) * P.ell_per_psi) : a0S0) *
            env64[2 * j],
        phd);
    bool more = true;
    while (more) {
        const double psi = fma((double)j, P.h, -P.psi_max);
        double aSh = a0S0, aS4 = a0S0;
        if (local) {
            aSh = sp.a0 * pd.S(fma(0.5, P.h, psi) * P.ell_per_psi);
            aS4 = sp.a0 * pd.S((psi + P.h) * P.ell_per_psi);
        }
        double dm, ds;
        rk4_q64(mu, s2, A1, aSh * env64[2 * j + 1], aS4 * env64[2 * j + 2], P.h, phd, tabd, dm, ds,
                chd);
        mu += dm;
        s2 += ds;
        ++j;
        if (j >= N) break;
        const double chi = A1.cpm * mu;
        cmx = fmaxf(cmx, (float)chi);
        more = __any(chi > (double)P.chi_fp64);
    }
    return j;
}

// The FP32 path of a sample from its FP64 draw.
template <bool MODES>
__device__ __forceinline__ Path<float, MODES> path32(const ShotParams &sp,
                                                     const Path<double, MODES> &pd, double thx,
                                                     double thy) {
    Path<float, MODES> pf;
    pf.xc = (float)pd.xc;
    pf.yc = (float)pd.yc;
    pf.thx = (float)thx;
    pf.thy = (float)thy;
    pf.zstar = (float)pd.zstar;
    pf.inv_w0sq = sp.inv_w0sqf;
    pf.inv_zR = sp.inv_zRf;
    pf.mode = sp.mode;
    pf.mm = sp.mode_m;
    pf.mn = sp.mode_n;
    pf.inv_norm = sp.mode_inv_normf;
    return pf;
}

// The amplitudes' spatial parts at the middle and end of FP32 step j.  Local
// amplitude: one spatial factor per step, at psi_{j+2}; the stage-2/3 value at
// psi_j + h/2 is the quadratic through psi_j (aS_prev), psi_{j+1} (aS_next) and
// psi_{j+2} (error of order h^3 times the third derivative of S, far below
// FP32 rounding).
template <bool MODES>
__device__ __forceinline__ void mid_end32(const BatchParams &P, const ShotParams &sp,
                                          const Path<float, MODES> &pf, float a0f, float a0S0f,
                                          bool local, int j, float &aS_prev, float &aS_next,
                                          float &aSh, float &aS4) {
    aSh = aS4 = a0S0f;
    if (local && sp.mid_interp) {
        const float psi2 = fmaf((float)(j + 2), P.hf, P.psi0f);
        const float aS_far = a0f * pf.S(psi2 * P.ellf);
        aS4 = aS_next;
        aSh = fmaf(0.375f, aS_prev, fmaf(0.75f, aS4, -0.125f * aS_far));
        aS_next = aS_far;
    } else if (local) {  // coarse steps: both points exactly
        const float psi = fmaf((float)j, P.hf, P.psi0f);
        aSh = a0f * pf.S(fmaf(0.5f, P.hf, psi) * P.ellf);
        aS4 = a0f * pf.S((psi + P.hf) * P.ellf);
    }
    aS_prev = aS4;
}

// The final state of sample i.
__device__ __forceinline__ void store_state(const BatchParams &P, const ShotParams &sp, int64_t i,
                                            double mu_f, double s2_f, double S0, double g0,
                                            double thx, double thy, float cmx) {
    const int64_t k = sp.state_off + i;
    P.st.mu[k] = mu_f;
    P.st.s2[k] = s2_f;
    P.st.S0[k] = S0;
    P.st.g0[k] = g0;
    P.st.thx[k] = thx;
    P.st.thy[k] = thy;
    P.st.cmx[k] = cmx;
}

// N steps of the classical model, step(eh, e4) with the envelope at the step's
// middle and end.  A step is some thirty dependent operations, less than the
// latency of a scalar read: small launches (a wavefront alone on its SIMD)
// waited for the envelope at every step.  It is read four steps at a time,
// while the four steps before are taken: 10^4 samples x 512 steps with a fixed
// amplitude 64 -> 42 us (FP64 76 -> 44 us, with the spatial factor 170 -> 136 us).
template <class T, class Step>
__device__ __forceinline__ void classical_steps(const T *__restrict__ env, int N, Step step) {
    constexpr int K = 4;
    int j = 0;
    if (N >= K) {
        T e[2 * K];
#pragma unroll
        for (int q = 0; q < 2 * K; ++q) {
            e[q] = env[1 + q];
            asm volatile("" : "+s"(e[q]));  // (or the reads move back to their uses)
        }
        for (; j + K <= N; j += K) {
            const T *p = env + (j + 2 * K <= N ? 2 * (j + K) + 1 : 1);
            T n[2 * K];
#pragma unroll
            for (int q = 0; q < 2 * K; ++q) n[q] = p[q];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < K; ++q) step(j + q, e[2 * q], e[2 * q + 1]);
#pragma unroll
            for (int q = 0; q < 2 * K; ++q) e[q] = n[q];
        }
    }
    for (; j < N; ++j) step(j, env[2 * j + 1], env[2 * j + 2]);
}

template <int PREC, bool QUANTUM, bool LOCAL, bool NODES, bool MODES, class Tab>
__device__ __forceinline__ void phase_sample(const BatchParams &P, const ShotParams &sp, int64_t i,
                                             const float *__restrict__ env32,
                                             const double *__restrict__ env64,
                                             const float *tab32, const Tab &tabd, int &flags,
                                             int &nprom) {
    const Phys<float> phf{P.Kf, P.CDf, P.two_over_aSf};
    const Phys<double> phd{P.K, P.CD, P.two_over_aS};
    const int N = P.n_steps;
    const bool local = LOCAL && !sp.plane_wave;
    const float chi_top = (float)(1 << (kEMax + 1));  // end of the tabulated range

    // ---- sample and geometry (FP64, once per sample) ----
    double g0, thx = 0.0, thy = 0.0, S0;
    Path<double, MODES> pd{};
    if (NODES) {
        static_assert(!NODES || !LOCAL, "nodes carry a fixed amplitude");
        const int k = (int)(i / sp.n_gnode);
        const int m = (int)(i - (int64_t)k * sp.n_gnode);
        S0 = (double)k / (double)(sp.n_anode - 1);
        g0 = sp.gamma0;
        if (sp.n_gnode > 1) {
#pragma clang fp contract(off)
            g0 = sp.g_node_lo + (double)m * sp.g_node_step;  // rounded twice, as defined
        }
    } else {
        draw_sample<MODES>(sp, P.key0, P.key1, i, g0, thx, thy, pd, S0);
    }
    const double a0S0 = sp.a0 * S0;

    double mu_f, s2_f;
    float cmx = 0.0f;     // largest chi at a step start for this sample
    float chi_hi = 0.0f;  // largest chi of the table reads (range check)
    if (PREC == PREC_F64) {
        double mu = g0, s2 = 0.0, chd = 0.0;
        // the amplitude at a step's end is the next one's start
        double a1 = (local ? sp.a0 * pd.S(-P.psi_max * P.ell_per_psi) : a0S0) * env64[0];
        auto mid_end = [&](int j, double &aSh, double &aS4) {
            const double psi = fma((double)j, P.h, -P.psi_max);
            aSh = aS4 = a0S0;
            if (local) {
                aSh = sp.a0 * pd.S(fma(0.5, P.h, psi) * P.ell_per_psi);
                aS4 = sp.a0 * pd.S((psi + P.h) * P.ell_per_psi);
            }
        };
        if constexpr (QUANTUM) {
            AmpFactors<double> A1(a1, phd);
            for (int j = 0; j < N; ++j) {
                double aSh, aS4;
                mid_end(j, aSh, aS4);
                const double ah = aSh * env64[2 * j + 1];
                const double a4 = aS4 * env64[2 * j + 2];
                cmx = fmaxf(cmx, (float)(A1.cpm * mu));
                double dm, ds;
                rk4_q64(mu, s2, A1, ah, a4, P.h, phd, tabd, dm, ds, chd);
                mu += dm;
                s2 += ds;
            }
        } else {
            classical_steps(env64, N, [&](int j, double eh, double e4) {
                double aSh, aS4;
                mid_end(j, aSh, aS4);
                const double ah = aSh * eh, a4 = aS4 * e4;
                cmx = fmaxf(cmx, (float)(P.two_over_aS * mu * fabs(a1)));
                mu += rk4_classical(mu, a1, ah, a4, P.h, phd);
                a1 = a4;
            });
        }
        mu_f = mu;
        s2_f = s2;
        chi_hi = (float)chd;
    } else {
        const Path<float, MODES> pf = path32(sp, pd, thx, thy);
        const float a0f = sp.a0f;
        const float a0S0f = (float)a0S0;
        float mu = (float)g0, mu_lo = (float)(g0 - (double)mu), s2 = 0.0f, s2_lo = 0.0f;
        // the part of g0 that the FP32 pair cannot hold: restored at the end,
        // or taken into the state by the first FP64 step
        double g0_rest = (g0 - (double)mu) - (double)mu_lo;
        double chd = 0.0;
        const float h6 = P.hf * (1.0f / 6.0f);
        float aS_prev = local ? a0f * pf.S(P.psi0f * P.ellf) : a0S0f;
        RadCell32 carry;
        AmpQ amp1;  // amplitude factors of the next stage 1
        if (QUANTUM) {
            amp1 = AmpQ(aS_prev * env32[0], phf);
            rad_lookup32(tab32, amp1.cpm * mu, carry);
        }
        float aS_next = local ? a0f * pf.S((P.psi0f + P.hf) * P.ellf) : a0S0f;
        auto mid_end = [&](int j, float &aSh, float &aS4) {
            mid_end32(P, sp, pf, a0f, a0S0f, local, j, aS_prev, aS_next, aSh, aS4);
        };
        if constexpr (!QUANTUM) {
            float a1 = aS_prev * env32[0];
            auto step = [&](int j, float eh, float e4) {
                float aSh, aS4;
                mid_end(j, aSh, aS4);
                const float ah = aSh * eh, a4 = aS4 * e4;
                cmx = fmaxf(cmx, phf.two_over_aS * mu * fabsf(a1));
                comp_add(mu, mu_lo, rk4_classical(mu, a1, ah, a4, P.hf, phf));
                a1 = a4;
            };
            if constexpr (!LOCAL) {
                classical_steps(env32, N, step);
            } else {  // (the spatial factor hides the reads: 2^20 samples 558 us, 666 so)
#pragma clang loop unroll_count(2)
                for (int j = 0; j < N; ++j) step(j, env32[2 * j + 1], env32[2 * j + 2]);
            }
        }
        auto step32 = [&](int j, auto round) {
            float aSh, aS4;
            mid_end(j, aSh, aS4);
            const float ah = aSh * env32[2 * j + 1];
            const float a4 = aS4 * env32[2 * j + 2];
            if (PREC != PREC_F32MIX) cmx = fmaxf(cmx, amp1.cpm * mu);
            float dm, ds;
            rk4_q32<decltype(round)::value>(mu, s2, amp1, AmpQ(ah, phf), AmpQ(a4, phf), P.hf, tab32,
                                            carry, dm, ds, chi_hi);
            comp_add(mu, mu_lo, h6, dm);
            comp_add(s2, s2_lo, h6, ds);
        };
        // two steps an iteration: the loop's bookkeeping and the moves of the
        // carried values at its back edge are halved (FP32 quantum pass 3%
        // faster; four steps no faster, with spills)
        if constexpr (QUANTUM && PREC == PREC_F32) {
            if constexpr (LOCAL) {
                q32_steps(0, N, step32);
            } else {
#pragma clang loop unroll_count(2)
                for (int j = 0; j < N; ++j) step32(j, std::false_type{});
            }
        }
        if constexpr (QUANTUM && PREC == PREC_F32MIX) {
            for (int j = 0; j < N;) {
                const float chi1 = amp1.cpm * mu;
                cmx = fmaxf(cmx, chi1);
                if (__any(chi1 > P.chi_fp64)) {
                    // FP64 steps while any lane of the wavefront has chi above
                    // the threshold at the step start (uniform loop); the FP32
                    // state, amplitudes and cell are rebuilt at the exit step
                    double mud = ((double)mu + (double)mu_lo) + g0_rest;
                    double s2d = (double)s2 + (double)s2_lo;
                    g0_rest = 0.0;
                    const int j0 = j;
                    j = fp64_segment(P, sp, pd, local, a0S0, env64, j, tabd, mud, s2d,
                                              cmx, chd);
                    nprom += j - j0;  // wave-uniform
                    mu = (float)mud;
                    mu_lo = (float)(mud - (double)mu);
                    s2 = (float)s2d;
                    s2_lo = (float)(s2d - (double)s2);
                    if (local) {
                        aS_prev = a0f * pf.S(fmaf((float)j, P.hf, P.psi0f) * P.ellf);
                        aS_next = a0f * pf.S(fmaf((float)(j + 1), P.hf, P.psi0f) * P.ellf);
                    }
                    if (j < N) {
                        amp1 = AmpQ(aS_prev * env32[2 * j], phf);
                        rad_lookup32(tab32, amp1.cpm * mu, carry);
                    }
                    continue;
                }
                step32(j, std::false_type{});
                ++j;
            }
        }
        mu_f = ((double)mu + (double)mu_lo) + g0_rest;
        s2_f = (double)s2 + (double)s2_lo;
        chi_hi = fmaxf(chi_hi, (float)chd);
    }
    {
        // chi at the end of the last step (the pulse tail)
        const double aN = (local ? sp.a0 * pd.S(P.psi_max * P.ell_per_psi) : a0S0) * env64[2 * N];
        cmx = fmaxf(cmx, (float)(P.two_over_aS * mu_f * fabs(aN)));
    }
    if (QUANTUM && !(chi_hi < chi_top)) flags |= kFlagRange;
    if (!(mu_f > 0.0) || !isfinite(mu_f) || !isfinite(s2_f)) flags |= kFlagNonFinite;
    store_state(P, sp, i, mu_f, s2_f, S0, g0, thx, thy, cmx);
}

// FP32 passes and classical FP64 passes: blocks take items of kPhaseBlock
// samples.
// DRAW: node passes of the reconstruction of few blocks.  Their wavefronts have
// long chains and leave the device idle (61 x 64 nodes: 61 wavefronts, 376 us of
// 1024 steps), so the launch's other blocks draw the samples meanwhile (2^22
// samples: about 100 us as a pass of their own), one block a CU, since beside
// other wavefronts a node's steps take longer (the launch 389 us, 426 us without).
template <int PREC, bool QUANTUM, bool LOCAL, bool NODES = false, bool MODES = false,
          bool DRAW = false>
__global__ __launch_bounds__(kPhaseBlock)
__attribute__((amdgpu_waves_per_eu((PREC == PREC_F32 && QUANTUM && !DRAW) ? 4 : 1))) void phase_kernel(BatchParams P,
                                                            const float *__restrict__ env32,
                                                            const double *__restrict__ env64) {
    static_assert(PREC == PREC_F32 || !QUANTUM, "phase64_kernel");
    __shared__ __align__(16) float tab32[QUANTUM ? kCells32 * kCellVals : 4];
    __shared__ int64_t slot;
    // quantum passes: the lanes take the item's samples in order of their chi
    // scale (chi_order32), so that neighbouring lanes read nearby table cells
    constexpr bool kOrder = QUANTUM && !NODES;
    __shared__ float okey[kOrder ? kPhaseBlock : 1];
    __shared__ unsigned short oidx[kOrder ? kPhaseBlock : 1];
    if (QUANTUM) {
        const float4 *src = reinterpret_cast<const float4 *>(P.rad32);
        float4 *dst = reinterpret_cast<float4 *>(tab32);
        for (int k = threadIdx.x; k < kCells32 * kCellVals / 4; k += blockDim.x) dst[k] = src[k];
        __syncthreads();
    }
    const NoTable tabd;
    int s_prev = 0;  // the shot of the block's previous item
    for (;;) {
        const int64_t item = next_item(&P.queue[0], &slot);
        if (item >= P.n_items) break;
        const int s = __builtin_amdgcn_readfirstlane(
            find_shot_from(P.shots, P.n_shots, item, false, s_prev));
        s_prev = s;
        const ShotParams &sp = P.shots[s];
        const int64_t base = (item - sp.item0) * kPhaseBlock;
        int off = threadIdx.x;
        if constexpr (kOrder) {
            chi_order32<kPhaseBlock, kPhaseBlock>(sp, P.key0, P.key1, base, sp.n_samples, okey,
                                                  oidx);
            off = oidx[threadIdx.x];
        }
        const int64_t i = base + off;
        if (i < sp.n_samples) {
            int flags = 0, nprom = 0;
            phase_sample<PREC, QUANTUM, LOCAL, NODES, MODES>(P, sp, i, env32, env64, tab32, tabd,
                                                             flags, nprom);
            if (flags) atomicOr(&P.flags[s], flags);
        }
    }
    if constexpr (DRAW) draw_samples(P);
}

// The draws by themselves, before the other node passes.
__global__ __launch_bounds__(kPhaseBlock) void draw_kernel(BatchParams P) { draw_samples(P); }

// Small FP32 quantum launches with the local amplitude: at most an item a CU, so
// that a wavefront of the kernel above would be alone on its SIMD.  Such a
// wavefront issues an instruction in four to five clocks, where two issue one in
// little more than two, and its steps are one dependent chain.  Here every
// wavefront of samples has a helper on its SIMD, which forms the amplitude factors
// (the spatial factor, the envelope: 45 of a step's 180 instructions, none of
// which needs the state) kPairSteps ahead and passes them through LDS (two
// buffers, a barrier of the block a buffer).  5003 samples x 512 steps 237 ->
// 197 us, 50,001 248 -> 214 us; from 257 items on (a second round; 131,072 samples
// 416 us, 297 us above) the kernel above is the better one.
// The results are the same bits (rk4_q32, mid_end32 and q32_steps are shared).
constexpr int kPairSteps = 8;
constexpr int kPairBlock = 2 * kPhaseBlock;
static_assert(kPairSteps % 2 == 0, "a buffer begins with an even step");

struct PairLds {
    float4 m[2][kPhaseBlock / 64][kPairSteps][64];  // at the middle nu, cd, cpm; at the end nu
    float2 e[2][kPhaseBlock / 64][kPairSteps][64];  // at the end cd, cpm
};

__global__ __launch_bounds__(kPairBlock) void phase_pair_kernel(BatchParams P,
                                                                const float *__restrict__ env32,
                                                                const double *__restrict__ env64) {
    __shared__ __align__(16) float tab32[kCells32 * kCellVals];
    __shared__ int64_t slot;
    extern __shared__ __align__(16) unsigned char pair_lds[];
    PairLds &B = *reinterpret_cast<PairLds *>(pair_lds);
    {
        const float4 *src = reinterpret_cast<const float4 *>(P.rad32);
        float4 *dst = reinterpret_cast<float4 *>(tab32);
        for (int k = threadIdx.x; k < kCells32 * kCellVals / 4; k += blockDim.x) dst[k] = src[k];
        __syncthreads();
    }
    constexpr int kPairs = kPhaseBlock / 64;
    const Phys<float> phf{P.Kf, P.CDf, P.two_over_aSf};
    const int N = P.n_steps, nbuf = (N + kPairSteps - 1) / kPairSteps;
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), pair = wid % kPairs;
    int s_prev = 0;  // the shot of the block's previous item
    for (;;) {
        const int64_t item = next_item(&P.queue[0], &slot);
        if (item >= P.n_items) break;
        const int s = __builtin_amdgcn_readfirstlane(
            find_shot_from(P.shots, P.n_shots, item, false, s_prev));
        s_prev = s;
        const ShotParams &sp = P.shots[s];
        const bool local = !sp.plane_wave;
        // (lanes past the samples take the last one: every wavefront meets the
        // same barriers)
        const int64_t k = (item - sp.item0) * kPhaseBlock + 64 * pair + lane;
        const bool live = k < sp.n_samples;
        const int64_t i = live ? k : sp.n_samples - 1;
        double g0, thx, thy, S0;
        Path<double, false> pd{};
        draw_sample<false>(sp, P.key0, P.key1, i, g0, thx, thy, pd, S0);
        const Path<float, false> pf = path32(sp, pd, thx, thy);
        const float a0f = sp.a0f;
        const double a0S0 = sp.a0 * S0;
        const float a0S0f = (float)a0S0;
        float aS_prev = local ? a0f * pf.S(P.psi0f * P.ellf) : a0S0f;
        if (wid >= kPairs) {  // the helpers
            float aS_next = local ? a0f * pf.S((P.psi0f + P.hf) * P.ellf) : a0S0f;
            auto fill = [&](int c) {
                const int j0 = c * kPairSteps, j1 = min(N, j0 + kPairSteps);
#pragma unroll 2
                for (int j = j0; j < j1; ++j) {
                    float aSh, aS4;
                    mid_end32(P, sp, pf, a0f, a0S0f, local, j, aS_prev, aS_next, aSh, aS4);
                    const AmpQ Ah(aSh * env32[2 * j + 1], phf), A4(aS4 * env32[2 * j + 2], phf);
                    B.m[c & 1][pair][j - j0][lane] = make_float4(Ah.nu, Ah.cd, Ah.cpm, A4.nu);
                    B.e[c & 1][pair][j - j0][lane] = make_float2(A4.cd, A4.cpm);
                }
            };
            fill(0);
            __syncthreads();
            for (int c = 0; c < nbuf; ++c) {
                if (c + 1 < nbuf) fill(c + 1);
                __syncthreads();
            }
        } else {
            float mu = (float)g0, mu_lo = (float)(g0 - (double)mu), s2 = 0.0f, s2_lo = 0.0f;
            const double g0_rest = (g0 - (double)mu) - (double)mu_lo;
            const float h6 = P.hf * (1.0f / 6.0f);
            float cmx = 0.0f, chi_hi = 0.0f;
            AmpQ amp1(aS_prev * env32[0], phf);
            RadCell32 carry;
            rad_lookup32(tab32, amp1.cpm * mu, carry);
            __syncthreads();
            for (int c = 0; c < nbuf; ++c) {
                const int j0 = c * kPairSteps;
                q32_steps(j0, min(N, j0 + kPairSteps), [&](int j, auto round) {
                    const float4 m = B.m[c & 1][pair][j - j0][lane];
                    const float2 e = B.e[c & 1][pair][j - j0][lane];
                    AmpQ Ah, A4;
                    Ah.nu = m.x;
                    Ah.nu2 = 2.0f * m.x;
                    Ah.cd = m.y;
                    Ah.cpm = m.z;
                    A4.nu = m.w;
                    A4.nu2 = 2.0f * m.w;
                    A4.cd = e.x;
                    A4.cpm = e.y;
                    cmx = fmaxf(cmx, amp1.cpm * mu);
                    float dm, ds;
                    rk4_q32<decltype(round)::value>(mu, s2, amp1, Ah, A4, P.hf, tab32, carry, dm,
                                                    ds, chi_hi);
                    comp_add(mu, mu_lo, h6, dm);
                    comp_add(s2, s2_lo, h6, ds);
                });
                __syncthreads();
            }
            const double mu_f = ((double)mu + (double)mu_lo) + g0_rest;
            const double s2_f = (double)s2 + (double)s2_lo;
            // chi at the end of the last step (the pulse tail)
            const double aN =
                (local ? sp.a0 * pd.S(P.psi_max * P.ell_per_psi) : a0S0) * env64[2 * N];
            cmx = fmaxf(cmx, (float)(P.two_over_aS * mu_f * fabs(aN)));
            if (live) {
                int flags = 0;
                if (!(chi_hi < (float)(1 << (kEMax + 1)))) flags |= kFlagRange;
                if (!(mu_f > 0.0) || !isfinite(mu_f) || !isfinite(s2_f)) flags |= kFlagNonFinite;
                store_state(P, sp, i, mu_f, s2_f, S0, g0, thx, thy, cmx);
                if (flags) atomicOr(&P.flags[s], flags);
            }
        }
    }
}

// Quantum passes with FP64 steps (all of them, or where chi is high).  One
// block a CU holds the FP64 table's cells that the launch reaches in LDS (and
// the FP32 table); its wavefronts take items of 64 samples each on their own,
// in passes with FP32 steps in order of the group's chi scale (order_kernel).
// Bound by FP64 issue and, in FP64 passes whose lanes are not ordered, LDS bank
// conflicts (VALU busy 0.79 of the time at 1.95 GHz, 7 conflict cycles an LDS
// instruction, by counters; see `ordered` in the host code): with the table read
// a wavefront at a time from L2 through LDS staging rows, two wavefronts a SIMD,
// 2^20 FP64 samples x 512 steps took 8.8 ms, now 4.9 ms; 5000 samples 0.86 and
// 0.49 ms; eight quantum shots of 2^18 x 1024 with FP64 steps 17.8 and 11.4 ms.
// Four wavefronts a SIMD in 128 registers in FP64 passes; three in 168 with FP32
// steps beside (at four the FP32 steps spill: 23.4 ms; at two 12.7 ms).
template <int PREC>
constexpr int phase64_block() {
    return PREC == PREC_F32MIX ? 768 : 1024;
}

template <int PREC, bool LOCAL, bool NODES, bool MODES>
__global__ __launch_bounds__(phase64_block<PREC>()) void phase64_kernel(
    BatchParams P, const float *__restrict__ env32, const double *__restrict__ env64) {
    constexpr bool kMix = PREC == PREC_F32MIX;
    constexpr int kWin = kMix ? kWinMix : kWin64;
    extern __shared__ double2 win[];  // [8][kWin]
    __shared__ __align__(16) float tab32[kMix ? kCells32 * kCellVals : 4];
    const TabWindow<kWin, 4> tabd(win, P.rad64);
    if (kMix) {
        const float4 *src = reinterpret_cast<const float4 *>(P.rad32);
        float4 *dst = reinterpret_cast<float4 *>(tab32);
        for (int k = threadIdx.x; k < kCells32 * kCellVals / 4; k += blockDim.x) dst[k] = src[k];
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    constexpr int kPer = kPhaseBlock / 64;
    int s_prev = 0;  // the shot of the wavefront's previous item
    for (;;) {
        unsigned int taken = 0;
        if (lane == 0) taken = atomicAdd(&P.queue[0], 1u);
        const int64_t item = __builtin_amdgcn_readfirstlane(taken);
        if (item >= kPer * P.n_items) break;
        const int s = __builtin_amdgcn_readfirstlane(
            find_shot_from(P.shots, P.n_shots, item / kPer, false, s_prev));
        s_prev = s;
        const ShotParams &sp = P.shots[s];
        const int64_t k = item - kPer * sp.item0;
        int64_t i = 64 * k + lane;
        bool live = i < sp.n_samples;
        if (!NODES && (kMix || P.order != nullptr)) {
            if (64 * k >= sp.n_samples) continue;
            const int64_t first = ordered_round<64>(sp.n_samples, k);
            const int64_t base = first & ~(kChiGroup - 1ll);
            const int cnt = (int)min((int64_t)kChiGroup, sp.n_samples - base);
            const int rank = (int)(first - base) + lane;
            live = rank < cnt;
            i = ordered_sample(P, sp, base, cnt, rank);
        }
        if (live) {
            int flags = 0, nprom = 0;
            phase_sample<PREC, true, LOCAL, NODES, MODES>(P, sp, i, env32, env64, tab32, tabd,
                                                          flags, nprom);
            if (flags) atomicOr(&P.flags[s], flags);
            // FP64 wave-steps of the wavefronts of the shot
            if (kMix && P.fp64_steps != nullptr && nprom > 0 && lane == 0)
                atomicAdd(&P.fp64_steps[s], (unsigned long long)nprom);
        }
    }
}

// ===========================================================================
// Deposit kernel: final states -> observables -> histograms and moments
// ===========================================================================
// Exclusive prefix sum over the block of one value a thread (256 threads);
// *total receives the sum.
__device__ __forceinline__ unsigned int block_scan(unsigned int v, unsigned int *wsum,
                                                   unsigned int *total) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    unsigned int x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[wid] = x;
    __syncthreads();
    unsigned int before = 0, all = 0;
    for (int w = 0; w < kDepBlock / 64; ++w) {
        if (w < wid) before += wsum[w];
        all += wsum[w];
    }
    __syncthreads();  // wsum is reused by the next scan
    *total = all;
    return before + x - v;
}

// Bin masses of one histogram of n bins from the edge accumulators of a tile
// (see wave_deposit): edge e carries T(e) = Q[e] (- QU[-e]) + 2^32 C(e), C(e) =
// sum_(c <= e) cnt[c]; bin b gets T(b+1) - T(b), the underflow T(0), the
// overflow 2^32 S - T(n) with S = sum of all cnt (every sample counts once).
// Added to the global words G[0 .. n+1] (bins, underflow, overflow).
template <bool SPLIT>
__device__ void flush_edges(const unsigned long long *Q, const unsigned long long *QU,
                            const unsigned int *cnt, int n, unsigned long long *G,
                            unsigned int *wsum) {
    auto q = [&](int e) { return SPLIT ? Q[e] - QU[-e] : Q[e]; };
    const int m = (n + 2 + kDepBlock - 1) / kDepBlock;  // cnt entries a thread
    const int c0 = threadIdx.x * m, c1 = min(c0 + m, n + 2);
    unsigned int local = 0;
    for (int c = c0; c < c1; ++c) local += cnt[c];
    unsigned int S;
    unsigned int C = block_scan(local, wsum, &S);
    const unsigned long long one = kOne;
    unsigned long long prev = c0 >= 1 && c0 <= n + 1 ? q(c0 - 1) + one * C : 0ull;
    for (int e = c0; e < c1 && e <= n; ++e) {
        C += cnt[e];
        const unsigned long long T = q(e) + one * C;
        const long long mass = (long long)(e == 0 ? T : T - prev);
        const int bin = e == 0 ? n : e - 1;
        if (mass > 0) atomicAdd(&G[bin], (unsigned long long)mass);
        if (e == n) {
            const long long over = (long long)(one * S - T);
            if (over > 0) atomicAdd(&G[n + 1], (unsigned long long)over);
        }
        prev = T;
    }
}

// FP64 shadow, histogram level: the bin masses of a sample's law (its own law
// convolved with the deposit kernel, as deposited) from its FP32 state minus
// those from its FP64 state, added to D[n + 2] (bins, underflow n, overflow
// n + 1) in signed fixed point of 2^-40 (the differences are small: units of
// 2^-32 would round most of them away; a word holds up to 2^23 whole masses).  Both laws' CDFs are evaluated exactly
// in FP64, so the difference is that of the two trajectories alone.  Only the
// CDF difference at each edge matters: edge j adds it to the mass below
// (bin j - 1, or the underflow) and subtracts it from the mass above (bin j,
// or the overflow); edges beyond 9 standard deviations of both laws add
// nothing at FP64 precision.
__device__ double law_cdf64(double t, double s, int dep, double ksig, double w) {
    const double r = 0.70710678118654752440;
    if (dep == 2) {  // GAUSS: N(0, s^2 + (ksig bins)^2)
        const double se = sqrt(fma(s, s, (ksig * w) * (ksig * w)));
        return 0.5 * erfc(-t * r / se);
    }
    if (dep == 1) {  // CIC: box one bin wide (x) N(0, s^2)
        const double h = 0.5 * w;
        if (!(s > 0.0)) return fmin(fmax((t + h) / w, 0.0), 1.0);
        auto psi = [&](double x) {  // Int_-inf^x Phi(u / s) du
            return x * 0.5 * erfc(-x * r / s) + s * 0.39894228040143267794 * exp(-0.5 * (x / s) * (x / s));
        };
        return fmin(fmax((psi(t + h) - psi(t - h)) / w, 0.0), 1.0);
    }
    if (!(s > 0.0)) return t > 0.0 ? 1.0 : 0.0;  // POINT: a value on an edge goes up
    return 0.5 * erfc(-t * r / s);
}

__device__ __forceinline__ void shadow_law_diff(double v32, double s32, double v64, double s64, int dep,
                                double ksig, double lo, double w, int n,
                                unsigned long long *D) {
    double reach = 9.0 * fmax(s32, s64) + w;
    if (dep == 2) reach += 9.0 * ksig * w;
    const double a = fmin(v32, v64) - reach, b = fmax(v32, v64) + reach;
    const int ja = (int)fmin(fmax(ceil((a - lo) / w), 0.0), (double)n + 1.0);
    const int jb = (int)fmin(fmax(floor((b - lo) / w), -1.0), (double)n);
    for (int j = ja; j <= jb; ++j) {
        const double e = fma((double)j, w, lo);
        const double d = law_cdf64(e - v32, s32, dep, ksig, w) - law_cdf64(e - v64, s64, dep, ksig, w);
        const long long q = llrint(d * 1099511627776.0);
        if (q == 0) continue;
        atomicAdd(&D[j == 0 ? n : j - 1], (unsigned long long)q);
        atomicAdd(&D[j == n ? n + 1 : j], (unsigned long long)(-q));
    }
}

// One lane per shadowed sample, over the work items of the shadow view
// (P.shots; an item lies within one shot; the FP32 state of shadowed sample q
// is src_off + q draw_stride, its FP64 state state_off + q in P.sst): the law
// differences summed per item in LDS, then added to the shot's words.  A
// kernel of its own keeps the FP64 CDFs off the deposit's register budget.
__global__ __launch_bounds__(kPhaseBlock) void shadow_diff_kernel(BatchParams P, int64_t n_items) {
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned long long *D = reinterpret_cast<unsigned long long *>(smem);
    for (int64_t item = blockIdx.x; item < n_items; item += gridDim.x) {
        const int s = __builtin_amdgcn_readfirstlane(find_shot(P.shots, P.n_shots, item, false));
        const ShotParams &sv = P.shots[s];
        const int nd = sv.n_e + 2 + sv.n_th + 2;
        for (int k = threadIdx.x; k < nd; k += blockDim.x) D[k] = 0ull;
        __syncthreads();
        const int64_t q = (item - sv.item0) * kPhaseBlock + threadIdx.x;
        if (q < sv.n_samples) {
            const int64_t k32 = sv.src_off + q * sv.draw_stride, k64 = sv.state_off + q;
            const double mu_f = P.st.mu[k32], s2_f = P.st.s2[k32];
            const double m64 = P.sst.mu[k64];
            if (mu_f > 0.0 && isfinite(mu_f) && isfinite(s2_f) && m64 > 0.0) {
                const double thx_m = 1e3 * P.st.thx[k32];
                const double sigf = sqrt(fmax(s2_f, 0.0)), s64 = sqrt(fmax(P.sst.s2[k64], 0.0));
                // Sec. 5.2 broadening of either state, as deposited
                const double c = 1e3 * P.c_theta * 0.79788456080286535588 * sv.a0 * P.st.S0[k32];
                const double sth32 = c * sigf / (mu_f * mu_f), sth64 = c * s64 / (m64 * m64);
                shadow_law_diff(mu_f, sigf, m64, s64, P.deposit, P.ksig_bins, sv.e_lo, sv.e_w,
                                sv.n_e, D);
                shadow_law_diff(thx_m, sth32, thx_m, sth64, P.deposit, P.ksig_bins, sv.th_lo,
                                sv.th_w, sv.n_th, D + sv.n_e + 2);
            }
        }
        __syncthreads();
        unsigned long long *G = P.shdiff + sv.shd_off;
        for (int k = threadIdx.x; k < nd; k += blockDim.x)
            if (D[k]) atomicAdd(&G[k], D[k]);
        __syncthreads();  // the next item clears D
    }
}

// Held to 80 VGPRs (six waves per SIMD): the runs are bound by LDS atomics and
// FP32 issue in turn, and more waves fill both (focused laws, 2^22 samples, with
// four / five / six waves: 706 / 671 / 661 us; the spills at six are block
// constants, stored once and read back a round).  The moment sums of a round are
// formed before the laws are walked rather than carried through them.
// SPLIT: the runs' upper-side tails in arrays of their own (16 bytes an edge
// instead of 8; histograms of up to 64 KB of LDS words take it).
// Small launches are bound by the rounds of 256 samples that a block takes one
// after another (about 28 us each: the laws of 64 samples by one wavefront), so
// the work item shrinks with the launch (default_dep_tile): 5003 samples 440 ->
// 39 us, 2^18 445 -> 106 us, 2^20 447 -> 219 us (focused laws; items of 4096
// before).
// NODES: a sample's final state is the bilinear interpolant of its shot's nodes
// (four reads, L2-resident, beside some 6,000 vector instructions of a round: a
// pass of its own that wrote the states took 75 us more at 2^22 samples).
template <bool SPLIT, bool NODES>
__global__ __launch_bounds__(kDepBlock) __attribute__((amdgpu_waves_per_eu(NODES ? 5 : 6))) void deposit_kernel(
    BatchParams P) {
    constexpr int kGroups = kDepBlock / 64;        // wavefronts
    constexpr int kRounds = kMomTile / kDepBlock;  // rounds of a moment tile
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int64_t slot;
    __shared__ double red[kRounds][kGroups][P_N];
    __shared__ float redmax[kGroups];
    __shared__ double redsh[kGroups][2];
    __shared__ unsigned int wsum[kDepBlock / 64];
    __shared__ int4 wrec[kDepBlock];
    __shared__ int2 wext[kDepBlock];
    __shared__ int woff[kDepBlock], wmark[kDepBlock];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const WaveLaws WL{wrec + 64 * wid, wext + 64 * wid, woff + 64 * wid, wmark + 64 * wid};
    WL.mark[lane] = -1;
    int s_prev = 0;  // the shot of the block's previous item
    for (;;) {
        const int64_t item = next_item(&P.queue[1], &slot);
        if (item >= P.n_ditems) break;
        const int s = __builtin_amdgcn_readfirstlane(
            find_shot_from(P.shots, P.n_shots, item, true, s_prev));
        s_prev = s;
        const ShotParams &sp = P.shots[s];
        const ShotOut &so = P.outs[s];
        const int nh_e = sp.n_e + 2, nh_t = sp.n_th + 2;
        // LDS: edge weights Qe [n_e + 1], Qt [n_th + 1] (u64; SPLIT: and the
        // upper tails QeU [n_e + 1], QtU [n_th + 1], backwards); counters ce [n_e + 2],
        // ct [n_th + 2], ca [n_a] (u32)
        unsigned long long *Qe = reinterpret_cast<unsigned long long *>(smem);
        unsigned long long *Qt = Qe + sp.n_e + 1;
        unsigned long long *QeU = Qt + sp.n_th + 1;
        unsigned long long *QtU = QeU + (SPLIT ? sp.n_e + 1 : 0);
        unsigned int *ce =
            reinterpret_cast<unsigned int *>(SPLIT ? QtU + sp.n_th + 1 : QeU);
        unsigned int *ct = ce + nh_e;
        unsigned int *ca = ct + nh_t;
        const int nq = (SPLIT ? 2 : 1) * (sp.n_e + 1 + sp.n_th + 1), nc = nh_e + nh_t + sp.n_a;
        for (int k = threadIdx.x; k < nq; k += kDepBlock) Qe[k] = 0ull;
        for (int k = threadIdx.x; k < nc; k += kDepBlock) ce[k] = 0u;
        __syncthreads();

        int flags = 0;
        const int64_t i0 = (item - sp.ditem0) * P.dep_tile;
        const int64_t i1 = i0 + P.dep_tile < sp.n_samples ? i0 + P.dep_tile : sp.n_samples;
        const float hfe = (float)(0.5 * sp.e_w), hft = (float)(0.5 * sp.th_w);
        const double inv_we = 1.0 / sp.e_w, inv_wt = 1.0 / sp.th_w;
        for (int64_t t0 = i0; t0 < i1; t0 += P.mom_row) {
            const int64_t t1 = t0 + P.mom_row < i1 ? t0 + P.mom_row : i1;
            float chimax = 0.0f;
            double emu = 0.0, esig = 0.0;  // FP64 shadow: largest differences
            // every lane runs every round (the wavefront deposit needs them all)
            int round = 0;
            for (int64_t base = t0; base < t1; base += kDepBlock, ++round) {
                const int64_t i = base + threadIdx.x;
                bool law = false;  // the sample deposits N(v_e, s_e^2) and N(v_t, s_t^2)
                double v_e = 0.0, s_e = 0.0, v_t = 0.0, s_t = 0.0;
                double acc[P_N];  // the round's moment sums
#pragma unroll
                for (int m = 0; m < P_N; ++m) acc[m] = 0.0;
                if (i < i1) {
                    const int64_t k = sp.state_off + i;
                    const double S0 = P.st.S0[k], g0 = P.st.g0[k];
                    const double thx_m = 1e3 * P.st.thx[k], thy_m = 1e3 * P.st.thy[k];
                    double mu_f, s2_f;
                    float cmx;
                    if constexpr (NODES) {
                        const NodeCell c(sp, S0, g0);
                        double cm = 0.0;
                        mu_f = s2_f = 0.0;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const int64_t g = sp.node_off + c.n[j];
                            mu_f += c.w[j] * P.nst.mu[g];
                            s2_f += c.w[j] * P.nst.s2[g];
                            cm += c.w[j] * (double)P.nst.cmx[g];
                        }
                        cmx = (float)cm;
                    } else {
                        mu_f = P.st.mu[k];
                        s2_f = P.st.s2[k];
                        cmx = P.st.cmx[k];
                    }
                    if (!(mu_f > 0.0) || !isfinite(mu_f) || !isfinite(s2_f)) {
                        flags |= kFlagNonFinite;  // also raised by the phase kernel
                    } else {
                        chimax = fmaxf(chimax, cmx);
                        // Sec. 5.2: the direction is kept, the stochastic broadening
                        // c_theta sqrt(2/pi) a0,eff sigma_f / gamma_f^2 acts in x
                        const double sigf = sqrt(fmax(s2_f, 0.0));
                        const double a_eff = sp.a0 * S0;
                        // 1 / mu_f^2 and 1 / g0 by the hardware reciprocal
                        // and two Newton steps (FP64 rounding)
                        const double mu2 = mu_f * mu_f;
                        double imu2 = __builtin_amdgcn_rcp(mu2), ig0 = __builtin_amdgcn_rcp(g0);
                        imu2 = fma(fma(-mu2, imu2, 1.0), imu2, imu2);
                        imu2 = fma(fma(-mu2, imu2, 1.0), imu2, imu2);
                        ig0 = fma(fma(-g0, ig0, 1.0), ig0, ig0);
                        ig0 = fma(fma(-g0, ig0, 1.0), ig0, ig0);
                        const double sigth =
                            1e3 * P.c_theta * 0.79788456080286535588 * a_eff * sigf * imu2;
                        law = true;
                        v_e = mu_f;
                        s_e = sigf;
                        v_t = thx_m;
                        s_t = sigth;
                        {
                            int ka = (int)floor(S0 * (double)sp.n_a);
                            ka = min(max(ka, 0), sp.n_a - 1);
                            atomicAdd(&ca[ka], 1u);
                        }
                        const double de = mu_f - sp.gamma0;
                        acc[P_S1E] = de;
                        acc[P_S2E] = fma(de, de, fmax(s2_f, 0.0));
                        acc[P_S1X] = thx_m;
                        acc[P_S2X] = fma(thx_m, thx_m, sigth * sigth);
                        acc[P_S1Y] = thy_m;
                        acc[P_S2Y] = thy_m * thy_m;
                        acc[P_SAEFF] = a_eff;
                        acc[P_SRAD] = fma(-mu_f, ig0, 1.0);
                        acc[P_SSIGF] = sigf;
                        if (sp.shadow_stride > 0 && i % sp.shadow_stride == 0) {
                            // the same sample integrated in FP64
                            const int64_t q = sp.shadow_off + i / sp.shadow_stride;
                            const double m64 = P.sst.mu[q];
                            const double s64 = sqrt(fmax(P.sst.s2[q], 0.0));
                            if (m64 > 0.0) {
                                const double d = mu_f - m64;
                                acc[P_SHN] = 1.0;
                                acc[P_SHMU] = d / m64;
                                acc[P_SHG] = d;
                                emu = fmax(emu, fabs(d) / m64);
                                esig = fmax(esig, fabs(sigf - s64) / m64);
                            }
                        }

                        if (so.samples != nullptr && i % so.rec_stride == 0 &&
                            i / so.rec_stride < so.rec_n) {
                            double *r = so.samples + (i / so.rec_stride) * 11;
                            r[0] = mu_f;
                            r[1] = s2_f;
                            r[2] = thx_m;
                            r[3] = thy_m;
                            r[4] = sigth;
                            r[5] = a_eff;
                            r[6] = cmx;
                            r[7] = g0;
                            r[8] = 0.0;
                            r[9] = 0.0;
                            r[10] = 0.0;
                        }
                    }
                }
#pragma unroll
                for (int m = 0; m < P_N; ++m) {
                    if (m >= P_SHN && sp.shadow_stride == 0) break;
                    const double v = wave_sum_last(acc[m]);
                    if (lane == 63) red[round][wid][m] = v;
                }
                LawLane le{-1, 0, -1, 0, 0.0f, 0.0f, 0.0f}, lt = le;
                if (law) {
                    le = law_setup(v_e, s_e, P.deposit, P.ksig_bins, sp.e_lo, sp.e_w, inv_we,
                                   sp.n_e);
                    lt = law_setup(v_t, s_t, P.deposit, P.ksig_bins, sp.th_lo, sp.th_w, inv_wt,
                                   sp.n_th);
                }
                wave_deposit<SPLIT>(le, P.deposit, sp.e_w, hfe, Qe, QeU + sp.n_e, ce, WL);
                wave_deposit<SPLIT>(lt, P.deposit, sp.th_w, hft, Qt, QtU + sp.n_th, ct, WL);
            }

            // ---- one row of moment sums (fixed order) ----
            const float wm = wave_max(chimax);
            if (lane == 0) redmax[wid] = wm;
            if (sp.shadow_stride > 0) {
                const double we = wave_max(emu), ws = wave_max(esig);
                if (lane == 0) {
                    redsh[wid][0] = we;
                    redsh[wid][1] = ws;
                }
            }
            __syncthreads();
            double *part = P.partials + (size_t)(sp.mtile0 + t0 / P.mom_row);
            if (threadIdx.x < P_N) {
                double tile = 0.0;
                if (threadIdx.x >= P_SHN && sp.shadow_stride == 0) round = 0;
                for (int r = 0; r < round; ++r) {
                    double sum = red[r][0][threadIdx.x];
                    for (int g = 1; g < kGroups; ++g) sum += red[r][g][threadIdx.x];
                    tile = r == 0 ? sum : tile + sum;
                }
                part[(size_t)threadIdx.x * P.n_mtiles] = tile;
            }
            if (threadIdx.x == 0) {
                float m = 0.0f;
                double e0 = 0.0, e1 = 0.0;
                for (int g = 0; g < kGroups; ++g) {
                    m = fmaxf(m, redmax[g]);
                    if (sp.shadow_stride > 0) {
                        e0 = fmax(e0, redsh[g][0]);
                        e1 = fmax(e1, redsh[g][1]);
                    }
                }
                part[(size_t)kPMaxChi * P.n_mtiles] = m;
                part[(size_t)kPMaxEmu * P.n_mtiles] = e0;
                part[(size_t)kPMaxEsig * P.n_mtiles] = e1;
            }
            __syncthreads();  // red is rewritten by the next row
        }
        if (flags) atomicOr(&P.flags[s], flags);
        unsigned long long *G = P.hist + sp.hist_off;
        flush_edges<SPLIT>(Qe, QeU + sp.n_e, ce, sp.n_e, G, wsum);
        flush_edges<SPLIT>(Qt, QtU + sp.n_th, ct, sp.n_th, G + nh_e, wsum);
        for (int k = threadIdx.x; k < sp.n_a; k += kDepBlock)
            if (ca[k]) atomicAdd(&G[nh_e + nh_t + k], kOne * ca[k]);
        __syncthreads();  // the next item clears the LDS words
    }
}

// ===========================================================================
// Finalize: one block per shot, fixed-order reduction of its moment rows
// ===========================================================================
// Bound by latency (one block).  One wavefront a column of the moment rows
// (stored column after column): lane l adds the tiles l, l + 64, ..., then the
// wavefront's sum: 16.3 -> 4.8 us at 5003 samples, 52 -> 11 us at 2^22 (23 us with
// four rows in flight), against a block that took the columns in turn, each with
// a tree of eight barriers.
constexpr int kFinBlock = 64 * 16;
static_assert(kPartials <= kFinBlock / 64, "a wavefront a column");

__global__ __launch_bounds__(kFinBlock) void finalize_kernel(BatchParams P) {
    const int s = blockIdx.x;
    const ShotParams &sp = P.shots[s];
    const ShotOut &so = P.outs[s];
    const int64_t nrow = (sp.n_samples + P.mom_row - 1) / P.mom_row;
    const int per = kMomTile / P.mom_row;  // rows of a moment tile
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __shared__ double sums[kPartials];
    __shared__ double tree[256];
    if (wid < kPartials) {
        const double *col = P.partials + (size_t)wid * P.n_mtiles + sp.mtile0;
        const bool mx = wid >= P_N;
        double acc = 0.0;
        if (per == 1) {
            // (sixteen rows in flight a lane)
#pragma unroll 16
            for (int64_t b = lane; b < nrow; b += 64) acc = mx ? fmax(acc, col[b]) : acc + col[b];
        } else {
#pragma unroll 4
            for (int64_t b = (int64_t)lane * per; b < nrow; b += 64 * per) {
                double v = col[b];
                for (int r = 1; r < per && b + r < nrow; ++r)
                    v = mx ? fmax(v, col[b + r]) : v + col[b + r];
                acc = mx ? fmax(acc, v) : acc + v;
            }
        }
        acc = mx ? wave_max(acc) : wave_sum(acc);
        if (lane == 0) sums[wid] = acc;
    }
    const int nh_e = sp.n_e + 2, nh_t = sp.n_th + 2;
    const unsigned long long *H = P.hist + sp.hist_off;
    const double scale = 1.0 / 4294967296.0;
    for (int k = threadIdx.x; k < nh_e; k += kFinBlock) so.energy_hist[k] = (double)H[k] * scale;
    for (int k = threadIdx.x; k < nh_t; k += kFinBlock)
        so.angle_hist[k] = (double)H[nh_e + k] * scale;
    for (int k = threadIdx.x; k < sp.n_a; k += kFinBlock)
        so.a0eff_hist[k] = (double)H[nh_e + nh_t + k] * scale;
    __syncthreads();
    // FP64 shadow, histogram level: L1 and largest bin of the summed law
    // differences, energy then angle, per shadowed sample
    __shared__ double shd[4];
    if (sp.shadow_stride > 0 && sums[P_SHN] > 0.0) {
        const unsigned long long *D = P.shdiff + sp.shd_off;
        for (int h = 0; h < 2; ++h) {
            const int n0 = h == 0 ? 0 : nh_e, n1 = h == 0 ? nh_e : nh_e + nh_t;
            double l1 = 0.0, mx = 0.0;
            if (threadIdx.x < 256)
                for (int k = n0 + threadIdx.x; k < n1; k += 256) {
                    const double v = fabs((double)(long long)D[k]) * (1.0 / 1099511627776.0);
                    l1 += v;
                    mx = fmax(mx, v);
                }
            for (int part = 0; part < 2; ++part) {
                if (threadIdx.x < 256) tree[threadIdx.x] = part == 0 ? l1 : mx;
                __syncthreads();
                for (int w = 128; w > 0; w >>= 1) {
                    if (threadIdx.x < w) {
                        const double o = tree[threadIdx.x + w];
                        tree[threadIdx.x] = part == 0 ? tree[threadIdx.x] + o : fmax(tree[threadIdx.x], o);
                    }
                    __syncthreads();
                }
                if (threadIdx.x == 0) shd[2 * h + part] = tree[0] / sums[P_SHN];
                __syncthreads();
            }
        }
    }
    if (threadIdx.x == 0) {
        double *M = so.moments;
        for (int m = 0; m < kMoments; ++m) M[m] = 0.0;
        const double W = (double)sp.n_samples;
        M[0] = W;
        if (sp.n_samples > 0) {
            const double m1 = sums[P_S1E] / W;
            M[1] = sp.gamma0 + m1;
            M[2] = sqrt(fmax(sums[P_S2E] / W - m1 * m1, 0.0));
            M[3] = sums[P_S1X] / W;
            M[4] = sqrt(sums[P_S2X] / W);
            M[5] = sums[P_S1Y] / W;
            M[6] = sqrt(sums[P_S2Y] / W);
            M[7] = sums[P_SAEFF] / W;
            M[8] = sums[kPMaxChi];
            M[9] = sums[P_SRAD] / W;
            M[10] = sums[P_SSIGF] / W;
            const double ns = sums[P_SHN];
            if (ns > 0.0) {
                M[11] = ns;
                M[12] = sums[kPMaxEmu];
                M[13] = sums[P_SHMU] / ns;
                M[14] = sums[kPMaxEsig];
                M[15] = sums[P_SHG] / ns;
                for (int q = 0; q < 4; ++q) M[16 + q] = shd[q];
            }
        }
        // share of the wavefront phase steps taken in FP64
        if (P.fp64_steps == nullptr)
            M[20] = -1.0;
        else if (P.prec == PREC_F64)
            M[20] = 1.0;
        else
            M[20] = (double)P.fp64_steps[s] /
                    ((double)((sp.n_samples + 63) / 64) * (double)P.n_steps);
        const int fl = P.flags[s];
        *so.status = (fl & kFlagNonFinite) ? 4 : ((fl & kFlagRange) ? 6 : 0);
    }
}

// ===========================================================================
// Set-up kernel: envelope x carrier table, clear of the accumulators (n words),
// the shot table if it came along by value.  One launch in place of a copy and
// two kernels: a call of 10^4 plane-wave samples takes 8 us less.
// ===========================================================================
constexpr int kSetupBlock = 256;

__global__ __launch_bounds__(kSetupBlock) void setup_kernel(
    SetupTab tab, int tab_words, unsigned long long *shot_tab, unsigned long long *accum, size_t n,
    double psi_max, double h, int n_steps, int envelope, double omega_tau, float *env32,
    double *env64) {
    const size_t i = (size_t)blockIdx.x * kSetupBlock + threadIdx.x;
    if (i < (size_t)tab_words) shot_tab[i] = tab.w[i];
    for (size_t w = i; w < n; w += (size_t)gridDim.x * kSetupBlock) accum[w] = 0ull;
    if (i > 2 * (size_t)n_steps) return;
    const int k = (int)i;
    const double psi = fma((double)k, 0.5 * h, -psi_max);
    double f;
    if (envelope == 0) {
        const double u = psi / omega_tau;
        f = exp(-2.0 * 0.69314718055994530942 * u * u);
    } else {
        if (fabs(psi) > omega_tau) {
            f = 0.0;
        } else {
            const double s = sinpi((psi + omega_tau) / (2.0 * omega_tau));
            f = s * s;
        }
    }
    const double e = f * cos(psi);
    env64[k] = e;
    env32[k] = (float)e;
}

// Passes with FP64 steps.  A wavefront steps in FP64 when any of its lanes
// needs it, so its lanes should hold samples of similar chi: the samples of a
// group are taken in increasing order of S0 gamma0, the chi scale of a sample
// at its collision point (ties by index; the Gaussian focus's factor also
// orders samples of a higher mode: any order gives the same results up to the
// FP64-step choice).  One block a group: keys from the FP64 draw, then a
// bitonic sort in LDS of (key, offset) words, padded to a power of two.
// A kernel of its own, so that the rounds of a group can go to any blocks of
// the pass (a group a block left most CUs idle below 2^20 samples: 2^18 samples
// of a quantum shot, 2048 steps, 15.0 -> 6.4 ms), and the pass keeps no LDS for
// it.  28 us for 128 groups, 110 us for 1024.
constexpr int kOrderBlock = kChiGroup / 2;
// Most blocks of a launch, which take group after group (2^36 samples are 2^25
// groups or more; a grid holds less than 2^32 threads).
constexpr int kOrderGrid = 4096;

__global__ __launch_bounds__(kOrderBlock) void order_kernel(BatchParams P) {
    __shared__ unsigned long long w[kChiGroup];
    for (int64_t group = blockIdx.x; group < P.n_gitems; group += gridDim.x) {
        const int s = __builtin_amdgcn_readfirstlane(find_group_shot(P.shots, P.n_shots, group));
        const ShotParams &sp = P.shots[s];
        const int64_t base = (group - sp.gitem0) * kChiGroup;
        const int cnt = (int)min((int64_t)kChiGroup, sp.n_samples - base);
        int m = 64;  // words sorted
        while (m < cnt) m <<= 1;
        __syncthreads();  // the previous group's words have been read
        for (int q = threadIdx.x; q < m; q += kOrderBlock) {
            uint32_t key = 0xffffffffu;  // past the samples
            if (q < cnt) {
                double g0, thx, thy, S0;
                Path<double, false> pd{};
                draw_sample<false>(sp, P.key0, P.key1, base + q, g0, thx, thy, pd, S0);
                // the float's bits in increasing order (+0: one zero)
                const uint32_t b = __float_as_uint((float)(S0 * g0) + 0.0f);
                key = b & 0x80000000u ? ~b : b | 0x80000000u;
            }
            w[q] = ((unsigned long long)key << 32) | (unsigned int)q;
        }
        __syncthreads();
        for (int k = 2; k <= m; k <<= 1)
            for (int j = k >> 1; j > 0; j >>= 1) {
                // pairs at most 64 apart stay within the 128 words of a wavefront
                if (j >= 64)
                    __syncthreads();
                else
                    wave_sync_lds();
                if (threadIdx.x < m / 2) {
                    const int t = (int)threadIdx.x, a = ((t & -j) << 1) | (t & (j - 1)), b = a + j;
                    const unsigned long long x = w[a], y = w[b];
                    if ((x > y) == ((a & k) == 0)) {
                        w[a] = y;
                        w[b] = x;
                    }
                }
            }
        __syncthreads();
        for (int q = threadIdx.x; q < cnt; q += kOrderBlock)
            P.order[sp.state_off + base + q] = (uint16_t)w[q];
    }
}

// ===========================================================================
// Launchers
// ===========================================================================
hipError_t launch_setup(const SetupTab *tab, size_t tab_bytes, unsigned char *shot_tab,
                        unsigned long long *accum, size_t n64, double psi_max, double h,
                        int n_steps, int envelope, double omega_tau, float *env32, double *env64,
                        hipStream_t s) {
    if (tab_bytes > sizeof(SetupTab) || tab_bytes % 8 != 0) return hipErrorInvalidValue;
    const int words = tab ? (int)(tab_bytes / 8) : 0;
    // a thread an envelope point or table word; the accumulators by 1024 blocks at most
    const size_t need = std::max((size_t)2 * n_steps + 1, (size_t)words);
    const size_t blocks = std::max((need + kSetupBlock - 1) / kSetupBlock,
                                   std::min((n64 + kSetupBlock - 1) / kSetupBlock, (size_t)1024));
    static const SetupTab none{};
    setup_kernel<<<(unsigned)blocks, kSetupBlock, 0, s>>>(
        tab ? *tab : none, words, reinterpret_cast<unsigned long long *>(shot_tab), accum, n64,
        psi_max, h, n_steps, envelope, omega_tau, env32, env64);
    return hipGetLastError();
}

hipError_t launch_order(const BatchParams &p, hipStream_t s) {
    if (p.n_gitems < 1) return hipSuccess;
    order_kernel<<<(unsigned)std::min(p.n_gitems, (int64_t)kOrderGrid), kOrderBlock, 0, s>>>(p);
    return hipGetLastError();
}

template <int PREC, bool LOCAL, bool NODES, bool MODES>
static PassKernel phase64_of() {
    return {reinterpret_cast<const void *>(&phase64_kernel<PREC, LOCAL, NODES, MODES>),
            phase64_block<PREC>(),
            sizeof(double2) * 8 * (PREC == PREC_F32MIX ? kWinMix : kWin64), true};
}

template <int PREC, bool QUANTUM, bool LOCAL, bool NODES, bool MODES>
static PassKernel phase_of() {
    if constexpr (QUANTUM && PREC != PREC_F32)
        return phase64_of<PREC, LOCAL, NODES, MODES>();
    else
        return {reinterpret_cast<const void *>(&phase_kernel<PREC, QUANTUM, LOCAL, NODES, MODES>),
                kPhaseBlock, 0, false};
}

// modes: some shot of the launch uses a higher transverse mode
template <int PREC, bool QUANTUM>
static PassKernel select_phase(bool local, bool modes) {
    if (local)
        return modes ? phase_of<PREC, QUANTUM, true, false, true>()
                     : phase_of<PREC, QUANTUM, true, false, false>();
    return modes ? phase_of<PREC, QUANTUM, false, false, true>()
                 : phase_of<PREC, QUANTUM, false, false, false>();
}

hipError_t launch_phase(const BatchParams &p, const float *env32, const double *env64, int prec,
                        int rr, int amp, hipStream_t s) {
    const bool q = rr == 1, l = amp == 1, m = p.any_mode != 0;
    if (prec == PREC_F32MIX && !q) prec = PREC_F32;  // no radiation table, no promotion
    PassKernel k{};
    int device = 0, ncu = 0;
    hipError_t e = hipGetDevice(&device);
    if (e == hipSuccess)
        e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess) return e;
    if (prec == PREC_F32 && q && l && !m && p.n_items <= ncu) {
        k = {reinterpret_cast<const void *>(&phase_pair_kernel), kPairBlock, sizeof(PairLds), false};
        e = hipFuncSetAttribute(k.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.lds);
        if (e != hipSuccess) return e;
    } else if (prec == PREC_F32) {
        k = q ? select_phase<PREC_F32, true>(l, m) : select_phase<PREC_F32, false>(l, m);
    }
    if (prec == PREC_F64) k = q ? select_phase<PREC_F64, true>(l, m) : select_phase<PREC_F64, false>(l, m);
    if (prec == PREC_F32MIX) k = select_phase<PREC_F32MIX, true>(l, m);
    if (!k.fn) return hipErrorInvalidValue;
    return run_pass(k, p, env32, env64, p.phase_cap, s);
}

hipError_t launch_phase_nodes(const BatchParams &p, const float *env32, const double *env64,
                              int prec, int rr, hipStream_t s) {
    const bool q = rr == 1;
    if (prec == PREC_F32MIX && !q) prec = PREC_F32;
    int device = 0, ncu = 0;
    hipError_t e = hipGetDevice(&device);
    if (e == hipSuccess)
        e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess) return e;
    BatchParams pn = p;
    const bool wide = q && prec != PREC_F32;
    PassKernel k{};
    if (!wide && p.n_items <= ncu) {
        // with the draws: LDS for one block a CU
        k = {prec == PREC_F64
                 ? reinterpret_cast<const void *>(
                       &phase_kernel<PREC_F64, false, false, true, false, true>)
             : q ? reinterpret_cast<const void *>(
                       &phase_kernel<PREC_F32, true, false, true, false, true>)
                 : reinterpret_cast<const void *>(
                       &phase_kernel<PREC_F32, false, false, true, false, true>),
             kPhaseBlock, 84 * 1024, false};
        e = hipFuncSetAttribute(k.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.lds);
        if (e != hipSuccess) return e;
    } else {
        if (prec == PREC_F32)
            k = q ? phase_of<PREC_F32, true, false, true, false>()
                  : phase_of<PREC_F32, false, false, true, false>();
        if (prec == PREC_F64)
            k = q ? phase_of<PREC_F64, true, false, true, false>()
                  : phase_of<PREC_F64, false, false, true, false>();
        if (prec == PREC_F32MIX) k = phase_of<PREC_F32MIX, true, false, true, false>();
        if (!k.fn) return hipErrorInvalidValue;
        int grid = 0;
        e = resident_grid(reinterpret_cast<const void *>(&draw_kernel), kPhaseBlock, 0,
                          (p.n_draws + kPhaseBlock / 64 - 1) / (kPhaseBlock / 64), &grid);
        if (e != hipSuccess) return e;
        draw_kernel<<<grid, kPhaseBlock, 0, s>>>(p);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        pn.n_draws = 0;
    }
    return run_pass(k, pn, env32, env64, p.phase_cap, s);
}

// edge weights (u64, one per edge) and counters (u32, one per bin and two
// more) of the deposit kernel: at most 12 bytes a histogram word (20 with the
// runs' upper tails apart)
size_t deposit_lds_bytes(int max_hist_words) { return (size_t)max_hist_words * 12; }

hipError_t launch_deposit(const BatchParams &p, int max_hist_words, bool nodes, hipStream_t s) {
    const bool split = (size_t)max_hist_words * 20 <= 64 * 1024;
    const void *fn = split ? (nodes ? reinterpret_cast<const void *>(&deposit_kernel<true, true>)
                                    : reinterpret_cast<const void *>(&deposit_kernel<true, false>))
                           : (nodes ? reinterpret_cast<const void *>(&deposit_kernel<false, true>)
                                    : reinterpret_cast<const void *>(&deposit_kernel<false, false>));
    const size_t lds = (size_t)max_hist_words * (split ? 20 : 12);
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    int grid = 0;
    e = resident_grid(fn, kDepBlock, lds, p.n_ditems, &grid, p.dep_cap);
    if (e != hipSuccess) return e;
    BatchParams pc = p;
    void *args[] = {&pc};
    return hipLaunchKernel(fn, dim3((unsigned)grid), dim3(kDepBlock), args, lds, s);
}

hipError_t launch_shadow_diff(const BatchParams &p, int64_t n_items, int max_hist_words,
                              hipStream_t s) {
    if (n_items <= 0) return hipSuccess;
    const int grid = (int)(n_items < 2048 ? n_items : 2048);
    shadow_diff_kernel<<<grid, kPhaseBlock, (size_t)max_hist_words * 8, s>>>(p, n_items);
    return hipGetLastError();
}

hipError_t launch_finalize(const BatchParams &p, hipStream_t s) {
    finalize_kernel<<<p.n_shots, kFinBlock, 0, s>>>(p);
    return hipGetLastError();
}

}  // namespace qs
