// qs_factor.hip -- plane-wave reconstruction of the A0EFF forward pass.
//
// Sec. 3.2 rebuilds the 3D spectrum from plane-wave runs over a uniform set
// of a0,eff values weighted by dN_b/da0,eff, and Sec. 3.3 applies it to the
// quantum case.  With the amplitude frozen at a0,eff, a sample's trajectory
// depends only on (a0,eff, gamma0_i), so the plane-wave runs are made once per
// node of an (a0,eff, gamma0) grid and every sample takes their result at its
// own coordinates:
//
//   node pass      (qs_kernels.hip, phase kernel in node mode): the moment
//                  system at every node a_k = a0 k / (K - 1), gamma_m; beside
//                  it each sample draws its coordinates as in the direct pass;
//   deposit        (qs_kernels.hip): each sample takes the bilinear interpolant
//                  of the nodes' final mean, variance and largest chi, and is
//                  deposited as in the direct pass; finalize is unchanged;
//   node weights   (here, for shots that ask): the bilinear weights summed over
//                  the samples (32.32 fixed point, in LDS), the discrete joint
//                  distribution of (a0,eff, gamma0).
//
// Only the node pass has a phase loop: K M trajectories instead of one per
// sample, few wavefronts on a mostly idle device, which the draws (Philox, one
// spatial factor a sample: 840 vector instructions, bound by FP64 issue) fill.
#include "qs_device.h"

namespace qs {

// The node weights of the shots that ask for them.  One block per deposit tile
// (dep_tile samples of one shot); dynamic LDS: the weights of the tile's shot.
__global__ __launch_bounds__(kDepBlock) void node_weights_kernel(BatchParams P) {
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned long long *Hn = reinterpret_cast<unsigned long long *>(smem);
    const int64_t item = blockIdx.x;
    const int s = __builtin_amdgcn_readfirstlane(find_shot(P.shots, P.n_shots, item, true));
    const ShotParams &sp = P.shots[s];
    if (P.outs[s].node_weights == nullptr) return;
    const int n_nodes = sp.n_anode * sp.n_gnode;
    for (int k = threadIdx.x; k < n_nodes; k += blockDim.x) Hn[k] = 0ull;
    __syncthreads();
    const int64_t i0 = (item - sp.ditem0) * P.dep_tile;
    const int64_t i1 = i0 + P.dep_tile < sp.n_samples ? i0 + P.dep_tile : sp.n_samples;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
        const int64_t o = sp.state_off + i;
        const NodeCell c(sp, P.st.S0[o], P.st.g0[o]);
        // the four weights rounded to 2^-32 so that they add up to exactly
        // one sample; the rounding remainder (at most two units) goes to
        // the largest
        unsigned long long q[4];
        long long rest = (long long)kOne;
        int big = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            q[j] = (unsigned long long)llrint(c.w[j] * 4294967296.0);
            rest -= (long long)q[j];
            if (c.w[j] > c.w[big]) big = j;
        }
        q[big] = (unsigned long long)((long long)q[big] + rest);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (q[j]) atomicAdd(&Hn[c.n[j]], q[j]);
    }
    __syncthreads();
    unsigned long long *G = P.hist + sp.hist_off + sp.n_e + 2 + sp.n_th + 2 + sp.n_a;
    for (int k = threadIdx.x; k < n_nodes; k += blockDim.x) {
        const unsigned long long v = Hn[k];
        if (v) atomicAdd(&G[k], v);
    }
}

// Node records and weights of the shots that ask for them (one block a shot).
__global__ __launch_bounds__(256) void node_outputs_kernel(BatchParams P) {
    const int s = blockIdx.x;
    const ShotParams &sp = P.shots[s];
    const ShotOut &so = P.outs[s];
    const int K = sp.n_anode, M = sp.n_gnode;
    if (so.node_weights) {
        const unsigned long long *H = P.hist + sp.hist_off + sp.n_e + 2 + sp.n_th + 2 + sp.n_a;
        for (int n = threadIdx.x; n < K * M; n += blockDim.x)
            so.node_weights[n] = (double)H[n] * (1.0 / 4294967296.0);
    }
    if (so.node_states) {
        for (int n = threadIdx.x; n < K * M; n += blockDim.x) {
            const int64_t g = sp.node_off + n;
            double *r = so.node_states + (size_t)n * kNodeFields;
            r[0] = sp.a0 * ((double)(n / M) / (double)(K - 1));
            r[1] = P.nst.g0[g];
            r[2] = P.nst.mu[g];
            r[3] = P.nst.s2[g];
            r[4] = (double)P.nst.cmx[g];
        }
    }
}

hipError_t launch_node_weights(const BatchParams &p, int weight_words, hipStream_t s) {
    if (p.n_ditems < 1 || weight_words < 1) return hipSuccess;
    const void *fn = reinterpret_cast<const void *>(&node_weights_kernel);
    const size_t lds = (size_t)weight_words * 8;
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    node_weights_kernel<<<(unsigned)p.n_ditems, kDepBlock, lds, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_node_outputs(const BatchParams &p, hipStream_t s) {
    node_outputs_kernel<<<p.n_shots, 256, 0, s>>>(p);
    return hipGetLastError();
}

}  // namespace qs
