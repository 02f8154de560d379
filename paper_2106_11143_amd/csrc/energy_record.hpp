// Fixed-order sum of workgroups' energy terms into a record (device code).
#pragma once
#include <hip/hip_runtime.h>

#include "step_common.hpp"

namespace cb {

// Sums nb workgroups' energy terms [nb][3] in a fixed order (each thread's
// strided share, a butterfly over each wave, the waves in wave order) into
// out: with what = REC_ALL, out[0..3] = K, U_C, U_trap, E; with REC_UC, U_C;
// with REC_UPOT, U_C + U_trap.  Every thread of the workgroup calls it.
template <int W>
__device__ __forceinline__ void energy_record(int nb, const double* __restrict__ eblk, double* __restrict__ out,
                                            int what) {
    __shared__ double sh[W][3];
    double e[3] = {0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < nb; b += 64 * W)
#pragma unroll
        for (int c = 0; c < 3; ++c) e[c] += eblk[(size_t)b * 3 + c];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) e[c] += __shfl_xor(e[c], o);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int c = 0; c < 3; ++c) sh[threadIdx.x >> 6][c] = e[c];
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < W; ++w)
#pragma unroll
            for (int c = 0; c < 3; ++c) e[c] += sh[w][c];
        if (what == REC_UC) {
            out[0] = e[1];
        } else if (what == REC_UPOT) {
            out[0] = e[1] + e[2];
        } else {
            out[0] = e[0];
            out[1] = e[1];
            out[2] = e[2];
            out[3] = e[0] + e[1] + e[2];
        }
    }
}

template <int W>
__global__ void __launch_bounds__(64 * W) k_energy_record(int nb, const double* __restrict__ eblk,
                                                         double* __restrict__ out, int what) {
    energy_record<W>(nb, eblk, out, what);
}

// Records of the runs of an ensemble, run r = blockIdx.x: runs[r] = its first
// block and its blocks.
template <int W>
__global__ void __launch_bounds__(64 * W) k_ens_record(const int2* __restrict__ runs,
                                                      const double* __restrict__ eblk, long long nrec, long long rec,
                                                      double* __restrict__ energies) {
    const int2 ru = runs[blockIdx.x];
    energy_record<W>(ru.y, eblk + (size_t)ru.x * 3, energies + ((size_t)blockIdx.x * nrec + rec) * 4, REC_ALL);
}

}  // namespace cb
