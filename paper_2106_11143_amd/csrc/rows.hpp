// Whole rows of the all-pairs sum in one launch (device code): a workgroup
// takes I ions against every ion j of the run, lanes holding the j's, and
// finishes what depends on the sums (forces, gradient, or trap, kick and
// drift) itself.
//
// What bounds small runs is not the pairs but the launches and the round
// trips of partial sums between them: one step of 1024 ions is 1e6 pairs,
// 0.6 us of the chip's FP64 rate, and took 9.5 us (11.0 with energy records)
// as a pair launch with j-split partials in memory and an epilogue launch
// that read them back.  Here no partial leaves the workgroup: with I = 4 ions
// per workgroup 1024 ions are 256 workgroups, one per CU, each lane holds its
// j's pairs with the I ions in registers (4 independent chains of FP64 work),
// and the step is one launch of coalesced loads, pairs, one reduction and the
// update: 4.9 (5.3) us, of which about 2 are the launch (which rows_run.hpp
// saves for a run of several steps).  Larger runs
// take I = 8, which halves the j loads and the reductions per pair (4096
// ions: 16.5 us per step; 19.1 with I = 4, and 21.4 as two launches); from
// about 8192 ions the direct pair kernel is as fast (54 us).
#pragma once
#include <hip/hip_runtime.h>

#include "rsqrt.hpp"
#include "step_common.hpp"
#include "wave_reduce.hpp"

namespace cb {

// p[i] at a uniform i, by a scalar load: no launch writes the positions it
// reads, which the compiler cannot see past its stores to the other buffers.
__device__ __forceinline__ double uniform_load(const double* p, int i) {
    return ((const __attribute__((address_space(4))) double*)(p))[i];
}

// One j per lane against the I ions (uniform: SGPR operands).  MASK: the
// self pair and lanes past the run (j >= n) add nothing.
template <int PREC, int I, bool POT, bool MASK>
__device__ __forceinline__ void rows_block(double xj, double yj, double zj, double qj, int j, int n, int i0,
                                           const double (&xi)[I], const double (&yi)[I], const double (&zi)[I],
                                           double eps2, const SeriesK& K, double (&f)[I][POT ? 4 : 3]) {
#pragma unroll
    for (int u = 0; u < I; ++u) {
        const double dx = xi[u] - xj, dy = yi[u] - yj, dz = zi[u] - zj;
        const double r2 = __builtin_fma(dx, dx, __builtin_fma(dy, dy, __builtin_fma(dz, dz, eps2)));
        double s = 0.0, y = 0.0;
        inv_r<PREC, true, POT>(r2, qj, K, s, y);
        if (MASK) {
            const bool off = j == i0 + u || j >= n;
            s = off ? 0.0 : s;
            if (POT) y = off ? 0.0 : y;
        }
        f[u][0] = __builtin_fma(dx, s, f[u][0]);
        f[u][1] = __builtin_fma(dy, s, f[u][1]);
        f[u][2] = __builtin_fma(dz, s, f[u][2]);
        if constexpr (POT) f[u][3] = __builtin_fma(qj, y, f[u][3]);
        // four pairs in flight: the empty asm keeps the compiler from
        // interleaving all I of them (205 VGPRs at I = 8 without it)
        if (u % 4 == 3 && u + 1 < I) {
#pragma unroll
            for (int v = u - 3; v <= u; ++v) asm volatile("" : "+v"(f[v][0]), "+v"(f[v][1]), "+v"(f[v][2]));
        }
    }
}

// Waves per SIMD the register budget is sized for.
template <int PREC, int I, bool POT>
constexpr int rows_waves() {
    return PREC == PREC_IEEE ? 2 : (POT && I > 4 ? 3 : 4);
}

// LDS of one workgroup of W waves: the waves' sums of each ion, and for more
// than 4 ions a reduction buffer per wave.
template <int I, int W, bool POT>
struct RowsLds {
    static constexpr int kC = POT ? 4 : 3;
    static constexpr int kVals = 4 * kC;  // sums of 4 ions, reduced together
    double red[I > 4 ? W : 1][I > 4 ? kVals * kRedStride : 1];
    double sum[W][I * kC];
};

// The sums over the wave's lanes of its f to lds.sum[w] (component c of ion u
// at u kC + c), and a barrier.  With 4 ions they go across the lanes by swaps
// and DPP, which wait for nobody; through LDS (lds_reduce), the sums of a
// workgroup of 8 waves queue for its bandwidth (115 KB per call).
template <int I, int W, bool POT>
__device__ __forceinline__ void rows_wave_sums(const double (&f)[I][POT ? 4 : 3], RowsLds<I, W, POT>& lds) {
    static_assert(I % 4 == 0, "ions per workgroup in fours");
    constexpr int C = POT ? 4 : 3, NV = 4 * C;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (I == 4) {
        double v[12], o[3], p = 0.0;
#pragma unroll
        for (int k = 0; k < 12; ++k) v[k] = f[k / 3][k % 3];
        reduce_scatter12(v, o);
        if constexpr (POT) {
            const double y[4] = {f[0][3], f[1][3], f[2][3], f[3][3]};
            p = reduce_scatter4(y);
        }
        const int c = lane & 15;
        if (c < C) lds.sum[w][(lane >> 4) * C + c] = c == 0 ? o[0] : (c == 1 ? o[1] : (c == 2 ? o[2] : p));
    } else {
#pragma unroll
        for (int h = 0; h < I / 4; ++h) {
            double v[NV];
#pragma unroll
            for (int k = 0; k < NV; ++k) v[k] = f[4 * h + k / C][k % C];
            const double o = lds_reduce<NV>(v, lds.red[w]);
            if ((lane & 3) == 0 && (lane >> 2) < NV) lds.sum[w][h * NV + (lane >> 2)] = o;
        }
    }
    __syncthreads();
}

// Value k of lds.sum over the waves, in wave order.
template <int I, int W, bool POT>
__device__ __forceinline__ double rows_sum(const RowsLds<I, W, POT>& lds, int k) {
    double a = lds.sum[0][k];
#pragma unroll
    for (int u = 1; u < W; ++u) a += lds.sum[u][k];
    return a;
}

// Sums over j of ions i0 .. i0 + I - 1 (indices from n on repeat the last
// ion) of a run of n at X, Y, Z with charges Q, by a workgroup of W waves:
// q_j d r^-3 (three components) and, with POT, q_j / r.  Wave w takes the
// blocks of 64 j's w, w + W, ...; its lanes' sums are added by rows_wave_sums
// and the waves' in wave order, so the result does not depend on timing.  Every
// thread calls it; thread t < I returns ion t's sums in out.
template <int PREC, int I, int W, bool POT>
__device__ __forceinline__ void rows_sums(int n, const double* __restrict__ X, const double* __restrict__ Y,
                                          const double* __restrict__ Z, const double* __restrict__ Q, int i0,
                                          double eps2, RowsLds<I, W, POT>& lds, double (&out)[4]) {
    constexpr int C = POT ? 4 : 3;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double xi[I], yi[I], zi[I];
#pragma unroll
    for (int u = 0; u < I; ++u) {
        const int i = min(i0 + u, n - 1);
        xi[u] = uniform_load(X, i);
        yi[u] = uniform_load(Y, i);
        zi[u] = uniform_load(Z, i);
    }
    double f[I][C];
#pragma unroll
    for (int u = 0; u < I; ++u)
#pragma unroll
        for (int c = 0; c < C; ++c) f[u][c] = 0.0;
    const SeriesK K;
    int jb = w * 64;
    if (jb < n) {
        int jc = min(jb + lane, n - 1);
        double xj = X[jc], yj = Y[jc], zj = Z[jc], qj = Q[jc];
        for (; jb < n; jb += 64 * W) {
            // the next block's loads are in flight during this block's pairs
            jc = min(jb + 64 * W + lane, n - 1);
            const double xn = X[jc], yn = Y[jc], zn = Z[jc], qn = Q[jc];
            if (jb + 64 > n || (jb < i0 + I && jb + 64 > i0))
                rows_block<PREC, I, POT, true>(xj, yj, zj, qj, jb + lane, n, i0, xi, yi, zi, eps2, K, f);
            else
                rows_block<PREC, I, POT, false>(xj, yj, zj, qj, jb + lane, n, i0, xi, yi, zi, eps2, K, f);
            xj = xn;
            yj = yn;
            zj = zn;
            qj = qn;
        }
    }
    rows_wave_sums<I, W, POT>(f, lds);
    if (threadIdx.x < I) {
#pragma unroll
        for (int c = 0; c < C; ++c) out[c] = rows_sum<I, W, POT>(lds, threadIdx.x * C + c);
    }
}

}  // namespace cb
