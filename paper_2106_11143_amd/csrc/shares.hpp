// Newton's third law for one run of some thousand ions, or an ensemble of runs
// (device code): the triangles of pairs cut into equal shares, one per
// workgroup.
//
// Ions are cut into i-blocks of IB = 64 P; row I is block I against the ions
// j >= I IB, its own block (the diagonal, of which the pairs j > i count)
// first.  The rows, one after the other, are cut into units of kShareJ j's,
// and the units into as many equal contiguous shares as the launch has
// workgroups.  A workgroup takes each row that its share touches in turn: a
// lane holds P ions of the row's block, and the four waves a quarter each of
// the share's j's (uniform, pair_sym.hpp's groups of 4 j's, whose reactions
// are summed over the wave through LDS).  The waves' i sums are added in LDS
// and stored once per share and row, so the i partials number workgroups plus
// rows, whatever n.  A second launch adds, per ion, its row's i sums and its
// column's reactions in a fixed order and finishes (forces, gradient, or
// trap, kick and drift).
//
// What bounds these sizes is how evenly the pairs share the chip: one-wave
// tiles of 256 x 256 ions (42 us of a SIMD each) leave some SIMDs a tile more
// than others, and the direct kernel evaluates every pair twice.  Equal
// shares, all resident at once, end together: 12001 ions of one charge take
// 71.7 us per evaluation (64 us of it the pair launch, 50 at the FP64 issue
// rate) against 104 with the direct kernel, 20001 168 against 210 with tiles.
#pragma once
#include <hip/hip_runtime.h>

#include "pair_sym.hpp"

namespace cb {

constexpr int kShareWaves = 4;
constexpr int kShareJ = 4 * kGroupJ;  // j's per unit: one group per wave

// The cut of n ions in i-blocks of IB into N shares: the first `more` shares
// hold len + 1 units, the others len.
struct ShareCut {
    int n, IB, C;  // C: units of row 0
    int nI;        // rows
    int U, N;      // units, shares (N <= U)
    int len, more;
};

// The rows alone (N, len and more unset).
__host__ __device__ __forceinline__ ShareCut share_rows(int n, int P) {
    ShareCut c{};
    c.n = n;
    c.IB = 64 * P;
    c.C = (n + kShareJ - 1) / kShareJ;
    c.nI = (n + c.IB - 1) / c.IB;
    c.U = c.nI * c.C - c.IB / kShareJ * (c.nI * (c.nI - 1) / 2);
    return c;
}

// U units into at most maxN shares.
__host__ __device__ __forceinline__ void share_units(ShareCut& c, int U, int maxN) {
    c.U = U;
    c.N = maxN < c.U ? maxN : c.U;
    c.len = (int)((unsigned)c.U / (unsigned)c.N);
    c.more = c.U - c.len * c.N;
}

__host__ __device__ __forceinline__ ShareCut share_cut(int n, int P, int maxN) {
    ShareCut c = share_rows(n, P);
    share_units(c, c.U, maxN);
    return c;
}

// First unit of row I (of nI: all units), its number of units, the first
// unit of share g, and the share of unit u.
__host__ __device__ __forceinline__ int row_unit(const ShareCut& c, int I) {
    return I * c.C - c.IB / kShareJ * (I * (I - 1) / 2);
}
__host__ __device__ __forceinline__ int row_units(const ShareCut& c, int I) { return c.C - c.IB / kShareJ * I; }
__host__ __device__ __forceinline__ int share_unit(const ShareCut& c, int g) {
    return g * c.len + (g < c.more ? g : c.more);
}
__host__ __device__ __forceinline__ int unit_share(const ShareCut& c, int u) {
    const int big = c.more * (c.len + 1);  // units of the longer shares
    return u < big ? (int)((unsigned)u / (unsigned)(c.len + 1)) : c.more + (int)((unsigned)(u - big) / (unsigned)c.len);
}

// Pairs of one wave: j's [j0, j1) against the lane's P ions of the block at
// jb, reactions to Rt[c * stride + j - jb], i sums into ia, pair energy into
// pe.  DIAG: j's of the block itself, EY: energies from r^-1 (see sym_group).
template <int PREC, int P, bool UNI, bool POT, bool DIAG, bool EY>
__device__ __forceinline__ void share_wave(const double* __restrict__ x, const double* __restrict__ y,
                                           const double* __restrict__ z, const double* __restrict__ q, double eps2,
                                           int j0, int j1, int jb, int stride, const double (&xi)[P],
                                           const double (&yi)[P], const double (&zi)[P], const double (&qi)[P],
                                           double qI, double qJ, double (&ia)[P][3], double& pe,
                                           double* __restrict__ red, double* __restrict__ Rt) {
    const SeriesK K;
    const int jfull = j0 + (j1 - j0) / kGroupJ * kGroupJ;
    int jg = j0;
    if (jg < jfull) {
        JGroupT<!UNI> cur;
        load_group<false>(cur, jg, 0, x, y, z, q);
        for (; jg < jfull; jg += kGroupJ) {
            JGroupT<!UNI> nxt;
            const int jn = jg + kGroupJ;
            // the last request is waited for before the next is made: after it
            // a wait would be for both (12001 ions 71.5 -> 71.0 us)
            __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0), the other counters unwaited
            __builtin_amdgcn_sched_barrier(0);
            load_group<false>(nxt, jn < jfull ? jn : jg, 0, x, y, z, q);
            __builtin_amdgcn_sched_barrier(0);  // keep the requests ahead of the arithmetic
            sym_group<PREC, P, 1, false, UNI, POT, DIAG, EY>(cur, jg, kGroupJ, jb, stride, eps2, xi, yi, zi, qi, ia, pe,
                                                             K, qI, Rt, red, jb);
            cur = nxt;
        }
    }
    if (jg < j1) {  // the last, partial group: j's from j1 on are masked
        JGroupT<!UNI> tail;
        load_group<true>(tail, jg, j1 - jg - 1, x, y, z, q);
        sym_group<PREC, P, 1, true, UNI, POT, DIAG, EY>(tail, jg, j1 - jg, jb, stride, eps2, xi, yi, zi, qi, ia, pe, K,
                                                        qI, Rt, red, jb);
    }
    if constexpr (UNI) {
        const double sc = qI * qJ;
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int c = 0; c < 3; ++c) ia[p][c] *= sc;
        if constexpr (POT) pe *= sc;
    }
}

// LDS of one workgroup: a reduction buffer per wave, then (after a row's
// pairs) the waves' i sums.
template <int P>
union ShareLds {
    double red[kShareWaves][12 * kRedStride];
    double sum[kShareWaves][3 * 64 * P];
};

// Units [ua, ub) of the nu of row I of a run of n ions, by the workgroup: i
// sums to Pt[3][IB], reactions to Rt[c nu kShareJ + j - I IB], the pair energy
// (POT) to Et[0].
template <int PREC, int P, bool POT, bool EY>
__device__ __forceinline__ void share_row(int n, const double* __restrict__ x, const double* __restrict__ y,
                                          const double* __restrict__ z, const double* __restrict__ q, double eps2,
                                          int I, int nu, int ua, int ub, ShareLds<P>& lds, double (&esum)[kShareWaves],
                                          double* __restrict__ Pt, double* __restrict__ Rt, double* __restrict__ Et) {
    constexpr int IB = 64 * P;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ib = I * IB;
    double xi[P], yi[P], zi[P], qi[P], ia[P][3], pe = 0.0;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int i = min(ib + p * 64 + lane, n - 1);
        xi[p] = x[i];
        yi[p] = y[i];
        zi[p] = z[i];
        qi[p] = q[i];
        ia[p][0] = ia[p][1] = ia[p][2] = 0.0;
    }
    // the wave's j's: the w-th quarter, a whole group per unit
    const int j0 = min(n, ib + ua * kShareJ + w * (ub - ua) * kGroupJ);
    const int j1 = min(n, j0 + (ub - ua) * kGroupJ);
    const int jd = ib + IB;  // the block's own ions end here
    const int stride = nu * kShareJ;
    const int jo = max(j0, jd);
    if (j1 > jo) {
        double qI, qJ;
        if (tile_charges<P>(qi, q, jo, j1, qI, qJ))
            share_wave<PREC, P, true, POT, false, EY>(x, y, z, q, eps2, jo, j1, ib, stride, xi, yi, zi, qi, qI, qJ, ia, pe,
                                                  lds.red[w], Rt);
        else
            share_wave<PREC, P, false, POT, false, EY>(x, y, z, q, eps2, jo, j1, ib, stride, xi, yi, zi, qi, 1.0, 1.0, ia,
                                                   pe, lds.red[w], Rt);
    }
    if (j0 < min(j1, jd))
        share_wave<PREC, P, false, POT, true, EY>(x, y, z, q, eps2, j0, min(j1, jd), ib, stride, xi, yi, zi, qi, 1.0, 1.0,
                                              ia, pe, lds.red[w], Rt);
    if constexpr (POT) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) pe += __shfl_xor(pe, o);
        if (lane == 0) esum[w] = pe;
    }
    __syncthreads();  // the reduction buffers become the waves' sums
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int p = 0; p < P; ++p) lds.sum[w][c * IB + p * 64 + lane] = ia[p][c];
    __syncthreads();
    for (int k = threadIdx.x; k < 3 * IB; k += 64 * kShareWaves) {
        double a = lds.sum[0][k];
#pragma unroll
        for (int v = 1; v < kShareWaves; ++v) a += lds.sum[v][k];
        Pt[k] = a;
    }
    if (POT && threadIdx.x == 0) Et[0] = (esum[0] + esum[1]) + (esum[2] + esum[3]);
}

// Share blockIdx.x of the cut.  i sums of row I to Pi[blockIdx.x + I][3][IB],
// reactions of row I on its j's to R[3 row_unit(I) kShareJ + c row_units(I)
// kShareJ + j - I IB], pair energies (POT) to Et[blockIdx.x + I].  cut: the
// run's.
template <int PREC, int P, bool POT, bool EY>
__global__ void __launch_bounds__(64 * kShareWaves, (sym_waves<PREC, P, POT>()))
    k_share_pairs(ShareCut cut, const double* __restrict__ x, const double* __restrict__ y,
                  const double* __restrict__ z, const double* __restrict__ q, double eps2, double* __restrict__ Pi,
                  double* __restrict__ R, double* __restrict__ Et) {
    __shared__ __align__(16) ShareLds<P> lds;
    __shared__ double esum[kShareWaves];
    const int g = blockIdx.x;
    int u = share_unit(cut, g);
    const int uend = share_unit(cut, g + 1);
    int I = 0;  // the row of unit u
    {
        int hi = cut.nI - 1;
        while (I < hi) {
            const int mid = (I + hi + 1) / 2;
            if (row_unit(cut, mid) <= u) I = mid;
            else hi = mid - 1;
        }
    }
    for (; u < uend; ++I) {
        const int u0 = row_unit(cut, I), nu = row_units(cut, I);
        const int ue = min(uend, u0 + nu);  // this share's units of the row: [u, ue)
        const size_t slot = (size_t)(g + I);
        share_row<PREC, P, POT, EY>(cut.n, x, y, z, q, eps2, I, nu, u - u0, ue - u0, lds, esum, Pi + slot * 3 * 64 * P,
                                R + (size_t)3 * u0 * kShareJ, Et + slot);
        u = ue;
        if (u < uend) __syncthreads();  // the next row rewrites the buffers
    }
}

// The rows of many runs, one run after the other, in equal shares.  runs[r]:
// its first ion, its ions, its first row and first unit among all rows and
// units; first[g]: the run and the row (of the run) where share g starts.
// cut: N, len and more of all units.  i sums, reactions and pair energies as
// above, with rows and units counted over all runs.
template <int PREC, int P, bool POT>
__global__ void __launch_bounds__(64 * kShareWaves, (sym_waves<PREC, P, POT>()))
    k_share_pairs_ens(ShareCut all, const int4* __restrict__ runs, const int2* __restrict__ first,
                      const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
                      const double* __restrict__ q, double eps2, double* __restrict__ Pi, double* __restrict__ R,
                      double* __restrict__ Et) {
    __shared__ __align__(16) ShareLds<P> lds;
    __shared__ double esum[kShareWaves];
    const int g = blockIdx.x;
    int u = share_unit(all, g);
    const int uend = share_unit(all, g + 1);
    const int2 at = first[g];
    int r = at.x, I = at.y;
    while (u < uend) {
        const int4 ru = runs[r];
        const ShareCut cut = share_rows(ru.y, P);
        for (; I < cut.nI && u < uend; ++I) {
            const int u0 = ru.w + row_unit(cut, I), nu = row_units(cut, I);
            const int ue = min(uend, u0 + nu);
            const size_t slot = (size_t)(g + ru.z + I);
            share_row<PREC, P, POT, POT && energy_y<PREC>()>(ru.y, x + ru.x, y + ru.x, z + ru.x, q + ru.x, eps2, I, nu, u - u0, ue - u0, lds,
                                    esum, Pi + slot * 3 * 64 * P, R + (size_t)3 * u0 * kShareJ, Et + slot);
            u = ue;
            if (u < uend) __syncthreads();
        }
        ++r;
        I = 0;
    }
}

}  // namespace cb
