// Launch sequence of the Newton's-third-law force stage (tile table, pair
// kernel, finish) for every precision, i-particles-per-lane count and
// reaction-sum variant.
#include <hip/hip_runtime.h>

#include "internal.hpp"
#include "pair_sym.hpp"

namespace cb {

constexpr int kPlanThreads = 1024;

// Tile table, one workgroup (sym_plan_fill in pair_sym.hpp).
__global__ void __launch_bounds__(kPlanThreads) k_sym_plan(int n, int IB, int JL, int W, int nI,
                                                           int* __restrict__ rowstart, int2* __restrict__ tiles,
                                                           int G0) {
    sym_plan_fill<kPlanThreads>(n, IB, JL, W, nI, rowstart, tiles, G0);
}

static size_t al256(size_t b) { return (b + 255) / 256 * 256; }

static int sym_groups(int64_t n, int IB, int W) {
    const int nI = (int)((n + IB - 1) / IB);
    return (nI + W - 1) / W;
}

int64_t sym_tiles(int64_t n, int IB, int JL, int W) {
    const int nG = sym_groups(n, IB, W);
    int64_t T = 0;
    for (int G = 0; G < nG; ++G) T += sym_nseg((int)n, IB, JL, G * W);
    return T;
}

// Workspace carve-up: rowstart[nG+1] | tiles[T] | Pi[T][W][3][IB] |
// R[T][3][JL] (| Et[T][W], the tiles' pair energies, with the energy)
size_t sym_ws_bytes(int64_t n, int p, int jl, bool pot, int W) {
    const int IB = 64 * p;
    const int64_t T = sym_tiles(n, IB, jl, W);
    const size_t TW = (size_t)W * T;
    return sym_plan_bytes(n, IB, jl, W) + al256(sizeof(double) * 3 * IB * (TW + 1)) +
           al256(sizeof(double) * 3 * (size_t)jl * (T + 1)) + (pot ? al256(sizeof(double) * (TW + 1)) : 0);
}

template <int PREC, int P, int RED, bool POT>
static void go_sym(int n, int JL, int64_t T, const double* x, const double* y, const double* z, const double* q,
                   double eps2, const int2* tiles, double* Pi, double* R, double* Et, hipStream_t st) {
    k_pair_sym<PREC, P, RED, POT><<<(unsigned)T, 64, 0, st>>>(n, x, y, z, q, eps2, JL, tiles, Pi, R, Et);
}

template <int PREC, int RED, bool POT>
static bool go_sym_p(int P, int n, int JL, int64_t T, const double* x, const double* y, const double* z,
                     const double* q, double eps2, const int2* tiles, double* Pi, double* R, double* Et,
                     hipStream_t st) {
    switch (P) {
        case 2: go_sym<PREC, 2, RED, POT>(n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st); return true;
        case 3: go_sym<PREC, 3, RED, POT>(n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st); return true;
        case 4: go_sym<PREC, 4, RED, POT>(n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st); return true;
        case 5: go_sym<PREC, 5, RED, POT>(n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st); return true;
        case 6: go_sym<PREC, 6, RED, POT>(n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st); return true;
        case 8: go_sym<PREC, 8, RED, POT>(n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st); return true;
        default: return false;
    }
}

// red: 1 = reactions summed through LDS, 0 = by permutes; the energy's
// variant sums them through LDS.
template <int PREC>
static bool go_sym_pr(int P, int red, bool pot, int n, int JL, int64_t T, const double* x, const double* y,
                      const double* z, const double* q, double eps2, const int2* tiles, double* Pi, double* R,
                      double* Et, hipStream_t st) {
    if (pot) return go_sym_p<PREC, 1, true>(P, n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st);
    return red ? go_sym_p<PREC, 1, false>(P, n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st)
               : go_sym_p<PREC, 0, false>(P, n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st);
}

// The row-group kernel (kSymRows i-blocks per workgroup), for P = 4, 6, 8.
// EY: the energies from r^-1 itself (the bands, with kBandP ions per lane).
template <int PREC, bool POT, bool EY>
static bool go_sym_rows(int P, int n, int JL, int64_t T, const double* x, const double* y, const double* z,
                        const double* q, double eps2, const int2* tiles, double* Pi, double* R, double* Et,
                        hipStream_t st) {
    const unsigned g = (unsigned)T, b = 64 * kSymRows;
    if constexpr (EY) {
        if (P != kBandP) return false;
        k_pair_sym_rows<PREC, kBandP, POT, true><<<g, b, 0, st>>>(n, x, y, z, q, eps2, JL, tiles, Pi, R, Et);
        return true;
    }
    switch (P) {
        case 4: k_pair_sym_rows<PREC, 4, POT><<<g, b, 0, st>>>(n, x, y, z, q, eps2, JL, tiles, Pi, R, Et); return true;
        case 6: k_pair_sym_rows<PREC, 6, POT><<<g, b, 0, st>>>(n, x, y, z, q, eps2, JL, tiles, Pi, R, Et); return true;
        case 8: k_pair_sym_rows<PREC, 8, POT><<<g, b, 0, st>>>(n, x, y, z, q, eps2, JL, tiles, Pi, R, Et); return true;
        default: return false;
    }
}

template <int PREC, bool BAND>
static bool go_sym_rows_p(int P, bool pot, int n, int JL, int64_t T, const double* x, const double* y,
                          const double* z, const double* q, double eps2, const int2* tiles, double* Pi, double* R,
                          double* Et, hipStream_t st) {
    constexpr bool EY = BAND && energy_y<PREC>();
    return pot ? go_sym_rows<PREC, true, EY>(P, n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st)
               : go_sym_rows<PREC, false, false>(P, n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st);
}

template <int PREC, bool BAND>
static void go_finish(bool pot, unsigned nb, int n, int IB, int JL, int lgJL, int W, const double* x,
                      const double* y, const double* z, const double* q, double eps2, const int* rowstart,
                      const double* Pi, const double* R, const double* Et, double* F, double* phi, int G0, int G1,
                      hipStream_t st) {
    if (pot)
        k_sym_finish<PREC, true, BAND><<<nb, 64 * kFinishParts, 0, st>>>(n, IB, JL, lgJL, W, x, y, z, q, eps2,
                                                                         rowstart, Pi, R, Et, F, phi, G0, G1);
    else
        k_sym_finish<PREC, false, BAND><<<nb, 64 * kFinishParts, 0, st>>>(n, IB, JL, lgJL, W, x, y, z, q, eps2,
                                                                          rowstart, Pi, R, Et, F, phi, G0, G1);
}

// Finish of the whole triangle, or of the band of row groups [G0, G1).
template <bool BAND>
static cb_status finish(int prec, bool pot, unsigned nb, int n, int IB, int JL, int W, const double* x,
                        const double* y, const double* z, const double* q, double eps2, const int* rowstart,
                        const double* Pi, const double* R, const double* Et, double* F, double* phi, int G0, int G1,
                        hipStream_t st) {
    int lgJL = 0;
    while ((1 << lgJL) < JL) ++lgJL;
    switch (prec) {
        case PREC_FP64: go_finish<PREC_FP64, BAND>(pot, nb, n, IB, JL, lgJL, W, x, y, z, q, eps2, rowstart, Pi, R, Et, F, phi, G0, G1, st); break;
        case PREC_MIXED: go_finish<PREC_MIXED, BAND>(pot, nb, n, IB, JL, lgJL, W, x, y, z, q, eps2, rowstart, Pi, R, Et, F, phi, G0, G1, st); break;
        case PREC_IEEE: go_finish<PREC_IEEE, BAND>(pot, nb, n, IB, JL, lgJL, W, x, y, z, q, eps2, rowstart, Pi, R, Et, F, phi, G0, G1, st); break;
        default: go_finish<PREC_FP32, BAND>(pot, nb, n, IB, JL, lgJL, W, x, y, z, q, eps2, rowstart, Pi, R, Et, F, phi, G0, G1, st); break;
    }
    return check_launch("k_sym_finish");
}

template <bool BAND>
static bool go_rows_prec(int prec, int P, bool pot, int n, int JL, int64_t T, const double* x, const double* y,
                         const double* z, const double* q, double eps2, const int2* tiles, double* Pi, double* R,
                         double* Et, hipStream_t st) {
    switch (prec) {
        case PREC_FP64: return go_sym_rows_p<PREC_FP64, BAND>(P, pot, n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st);
        case PREC_MIXED: return go_sym_rows_p<PREC_MIXED, BAND>(P, pot, n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st);
        case PREC_IEEE: return go_sym_rows_p<PREC_IEEE, BAND>(P, pot, n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st);
        case PREC_FP32: return go_sym_rows_p<PREC_FP32, BAND>(P, pot, n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st);
        default: return false;
    }
}

size_t sym_plan_bytes(int64_t n, int IB, int JL, int W) {
    const int64_t nG = sym_groups(n, IB, W);
    return al256(sizeof(int) * (nG + 1)) + al256(sizeof(int2) * (sym_tiles(n, IB, JL, W) + 1));
}

cb_status sym_plan(int n, int IB, int JL, void* ws, SymPlan* out, hipStream_t st, int W, bool filled) {
    const int nI = (n + IB - 1) / IB;
    if (nI > kPlanMaxRows) return fail(CB_EINVAL, "sym_plan: n = %d is too large for the symmetric kernels", n);
    const int nG = sym_groups(n, IB, W);
    out->T = sym_tiles(n, IB, JL, W);
    char* base = static_cast<char*>(ws);
    out->rowstart = reinterpret_cast<int*>(base);
    base += al256(sizeof(int) * (nG + 1));
    out->tiles = reinterpret_cast<int2*>(base);
    out->bytes = sym_plan_bytes(n, IB, JL, W);
    if (filled) return CB_OK;
    k_sym_plan<<<1, kPlanThreads, 0, st>>>(n, IB, JL, W, nG, out->rowstart, out->tiles, 0);
    return check_launch("k_sym_plan");
}

cb_status launch_pair_sym(int prec, const LaunchCfg& c, int n, const double* x, const double* y, const double* z,
                          const double* q, double eps2, void* ws, double* F, hipStream_t st, double* phi,
                          bool plan_filled) {
    const int P = c.p, JL = c.splits, IB = 64 * P, W = sym_rows(c.algo);
    if (!is_sym(c.algo) || !sym_cfg_ok(P, c.wg, JL) || (W > 1 && !sym_rows_p_ok(P)))
        return fail(CB_EINVAL, "launch_pair_sym: bad configuration");
    const int red = c.algo == ALGO_SYM ? 0 : 1;
    SymPlan plan;
    cb_status rc = sym_plan(n, IB, JL, ws, &plan, st, W, plan_filled);
    if (rc) return rc;
    const int64_t T = plan.T;
    int* rowstart = plan.rowstart;
    const int2* tiles = plan.tiles;
    const bool pot = phi != nullptr;
    char* base = static_cast<char*>(ws) + plan.bytes;
    double* Pi = reinterpret_cast<double*>(base);
    base += al256(sizeof(double) * 3 * IB * ((size_t)W * T + 1));
    double* R = reinterpret_cast<double*>(base);
    base += al256(sizeof(double) * 3 * (size_t)JL * (T + 1));
    double* Et = pot ? reinterpret_cast<double*>(base) : nullptr;
    if (T > 0 && W > 1) {
        const bool okk = go_rows_prec<false>(prec, P, pot, n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st);
        if (!okk) return fail(CB_EINVAL, "launch_pair_sym: unsupported precision %d / p %d", prec, P);
        if ((rc = check_launch("k_pair_sym_rows"))) return rc;
    } else if (T > 0) {
        bool okk = false;
        switch (prec) {
            case PREC_FP64: okk = go_sym_pr<PREC_FP64>(P, red, pot, n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st); break;
            case PREC_MIXED: okk = go_sym_pr<PREC_MIXED>(P, red, pot, n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st); break;
            case PREC_IEEE: okk = go_sym_pr<PREC_IEEE>(P, red, pot, n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st); break;
            case PREC_FP32: okk = go_sym_pr<PREC_FP32>(P, red, pot, n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st); break;
            default: break;
        }
        if (!okk) return fail(CB_EINVAL, "launch_pair_sym: unsupported precision %d / p %d", prec, P);
        if ((rc = check_launch("k_pair_sym"))) return rc;
    }
    return finish<false>(prec, pot, (unsigned)((n + 63) / 64), n, IB, JL, W, x, y, z, q, eps2, rowstart, Pi, R, Et, F,
                         phi, 0, 0, st);
}

// Row groups of the band that starts at group G0 with at most ws_bytes of
// tables and partials (at least one group): its tiles to *T.
static int band_groups(int64_t n, int G0, bool pot, size_t ws_bytes, int64_t* T) {
    constexpr int IB = 64 * kBandP, W = kSymRows;
    const int nG = sym_groups(n, IB, W);
    const size_t per_tile = sizeof(int2) + sizeof(double) * (3 * IB * W + 3 * (size_t)kBandJL + (pot ? W : 0));
    const size_t fixed = 4 * 256 + sizeof(int) * (kPlanMaxRows + 1);  // rowstart and the roundings
    int G = G0;
    *T = 0;
    while (G < nG && G - G0 < kPlanMaxRows) {
        const int64_t t = sym_nseg((int)n, IB, kBandJL, G * W);
        if (G > G0 && fixed + per_tile * (size_t)(*T + t) > ws_bytes) break;
        *T += t;
        ++G;
    }
    return G - G0;
}

cb_status launch_pair_sym_bands(int prec, int n, const double* x, const double* y, const double* z, const double* q,
                                double eps2, void* ws, size_t ws_bytes, double* F, hipStream_t st, double* phi) {
    constexpr int P = kBandP, JL = kBandJL, IB = 64 * P, W = kSymRows;
    const int nG = sym_groups(n, IB, W);
    const bool pot = phi != nullptr;
    for (int G0 = 0; G0 < nG;) {
        int64_t T = 0;
        const int ng = band_groups(n, G0, pot, ws_bytes, &T), G1 = G0 + ng;
        char* base = static_cast<char*>(ws);
        auto carve = [&](size_t bytes) {
            char* p = base;
            base += al256(bytes);
            return p;
        };
        int* rowstart = reinterpret_cast<int*>(carve(sizeof(int) * (ng + 1)));
        int2* tiles = reinterpret_cast<int2*>(carve(sizeof(int2) * T));
        double* Pi = reinterpret_cast<double*>(carve(sizeof(double) * 3 * IB * W * T));
        double* R = reinterpret_cast<double*>(carve(sizeof(double) * 3 * JL * T));
        double* Et = pot ? reinterpret_cast<double*>(carve(sizeof(double) * W * T)) : nullptr;
        if (base > static_cast<char*>(ws) + ws_bytes)
            return fail(CB_ENOWS, "launch_pair_sym_bands: workspace too small for one row group at n = %d", n);
        k_sym_plan<<<1, kPlanThreads, 0, st>>>(n, IB, JL, W, ng, rowstart, tiles, G0);
        cb_status rc = check_launch("k_sym_plan");
        if (rc) return rc;
        if (T > 0) {
            if (!go_rows_prec<true>(prec, P, pot, n, JL, T, x, y, z, q, eps2, tiles, Pi, R, Et, st))
                return fail(CB_EINVAL, "launch_pair_sym_bands: unsupported precision %d", prec);
            if ((rc = check_launch("k_pair_sym_rows"))) return rc;
        }
        const int k0 = G0 * W * IB;
        if ((rc = finish<true>(prec, pot, (unsigned)((n - k0 + 63) / 64), n, IB, JL, W, x, y, z, q, eps2, rowstart, Pi, R,
                               Et, F, phi, G0, G1, st)))
            return rc;
        G0 = G1;
    }
    return CB_OK;
}

}  // namespace cb
