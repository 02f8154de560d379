// Forces, gradients and velocity-Verlet steps of one run on equal shares of
// its Newton's-third-law pairs (shares.hpp): a pair launch and a launch that
// finishes each ion.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "energy_record.hpp"
#include "internal.hpp"
#include "shares.hpp"
#include "step_ion.hpp"

namespace cb {

struct ShareStep {
    int n;
    ShareCut cut;  // k_share_pairs'
    const double *Pi, *R, *Et;
    double *x, *y, *z;     // positions (a drift moves them in place)
    double *xn, *yn, *zn;  // = x, y, z
    const double *q, *m;   // m NULL: no trap term (EPI_GRAD)
    double *vx, *vy, *vz, *ax, *ay, *az;
    double *fx, *fy, *fz;  // EPI_FORCES, EPI_GRAD
    TrapK k;
    double gamma, dt;
    unsigned mode;
    double* eblk;  // [workgroups][3] energy sums (EPI_ENERGY)
    const double* eprev;  // an earlier record's sums, added by one extra workgroup into eprev_out
    double* eprev_out;
    int nprev;
    unsigned* flags;
};

// 64 ions of one block per workgroup: wave w adds the w-th part of the ions'
// i sums (the shares of their row) and of their reactions (the rows above and its own),
// wave 0 the waves' parts in order; then forces, gradient, or trap, kick and
// drift as the mode says.  The partials were just written by other CUs:
// several are in flight per wave.
constexpr int kFinWaves = 8, kFinPi = 3, kFinR = 6;

// A run among several (a single one is at zero): its first ion, row and unit,
// and its trap.
struct ShareRun {
    int o, row, unit;
    TrapK k;
    double gamma;
};

// The 64 ions from k0 on of a run of cut.n ions, by FW waves; their energy
// sums (POT) to eblk.
template <bool POT, int FW>
__device__ __forceinline__ void share_finish_ions(const ShareStep& S, const ShareCut& cut, const ShareRun& run, int k0,
                                                  double (&red)[FW][6][64], double* __restrict__ eblk) {
    const int IB = cut.IB;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kl = k0 + lane, kc = min(kl, cut.n - 1), k = run.o + kl;
    const int B = k0 / IB, off = kc - B * IB;
    const unsigned mode = S.mode;
    const bool own = w == 0 && kl < cut.n;
    const bool step =
        (mode & (EPI_ACCEL | EPI_KICK | EPI_DRIFT)) || ((mode & EPI_ENERGY) && !(mode & (EPI_GRAD | EPI_UPOT)));
    // the row's slots: its shares, each at slot share + row
    const int u0 = run.unit + row_unit(cut, B), row = run.row + B;
    const int s0 = unit_share(cut, u0) + row, s1 = unit_share(cut, u0 + row_units(cut, B) - 1) + row + 1;
    IonState s{};
    double x = 0.0, y = 0.0, z = 0.0, qk = 0.0;
    if (own) {
        qk = S.q[k];
        if (step || S.m) {
            x = S.x[k];
            y = S.y[k];
            z = S.z[k];
        }
        if (step) s = load_ion(S, k);
        else if (S.m) s.m = S.m[k];
    }
    double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (mode & (EPI_ACCEL | EPI_KICK | EPI_FORCES | EPI_GRAD)) {
        // part w of the row's slots [s0, s1) and of the rows 0 .. B, kFinPi and
        // kFinR of them requested together
        auto part = [&](int a, int b, int& lo, int& hi) {
            const int len = (b - a + FW - 1) / FW;
            lo = min(b, a + w * len);
            hi = min(b, lo + len);
        };
        int tp, tpe, tr, tre;
        part(s0, s1, tp, tpe);
        part(0, B + 1, tr, tre);
        for (; tp < tpe || tr < tre; tp += kFinPi, tr += kFinR) {
            double d[kFinPi][3], e[kFinR][3];
#pragma unroll
            for (int i = 0; i < kFinPi; ++i) {
                const double* p = S.Pi + (size_t)max(s0, min(tp + i, tpe - 1)) * 3 * IB + off;
                d[i][0] = p[0];
                d[i][1] = p[IB];
                d[i][2] = p[2 * IB];
            }
#pragma unroll
            for (int i = 0; i < kFinR; ++i) {
                const int I = max(0, min(tr + i, tre - 1)), stride = row_units(cut, I) * kShareJ;
                const double* p = S.R + (size_t)3 * (run.unit + row_unit(cut, I)) * kShareJ + (kc - I * IB);
                e[i][0] = p[0];
                e[i][1] = p[stride];
                e[i][2] = p[2 * (size_t)stride];
            }
#pragma unroll
            for (int i = 0; i < kFinPi; ++i)
                if (tp + i < tpe)
#pragma unroll
                    for (int c = 0; c < 3; ++c) v[c] += d[i][c];
#pragma unroll
            for (int i = 0; i < kFinR; ++i)
                if (tr + i < tre)
#pragma unroll
                    for (int c = 0; c < 3; ++c) v[3 + c] += e[i][c];
        }
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) red[w][c][lane] = v[c];
    __syncthreads();
    if (w != 0) return;
#pragma unroll
    for (int u = 1; u < FW; ++u)
#pragma unroll
        for (int c = 0; c < 6; ++c) v[c] += red[u][c][lane];
    double eK = 0.0, eC = 0.0, eT = 0.0;
    if (own) {
        const double Fx = kCoulomb * (v[0] - qk * v[3]);
        const double Fy = kCoulomb * (v[1] - qk * v[4]);
        const double Fz = kCoulomb * (v[2] - qk * v[5]);
        bool ok = true;
        if (mode & EPI_FORCES) {
            S.fx[k] = Fx;
            S.fy[k] = Fy;
            S.fz[k] = Fz;
            ok = finite3(Fx, Fy, Fz);
        } else if (step) {
            step_ion(S, run.k, run.gamma, k, s, x, y, z, qk, Fx, Fy, Fz, 0.0, eK, eC, eT);
        } else {
            if (mode & EPI_GRAD) {
                const double gx = __builtin_fma(s.m * run.k.kx, x, -Fx);
                const double gy = __builtin_fma(s.m * run.k.ky, y, -Fy);
                const double gz = __builtin_fma(s.m * run.k.kz, z, -Fz);
                S.fx[k] = gx;
                S.fy[k] = gy;
                S.fz[k] = gz;
                ok = finite3(gx, gy, gz);
            }
            if (POT) eT = 0.5 * s.m * (run.k.kx * x * x + run.k.ky * y * y + run.k.kz * z * z);
        }
        if (POT) {
            // each share of the block's row gives its pair energy to one ion
            eC = 0.0;
            for (int t = s0 + off; t < s1; t += IB) eC += S.Et[t];
            eC *= kCoulomb;
            ok = ok && __builtin_isfinite(eC) && __builtin_isfinite(eT);
        }
        if (!ok) atomicOr(S.flags, 1u);
    }
    if (POT) {
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) {
            eK += __shfl_xor(eK, d);
            eC += __shfl_xor(eC, d);
            eT += __shfl_xor(eT, d);
        }
        if (lane == 0) {
            eblk[0] = eK;
            eblk[1] = eC;
            eblk[2] = eT;
        }
    }
}

template <bool POT>
__global__ void __launch_bounds__(64 * kFinWaves) k_share_finish(ShareStep S) {
    __shared__ double red[kFinWaves][6][64];
    if (S.eprev && blockIdx.x == gridDim.x - 1)
        energy_record<kFinWaves>(S.nprev, S.eprev, S.eprev_out, REC_ALL);
    else
        share_finish_ions<POT, kFinWaves>(S, S.cut, ShareRun{0, 0, 0, S.k, S.gamma}, blockIdx.x * 64, red,
                                          POT ? S.eblk + (size_t)blockIdx.x * 3 : nullptr);
}

// The same for the runs of k_share_pairs_ens.  chunks[blockIdx.x]: run and
// first ion (of the run) of the workgroup's 64.
template <bool POT, int FW>
__global__ void __launch_bounds__(64 * FW) k_share_finish_ens(ShareStep S, const int4* __restrict__ runs,
                                                             const int2* __restrict__ chunks,
                                                             const cb_trap* __restrict__ traps, double t0,
                                                             long long step) {
    __shared__ double red[FW][6][64];
    const int2 ch = chunks[blockIdx.x];
    const int4 ru = runs[ch.x];
    ShareCut cut = share_rows(ru.y, S.cut.IB / 64);
    cut.len = S.cut.len;
    cut.more = S.cut.more;
    const cb_trap& tr = traps[ch.x];
    share_finish_ions<POT, FW>(S, cut, ShareRun{ru.x, ru.z, ru.w, trap_k(tr, step_time(t0, S.dt, step)), tr.gamma},
                               ch.y, red, POT ? S.eblk + (size_t)blockIdx.x * 3 : nullptr);
}

// ----------------------------------------------------------------- host

static size_t al(size_t b) { return (b + 255) / 256 * 256; }

// Shape at n ions.  Four ions per lane and 1024 shares, all resident at once
// (4 waves on each of the 1024 SIMDs); 2048 from 18000 ions, where a second
// round costs less than the uneven end of longer shares; eight ions per lane
// from 28000, where half the reaction sums per pair count more, in 2 rounds of
// the 768 workgroups that then fit at once, or 3 (us per evaluation on
// MI355X, P 4 with 1024 / 2048 shares: 8192 ions 42.7 / 46.7, 12001 70.8 / 71.5,
// 20001 173 / 168, 24576 248 / 242, 32768 427 / 417; P 8 with 768 / 1536 / 2304:
// 32768 ions 415 / 404 / 407, 40000 607 / 588 / 585, 49152 906 / 884 / 865).  With
// the energy, P = 8 does not fit its registers (49152 ions: 1180 against 1007
// with P = 4).
struct ShareShape {
    int P, N;
};

static ShareShape share_shape(int64_t n, bool pot) {
    if (n >= 28000 && !pot) return {8, n < 45056 ? 1536 : 2304};
    return {4, n < 18000 ? 1024 : 2048};
}

struct ShareWs {
    double *Pi, *R, *Et, *eblk[2];
    size_t bytes;
};

// Two sets of energy sums (at the same place for either shape) | Pi | R | Et.
// ws NULL: the size alone.
static ShareWs share_carve(int64_t n, bool pot, void* ws) {
    const ShareShape h = share_shape(n, pot);
    const ShareCut c = share_cut((int)n, h.P, h.N);
    const size_t slots = (size_t)c.N + c.nI, nb = (size_t)((n + 63) / 64);
    size_t at = 0;
    auto carve = [&](size_t doubles) {
        const size_t p = at;
        at += al(sizeof(double) * doubles);
        return ws ? reinterpret_cast<double*>(static_cast<char*>(ws) + p) : nullptr;
    };
    ShareWs w;
    w.eblk[0] = carve(3 * nb);
    w.eblk[1] = carve(3 * nb);
    w.Pi = carve(3 * slots * c.IB);
    w.R = carve(3 * (size_t)c.U * kShareJ);
    w.Et = carve(slots);
    w.bytes = at;
    return w;
}

size_t share_ws_bytes(int64_t n, bool pot) {
    const size_t f = share_carve(n, false, nullptr).bytes;
    return pot ? std::max(f, share_carve(n, true, nullptr).bytes) : f;
}

// Energies from r^-1 itself (energy_y) below the sizes at which the tiles are
// configured, whose energies are r^2 r^-3 (mixed, 28000 ions: 322 us against 313).
constexpr int kShareEyMaxN = 16383;

template <int PREC, int P, bool POT, bool EY = false>
static void go_share(int n, int N, const double* x, const double* y, const double* z, const double* q, double eps2,
                     const ShareWs& W, hipStream_t st) {
    const ShareCut c = share_cut(n, P, N);
    k_share_pairs<PREC, P, POT, EY><<<(unsigned)c.N, 64 * kShareWaves, 0, st>>>(c, x, y, z, q, eps2, W.Pi, W.R, W.Et);
}

template <int PREC>
static void go_share_p(bool pot, int n, const double* x, const double* y, const double* z, const double* q,
                       double eps2, const ShareWs& W, hipStream_t st) {
    const ShareShape h = share_shape(n, pot);
    switch (h.P) {
        case 4:
            if (!pot) go_share<PREC, 4, false>(n, h.N, x, y, z, q, eps2, W, st);
            else if (energy_y<PREC>() && n <= kShareEyMaxN) go_share<PREC, 4, true, energy_y<PREC>()>(n, h.N, x, y, z, q, eps2, W, st);
            else go_share<PREC, 4, true>(n, h.N, x, y, z, q, eps2, W, st);
            break;
        default: go_share<PREC, 8, false>(n, h.N, x, y, z, q, eps2, W, st); break;
    }
}

static cb_status share_pairs(int prec, int64_t n, const double* x, const double* y, const double* z, const double* q,
                             double eps2, bool pot, const ShareWs& W, hipStream_t st) {
    switch (prec) {
        case CB_FP64: go_share_p<PREC_FP64>(pot, (int)n, x, y, z, q, eps2, W, st); break;
        case CB_MIXED: go_share_p<PREC_MIXED>(pot, (int)n, x, y, z, q, eps2, W, st); break;
        case CB_FP64_IEEE: go_share_p<PREC_IEEE>(pot, (int)n, x, y, z, q, eps2, W, st); break;
        default: go_share_p<PREC_FP32>(pot, (int)n, x, y, z, q, eps2, W, st); break;
    }
    return check_launch("k_share_pairs");
}

static cb_status share_finish(const ShareStep& S, hipStream_t st) {
    const unsigned g = (unsigned)((S.n + 63) / 64) + (S.eprev ? 1u : 0u);
    if (S.mode & EPI_ENERGY) k_share_finish<true><<<g, 64 * kFinWaves, 0, st>>>(S);
    else k_share_finish<false><<<g, 64 * kFinWaves, 0, st>>>(S);
    return check_launch("k_share_finish");
}

// The partials that S reads, as share_pairs left them.
static void share_use(ShareStep& S, int64_t n, bool pot, const ShareWs& W) {
    const ShareShape h = share_shape(n, pot);
    S.n = (int)n;
    S.cut = share_cut((int)n, h.P, h.N);
    S.Pi = W.Pi;
    S.R = W.R;
    S.Et = W.Et;
}

cb_status share_forces(int prec, int64_t n, const double* x, const double* y, const double* z, const double* q,
                       const double* m, const TrapK& k, double eps2, unsigned mode, double* fx, double* fy, double* fz,
                       double* u_out, void* ws, hipStream_t st) {
    const bool pot = u_out != nullptr;
    const ShareWs W = share_carve(n, pot, ws);
    ShareStep S{};
    share_use(S, n, pot, W);
    S.eblk = W.eblk[0];
    S.x = const_cast<double*>(x);  // read only in these modes
    S.y = const_cast<double*>(y);
    S.z = const_cast<double*>(z);
    S.q = q;
    S.m = m;
    S.k = k;
    S.fx = fx; S.fy = fy; S.fz = fz;
    S.mode = mode | (u_out ? EPI_ENERGY | EPI_UPOT : 0u);
    S.flags = flags_ptr();
    if (!S.flags) return fail(CB_EHIP, "share_forces: device flag symbol not found");
    cb_status rc = share_pairs(prec, n, x, y, z, q, eps2, pot, W, st);
    if (rc || (rc = share_finish(S, st)) || !u_out) return rc;
    k_energy_record<kFinWaves><<<1, 64 * kFinWaves, 0, st>>>((int)((n + 63) / 64), S.eblk, u_out, REC_UPOT);
    return check_launch("k_energy_record");
}

cb_status md_run_shares(int64_t n, const cb_state* s, const double* q, const double* m, const cb_trap* trap, double t0,
                        double dt, int64_t nsteps, double eps2, int32_t prec, uint32_t flags, double* energies,
                        int64_t every, void* ws, hipStream_t st) {
    const ShareWs W[2] = {share_carve(n, false, ws), share_carve(n, true, ws)};  // a plain step's, a record's
    ShareStep S{};
    S.x = S.xn = s->x;
    S.y = S.yn = s->y;
    S.z = S.zn = s->z;
    S.vx = s->vx; S.vy = s->vy; S.vz = s->vz;
    S.ax = s->ax; S.ay = s->ay; S.az = s->az;
    S.q = q;
    S.m = m;
    S.gamma = trap->gamma;
    S.dt = dt;
    S.flags = flags_ptr();
    if (!S.flags) return fail(CB_EHIP, "md_run: device flag symbol not found");
    const int nb = (int)((n + 63) / 64);
    int parity = 0;
    auto step = [&](int64_t k, unsigned mode, double* rec) -> cb_status {
        cb_status r;
        if ((mode & (EPI_ACCEL | EPI_KICK | EPI_ENERGY)) &&
            (r = share_pairs(prec, n, s->x, s->y, s->z, q, eps2, rec != nullptr, W[rec != nullptr], st)))
            return r;
        share_use(S, n, rec != nullptr, W[rec != nullptr]);
        S.k = trap_k(*trap, t0 + (double)k * dt);
        S.mode = mode;
        S.eblk = W[0].eblk[parity];
        if ((r = share_finish(S, st))) return r;
        // a record's sums are added by the next finish launch
        S.eprev = rec ? W[0].eblk[parity] : nullptr;
        S.eprev_out = rec;
        S.nprev = nb;
        if (rec) parity ^= 1;
        return CB_OK;
    };
    const bool rec0 = energies != nullptr;
    const bool init = (flags & CB_INIT_ACCEL) != 0;
    const unsigned mode0 = (init ? EPI_ACCEL : 0u) | (rec0 ? EPI_ENERGY : 0u) | (nsteps > 0 ? EPI_DRIFT : 0u);
    cb_status rc;
    if (mode0 && (rc = step(0, mode0, rec0 ? energies : nullptr))) return rc;
    for (int64_t k = 1; k <= nsteps; ++k) {
        const bool rec = rec0 && k % every == 0;
        if ((rc = step(k, EPI_KICK | (rec ? EPI_ENERGY : 0u) | (k < nsteps ? EPI_DRIFT : 0u),
                       rec ? energies + 4 * (k / every) : nullptr)))
            return rc;
    }
    if (S.eprev) {
        k_energy_record<kFinWaves><<<1, 64 * kFinWaves, 0, st>>>(nb, S.eprev, S.eprev_out, REC_ALL);
        if ((rc = check_launch("k_energy_record"))) return rc;
    }
    return ok();
}

// ------------------------------------------------------------- ensembles
constexpr int kEnsP = 4;  // ions per lane
// Shares, in two rounds of the 1024 workgroups that fit at once (us per step
// with 1024 / 2048 / 4096: 16 runs of 2048-4096 ions 81.8 / 79.6 / 87.2, 512 of
// 64-1024 128.6 / 124.8 / 125.8, 256 of 64-2048 188 / 183 / 182; a share per
// wave instead of per workgroup, 4096 and 8192: 89 / 90, 135 / 132, 192 / 190;
// 2 ions per lane and 1024 workgroups 86, 128, 200).
constexpr int kEnsShares = 2048;
constexpr size_t kEnsFinishFew = 4096;  // up to here 8 waves finish 64 ions, above 2

struct ShareEns {
    std::vector<int4> runs;    // k_share_pairs_ens'
    std::vector<int2> first, chunks, recs;
    ShareCut all{};
    size_t rows = 0, bytes = 0;
};

// Whether nrun runs can take equal shares, and their tables.
static bool share_ens(int32_t nrun, const int64_t* offsets, ShareEns& E) {
    if (share_ens_units(nrun, offsets) > 1e9) return false;  // (unit numbers are 32 bits)
    E.runs.resize(nrun);
    E.recs.resize(nrun);
    int u = 0;
    for (int r = 0; r < nrun; ++r) {
        const int n = (int)(offsets[r + 1] - offsets[r]);
        const ShareCut c = share_rows(n, kEnsP);
        E.runs[r] = make_int4((int)offsets[r], n, (int)E.rows, u);
        E.recs[r] = make_int2((int)E.chunks.size(), (n + 63) / 64);
        for (int k0 = 0; k0 < n; k0 += 64) E.chunks.push_back(make_int2(r, k0));
        E.rows += (size_t)c.nI;
        u += c.U;
    }
    E.all.IB = 64 * kEnsP;
    share_units(E.all, u, kEnsShares);
    E.first.reserve((size_t)E.all.N);
    int r = 0, I = 0;
    ShareCut c = share_rows(E.runs[0].y, kEnsP);
    for (int g = 0; g < E.all.N; ++g) {
        const int at = share_unit(E.all, g);
        while (at >= E.runs[r].w + c.U) {
            c = share_rows(E.runs[++r].y, kEnsP);
            I = 0;
        }
        while (at >= E.runs[r].w + row_unit(c, I) + row_units(c, I)) ++I;
        E.first.push_back(make_int2(r, I));
    }
    const size_t slots = (size_t)E.all.N + E.rows, nch = E.chunks.size();
    E.bytes = al(sizeof(int4) * nrun) + al(sizeof(int2) * E.first.size()) + al(sizeof(int2) * nch) +
              al(sizeof(int2) * nrun) + al(sizeof(cb_trap) * nrun) + al(sizeof(double) * 3 * slots * 64 * kEnsP) +
              al(sizeof(double) * 3 * (size_t)u * kShareJ) + al(sizeof(double) * slots) + al(sizeof(double) * 3 * nch);
    return true;
}

double share_ens_units(int32_t nrun, const int64_t* offsets) {
    double units = 0.0;
    for (int r = 0; r < nrun; ++r) units += share_rows((int)(offsets[r + 1] - offsets[r]), kEnsP).U;
    return units;
}

template <int PREC>
static void go_share_ens(bool pot, const ShareEns& E, const int4* runs, const int2* first, const cb_state* s,
                         const double* q, double eps2, double* Pi, double* R, double* Et, hipStream_t st) {
    const unsigned g = (unsigned)E.all.N;
    if (pot)
        k_share_pairs_ens<PREC, kEnsP, true><<<g, 64 * kShareWaves, 0, st>>>(E.all, runs, first, s->x, s->y, s->z, q, eps2, Pi, R, Et);
    else
        k_share_pairs_ens<PREC, kEnsP, false><<<g, 64 * kShareWaves, 0, st>>>(E.all, runs, first, s->x, s->y, s->z, q, eps2, Pi, R, Et);
}

template <int FW>
static void go_finish_ens(const ShareStep& S, unsigned g, const int4* runs, const int2* chunks, const cb_trap* traps,
                          double t0, long long step, hipStream_t st) {
    if (S.mode & EPI_ENERGY) k_share_finish_ens<true, FW><<<g, 64 * FW, 0, st>>>(S, runs, chunks, traps, t0, step);
    else k_share_finish_ens<false, FW><<<g, 64 * FW, 0, st>>>(S, runs, chunks, traps, t0, step);
}

cb_status md_run_shares_ensemble(int32_t nrun, const int64_t* offsets, const cb_state* s, const double* q,
                                 const double* m, const cb_trap* traps, double t0, double dt, int64_t nsteps,
                                 double eps2, int32_t prec, uint32_t flags, double* energies, int64_t every, void* ws,
                                 size_t ws_bytes, bool* taken, hipStream_t st) {
    ShareEns E;
    *taken = share_ens(nrun, offsets, E) && E.bytes <= ws_bytes;
    if (!*taken) return CB_OK;
    const size_t slots = (size_t)E.all.N + E.rows, nch = E.chunks.size();
    char* base = static_cast<char*>(ws);
    auto carve = [&](size_t bytes) {
        char* p = base;
        base += al(bytes);
        return p;
    };
    int4* d_runs = reinterpret_cast<int4*>(carve(sizeof(int4) * nrun));
    int2* d_first = reinterpret_cast<int2*>(carve(sizeof(int2) * E.first.size()));
    int2* d_chunks = reinterpret_cast<int2*>(carve(sizeof(int2) * nch));
    int2* d_recs = reinterpret_cast<int2*>(carve(sizeof(int2) * nrun));
    cb_trap* d_traps = reinterpret_cast<cb_trap*>(carve(sizeof(cb_trap) * nrun));
    double* Pi = reinterpret_cast<double*>(carve(sizeof(double) * 3 * slots * 64 * kEnsP));
    double* R = reinterpret_cast<double*>(carve(sizeof(double) * 3 * (size_t)E.all.U * kShareJ));
    double* Et = reinterpret_cast<double*>(carve(sizeof(double) * slots));
    double* eblk = reinterpret_cast<double*>(carve(sizeof(double) * 3 * nch));
    HostUpload up;
    up.add(d_runs, E.runs.data(), sizeof(int4) * nrun);
    up.add(d_first, E.first.data(), sizeof(int2) * E.first.size());
    up.add(d_chunks, E.chunks.data(), sizeof(int2) * nch);
    up.add(d_recs, E.recs.data(), sizeof(int2) * nrun);
    up.add(d_traps, traps, sizeof(cb_trap) * nrun);
    if (cb_status urc = up.run(st, "md_run")) return urc;
    ShareStep S{};
    S.cut = E.all;
    S.Pi = Pi;
    S.R = R;
    S.Et = Et;
    S.x = S.xn = s->x;
    S.y = S.yn = s->y;
    S.z = S.zn = s->z;
    S.vx = s->vx; S.vy = s->vy; S.vz = s->vz;
    S.ax = s->ax; S.ay = s->ay; S.az = s->az;
    S.q = q;
    S.m = m;
    S.dt = dt;
    S.eblk = eblk;
    S.flags = flags_ptr();
    if (!S.flags) return fail(CB_EHIP, "md_run: device flag symbol not found");
    const long long nrec = energies ? nsteps / every + 1 : 0;
    auto step = [&](int64_t k, unsigned mode, int64_t rec) -> cb_status {
        cb_status r;
        const bool pot = rec >= 0;
        if (mode & (EPI_ACCEL | EPI_KICK | EPI_ENERGY)) {
            switch (prec) {
                case CB_FP64: go_share_ens<PREC_FP64>(pot, E, d_runs, d_first, s, q, eps2, Pi, R, Et, st); break;
                case CB_MIXED: go_share_ens<PREC_MIXED>(pot, E, d_runs, d_first, s, q, eps2, Pi, R, Et, st); break;
                case CB_FP64_IEEE: go_share_ens<PREC_IEEE>(pot, E, d_runs, d_first, s, q, eps2, Pi, R, Et, st); break;
                default: go_share_ens<PREC_FP32>(pot, E, d_runs, d_first, s, q, eps2, Pi, R, Et, st); break;
            }
            if ((r = check_launch("k_share_pairs_ens"))) return r;
        }
        S.mode = mode;
        if (nch < kEnsFinishFew) go_finish_ens<8>(S, (unsigned)nch, d_runs, d_chunks, d_traps, t0, k, st);
        else go_finish_ens<2>(S, (unsigned)nch, d_runs, d_chunks, d_traps, t0, k, st);
        if ((r = check_launch("k_share_finish_ens")) || rec < 0) return r;
        k_ens_record<4><<<nrun, 256, 0, st>>>(d_recs, eblk, nrec, rec, energies);
        return check_launch("k_ens_record");
    };
    const unsigned mode0 = ((flags & CB_INIT_ACCEL) ? EPI_ACCEL : 0u) | (energies ? EPI_ENERGY : 0u) |
                           (nsteps > 0 ? EPI_DRIFT : 0u);
    cb_status rc;
    if (mode0 && (rc = step(0, mode0, energies ? 0 : -1))) return rc;
    for (int64_t k = 1; k <= nsteps; ++k) {
        const bool rec = energies && k % every == 0;
        if ((rc = step(k, EPI_KICK | (rec ? EPI_ENERGY : 0u) | (k < nsteps ? EPI_DRIFT : 0u), rec ? k / every : -1)))
            return rc;
    }
    return ok();
}

}  // namespace cb
