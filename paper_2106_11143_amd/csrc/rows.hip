// One launch per velocity-Verlet step of a small run (rows.hpp), and the host
// loop that runs md_step / md_run on it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <numeric>
#include <vector>

#include "energy_record.hpp"
#include "internal.hpp"
#include "rows.hpp"
#include "step_ion.hpp"

namespace cb {

struct RowParams {
    int n;
    const double *x, *y, *z;  // positions at this step (read)
    const double *q, *m;
    double *xn, *yn, *zn;     // positions after the drift (written; not x, y, z when other ions' are read)
    double *vx, *vy, *vz, *ax, *ay, *az;
    TrapK k;                  // the trap's spring constants at this step
    double gamma, dt, eps2;
    unsigned mode;            // EPI_ACCEL, EPI_KICK, EPI_DRIFT, EPI_ENERGY
    double* eblk;             // [gridDim.x][3] energy sums of the workgroups (EPI_ENERGY)
    // An earlier record's workgroup sums, added in order by one extra
    // workgroup of this launch into eprev_out (K, U_C, U_trap, E).
    const double* eprev;
    double* eprev_out;
    int nprev;
    unsigned* flags;
};

// The workgroup's energy sums (the I ions' terms in its first I threads) to
// eblk[blockIdx.x].
template <int I>
__device__ __forceinline__ void rows_energy(double eK, double eC, double eT, double* __restrict__ eblk) {
    if (threadIdx.x >= 64) return;
#pragma unroll
    for (int d = I / 2; d > 0; d >>= 1) {
        eK += __shfl_xor(eK, d);
        eC += __shfl_xor(eC, d);
        eT += __shfl_xor(eT, d);
    }
    if (threadIdx.x == 0) {
        eblk[(size_t)blockIdx.x * 3 + 0] = eK;
        eblk[(size_t)blockIdx.x * 3 + 1] = eC;
        eblk[(size_t)blockIdx.x * 3 + 2] = eT;
    }
}

// One step of the run: I ions per workgroup of W waves.  POT: a recording
// step.
template <int PREC, int I, int W, bool POT>
__device__ __forceinline__ void rows_step_block(const RowParams& P) {
    __shared__ __align__(16) RowsLds<I, W, POT> lds;
    const int i0 = blockIdx.x * I, k = i0 + (int)threadIdx.x;
    const bool own = threadIdx.x < I && k < P.n;
    // with 4 ions the ions' state is requested before the pairs; with 8 the
    // registers are worth more as waves in flight
    constexpr bool kAhead = I == 4;
    IonState s{};
    double x = 0.0, y = 0.0, z = 0.0, qk = 0.0;
    auto load = [&] {
        s = load_ion(P, k);
        x = P.x[k];
        y = P.y[k];
        z = P.z[k];
        qk = P.q[k];
    };
    if (kAhead && own) load();
    double o[4] = {0.0, 0.0, 0.0, 0.0};
    if (P.mode & (EPI_ACCEL | EPI_KICK | EPI_ENERGY))
        rows_sums<PREC, I, W, POT>(P.n, P.x, P.y, P.z, P.q, i0, P.eps2, lds, o);
    double eK = 0.0, eC = 0.0, eT = 0.0;
    if (own) {
        if (!kAhead) load();
        const double c = kCoulomb * qk;
        step_ion(P, P.k, P.gamma, k, s, x, y, z, qk, c * o[0], c * o[1], c * o[2], POT ? o[3] : 0.0, eK, eC, eT);
    }
    if (POT) rows_energy<I>(eK, eC, eT, P.eblk);
}

template <int PREC, int I, int W, bool POT>
__global__ void __launch_bounds__(64 * W, (rows_waves<PREC, I, POT>())) k_rows_step(RowParams P) {
    if (!P.eprev || blockIdx.x != gridDim.x - 1)
        rows_step_block<PREC, I, W, POT>(P);
    else
        energy_record<W>(P.nprev, P.eprev, P.eprev_out, REC_ALL);
}

// ------------------------------------------------- forces, gradient, energy
struct RowForceParams {
    int n;
    const double *x, *y, *z, *q;
    const double* m;  // NULL: no trap term
    TrapK k;
    double eps2;
    unsigned mode;          // EPI_FORCES or EPI_GRAD (outputs fx, fy, fz), EPI_ENERGY (U_C and U_trap sums)
    double *fx, *fy, *fz;
    double* eblk;           // [gridDim.x][3]
    unsigned* flags;
};

template <int PREC, int I, int W, bool POT>
__global__ void __launch_bounds__(64 * W, (rows_waves<PREC, I, POT>())) k_rows_forces(RowForceParams P) {
    __shared__ __align__(16) RowsLds<I, W, POT> lds;
    const int i0 = blockIdx.x * I, k = i0 + (int)threadIdx.x;
    double o[4] = {0.0, 0.0, 0.0, 0.0};
    rows_sums<PREC, I, W, POT>(P.n, P.x, P.y, P.z, P.q, i0, P.eps2, lds, o);
    double eK = 0.0, eC = 0.0, eT = 0.0;
    if (threadIdx.x < I && k < P.n) {
        const double c = kCoulomb * P.q[k];
        const double Fx = c * o[0], Fy = c * o[1], Fz = c * o[2];
        bool ok = true;
        if (P.mode & EPI_FORCES) {
            P.fx[k] = Fx;
            P.fy[k] = Fy;
            P.fz[k] = Fz;
            ok = finite3(Fx, Fy, Fz);
        } else {
            double x = 0.0, y = 0.0, z = 0.0, mk = 0.0;
            if (P.m) {
                x = P.x[k];
                y = P.y[k];
                z = P.z[k];
                mk = P.m[k];
            }
            if (P.mode & EPI_GRAD) {
                const double gx = __builtin_fma(mk * P.k.kx, x, -Fx);
                const double gy = __builtin_fma(mk * P.k.ky, y, -Fy);
                const double gz = __builtin_fma(mk * P.k.kz, z, -Fz);
                P.fx[k] = gx;
                P.fy[k] = gy;
                P.fz[k] = gz;
                ok = finite3(gx, gy, gz);
            }
            if (POT) {
                eC = 0.5 * c * o[3];
                eT = 0.5 * mk * (P.k.kx * x * x + P.k.ky * y * y + P.k.kz * z * z);
                ok = ok && __builtin_isfinite(eC) && __builtin_isfinite(eT);
            }
        }
        if (!ok) atomicOr(P.flags, 1u);
    }
    if (POT) rows_energy<I>(eK, eC, eT, P.eblk);
}

// --------------------------------------------------------------- ensembles
struct RowEnsParams {
    const int4* chunks;    // [gridDim.x] (run's first ion, run's ions, chunk's first ion within the run, run)
    const cb_trap* traps;  // [nrun]
    const double *x, *y, *z;
    const double *q, *m;
    double *xn, *yn, *zn;
    double *vx, *vy, *vz, *ax, *ay, *az;
    double t0, dt, eps2;
    long long step;
    unsigned mode;
    double* eblk;  // [chunks][3]
    unsigned* flags;
};

// One step of every run: a workgroup takes I ions of one run against the
// run's ions.
template <int PREC, int I, int W, bool POT>
__global__ void __launch_bounds__(64 * W, (rows_waves<PREC, I, POT>())) k_rows_ens(RowEnsParams P) {
    __shared__ __align__(16) RowsLds<I, W, POT> lds;
    const int4 ch = P.chunks[blockIdx.x];
    const int o = ch.x, n = ch.y, i0 = ch.z, kl = i0 + (int)threadIdx.x, k = o + kl;
    const bool own = threadIdx.x < I && kl < n;
    double f[4] = {0.0, 0.0, 0.0, 0.0};
    if (P.mode & (EPI_ACCEL | EPI_KICK | EPI_ENERGY))
        rows_sums<PREC, I, W, POT>(n, P.x + o, P.y + o, P.z + o, P.q + o, i0, P.eps2, lds, f);
    double eK = 0.0, eC = 0.0, eT = 0.0;
    if (own) {
        const cb_trap& tr = P.traps[ch.w];
        const double qk = P.q[k], c = kCoulomb * qk;
        step_ion(P, trap_k(tr, step_time(P.t0, P.dt, P.step)), tr.gamma, k, load_ion(P, k), P.x[k], P.y[k], P.z[k], qk,
                 c * f[0], c * f[1], c * f[2], POT ? f[3] : 0.0, eK, eC, eT);
    }
    if (POT) rows_energy<I>(eK, eC, eT, P.eblk);
}

// ----------------------------------------------------------------- host

static size_t al(size_t b) { return (b + 255) / 256 * 256; }

// The launches of a run of nsteps steps.  launch(step, mode, record, swap)
// enqueues one: `record` is the index of the energy record it makes (-1:
// none), and its drift lands in the other position buffer when `swap`
// (always when it reads other ions' positions), else in place.  The drifts
// of steps 1 .. nsteps - 1 swap the buffers; the first drift is placed so
// that the last one lands in the caller's arrays (a launch of its own when
// it would have to swap and must not).
template <class Launch>
static cb_status rows_steps(int64_t nsteps, bool init, bool records, int64_t every, Launch launch) {
    const unsigned read0 = (init ? EPI_ACCEL : 0u) | (records ? EPI_ENERGY : 0u);
    const bool odd = nsteps > 0 && (nsteps - 1) % 2 == 1;
    const int64_t rec0 = records ? 0 : -1;
    cb_status rc;
    if (read0 && odd) {
        if ((rc = launch((int64_t)0, read0 | EPI_DRIFT, rec0, true))) return rc;
    } else {
        if (read0 && (rc = launch((int64_t)0, read0, rec0, false))) return rc;
        if (nsteps > 0 && (rc = launch((int64_t)0, (unsigned)EPI_DRIFT, (int64_t)-1, odd))) return rc;
    }
    for (int64_t k = 1; k <= nsteps; ++k) {
        const bool rec = records && k % every == 0;
        const unsigned drift = k < nsteps ? EPI_DRIFT : 0u;
        if ((rc = launch(k, EPI_KICK | drift | (rec ? EPI_ENERGY : 0u), rec ? k / every : (int64_t)-1, drift != 0)))
            return rc;
    }
    return CB_OK;
}

// Shape of the single run's launch.
static bool rows_small(int64_t n) { return n <= kRowsSmallN; }
static int rows_blocks(int64_t n) {
    const int I = rows_small(n) ? 4 : 8;
    return (int)((n + I - 1) / I);
}

size_t md_rows_ws_bytes(int64_t n) {
    return al(sizeof(double) * 3 * (size_t)n) + 2 * al(sizeof(double) * 3 * (size_t)rows_blocks(n));
}

template <int PREC, int I, int W>
static void go_rows(const RowParams& P, unsigned g, hipStream_t st) {
    if (P.mode & EPI_ENERGY)
        k_rows_step<PREC, I, W, true><<<g, 64 * W, 0, st>>>(P);
    else
        k_rows_step<PREC, I, W, false><<<g, 64 * W, 0, st>>>(P);
}

template <int PREC>
static void go_rows_shape(const RowParams& P, unsigned g, hipStream_t st) {
    if (rows_small(P.n)) go_rows<PREC, 4, 8>(P, g, st);
    else go_rows<PREC, 8, 4>(P, g, st);
}

cb_status md_run_rows(int64_t n, const cb_state* s, const double* q, const double* m, const cb_trap* trap, double t0,
                      double dt, int64_t nsteps, double eps2, int32_t prec, uint32_t flags, double* energies,
                      int64_t every, void* ws, size_t ws_bytes, int spins, hipStream_t st) {
    if (ws_bytes < md_rows_ws_bytes(n)) return fail(CB_ENOWS, "md_run: workspace too small for the one-launch step");
    unsigned* fl = flags_ptr();
    if (!fl) return fail(CB_EHIP, "md_run: device flag symbol not found");
    char* base = static_cast<char*>(ws);
    double* pos2 = reinterpret_cast<double*>(base);
    base += al(sizeof(double) * 3 * (size_t)n);
    const int nb = rows_blocks(n);
    double* ebuf[2] = {reinterpret_cast<double*>(base),
                       reinterpret_cast<double*>(base + al(sizeof(double) * 3 * (size_t)nb))};
    double* bufA[3] = {s->x, s->y, s->z};
    double* bufB[3] = {pos2, pos2 + n, pos2 + 2 * n};
    double** cur = bufA;
    double** nxt = bufB;
    RowParams P{};
    P.n = (int)n;
    P.q = q;
    P.m = m;
    P.vx = s->vx; P.vy = s->vy; P.vz = s->vz;
    P.ax = s->ax; P.ay = s->ay; P.az = s->az;
    P.gamma = trap->gamma;
    P.dt = dt;
    P.eps2 = eps2;
    P.flags = fl;
    // the workgroups' energy sums of a record alternate between two buffers:
    // the next launch adds them
    const double* pend = nullptr;
    double* pend_out = nullptr;
    int parity = 0;
    auto launch = [&](int64_t step, unsigned mode, int64_t rec, bool swap) -> cb_status {
        double** out = swap ? nxt : cur;
        P.x = cur[0]; P.y = cur[1]; P.z = cur[2];
        P.xn = out[0]; P.yn = out[1]; P.zn = out[2];
        P.k = trap_k(*trap, t0 + (double)step * dt);
        P.mode = mode;
        P.eblk = ebuf[parity];
        P.eprev = pend;
        P.eprev_out = pend_out;
        P.nprev = nb;
        const unsigned g = (unsigned)(nb + (pend ? 1 : 0));
        switch (prec) {
            case CB_FP64: go_rows_shape<PREC_FP64>(P, g, st); break;
            case CB_MIXED: go_rows_shape<PREC_MIXED>(P, g, st); break;
            case CB_FP64_IEEE: go_rows_shape<PREC_IEEE>(P, g, st); break;
            default: go_rows_shape<PREC_FP32>(P, g, st); break;
        }
        const cb_status r = check_launch("k_rows_step");
        if (r) return r;
        pend = rec >= 0 ? ebuf[parity] : nullptr;
        pend_out = rec >= 0 ? energies + 4 * rec : nullptr;
        if (rec >= 0) parity ^= 1;
        if (swap) std::swap(cur, nxt);
        return CB_OK;
    };
    const bool init = (flags & CB_INIT_ACCEL) != 0;
    const bool resident = rows_run_fits(n, nsteps, ws_bytes);
    cb_status rc = rows_steps(resident ? 0 : nsteps, init, energies != nullptr, every, launch);
    if (rc) return rc;
    if (pend) {  // the last record, in the order of the launches' extra workgroups
        if (rows_small(n)) k_energy_record<8><<<1, 512, 0, st>>>(nb, pend, pend_out, REC_ALL);
        else k_energy_record<4><<<1, 256, 0, st>>>(nb, pend, pend_out, REC_ALL);
        if ((rc = check_launch("k_energy_record"))) return rc;
    }
    if (resident && (rc = rows_run(n, s, q, m, trap, t0, dt, nsteps, eps2, prec, energies, every, spins, ws, st)))
        return rc;
    return ok();
}

template <int PREC, int I, int W>
static void go_rows_forces(const RowForceParams& P, unsigned g, hipStream_t st) {
    if (P.mode & EPI_ENERGY)
        k_rows_forces<PREC, I, W, true><<<g, 64 * W, 0, st>>>(P);
    else
        k_rows_forces<PREC, I, W, false><<<g, 64 * W, 0, st>>>(P);
}

template <int PREC>
static void go_rows_forces_shape(const RowForceParams& P, unsigned g, hipStream_t st) {
    if (rows_small(P.n)) go_rows_forces<PREC, 4, 8>(P, g, st);
    else go_rows_forces<PREC, 8, 4>(P, g, st);
}

cb_status rows_forces(int prec, int64_t n, const double* x, const double* y, const double* z, const double* q,
                      const double* m, const TrapK& k, double eps2, unsigned mode, double* fx, double* fy, double* fz,
                      double* u_out, void* ws, hipStream_t st) {
    RowForceParams P{};
    P.n = (int)n;
    P.x = x; P.y = y; P.z = z;
    P.q = q;
    P.m = m;
    P.k = k;
    P.eps2 = eps2;
    P.mode = mode | (u_out ? EPI_ENERGY : 0u);
    P.fx = fx; P.fy = fy; P.fz = fz;
    P.eblk = static_cast<double*>(ws);
    P.flags = flags_ptr();
    if (!P.flags) return fail(CB_EHIP, "rows_forces: device flag symbol not found");
    const int nb = rows_blocks(n);
    switch (prec) {
        case CB_FP64: go_rows_forces_shape<PREC_FP64>(P, (unsigned)nb, st); break;
        case CB_MIXED: go_rows_forces_shape<PREC_MIXED>(P, (unsigned)nb, st); break;
        case CB_FP64_IEEE: go_rows_forces_shape<PREC_IEEE>(P, (unsigned)nb, st); break;
        default: go_rows_forces_shape<PREC_FP32>(P, (unsigned)nb, st); break;
    }
    cb_status rc = check_launch("k_rows_forces");
    if (rc || !u_out) return rc;
    k_energy_record<4><<<1, 256, 0, st>>>(nb, P.eblk, u_out, REC_UPOT);
    return check_launch("k_energy_record");
}

// Ions per workgroup of an ensemble's launch.
constexpr int kEnsI = 8;

template <int PREC, int W>
static void go_rows_ens(const RowEnsParams& P, unsigned g, hipStream_t st) {
    if (P.mode & EPI_ENERGY)
        k_rows_ens<PREC, kEnsI, W, true><<<g, 64 * W, 0, st>>>(P);
    else
        k_rows_ens<PREC, kEnsI, W, false><<<g, 64 * W, 0, st>>>(P);
}

// One wave per chunk where the chunks alone fill the chip's 1024 SIMDs, four
// below (us per step on MI355X, W = 1 / 2 / 4: 64 runs of 64-1024 ions, 4360
// chunks, 26.3 / 27.0 / 28.3; 512 of 64-512 57.2 / 61.6 / 73.1; 8 of 64-600,
// 340 chunks, 7.4 / 6.8 / 6.3; 4 of 30-100 5.2 / 4.9 / 4.8).
template <int PREC>
static void go_rows_ens_shape(const RowEnsParams& P, unsigned g, hipStream_t st) {
    if (g < 1024) go_rows_ens<PREC, 4>(P, g, st);
    else go_rows_ens<PREC, 1>(P, g, st);
}

cb_status md_run_rows_ensemble(int32_t nrun, const int64_t* offsets, const cb_state* s, const double* q,
                               const double* m, const cb_trap* traps, double t0, double dt, int64_t nsteps,
                               double eps2, int32_t prec, uint32_t flags, double* energies, int64_t every, void* ws,
                               size_t ws_bytes, hipStream_t st) {
    const size_t ntot = (size_t)offsets[nrun];
    // chunks of the largest runs first, so that the short ones fill the end
    // of the launch
    std::vector<int> order(nrun);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(),
                     [&](int a, int b) { return offsets[a + 1] - offsets[a] > offsets[b + 1] - offsets[b]; });
    std::vector<int2> runs(nrun);
    std::vector<int4> chunks;
    chunks.reserve(ntot / kEnsI + (size_t)nrun);
    for (int r : order) {
        const int o = (int)offsets[r], n = (int)(offsets[r + 1] - offsets[r]);
        const int c0 = (int)chunks.size();
        for (int i0 = 0; i0 < n; i0 += kEnsI) chunks.push_back(make_int4(o, n, i0, r));
        runs[r] = make_int2(c0, (int)chunks.size() - c0);
    }
    const size_t nch = chunks.size();
    const size_t need = al(sizeof(int4) * nch) + al(sizeof(int2) * nrun) + al(sizeof(cb_trap) * nrun) +
                        al(sizeof(double) * 3 * ntot) + al(sizeof(double) * 3 * nch);
    if (ws_bytes < need)
        return fail(CB_ENOWS, "md_run: the ensemble path needs %zu workspace bytes, has %zu", need, ws_bytes);
    unsigned* fl = flags_ptr();
    if (!fl) return fail(CB_EHIP, "md_run: device flag symbol not found");
    char* base = static_cast<char*>(ws);
    auto carve = [&](size_t bytes) {
        char* p = base;
        base += al(bytes);
        return p;
    };
    int4* d_chunks = reinterpret_cast<int4*>(carve(sizeof(int4) * nch));
    int2* d_runs = reinterpret_cast<int2*>(carve(sizeof(int2) * nrun));
    cb_trap* d_traps = reinterpret_cast<cb_trap*>(carve(sizeof(cb_trap) * nrun));
    double* pos2 = reinterpret_cast<double*>(carve(sizeof(double) * 3 * ntot));
    double* eblk = reinterpret_cast<double*>(carve(sizeof(double) * 3 * nch));
    HostUpload up;
    up.add(d_chunks, chunks.data(), sizeof(int4) * nch);
    up.add(d_runs, runs.data(), sizeof(int2) * nrun);
    up.add(d_traps, traps, sizeof(cb_trap) * nrun);
    if (cb_status urc = up.run(st, "md_run")) return urc;
    double* bufA[3] = {s->x, s->y, s->z};
    double* bufB[3] = {pos2, pos2 + ntot, pos2 + 2 * ntot};
    double** cur = bufA;
    double** nxt = bufB;
    RowEnsParams P{};
    P.chunks = d_chunks;
    P.traps = d_traps;
    P.q = q;
    P.m = m;
    P.vx = s->vx; P.vy = s->vy; P.vz = s->vz;
    P.ax = s->ax; P.ay = s->ay; P.az = s->az;
    P.t0 = t0;
    P.dt = dt;
    P.eps2 = eps2;
    P.eblk = eblk;
    P.flags = fl;
    const long long nrec = energies ? nsteps / every + 1 : 0;
    auto launch = [&](int64_t step, unsigned mode, int64_t rec, bool swap) -> cb_status {
        double** out = swap ? nxt : cur;
        P.x = cur[0]; P.y = cur[1]; P.z = cur[2];
        P.xn = out[0]; P.yn = out[1]; P.zn = out[2];
        P.step = step;
        P.mode = mode;
        const unsigned g = (unsigned)nch;
        switch (prec) {
            case CB_FP64: go_rows_ens_shape<PREC_FP64>(P, g, st); break;
            case CB_MIXED: go_rows_ens_shape<PREC_MIXED>(P, g, st); break;
            case CB_FP64_IEEE: go_rows_ens_shape<PREC_IEEE>(P, g, st); break;
            default: go_rows_ens_shape<PREC_FP32>(P, g, st); break;
        }
        cb_status r = check_launch("k_rows_ens");
        if (r) return r;
        if (swap) std::swap(cur, nxt);
        if (rec < 0) return CB_OK;
        k_ens_record<4><<<nrun, 256, 0, st>>>(d_runs, eblk, nrec, rec, energies);
        return check_launch("k_ens_record");
    };
    const cb_status rc = rows_steps(nsteps, (flags & CB_INIT_ACCEL) != 0, energies != nullptr, every, launch);
    return rc ? rc : ok();
}

}  // namespace cb
