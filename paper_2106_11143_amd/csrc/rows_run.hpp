// Many velocity-Verlet steps of a small run in one launch (device code).
//
// A step of some hundred ions is little work (1024 ions: 0.6 us of the chip's
// FP64 rate), and one launch per step (rows.hpp) spends most of its 4-5 us on
// the launch and on reading every ion's position and state afresh.  Here the
// workgroups stay: each keeps the state of its 4 ions, publishes their
// drifted positions and polls for the others', lanes holding the j's that
// they polled.  What bounds a step is a chain: a position's way through the
// memory that the dies share (0.45 us), the pairs, their sums and the update.
// The sums go across lanes and the update takes one component per lane for
// this chain's sake (150 ions 2.3 -> 1.9 us per step).
// us per step on MI355X, one launch per step / this (with a record at every
// step): 16 ions 3.8 / 1.6 (2.2), 150 3.8 / 1.8 (2.3), 512 4.2 / 2.1 (2.7),
// 1024 4.9 / 2.9 (3.6), 1200 6.1 / 4.4 (5.2), 1536 6.9 / 6.0.
//
// Positions travel without fences or counters: a word of `pub` holds either a
// bit pattern that no position has (a signalling NaN, which no arithmetic
// returns) or the position, so it says itself whether it has arrived.  Words
// are written and read by relaxed agent-scope atomics, past the L2s of the
// chip's eight dies.  pub is a ring of kRunRing steps: a workgroup that has
// read all of step s knows that every other has published it, and so has read
// all of step s - 1, whose own words it marks as not yet written; those words
// are written again kRunRing - 1 steps later, and its polls in between have
// waited for the mark.
//
// Workgroups that wait for each other have to be resident together.  A launch
// ahead of the run's admits it: the waves of the runs between their first
// launch and their last are counted on the device, and a run waits until its
// own fit beside them, with room for the uneven ways in which the CUs fill.
// Other kernels end by themselves, so an admitted run's workgroups all get
// their places.  What this does not see (another process's runs, a captured
// graph's launches between another stream's) is caught by a bound on every
// wait: a workgroup whose wait runs out raises `abort`, on which all of them
// end.  Nothing of the caller's is written meanwhile: k_rows_run_end commits
// the results, or if `abort` is up takes the same steps itself, in an order
// that needs no workgroup but those that have a place.  Its workgroups take the
// groups of four ions of step after step by a running number (a ticket) and
// wait for the steps before their own alone, whose tickets were taken earlier,
// by workgroups that run: the lowest ticket not yet done never waits, so every
// wait ends, with any number of them on the chip (us per step of a run that
// gave up, by one workgroup / so / a launch per step: 150 ions 56 / 4.7 / 5.9,
// 1024 603 / 8.7 / 6.0, 1280 815 / 12.1 / 6.9).
#pragma once
#include <hip/hip_runtime.h>

#include "rows.hpp"
#include "step_ion.hpp"

namespace cb {

constexpr int kRunSteps = 128;  // steps per launch: its kernel arguments hold their trap's spring constants
constexpr int kRunRing = 8;
constexpr int kTaken = 16, kDone = 32;  // (words, each in a line of its own)
constexpr unsigned long long kUnset = 0x7ff4'5a5a'7ff4'5a5aull;

struct RowRunParams {
    int n, nk;                 // ions, steps
    const double *q, *m;
    double *x, *y, *z, *vx, *vy, *vz, *ax, *ay, *az;  // the run's state
    double* pub;               // [kRunRing][3][n] positions after the last drifts
    double* out;               // [9][n] state after the last step: x y z vx vy vz ax ay az
    double* eblk;              // [records][nquads(n)][3] energy sums of four ions each
    unsigned* abort;           // give up; the waves this run was admitted with; at kTaken and kDone, tickets
    double gamma, dt, eps2;
    int every, phase;          // a record after step k (1 .. nk) where phase + k is a multiple of every (0: none)
    int spins;                 // polls of one wait for a position
    unsigned* flags;
    TrapK k[kRunSteps];        // the trap's spring constants at steps 1 .. nk
};

constexpr int run_quads(int n) { return (n + 3) / 4; }

__device__ __forceinline__ double poll(const double* p) {
    return __builtin_bit_cast(double, __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p),
                                                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void publish(double* p, double v) {
    unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    if (b == kUnset) b |= 1ull << 51;  // (still a NaN)
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void mark(double* p) {
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), kUnset, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool unset(double v) { return hi_u(v) == static_cast<unsigned>(kUnset >> 32); }

constexpr int kRunI = 4;  // ions per workgroup

template <int W, bool REC>
struct RunLds {
    union {
        RowsLds<kRunI, W, false> f;
        RowsLds<kRunI, W, REC> p;
    };
    // the ions' state, component by component (in registers it would be every
    // wave's, and spill): position, velocity, acceleration, mass, charge, and
    // a record's position
    double x[3][kRunI], v[3][kRunI], a[3][kRunI], m[kRunI], q[kRunI], r[3][kRunI];
    double k[kRunSteps][3];  // the trap's spring constants (an indexed kernel argument is a load from memory)
    int dead;
    unsigned ticket;
};

// rows_sums' wave sums over the positions X = [3][n] of one step, as they
// arrive.  False in every thread (the sums are then void) if a wait ran out.
// THERE: they have all arrived.
template <int PREC, int W, bool POT, bool THERE>
__device__ __forceinline__ bool run_sums(const RowRunParams& P, const double* X, int i0,
                                         const double (&xs)[3][kRunI], RowsLds<kRunI, W, POT>& lds, int& dead) {
    constexpr int C = POT ? 4 : 3, I = kRunI;
    const int n = P.n;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double f[I][C];
#pragma unroll
    for (int u = 0; u < I; ++u)
#pragma unroll
        for (int c = 0; c < C; ++c) f[u][c] = 0.0;
    const SeriesK K;
    int jb = w * 64;
    if (jb < n) {
        double xi[I], yi[I], zi[I];
#pragma unroll
        for (int u = 0; u < I; ++u) {
            xi[u] = uniform(xs[0][u]);
            yi[u] = uniform(xs[1][u]);
            zi[u] = uniform(xs[2][u]);
        }
        int jc = min(jb + lane, n - 1);
        double qj = P.q[jc], xj = poll(X + jc), yj = poll(X + n + jc), zj = poll(X + 2 * n + jc);
        for (; jb < n; jb += 64 * W) {
            for (int s = 0; !THERE && __any(unset(xj) || unset(yj) || unset(zj)); ++s) {
                const bool look = (s & 15) == 15;
                if (s >= P.spins ||
                    (look && __hip_atomic_load(P.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
                    if (lane == 0) {
                        dead = 1;
                        __hip_atomic_store(P.abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                    jb = n;
                    break;
                }
                xj = poll(X + jc);
                yj = poll(X + n + jc);
                zj = poll(X + 2 * n + jc);
            }
            if (jb >= n) break;
            // the next block is requested before this block's pairs
            const int jn = min(jb + 64 * W + lane, n - 1);
            double xn = 0.0, yn = 0.0, zn = 0.0, qn = 0.0;
            if (jb + 64 * W < n) {
                qn = P.q[jn];
                xn = poll(X + jn);
                yn = poll(X + n + jn);
                zn = poll(X + 2 * n + jn);
            }
            if (jb + 64 > n || (jb < i0 + I && jb + 64 > i0))
                rows_block<PREC, I, POT, true>(xj, yj, zj, qj, jb + lane, n, i0, xi, yi, zi, P.eps2, K, f);
            else
                rows_block<PREC, I, POT, false>(xj, yj, zj, qj, jb + lane, n, i0, xi, yi, zi, P.eps2, K, f);
            xj = xn;
            yj = yn;
            zj = zn;
            qj = qn;
            jc = jn;
        }
    }
    rows_wave_sums<I, W, POT>(f, lds);  // (a barrier: dead is known to all)
    return dead == 0;
}

// ONE: steps 1 .. nk of the ions' group blockIdx.x of kRunI, results to P.out.
// Else step ts (0: the first drift) of group tg, whose state is in P.out
// meanwhile, the last step's results to the run's state.  Thread t < 3 kRunI
// updates component t / kRunI of ion t % kRunI (as step_update does): one
// division in the chain from sums to positions instead of three.
template <int PREC, int W, bool REC, bool ONE>
__device__ __forceinline__ void rows_run(const RowRunParams& P, RunLds<W, REC>& lds, int ts = 0, int tg = 0) {
    constexpr int I = kRunI;
    const int n = P.n, t = threadIdx.x;
    // (one group, in loops of one turn: written without them the compiler spills
    // two registers in the chain, 1024 ions with records 3.4 -> 3.5 us per step)
    const int g0 = ONE ? (int)blockIdx.x : tg, g1 = g0 + 1;
    if (t == 0) lds.dead = ONE && __hip_atomic_load(P.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (t < P.nk) {
        lds.k[t][0] = P.k[t].kx;
        lds.k[t][1] = P.k[t].ky;
        lds.k[t][2] = P.k[t].kz;
    }
    const bool mine = t < 3 * I;
    const int c = mine ? t / I : 0, u = t % I;  // component and ion of the group
    const double h = 0.5 * P.dt, h2 = 0.5 * P.dt * P.dt;
    auto load = [&](int k, const double* X, const double* V, const double* A) {
        lds.x[c][u] = X[k];
        lds.v[c][u] = V[k];
        lds.a[c][u] = A[k];
        lds.m[u] = P.m[k];
        lds.q[u] = P.q[k];
    };
    auto save = [&](int k) {
        P.out[(size_t)c * n + k] = lds.x[c][u];
        P.out[(size_t)(3 + c) * n + k] = lds.v[c][u];
        P.out[(size_t)(6 + c) * n + k] = lds.a[c][u];
    };
    // (a step's results for other workgroups; nobody reads the run's state any
    // more when the last step's get there)
    auto pass = [&](int k, bool last) {
        publish(last ? (c == 0 ? P.x : (c == 1 ? P.y : P.z)) + k : P.out + (size_t)c * n + k, lds.x[c][u]);
        publish(last ? (c == 0 ? P.vx : (c == 1 ? P.vy : P.vz)) + k : P.out + (size_t)(3 + c) * n + k, lds.v[c][u]);
        publish(last ? (c == 0 ? P.ax : (c == 1 ? P.ay : P.az)) + k : P.out + (size_t)(6 + c) * n + k, lds.a[c][u]);
    };
    auto drift = [&](double* X, int k, bool own, double x, double v, double a, double m) {
        if (P.gamma == 0.0) {
            x = x + v * P.dt + h2 * a;
        } else {
            const double g = P.gamma / m;
            x = x + v * P.dt + h2 * (a - g * v);
        }
        if (own) publish(X + (size_t)c * n + k, x);
        lds.x[c][u] = x;
        if (own && !__builtin_isfinite(x)) atomicOr(P.flags, 1u);
    };
    for (int g = g0; (ONE || ts == 0) && g < g1; ++g) {  // the first drift
        const int k = min(g * I + u, n - 1);
        if (mine) {
            load(k, c == 0 ? P.x : (c == 1 ? P.y : P.z), c == 0 ? P.vx : (c == 1 ? P.vy : P.vz),
                 c == 0 ? P.ax : (c == 1 ? P.ay : P.az));
            drift(P.pub + (size_t)(1 % kRunRing) * 3 * n, k, g * I + u < n, lds.x[c][u], lds.v[c][u], lds.a[c][u],
                  lds.m[u]);
            if (!ONE && g * I + u < n) pass(k, false);
        }
    }
    if (!ONE && ts == 0) return;
    __syncthreads();
    if (lds.dead) return;  // (given up before this workgroup started, or not admitted)
    int rec = 0, due = REC ? P.phase : 0;
    if (REC && !ONE) {
        due += ts - 1;
        rec = due / P.every;
        due -= rec * P.every;
    }
    for (int s = ONE ? 1 : ts; s <= (ONE ? P.nk : ts); ++s) {
        const bool record = REC && ++due == P.every;
        auto ring = [&](int step) { return P.pub + (size_t)(step % kRunRing) * 3 * n; };
        const double* X = ring(s);
        for (int g = g0; g < g1; ++g) {
            const int i0 = g * I, k = min(i0 + u, n - 1);
            const bool own = i0 + u < n;
            if (!ONE) {
                if (mine) {
                    lds.x[c][u] = poll(P.out + (size_t)c * n + k);
                    lds.v[c][u] = poll(P.out + (size_t)(3 + c) * n + k);
                    lds.a[c][u] = poll(P.out + (size_t)(6 + c) * n + k);
                    lds.m[u] = P.m[k];
                    lds.q[u] = P.q[k];
                }
                __syncthreads();
            }
            bool live;
            if constexpr (REC) {
                if (record) live = run_sums<PREC, W, true, !ONE>(P, X, i0, lds.x, lds.p, lds.dead);
                else live = run_sums<PREC, W, false, !ONE>(P, X, i0, lds.x, lds.f, lds.dead);
            } else {
                live = run_sums<PREC, W, false, !ONE>(P, X, i0, lds.x, lds.f, lds.dead);
            }
            if (!live) return;
            double pot = 0.0;
            if (mine) {
                const double x = lds.x[c][u], m = lds.m[u], a = lds.a[c][u];
                double v = lds.v[c][u], o;
                if (REC && record) {
                    o = rows_sum<I, W, REC>(lds.p, u * (REC ? 4 : 3) + c);
                    if (c == 0) pot = rows_sum<I, W, REC>(lds.p, u * (REC ? 4 : 3) + (REC ? 3 : 0));
                } else {
                    o = rows_sum<I, W, false>(lds.f, u * 3 + c);
                }
                const double F = kCoulomb * lds.q[u] * o;
                const double an = F / m - lds.k[s - 1][c] * x;
                if (P.gamma == 0.0) {
                    v = v + h * (a + an);
                } else {
                    const double f = P.gamma / m, lo = 1.0 - f * h, hi = 1.0 + f * h;
                    v = (v * lo + h * (a + an)) / hi;
                }
                if (s < P.nk) drift(ring(s + 1), k, own, x, v, an, m);
                lds.v[c][u] = v;
                lds.a[c][u] = an;
                if (REC && record) lds.r[c][u] = x;
                if (ONE && own) mark(ring(s - 1) + (size_t)c * n + k);
                if (own && !(__builtin_isfinite(an) && __builtin_isfinite(v))) atomicOr(P.flags, 1u);
                if (!ONE && own) pass(k, s == P.nk);
            }
            __syncthreads();  // x is the next step's, the sums' LDS free
            if (REC && record && t < I) {  // the four ions' energies, while their positions travel
                double e[3];
                IonState st{lds.v[0][t], lds.v[1][t], lds.v[2][t], 0.0, 0.0, 0.0, lds.m[t]};
                double px = lds.r[0][t], py = lds.r[1][t], pz = lds.r[2][t];
                const TrapK kk{lds.k[s - 1][0], lds.k[s - 1][1], lds.k[s - 1][2]};
                const bool ok = step_update(EPI_ENERGY, kk, P.gamma, P.dt, st, px, py, pz, lds.q[t], 0.0, 0.0, 0.0, pot,
                                            e[0], e[1], e[2]);
                if (own && !ok) atomicOr(P.flags, 1u);
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    if (!own) e[b] = 0.0;
#pragma unroll
                    for (int d = I / 2; d > 0; d >>= 1) e[b] += __shfl_xor(e[b], d);
                    if (t == 0) P.eblk[((size_t)rec * run_quads(n) + g) * 3 + b] = e[b];
                }
            }
        }
        if (record) {
            ++rec;
            due = 0;
        }
    }
    if (ONE && mine && g0 * I + u < n) save(g0 * I + u);
}

// Waits until `before` tickets are done; the wait ends by itself (see above), its
// bound, of half a second, sets the flag.
constexpr int kTicketSpins = 1 << 20;

__device__ __forceinline__ void wait_tickets(const RowRunParams& P, unsigned before) {
    const unsigned* done = P.abort + kDone;
    for (int spin = 0; __hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < before; ++spin) {
        if (spin >= kTicketSpins) {
            atomicOr(P.flags, 1u);
            break;
        }
        __builtin_amdgcn_s_sleep(2);
    }
}

// Waits for the wave's stores.  What workgroups exchange here they write and
// read past the L2s (agent-scope atomics), so nothing is to be written back or
// dropped, as a fence would: by every wave that took 0.15 us a ticket, one
// after the other (1024 ions 40 us per step; by one thread 14, and so 7.5).
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The run's steps after giving up, by as many workgroups as run: ticket s G + g
// is step s of group g of G.  The positions of step s + 2 are written when all
// tickets of step s are done, so never over positions that are still read.
template <int PREC, int W, bool REC>
__device__ __forceinline__ void rows_run_tickets(const RowRunParams& P, RunLds<W, REC>& lds) {
    const unsigned groups = (unsigned)run_quads(P.n), all = groups * (unsigned)(P.nk + 1);
    for (;;) {
        if (threadIdx.x == 0) lds.ticket = atomicAdd(P.abort + kTaken, 1u);
        __syncthreads();
        const unsigned ticket = __builtin_amdgcn_readfirstlane(lds.ticket);
        if (ticket >= all) return;
        const unsigned s = ticket / groups;
        if (threadIdx.x == 0 && s > 0) wait_tickets(P, s * groups);
        __syncthreads();
        rows_run<PREC, W, REC, false>(P, lds, (int)s, (int)(ticket - s * groups));
        if (threadIdx.x == 0) {
            stores_done();  // (all of them are this wave's)
            atomicAdd(P.abort + kDone, 1u);
        }
        __syncthreads();
    }
}

// Two workgroups of 8 waves (four of 4) on each CU.
template <int PREC, int W, bool REC>
__global__ void __launch_bounds__(64 * W, 4) k_rows_run(RowRunParams P) {
    __shared__ __align__(16) RunLds<W, REC> lds;
    rows_run<PREC, W, REC, true>(P, lds);
}

// Waves of the runs admitted and not yet ended.
static __device__ unsigned g_run_waves;

// pub (len words) is marked as not yet written, and the run of `waves` waves
// admitted beside others up to `most` in all, or (after `polls` tries) given
// up; give_up: also when admitted.
static __global__ void __launch_bounds__(256) k_rows_run_begin(unsigned long long* __restrict__ pub, int len,
                                                               unsigned* __restrict__ abort, unsigned waves,
                                                               unsigned most, int polls, bool give_up) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    for (int k = i; k < len; k += gridDim.x * 256) pub[k] = kUnset;
    if (i != 0) return;
    unsigned got = 0;
    for (int s = 0; s < polls && !got; ++s) {
        const unsigned now = __hip_atomic_load(&g_run_waves, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (now + waves <= most && atomicCAS(&g_run_waves, now, now + waves) == now) got = waves;
        else __builtin_amdgcn_s_sleep(8);
    }
    abort[0] = got == 0 || give_up;
    abort[1] = got;
    abort[kTaken] = abort[kDone] = 0;
}

// The results of k_rows_run into the run's state, after its steps were taken
// here if it gave up.
template <int PREC, int W, bool REC>
__global__ void __launch_bounds__(64 * W, 4) k_rows_run_end(RowRunParams P) {
    __shared__ __align__(16) RunLds<W, REC> lds;
    if (blockIdx.x == 0 && threadIdx.x == 0 && P.abort[1]) atomicSub(&g_run_waves, P.abort[1]);
    if (P.abort[0]) {
        rows_run_tickets<PREC, W, REC>(P, lds);
        return;
    }
    double* const s[9] = {P.x, P.y, P.z, P.vx, P.vy, P.vz, P.ax, P.ay, P.az};
    for (int k = blockIdx.x * 64 * W + threadIdx.x; k < P.n; k += gridDim.x * 64 * W)
#pragma unroll
        for (int c = 0; c < 9; ++c) s[c][k] = P.out[(size_t)c * P.n + k];
}

}  // namespace cb
