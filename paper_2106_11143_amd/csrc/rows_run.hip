// Host side of the resident small runs (rows_run.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "energy_record.hpp"
#include "internal.hpp"
#include "rows_run.hpp"

namespace cb {

static size_t al(size_t b) { return (b + 255) / 256 * 256; }

// Four waves where the j's fill no more.
static int run_waves(int64_t n) { return n <= 256 ? 4 : 8; }

size_t rows_run_ws_bytes(int64_t n) {
    return 256 + al(sizeof(double) * 3 * kRunRing * (size_t)n) + al(sizeof(double) * 9 * (size_t)n) +
           al(sizeof(double) * 3 * kRunSteps * (size_t)run_quads((int)n));
}

static int cu_count() {
    int dev = 0, ncu = 0;
    return hipGetDevice(&dev) == hipSuccess &&
                   hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess
               ? ncu
               : 0;
}

// Waves that are admitted together: 12 of the 16 that a CU holds (128
// registers).  While a workgroup of 8 still waits for its place, the others
// admitted have less than that, so some CU has two of each SIMD's four free.
constexpr int kRunWavesPerCu = 12;
constexpr int kRunAdmitPolls = 1 << 13;  // some ms

// Up to 1280 ions: beyond, more than a few CUs hold two workgroups, whose pairs
// take twice as long (1536 ions 6.0 us per step against 6.9 with a launch
// each, and with a record at every step no less).  A run pays four launches
// for what a launch per step pays one at a time (150 ions, 4 / 6 / 8 / 12
// steps: 40 / 47 / 56 / 68 us with a launch each, 40 / 41 / 44 / 51 so; 1024
// ions 43 / 52 / 61 / 78 against 43 / 52 / 57 / 68).
bool rows_run_fits(int64_t n, int64_t nsteps, size_t ws_bytes) {
    return n <= kRowsRunMaxN && nsteps >= 6 + n / 256 && ws_bytes >= rows_run_ws_bytes(n) &&
           run_quads((int)n) * run_waves(n) <= kRunWavesPerCu * cu_count();
}

template <int W>
__global__ void __launch_bounds__(64 * W) k_rows_run_records(int nb, const double* __restrict__ eblk,
                                                            double* __restrict__ energies) {
    energy_record<W>(nb, eblk + (size_t)blockIdx.x * nb * 3, energies + (size_t)blockIdx.x * 4, REC_ALL);
}

// A run's launches follow each other without another run's of this process
// between them: streams may share a queue, where a launch waiting to be
// admitted would hold up the one it waits for.
static std::mutex run_mutex;

template <int PREC, int W, bool REC>
static void go_run(const RowRunParams& P, hipStream_t st) {
    const int len = kRunRing * 3 * P.n, quads = run_quads(P.n);
    const unsigned most = (unsigned)(kRunWavesPerCu * cu_count());
    std::lock_guard<std::mutex> lock(run_mutex);
    k_rows_run_begin<<<(unsigned)std::min(256, (len + 1023) / 1024), 256, 0, st>>>(
        reinterpret_cast<unsigned long long*>(P.pub), len, P.abort, (unsigned)(quads * W), most,
        P.spins < 0 ? 0 : kRunAdmitPolls, P.spins == 0);
    k_rows_run<PREC, W, REC><<<(unsigned)quads, 64 * W, 0, st>>>(P);
    k_rows_run_end<PREC, W, REC><<<(unsigned)quads, 64 * W, 0, st>>>(P);
}

template <int PREC>
static void go_run_shape(const RowRunParams& P, hipStream_t st) {
    if (run_waves(P.n) == 4) P.every > 0 ? go_run<PREC, 4, true>(P, st) : go_run<PREC, 4, false>(P, st);
    else P.every > 0 ? go_run<PREC, 8, true>(P, st) : go_run<PREC, 8, false>(P, st);
}

cb_status rows_run(int64_t n, const cb_state* s, const double* q, const double* m, const cb_trap* trap, double t0,
                   double dt, int64_t nsteps, double eps2, int32_t prec, double* energies, int64_t every, int spins,
                   void* ws, hipStream_t st) {
    RowRunParams P{};
    P.n = (int)n;
    P.q = q;
    P.m = m;
    P.x = s->x; P.y = s->y; P.z = s->z;
    P.vx = s->vx; P.vy = s->vy; P.vz = s->vz;
    P.ax = s->ax; P.ay = s->ay; P.az = s->az;
    P.gamma = trap->gamma;
    P.dt = dt;
    P.eps2 = eps2;
    P.spins = spins;
    P.flags = flags_ptr();
    if (!P.flags) return fail(CB_EHIP, "md_run: device flag symbol not found");
    char* base = static_cast<char*>(ws);
    P.abort = reinterpret_cast<unsigned*>(base);
    base += 256;
    P.pub = reinterpret_cast<double*>(base);
    base += al(sizeof(double) * 3 * kRunRing * (size_t)n);
    P.out = reinterpret_cast<double*>(base);
    base += al(sizeof(double) * 9 * (size_t)n);
    P.eblk = reinterpret_cast<double*>(base);
    const int nb = run_quads((int)n);
    for (int64_t k0 = 0; k0 < nsteps; k0 += P.nk) {
        P.nk = (int)std::min<int64_t>(kRunSteps, nsteps - k0);
        for (int a = 0; a < P.nk; ++a) P.k[a] = trap_k(*trap, t0 + (double)(k0 + a + 1) * dt);
        // the first record of these steps, and how many there are
        const int64_t r0 = energies ? k0 / every + 1 : 0, nrec = energies ? (k0 + P.nk) / every + 1 - r0 : 0;
        P.every = nrec ? (int)std::min<int64_t>(every, 2 * kRunSteps) : 0;
        P.phase = nrec ? (int)(P.every - std::min<int64_t>(r0 * every - k0, P.every)) : 0;
        switch (prec) {
            case CB_FP64: go_run_shape<PREC_FP64>(P, st); break;
            case CB_MIXED: go_run_shape<PREC_MIXED>(P, st); break;
            case CB_FP64_IEEE: go_run_shape<PREC_IEEE>(P, st); break;
            default: go_run_shape<PREC_FP32>(P, st); break;
        }
        if (nrec) k_rows_run_records<8><<<(unsigned)nrec, 512, 0, st>>>(nb, P.eblk, energies + 4 * r0);
        if (cb_status rc = check_launch("k_rows_run")) return rc;
    }
    return CB_OK;
}

}  // namespace cb
