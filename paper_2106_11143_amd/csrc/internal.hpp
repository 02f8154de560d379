// Host-side declarations shared by the translation units of the library.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <cstring>

#include "coulomb.h"

namespace cb {

struct TrapK;  // step_common.hpp

constexpr int kMaxSplits = 64;       // j-splits per launch
constexpr int kMaxVec = 8;           // HVP vectors per call
constexpr int kMaxBatchIons = 4096;  // ions per run in the batched kernel (LDS bound)
constexpr int kBatchGridMax = 2048;  // workgroups of one batched launch (force accumulator slots)
constexpr int kBatchWG = 512;        // threads per workgroup of the persistent batched kernel
constexpr int kBatchP = 4;           // ions per thread and register group in that kernel
constexpr int kEpiBlock = 256;       // threads per element-wise block
constexpr int kEpiMinIons = kEpiBlock / 16;  // ions per block of the widest epilogue (16 threads per ion)
// Threads per ion of the epilogue (k_epilogue<T>) of the all-pairs kernel's
// calls (forces, energy, gradient, md_step, md_run): in a run of at most
// 8192 ions whose pair launch leaves 16 or more j-split partials per ion, 8
// or 16 threads share each ion's sums, over 8 or 16 times the CUs (md_run
// with energies every step on MI355X: 1024 ions 14.5 -> 11.0 us per step,
// 2048 17.4 -> 14.3, 4096 28.5 -> 24.9, with 64 splits).
constexpr int epi_parts(int64_t n, int S) { return n > 8192 ? 1 : (S >= 32 ? 16 : (S >= 16 ? 8 : 1)); }
constexpr int64_t kMaxIons = int64_t(1) << 28;  // largest n any entry point accepts
constexpr int64_t kSymMaxN = int64_t(1) << 18;  // largest n for the symmetric kernel (partials grow as n^2)
constexpr int64_t kRowsMaxN = 6144;     // largest n that takes whole rows per workgroup by default (rows.hip)
constexpr int64_t kSharesMaxN = 57344;  // and equal shares of the pairs (shares.hip)
constexpr int kMaxDevices = 64;      // GPUs per process the per-device symbol tables hold

// ALGO_SYM and ALGO_SYM_LDS differ only in how the per-j reactions are summed
// over the wave (cross-lane permutes and DPP, or LDS).  ALGO_SYM_ROWS: as
// ALGO_SYM_LDS with kSymRows consecutive i-blocks per workgroup sharing each
// j-segment, their reactions added in LDS before one store.
// ALGO_SMALL (md_step / md_run of one run of at most kSmallRunMax ions):
// one launch per step, every pair direct (md_run_rows; up to kRowsRunMaxN ions
// and from some steps on, one launch for many steps).
enum : int { ALGO_DIRECT = 0, ALGO_SYM = 1, ALGO_SYM_LDS = 2, ALGO_SMALL = 3, ALGO_SYM_ROWS = 4 };

// What an entry's calls take: the launches of its algorithm and shape, or
// whole rows per workgroup (rows.hip), equal shares of the pairs (shares.hip)
// or the Newton's-third-law stage in bands (pair_sym.hip).
enum : int { PATH_CFG = 0, PATH_ROWS = 1, PATH_SHARES = 2, PATH_BANDS = 3 };

constexpr bool is_sym(int algo) { return algo == ALGO_SYM || algo == ALGO_SYM_LDS || algo == ALGO_SYM_ROWS; }

// i-blocks per workgroup of the row-group variant, and of the others.
constexpr int kSymRows = 4;
constexpr int sym_rows(int algo) { return algo == ALGO_SYM_ROWS ? kSymRows : 1; }
constexpr bool sym_rows_p_ok(int p) { return p == 4 || p == 6 || p == 8; }
constexpr int64_t kSymRowsMinN = 81920;  // the row-group tiles are the default from here

// Operations whose pair stage may take the Newton's-third-law kernels.
constexpr bool sym_op(int op) {
    return op == CB_OP_FORCES || op == CB_OP_ENERGY || op == CB_OP_MD_STEP || op == CB_OP_MD_RUN;
}

// Symmetric path launch parameters: i-particles per lane, j's per reaction
// group, segment lengths (powers of two).
constexpr int kSymP[] = {2, 3, 4, 5, 6, 8};
constexpr int kSymGroup = 4;
constexpr int kSymJL[] = {256, 512, 1024, 2048};

// Newton's-third-law Hessian-vector products (hvp.hip): i-particles per
// lane, segment lengths, the smallest n of the default, the largest n a
// tile table holds, and the workspace of the configuration.
constexpr int kHvpSymP[] = {1, 2, 4};
constexpr int kHvpSymJL[] = {64, 128, 256, 512};
constexpr int64_t kHvpSymMinN = 4096;
constexpr bool hvp_sym_cfg_ok(int p, int jl) {
    bool pk = false, jk = false;
    for (int v : kHvpSymP) pk = pk || v == p;
    for (int v : kHvpSymJL) jk = jk || v == jl;
    return pk && jk;
}
constexpr int64_t hvp_sym_max_n(int p) { return int64_t(2048) * 64 * p; }
// Passes of nvmax vectors that one launch evaluates together (more waves in
// flight than one pass of a small problem gives), and the passes a
// workspace for nvec vectors holds.
constexpr int kHvpSymPasses = 2;
constexpr int hvp_sym_passes(int nvec, int nvmax) {
    return nvec / nvmax < 1 ? 1 : (nvec / nvmax > kHvpSymPasses ? kHvpSymPasses : nvec / nvmax);
}
size_t hvp_sym_ws_bytes(int64_t n, int p, int jl, int npass);

constexpr bool sym_cfg_ok(int p, int g, int jl) {
    bool pk = false, jk = false;
    for (int v : kSymP) pk = pk || v == p;
    for (int v : kSymJL) jk = jk || v == jl;
    return pk && jk && g == kSymGroup;
}

struct LaunchCfg {
    int p;       // i-particles per lane
    int wg;      // direct: threads per workgroup; symmetric: j's per reaction group (4)
    int splits;  // direct: requested j-splits; symmetric: segment length JL
    int tuned;   // 1 if set by tuning or cb_set_config
    int algo;    // ALGO_DIRECT, ALGO_SYM or ALGO_SYM_LDS
    int path;    // PATH_CFG, or the path taken in its place (untuned entries, or a tuned one that was faster so)
    // A tuned entry's: the default path it was timed against.  At the sizes of
    // its bucket that have another, that one is taken (get_cfg).  -1: path holds
    // at every size.
    int base = -1;
};

struct WsLayout {
    size_t part, ppot, eblk, aux, batch, total;
};

cb_status fail(cb_status st, const char* fmt, ...);
cb_status ok();
cb_status check_launch(const char* what);
unsigned* flags_ptr();

// Host-to-device copies of tables a call builds on the host (run tables,
// traps).  On a stream that is not capturing, each copy reads its source
// directly (HIP consumes pageable sources before hipMemcpyAsync returns).
// On a capturing stream the sources are first copied into one host block
// that the graph under construction owns (a user object the graph retains,
// freed after the graph is destroyed), so every replay copies the same
// bytes again.  Sources must stay valid until run() returns.
class HostUpload {
  public:
    void add(void* dst, const void* src, size_t bytes);
    cb_status run(hipStream_t st, const char* what);

  private:
    struct Item {
        void* dst;
        const void* src;
        size_t bytes;
    };
    Item items_[8];
    int count_ = 0;
};

int n_bucket(int64_t n);
// Whether the one-wave 512 x 512 tiles that are configured from 32768 ions
// fill the 1024 SIMDs evenly (96% of the waves of their last round): then they
// beat equal shares, which else win (us per evaluation on MI355X, tiles /
// shares: 32768 ions, 2016 tiles, 408 / 410; 39900, 3003, 583 / 587; 46592, 4095,
// 760 / 784; 56832, 6105, 1121 / 1152; but 39424, 2926, 581 / 575; 33500, 2080,
// 548 / 426; 49152, 4560, 906 / 865).
constexpr bool tiles_fit(int64_t n) {
    const int64_t r = (n + 511) / 512, T = r * (r - 1) / 2, rounds = (T + 1023) / 1024;
    return n >= 32768 && 100 * T >= 96 * 1024 * rounds;
}

// The path of an untuned entry (us per md_run step on MI355X, rows / pair
// launch and epilogue: 150 ions 4.0 / 7.6, 1024 5.2 / 9.5, 2048 7.8 / 12.5,
// 4096 16.5 / 21.4, 6000 31.2 / 35.7, 8192 54.3 / 54.0; us per force
// evaluation, shares / configured: 7000 ions 37.6 / 39.4 (6144: rows 30.4),
// 8192 43.4 / 48.5, 12001 71.7 / 104, 16000 114 / 181, 20001 168 / 210, 24577 240 /
// 243, 27999 307 / 309, 30000 348 / 371, 33500 426 / 548, 40000 588 /
// 714, 49152 865 / 906, 57344 1161 / 1239, 65536 1490 / 1485).
//
// The energy alone takes the potential-only all-pairs launches where rows
// and shares, which sum the forces too, are slower (us per coulomb_energy, rows
// or shares / those: FP64 2000 ions 10.0 / 12.9, 2500 15.3 / 15.2, 3000 16.9 /
// 14.9, 4096 20.9 / 18.6, 5000 33.0 / 24.7, 6144 39.2 / 31.1, 6145 32.3 / 36.4,
// 8192 41.8 / 44.6; mixed 7000 35.1 / 33.6, 8192 42.6 / 40.1, 8704 46.2 / 44.3,
// 8800 46.5 / 49.3; the FP32 estimate 8193 37.4 / 33.3, 8704 39.7 / 37.0, 8800
// 39.9 / 40.2).
constexpr int64_t kPotAloneMinN = 2401;
constexpr int64_t pot_alone_max(int prec) { return prec == CB_MIXED || prec == CB_FP32_RSQ ? 8750 : kRowsMaxN; }
constexpr int default_path(int op, int64_t n, int prec) {
    if (op == CB_OP_ENERGY && n >= kPotAloneMinN && n <= pot_alone_max(prec)) return PATH_CFG;
    if (op != CB_OP_FORCES && op != CB_OP_ENERGY && op != CB_OP_MD_STEP && op != CB_OP_MD_RUN) return PATH_CFG;
    return n <= kRowsMaxN ? PATH_ROWS : n <= kSharesMaxN && !tiles_fit(n) ? PATH_SHARES : n > kSymMaxN ? PATH_BANDS : PATH_CFG;
}
LaunchCfg default_cfg(int op, int64_t n, int prec);
LaunchCfg direct_cfg(int op, int64_t n, int prec);
LaunchCfg get_cfg(int op, int64_t n, int prec);
// The path of a call.  CB_OP_GRAD: of the gradient with the energy, whose
// configuration is the energy's.
int path_of(int op, int64_t n, int prec);
void put_cfg(int op, int64_t n, int prec, LaunchCfg c);
void drop_cfg(int op, int64_t n, int prec);
bool valid_cfg(int op, const LaunchCfg& c);
int split_len(int64_t n, int splits);
int n_splits(int64_t n, int jlen);
// Workspace carve-up of an entry point; sized for the launch configuration
// get_cfg picks for (op, n, prec) at the time of the call.
WsLayout ws_layout(int op, int64_t n, int32_t nrun, int32_t nvec, int32_t prec);

bool trap_ok(const cb_trap* t, const char* who, cb_status* st);

// Tile table of the Newton's-third-law kernels (pair_sym.hip): row groups of
// W consecutive i-blocks of IB ions (W = 1: single rows), the j's above the
// group's first block cut into j-segments of JL.  sym_plan carves
// rowstart[nG+1] and tiles[T] (tile = (group, segment)) from the start of ws
// (sym_plan_bytes of it) and enqueues the kernel that fills them (unless
// filled: the same table is already in ws, written by an earlier call on the
// stream with the same n, IB, JL and W).
struct SymPlan {
    int* rowstart;
    int2* tiles;
    int64_t T;
    size_t bytes;
};
int64_t sym_tiles(int64_t n, int IB, int JL, int W = 1);
size_t sym_plan_bytes(int64_t n, int IB, int JL, int W = 1);
cb_status sym_plan(int n, int IB, int JL, void* ws, SymPlan* out, hipStream_t st, int W = 1, bool filled = false);

// Symmetric (Newton's third law) force path (pair_sym.hip): workspace bytes
// for (n, p, JL) and W rows per workgroup (pot: with the tiles' pair
// energies), and the launch sequence ending with finished forces F[3][n]
// and, when phi is set, each ion's share of the Coulomb energy, U_C = k_C
// sum_k phi[k].  plan_filled: ws already holds the tile table of (n, c), from
// an earlier launch on the stream (md_run's later steps).
size_t sym_ws_bytes(int64_t n, int p, int jl, bool pot = false, int W = 1);
cb_status launch_pair_sym(int prec, const LaunchCfg& c, int n, const double* x, const double* y, const double* z,
                          const double* q, double eps2, void* ws, double* F, hipStream_t st, double* phi = nullptr,
                          bool plan_filled = false);

// The same beyond kSymMaxN ions, where the partials of the whole triangle
// (they grow as n^2) do not fit: row-group tiles of kBandP and kBandJL, the
// triangle's row groups taken in bands whose partials fit ws_bytes, each band
// finished and added to F (and phi) before the next.  (ms per evaluation on
// MI355X, the direct kernel / bands: 262145 ions 36.9 / 23.4, 300001 48.3 /
// 30.0, 420000 94.6 / 59.5, ions grouped by charge; 50.1 / 32.6 at 300001 in
// seeded order.  Segments of 1024 or 2048 measured 0-3% slower.)
constexpr int kBandP = 8, kBandJL = 512;
cb_status launch_pair_sym_bands(int prec, int n, const double* x, const double* y, const double* z, const double* q,
                                double eps2, void* ws, size_t ws_bytes, double* F, hipStream_t st,
                                double* phi = nullptr);

// Forces, gradient (with u_out the energy) and md steps of n ions on equal shares
// of the pairs (shares.hip); arguments as rows_forces and md_run_rows, ws:
// share_ws_bytes(n, pot) bytes, pot: with the energy or records.
size_t share_ws_bytes(int64_t n, bool pot);
cb_status share_forces(int prec, int64_t n, const double* x, const double* y, const double* z, const double* q,
                    const double* m, const TrapK& k, double eps2, unsigned mode, double* fx, double* fy, double* fz,
                    double* u_out, void* ws, hipStream_t st);
cb_status md_run_shares(int64_t n, const cb_state* s, const double* q, const double* m, const cb_trap* trap, double t0,
                    double dt, int64_t nsteps, double eps2, int32_t prec, uint32_t flags, double* energies,
                    int64_t every, void* ws, hipStream_t st);

// Launches of the pair kernels (pair.hip).  The _range form evaluates the
// forces / potentials of the ions i0 .. i0 + ni - 1 only (partials indexed by
// i - i0); launch_pair is the whole range.
cb_status launch_pair_range(int prec, const LaunchCfg& c, bool force, bool pot, int n, int i0, int ni,
                            const double* x, const double* y, const double* z, const double* q, double eps2,
                            int jlen, double* part, double* ppot, hipStream_t st);
cb_status launch_pair(int prec, const LaunchCfg& c, bool force, bool pot, int n, const double* x,
                      const double* y, const double* z, const double* q, double eps2, int jlen, double* part,
                      double* ppot, hipStream_t st);
cb_status launch_hvp(int prec, const LaunchCfg& c, int nvec, int n, const double* x, const double* y,
                     const double* z, const double* q, const double* v, double eps2, int jlen, double* part,
                     hipStream_t st);

// Stepped ensemble md_run (ensemble.hip): supported (p, JL), a workspace
// bound over every split of ntot ions into nrun runs of at most
// kMaxBatchIons, and the driver.
bool ens_cfg_ok(int p, int jl);
size_t ens_ws_bound(int64_t ntot, int32_t nrun);
cb_status md_run_ensemble(int32_t nrun, const int64_t* offsets, const cb_state* s, const double* q,
                          const double* m, const cb_trap* traps, double t0, double dt, int64_t nsteps, double eps2,
                          int32_t prec, uint32_t flags, double* energies, int64_t every, int P, int JL, void* ws,
                          size_t ws_bytes, hipStream_t st);

// One run in one launch per step, whole rows per workgroup (rows.hip): every
// entry of ALGO_SMALL, and the untuned default up to kRowsMaxN ions.
// Workspace bytes and driver.
constexpr int64_t kSmallRunMax = 8192;     // largest run an ALGO_SMALL entry may hold
constexpr int64_t kSmallRunDefault = 256;  // the reported default is ALGO_SMALL up to here
constexpr int kSmallPartsMax = 32;
int small_parts(int64_t n);
constexpr int64_t kRowsSmallN = 1536;  // up to here 4 ions to a workgroup of 8 waves, above 8 to 4 waves
size_t md_rows_ws_bytes(int64_t n);
cb_status md_run_rows(int64_t n, const cb_state* s, const double* q, const double* m, const cb_trap* trap, double t0,
                      double dt, int64_t nsteps, double eps2, int32_t prec, uint32_t flags, double* energies,
                      int64_t every, void* ws, size_t ws_bytes, int spins, hipStream_t st);

// Its steps by workgroups that stay resident (rows_run.hpp): whether a run
// takes them, and the steps themselves, from accelerations at t0 on; spins:
// polls of one wait for a position before the launch gives up (its end then
// takes the steps, in an order that waits for no workgroup without a place).
// Some ms, several times what a run of another process may hold the places,
// since only the wait for a place can be long (us per step of two processes
// with runs of 1280 ions, alone 4.4: 8.4 while each waits for the other's runs,
// 25 with 2^11 polls, which give up on them).
constexpr int64_t kRowsRunMaxN = 1280;
constexpr int kRunSpins = 1 << 13;
size_t rows_run_ws_bytes(int64_t n);
bool rows_run_fits(int64_t n, int64_t nsteps, size_t ws_bytes);
cb_status rows_run(int64_t n, const cb_state* s, const double* q, const double* m, const cb_trap* trap, double t0,
                   double dt, int64_t nsteps, double eps2, int32_t prec, double* energies, int64_t every, int spins,
                   void* ws, hipStream_t st);

// Forces (mode EPI_FORCES) or gradient (EPI_GRAD) of n ions in one launch,
// and with u_out the energy U_C (+ U_trap with m) in a second; ws (with u_out
// only): 3 doubles per workgroup of 4 ions or more.
cb_status rows_forces(int prec, int64_t n, const double* x, const double* y, const double* z, const double* q,
                      const double* m, const TrapK& k, double eps2, unsigned mode, double* fx, double* fy, double* fz,
                      double* u_out, void* ws, hipStream_t st);
// md_run of an ensemble on equal shares of its runs' pairs (shares.hip), and
// the units of 256 ions by 16 that they hold.  *taken: whether its tables and
// partials fit ws_bytes (else nothing is done).
double share_ens_units(int32_t nrun, const int64_t* offsets);
cb_status md_run_shares_ensemble(int32_t nrun, const int64_t* offsets, const cb_state* s, const double* q,
                                 const double* m, const cb_trap* traps, double t0, double dt, int64_t nsteps,
                                 double eps2, int32_t prec, uint32_t flags, double* energies, int64_t every, void* ws,
                                 size_t ws_bytes, bool* taken, hipStream_t st);
// md_run_rows for an ensemble of runs, one launch per step over all of them.
cb_status md_run_rows_ensemble(int32_t nrun, const int64_t* offsets, const cb_state* s, const double* q,
                               const double* m, const cb_trap* traps, double t0, double dt, int64_t nsteps,
                               double eps2, int32_t prec, uint32_t flags, double* energies, int64_t every, void* ws,
                               size_t ws_bytes, hipStream_t st);

// Batched md_run (batched.hip): picks the persistent kernel or the stepped
// ensemble path.
cb_status md_run_batched(int32_t nrun, const int64_t* offsets, const cb_state* s, const double* q,
                         const double* m, const cb_trap* traps, double t0, double dt, int64_t nsteps,
                         double eps2, int32_t prec, uint32_t flags, double* energies, int64_t every, void* ws,
                         size_t ws_bytes, hipStream_t st);

}  // namespace cb
