// Velocity-Verlet update of one ion (paper, section 2) from its finished
// Coulomb force, shared by the kernels that fuse it with the force sums.
#pragma once
#include <hip/hip_runtime.h>

#include "step_common.hpp"

namespace cb {

// What an ion's update reads besides its position, held in registers (loaded
// ahead of the force sums where a kernel is bound by latency).
struct IonState {
    double vx, vy, vz, ax, ay, az, m;
};

template <class Params>
__device__ __forceinline__ IonState load_ion(const Params& P, int i) {
    return IonState{P.vx[i], P.vy[i], P.vz[i], P.ax[i], P.ay[i], P.az[i], P.m[i]};
}

// Trap, kick and drift (as mode says) of an ion at (x, y, z) with charge qk,
// state s, Coulomb force (Fx, Fy, Fz) and pot = sum_j q_j / r, in a trap of
// spring constants kk and friction gamma: s and the position become the new
// ones, its energy terms (EPI_ENERGY) go to eK, eC, eT.  False if a result is
// not finite.
__device__ __forceinline__ bool step_update(unsigned mode, const TrapK& kk, double gamma, double dt, IonState& s,
                                            double& x, double& y, double& z, double qk, double Fx, double Fy,
                                            double Fz, double pot, double& eK, double& eC, double& eT) {
    const double mi = s.m;
    bool ok = true;
    if (mode & (EPI_ACCEL | EPI_KICK)) {
        const double anx = Fx / mi - kk.kx * x;
        const double any = Fy / mi - kk.ky * y;
        const double anz = Fz / mi - kk.kz * z;
        if (mode & EPI_KICK) {
            const double h = 0.5 * dt;
            if (gamma == 0.0) {
                s.vx = s.vx + h * (s.ax + anx);
                s.vy = s.vy + h * (s.ay + any);
                s.vz = s.vz + h * (s.az + anz);
            } else {  // friction -g v by the trapezoidal rule, g = Gamma / m_i
                const double g = gamma / mi, lo = 1.0 - g * h, hi = 1.0 + g * h;
                s.vx = (s.vx * lo + h * (s.ax + anx)) / hi;
                s.vy = (s.vy * lo + h * (s.ay + any)) / hi;
                s.vz = (s.vz * lo + h * (s.az + anz)) / hi;
            }
        }
        s.ax = anx;
        s.ay = any;
        s.az = anz;
        ok = finite3(s.ax, s.ay, s.az) && finite3(s.vx, s.vy, s.vz);
    }
    if (mode & EPI_ENERGY) {
        // (fused by hand: every kernel that records gives the same bits)
        const double kx = kk.kx * x, ky = kk.ky * y, kz = kk.kz * z;
        eK = 0.5 * mi * __builtin_fma(s.vz, s.vz, __builtin_fma(s.vy, s.vy, s.vx * s.vx));
        eC = 0.5 * kCoulomb * qk * pot;
        eT = 0.5 * mi * __builtin_fma(kz, z, __builtin_fma(ky, y, kx * x));
        ok = ok && finite3(eK, eC, eT);
    }
    if (mode & EPI_DRIFT) {
        const double h2 = 0.5 * dt * dt;
        if (gamma == 0.0) {
            x = x + s.vx * dt + h2 * s.ax;
            y = y + s.vy * dt + h2 * s.ay;
            z = z + s.vz * dt + h2 * s.az;
        } else {  // the drift sees the friction acceleration -g v too
            const double g = gamma / mi;
            x = x + s.vx * dt + h2 * (s.ax - g * s.vx);
            y = y + s.vy * dt + h2 * (s.ay - g * s.vy);
            z = z + s.vz * dt + h2 * (s.az - g * s.vz);
        }
        ok = ok && finite3(x, y, z);
    }
    return ok;
}

// The same for ion i of P's arrays, results to P's arrays (positions to xn,
// yn, zn), P.mode and P.dt; non-finite results set the flag.
template <class Params>
__device__ __forceinline__ void step_ion(const Params& P, const TrapK& kk, double gamma, int i, IonState s, double x,
                                         double y, double z, double qk, double Fx, double Fy, double Fz, double pot,
                                         double& eK, double& eC, double& eT) {
    const unsigned mode = P.mode;
    const bool ok = step_update(mode, kk, gamma, P.dt, s, x, y, z, qk, Fx, Fy, Fz, pot, eK, eC, eT);
    if (mode & EPI_KICK) {
        P.vx[i] = s.vx;
        P.vy[i] = s.vy;
        P.vz[i] = s.vz;
    }
    if (mode & (EPI_ACCEL | EPI_KICK)) {
        P.ax[i] = s.ax;
        P.ay[i] = s.ay;
        P.az[i] = s.az;
    }
    if (mode & EPI_DRIFT) {
        P.xn[i] = x;
        P.yn[i] = y;
        P.zn[i] = z;
    }
    if (!ok) atomicOr(P.flags, 1u);
}

}  // namespace cb
