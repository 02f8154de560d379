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

// Trap, kick and drift (as P.mode says) of ion i (index into P's arrays) at
// (x, y, z) with charge qk, state s, Coulomb force (Fx, Fy, Fz) and pot =
// sum_j q_j / r, in a trap of spring constants kk and friction gamma; its
// energy terms (EPI_ENERGY) go to eK, eC, eT.  Non-finite results set the
// flag.
template <class Params>
__device__ __forceinline__ void step_ion(const Params& P, const TrapK& kk, double gamma, int i, IonState s, double x,
                                         double y, double z, double qk, double Fx, double Fy, double Fz, double pot,
                                         double& eK, double& eC, double& eT) {
    const unsigned mode = P.mode;
    double vx = s.vx, vy = s.vy, vz = s.vz;
    double ax = s.ax, ay = s.ay, az = s.az;
    const double mi = s.m;
    bool ok = true;
    if (mode & (EPI_ACCEL | EPI_KICK)) {
        const double anx = Fx / mi - kk.kx * x;
        const double any = Fy / mi - kk.ky * y;
        const double anz = Fz / mi - kk.kz * z;
        if (mode & EPI_KICK) {
            const double h = 0.5 * P.dt;
            if (gamma == 0.0) {
                vx = vx + h * (ax + anx);
                vy = vy + h * (ay + any);
                vz = vz + h * (az + anz);
            } else {  // friction -g v by the trapezoidal rule, g = Gamma / m_i
                const double g = gamma / mi, lo = 1.0 - g * h, hi = 1.0 + g * h;
                vx = (vx * lo + h * (ax + anx)) / hi;
                vy = (vy * lo + h * (ay + any)) / hi;
                vz = (vz * lo + h * (az + anz)) / hi;
            }
            P.vx[i] = vx;
            P.vy[i] = vy;
            P.vz[i] = vz;
        }
        ax = anx;
        ay = any;
        az = anz;
        P.ax[i] = ax;
        P.ay[i] = ay;
        P.az[i] = az;
        ok = finite3(ax, ay, az) && finite3(vx, vy, vz);
    }
    if (mode & EPI_ENERGY) {
        eK = 0.5 * mi * (vx * vx + vy * vy + vz * vz);
        eC = 0.5 * kCoulomb * qk * pot;
        eT = 0.5 * mi * (kk.kx * x * x + kk.ky * y * y + kk.kz * z * z);
        ok = ok && finite3(eK, eC, eT);
    }
    if (mode & EPI_DRIFT) {
        const double dt = P.dt, h2 = 0.5 * dt * dt;
        if (gamma == 0.0) {
            x = x + vx * dt + h2 * ax;
            y = y + vy * dt + h2 * ay;
            z = z + vz * dt + h2 * az;
        } else {  // the drift sees the friction acceleration -g v too
            const double g = gamma / mi;
            x = x + vx * dt + h2 * (ax - g * vx);
            y = y + vy * dt + h2 * (ay - g * vy);
            z = z + vz * dt + h2 * (az - g * vz);
        }
        P.xn[i] = x;
        P.yn[i] = y;
        P.zn[i] = z;
        ok = ok && finite3(x, y, z);
    }
    if (!ok) atomicOr(P.flags, 1u);
}

}  // namespace cb
