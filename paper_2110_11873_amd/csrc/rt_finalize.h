// rt_finalize.h -- the operator's last step at one depth point (device code
// shared by the finalize pass and the sweep of slabs that one block holds).
#pragma once

#include "rt_internal.h"

namespace rt {

// sigma_out at point k of slab atm from its quadrature sums over the
// sweep's blocks (J0, J2): the source part of the quadrature and the
// scattering step (operator), or the right-hand side.
__device__ inline void finalize_point(const SweepArgs &a, int atm, const AtmDesc &at, int k,
                                      double J0, double J2) {
    const int kk = at.doff + k;
    const long long e = 2LL * kk;
    double o0, o2;
    if (a.mode == 0) {
        double z0 = a.sig_in[e], z2 = a.sig_in[e + 1];
        if (a.scale) {
            z0 *= a.scale[e];
            z2 *= a.scale[e + 1];
        }
        // source part of the quadrature: sum over all rays of q S
        const double4 Q = a.Qs[atm];
        J0 += z0 * Q.x + z2 * Q.y;
        J2 += z0 * Q.y + z2 * Q.z;
        o0 = z0 - at.xi * J0;
        o2 = z2 - at.xi * at.W2 * J2;
    } else {
        o0 = at.xi * J0 + at.eps * a.B[kk];
        o2 = at.xi * at.W2 * J2;
    }
    a.sig_out[e] = o0;
    a.sig_out[e + 1] = o2;
}

}  // namespace rt
