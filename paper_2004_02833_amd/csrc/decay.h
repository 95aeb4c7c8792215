// Derivatives of the decay factors of eq. (5), for the transposed sweeps.
#pragma once
#include <hip/hip_runtime.h>

namespace pm {

// d beta / d c for beta = (1 - exp(-c tau))/c:  -tau^2 F(c tau) with
// F(z) = (1 - (1+z) e^{-z}) / z^2 = sum_k (-1)^k (k+1) z^k / (k+2)!,
// summed as a series for |z| < 1e-2 (truncation below 1e-16 relative).
__device__ __forceinline__ double dbeta_series(double z, double tau) {
    const double F = 0.5 + z * (-1.0 / 3.0 + z * (1.0 / 8.0 + z * (-1.0 / 30.0 + z * (1.0 / 144.0 - z / 840.0))));
    return -tau * tau * F;
}

// dL/dc of a coefficient with decay factors al, be over tau, from
// A = sum w u and B = sum w u' (w = be lam): lam u dal/dc + lam r dbe/dc,
// with c recovered from the factors, c = (1 - al) / be.  be = 0 is an opaque
// point (the mean of its cells' coefficients overflows): al, A and B are 0 and
// so is the derivative, where the quotients by be would be 0 / 0.
__device__ __forceinline__ double dl_dc(double A, double B, double al, double be, double tau) {
    const double om = 1.0 - al;
    const double db = om < 1e-2 ? dbeta_series(tau * om / be, tau) : (tau * al - be) * be / om;
    const double d = be == 0.0 ? 1.0 : be;
    return ((B - al * A) * (db / d) - tau * al * A) / d;
}

}  // namespace pm
