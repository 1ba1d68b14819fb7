// fn_env.h -- device functions shared by the envelope and determinant kernels.
#pragma once
#include "fn_internal.h"

namespace fn {

template <typename T>
__device__ inline T wave_sum(T v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// One nucleus' term of orbital column col's envelope at electron position
// xj: em = pi exp(-q) added to env, and with FL its contributions to the
// electron's gradient and Laplacian of the envelope (all FP64).
//   anisotropic: q = |Sigma d|, grad q = S d / q, S = Sigma^T Sigma,
//                lap q = (tr S - |S d|^2 / q^2) / q;
//   isotropic (Sigma = sigma I): q = |sigma| r with r = |d|,
//                grad q = |sigma| d / r, |grad q|^2 = sigma^2, lap q = 2 |sigma| / r.
template <typename T, bool FL>
__device__ __forceinline__ void env_add(const Sys &s, const T *theta, int64_t piof, int64_t sigof, int col, int m,
                                        const double *xj, double &env, double (&ge)[3], double &le)
{
    const double d[3] = {xj[0] - s.R[m][0], xj[1] - s.R[m][1], xj[2] - s.R[m][2]};
    if (s.iso) {
        const double sg = fabs((double)theta[sigof + (int64_t)col * s.M + m]);
        const double r = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
        const double em = (double)theta[piof + (int64_t)col * s.M + m] * exp(-(sg * r));
        env += em;
        if constexpr (FL) {
            const double gr = sg / r;
            for (int a = 0; a < 3; ++a) ge[a] -= em * gr * d[a];
            le += em * (sg * sg - 2.0 * gr);
        }
        return;
    }
    const T *Sgp = theta + sigof + ((int64_t)col * s.M + m) * 9;
    double sd[3], ad[3], Sg[9];
    for (int e = 0; e < 9; ++e) Sg[e] = (double)Sgp[e];
    for (int p = 0; p < 3; ++p) sd[p] = Sg[3 * p] * d[0] + Sg[3 * p + 1] * d[1] + Sg[3 * p + 2] * d[2];
    for (int a = 0; a < 3; ++a) ad[a] = Sg[a] * sd[0] + Sg[3 + a] * sd[1] + Sg[6 + a] * sd[2];
    const double qd = sqrt(sd[0] * sd[0] + sd[1] * sd[1] + sd[2] * sd[2]);
    const double em = (double)theta[piof + (int64_t)col * s.M + m] * exp(-qd);
    env += em;
    if constexpr (FL) {
        double trS = 0.0;
        for (int e = 0; e < 9; ++e) trS += Sg[e] * Sg[e];
        const double iq = 1.0 / qd;
        const double ad2 = ad[0] * ad[0] + ad[1] * ad[1] + ad[2] * ad[2];
        const double lq = (trS - ad2 * iq * iq) * iq;
        const double gq2 = ad2 * iq * iq;
        for (int a = 0; a < 3; ++a) ge[a] -= em * ad[a] * iq;
        le += em * (gq2 - lq);
    }
}

}  // namespace fn
