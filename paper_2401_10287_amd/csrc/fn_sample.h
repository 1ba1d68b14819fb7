// fn_sample.h -- the sampler's proposal (Electron Sampler section of the paper),
// shared by the kernels of fn_mc.hip and the small-network walk.
#pragma once
#include "fn_internal.h"
#include "fn_kernels.h"

namespace fn {

// Deviate pair d of walker w (d < ceil(3N/2): coordinates 2 d and 2 d + 1,
// x' = x + sigma z rounded as a product and then a sum, no fused
// multiply-add), or its accept uniform (d == ceil(3N/2)).  The generator
// counter takes the walker's index within its own job, wl.
__device__ inline void propose_item(const double *x, int64_t w, int64_t wl, int d, int n3, double sigma, uint32_t k0,
                                    uint32_t k1, uint32_t step, uint32_t stream_id, const double *z_ext,
                                    const double *u_ext, double *xp, double *u)
{
#pragma clang fp contract(off)
    const int D = (n3 + 1) / 2;
    if (d == D) {
        if (u_ext) {
            u[w] = u_ext[w];
        } else {
            uint32_t c[4] = {0xFFFFFFFFu, (uint32_t)wl, step, stream_id};
            philox4x32_10(c, k0, k1);
            u[w] = word_pair_to_unit(c[0], c[1]);
        }
        return;
    }
    double z0, z1;
    if (z_ext) {
        z0 = z_ext[w * n3 + 2 * d];
        z1 = 2 * d + 1 < n3 ? z_ext[w * n3 + 2 * d + 1] : 0.0;
    } else {
        uint32_t c[4] = {(uint32_t)d, (uint32_t)wl, step, stream_id};
        philox4x32_10(c, k0, k1);
        const double u1 = word_pair_to_unit(c[0], c[1]), u2 = word_pair_to_unit(c[2], c[3]);
        const double rad = sqrt(-2.0 * log(u1));
        const double ang = 2.0 * M_PI * u2;
        z0 = rad * cos(ang);
        z1 = rad * sin(ang);
    }
    const double s0 = sigma * z0;
    xp[w * n3 + 2 * d] = x[w * n3 + 2 * d] + s0;
    if (2 * d + 1 < n3) {
        const double s1 = sigma * z1;
        xp[w * n3 + 2 * d + 1] = x[w * n3 + 2 * d + 1] + s1;
    }
}

// the job of walker w: the last one with w0 <= w
__device__ inline int group_job(const GroupTable &g, int64_t w)
{
    int lo = 0, hi = g.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (g.w0[mid] <= w) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

}  // namespace fn
