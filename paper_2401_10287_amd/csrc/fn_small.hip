// fn_small.hip -- log|psi| and the Metropolis walk of small FP64 networks (up
// to 4 electrons, layers of up to 64, all parameters in LDS) in one launch.
//
// What bounds it: latency.  Layer by layer, a move of the 2-electron network
// (2 layers 32/8, 2 determinants, 256 walkers) is 12 launches of 3 to 30 us for
// some 20 kFLOP per walker.  Here a wave owns a walker: the parameters are
// copied to LDS once per workgroup, every stage runs over its items with the
// lanes of the wave and hands its results on through LDS, and the moves of a
// call follow each other without leaving the kernel (walkers do not interact).
// 256 walkers: log|psi| 67 -> 15 us per call, ten moves 700 -> 120 us.
#include "fn_env.h"
#include "fn_internal.h"
#include "fn_kernels.h"
#include "fn_sample.h"

namespace fn {

namespace {

constexpr int SM_ELEC = 4, SM_W1 = 64, SM_W2 = 32, SM_DET = 16;

__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// offsets in doubles of a wave's scratch
struct SmallScratch {
    int x, xp, u, h[2], g, p[2], gi, A, total;
};
__host__ __device__ inline SmallScratch small_scratch(const Sys &s)
{
    const int wm = s.w1 > 4 * s.M ? s.w1 : 4 * s.M, pm = s.w2 > 4 ? s.w2 : 4;
    SmallScratch c;
    int o = 0;
    c.x = o; o += 3 * SM_ELEC;
    c.xp = o; o += 3 * SM_ELEC;
    c.u = o; o += 2;
    for (int b = 0; b < 2; ++b) { c.h[b] = o; o += s.N * wm; }
    c.g = o; o += 2 * wm;
    for (int b = 0; b < 2; ++b) { c.p[b] = o; o += s.N * s.N * pm; }
    c.gi = o; o += s.N * 2 * pm;
    c.A = o; o += 2 * s.K * SM_ELEC * SM_ELEC;
    c.total = (o + 1) / 2 * 2;
    return c;
}

// sum_k a[k] V[k ld], k < n, four chains
__device__ __forceinline__ void dot4(const double *a, const double *V, int ld, int n, double (&c)[4])
{
    int k = 0;
    for (; k + 8 <= n; k += 8)
#pragma unroll
        for (int q = 0; q < 8; ++q) c[q & 3] = fma(a[k + q], V[(k + q) * ld], c[q & 3]);
    for (; k < n; ++k) c[0] = fma(a[k], V[k * ld], c[0]);
}

// log|psi| and its sign for the walker at xs (LDS); every lane gets them
__device__ __forceinline__ double small_log_psi(const Sys &s, const ParamLayout &P, const SmallScratch &c,
                                                const double *th, double *sc, const double *xs, int &sign)
{
    const int lane = threadIdx.x & 63;
    const int N = s.N, nu = s.nu, nd = s.nd, M = s.M, K = s.K, w1 = s.w1, w2 = s.w2;
    const double iu = nu > 0 ? 1.0 / nu : 0.0, id = nd > 0 ? 1.0 / nd : 0.0;
    double *h = sc + c.h[0], *hn = sc + c.h[1], *p = sc + c.p[0], *pn = sc + c.p[1], *g = sc + c.g, *gi = sc + c.gi;
    for (int it = lane; it < N * M; it += 64) {
        const int i = it / M, m = it - i * M;
        const double d0 = xs[3 * i] - s.R[m][0], d1 = xs[3 * i + 1] - s.R[m][1], d2 = xs[3 * i + 2] - s.R[m][2];
        double *q = h + 4 * it;
        q[0] = d0; q[1] = d1; q[2] = d2;
        q[3] = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
    }
    for (int it = lane; it < N * N; it += 64) {
        const int i = it / N, j = it - i * N;
        const double d0 = xs[3 * i] - xs[3 * j], d1 = xs[3 * i + 1] - xs[3 * j + 1], d2 = xs[3 * i + 2] - xs[3 * j + 2];
        double *q = p + 4 * it;
        q[0] = d0; q[1] = d1; q[2] = d2;
        q[3] = i == j ? 0.0 : sqrt(d0 * d0 + d1 * d1 + d2 * d2);
    }
    wave_order();
    for (int l = 0; l < s.L; ++l) {
        const int dh = layer_dh(s, l), dp = layer_dp(s, l);
        for (int it = lane; it < 2 * dh; it += 64) {
            const int sp = it >= dh, k = it - sp * dh;
            double v = 0.0;
            for (int j = sp ? nu : 0; j < (sp ? N : nu); ++j) v += h[j * dh + k];
            g[it] = v * (sp ? id : iu);
        }
        for (int it = lane; it < N * 2 * dp; it += 64) {
            const int i = it / (2 * dp), q = it - i * 2 * dp, sp = q >= dp, k = q - sp * dp;
            double v = 0.0;
            for (int j = sp ? nu : 0; j < (sp ? N : nu); ++j) v += p[(i * N + j) * dp + k];
            gi[it] = v * (sp ? id : iu);
        }
        wave_order();
        const double *V = th + P.V[l], *b = th + P.b[l];
        for (int it = lane; it < N * w1; it += 64) {
            const int i = it / w1, u = it - i * w1;
            double a[4] = {b[u], 0.0, 0.0, 0.0};
            dot4(h + i * dh, V + u, w1, dh, a);
            dot4(g, V + dh * w1 + u, w1, 2 * dh, a);
            dot4(gi + i * 2 * dp, V + 3 * dh * w1 + u, w1, 2 * dp, a);
            const double y = tanh((a[0] + a[1]) + (a[2] + a[3]));
            hn[it] = l >= 1 ? y + h[it] : y;
        }
        if (l + 1 < s.L) {
            const double *W = th + P.W2[l], *c2 = th + P.c2[l];
            for (int it = lane; it < N * N * w2; it += 64) {
                const int ij = it / w2, o = it - ij * w2;
                double a[4] = {c2[o], 0.0, 0.0, 0.0};
                dot4(p + ij * dp, W + o, w2, dp, a);
                const double y = tanh((a[0] + a[1]) + (a[2] + a[3]));
                pn[it] = l >= 1 ? y + p[it] : y;
            }
        }
        wave_order();
        double *t = h; h = hn; hn = t;
        t = p; p = pn; pn = t;
    }
    // orbital matrices A[spin][k][orbital][electron] (Eq. 4)
    double *A = sc + c.A;
    for (int sp = 0; sp < 2; ++sp) {
        const int n = sp ? nd : nu, j0 = sp ? nu : 0, kn = K * n;
        for (int it = lane; it < n * kn; it += 64) {
            const int jj = it / kn, col = it - jj * kn, k = col / n, io = col - k * n;
            double a[4] = {th[P.g[sp] + col], 0.0, 0.0, 0.0};
            dot4(h + (j0 + jj) * w1, th + P.w[sp] + col, kn, w1, a);
            double env = 0.0, ge[3], le;
            for (int m = 0; m < M; ++m) env_add<double, false>(s, th, P.pi[sp], P.sig[sp], col, m, xs + 3 * (j0 + jj), env, ge, le);
            A[((sp * K + k) * SM_ELEC + io) * SM_ELEC + jj] = ((a[0] + a[1]) + (a[2] + a[3])) * env;
        }
    }
    wave_order();
    // lane (spin, k): elimination with row pivoting on the matrix padded with the identity
    double sg = 0.0, lg = -INFINITY;
    if (lane < 2 * K) {
        const int n = lane < K ? nu : nd;
        const double *a = A + lane * SM_ELEC * SM_ELEC;
        double v[SM_ELEC][SM_ELEC];
#pragma unroll
        for (int r = 0; r < SM_ELEC; ++r)
#pragma unroll
            for (int q = 0; q < SM_ELEC; ++q) v[r][q] = r < n && q < n ? a[r * SM_ELEC + q] : (r == q ? 1.0 : 0.0);
        bool sing = false;
        int sn = 1;
        double ll = 0.0;
#pragma unroll
        for (int q = 0; q < SM_ELEC; ++q) {
            if (q < n) {
                int pr = q;
                double best = fabs(v[q][q]);
#pragma unroll
                for (int r = q + 1; r < SM_ELEC; ++r) {
                    const double t = fabs(v[r][q]);
                    if (r < n && t > best) { best = t; pr = r; }
                }
                sing = sing || best == 0.0;
#pragma unroll
                for (int r = q + 1; r < SM_ELEC; ++r) {
                    const bool sw = pr == r;
#pragma unroll
                    for (int y = 0; y < SM_ELEC; ++y) {
                        const double t = v[q][y];
                        v[q][y] = sw ? v[r][y] : t;
                        v[r][y] = sw ? t : v[r][y];
                    }
                }
                if (pr != q) sn = -sn;
                if (v[q][q] < 0.0) sn = -sn;
                ll += log(fabs(v[q][q]));
                const double ip = 1.0 / v[q][q];
#pragma unroll
                for (int r = q + 1; r < SM_ELEC; ++r) {
                    const double f = v[r][q] * ip;
#pragma unroll
                    for (int y = q + 1; y < SM_ELEC; ++y) v[r][y] -= f * v[q][y];
                }
            }
        }
        sg = sing ? 0.0 : (double)sn;
        lg = sing ? -INFINITY : ll;
    }
    // determinant k: spin-down factor from lane K + k; FP64 log-sum over k
    const int src = lane < K ? lane + K : lane;
    const double sd = __shfl(sg, src, 64), ld = __shfl(lg, src, 64);
    const double sk = lane < K ? sg * sd : 0.0, lk = sk != 0.0 ? lg + ld : -INFINITY;
    double lmax = lk;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) lmax = fmax(lmax, __shfl_xor(lmax, off, 64));
    const double sum = wave_sum(sk != 0.0 ? sk * exp(lk - lmax) : 0.0);
    const bool node = !(lmax > -INFINITY) || sum == 0.0 || !(sum == sum);
    sign = node ? 0 : (sum > 0 ? 1 : -1);
    return node ? -INFINITY : lmax + log(fabs(sum));
}

// n_steps = 0: log|psi| and sign of x; else the moves of the job table's
// walkers (or with the caller's deviates z, u), in place on x and log_abs
__global__ __launch_bounds__(256) void k_small_walk(Sys s, ParamLayout P, const double *theta, double *x, double *log_abs,
                                                    int8_t *sign, int64_t B, int n_steps, double sigma, GroupTable g,
                                                    const double *z, const double *u, int32_t *n_accept, int nw)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    double *th = (double *)smem_raw;
    const int64_t np = P.total;
    for (int64_t q = threadIdx.x; q < np; q += blockDim.x) th[q] = theta[q];
    __syncthreads();
    const SmallScratch c = small_scratch(s);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n3 = 3 * s.N, D = (n3 + 1) / 2;
    const int64_t w = (int64_t)blockIdx.x * nw + wave;
    if (wave >= nw || w >= B) return;
    double *sc = th + (np + 1) / 2 * 2 + wave * c.total, *xc = sc + c.x, *xp = sc + c.xp, *us = sc + c.u;
    if (lane < n3) xc[lane] = x[w * n3 + lane];
    wave_order();
    int sn;
    if (n_steps == 0) {
        const double lp = small_log_psi(s, P, c, th, sc, xc, sn);
        if (lane == 0) {
            log_abs[w] = lp;
            if (sign) sign[w] = (int8_t)sn;
        }
        return;
    }
    const int job = group_job(g, w);
    double lp = log_abs[w];
    int taken = 0;
    for (int k = 0; k < n_steps; ++k) {
        if (lane <= D)
            propose_item(xc, 0, w - g.w0[job], lane, n3, sigma, g.k0[job], g.k1[job], g.step[job] + (uint32_t)k, g.stream[job],
                         z ? z + ((int64_t)k * B + w) * n3 : nullptr, u ? u + (int64_t)k * B + w : nullptr, xp, us);
        wave_order();
        const double lpn = small_log_psi(s, P, c, th, sc, xp, sn);
        if (isfinite(lpn) && log(us[0]) <= 2.0 * (lpn - lp)) {
            lp = lpn;
            ++taken;
            if (lane < n3) xc[lane] = xp[lane];
        }
        wave_order();
    }
    if (lane < n3) x[w * n3 + lane] = xc[lane];
    if (lane == 0) {
        log_abs[w] = lp;
        if (n_accept) n_accept[w] += taken;
    }
}

}  // namespace

namespace {

size_t small_lds(const Sys &s, const ParamLayout &P, int nw)
{
    return ((size_t)(P.total + 1) / 2 * 2 + (size_t)nw * small_scratch(s).total) * sizeof(double);
}

// walkers of a workgroup: one while that leaves CUs idle; beyond, up to four share
// the parameters (all four waves copy them in either case)
int small_waves(const Sys &s, const ParamLayout &P, int64_t B)
{
    int nw = B <= 256 ? 1 : (B <= 512 ? 2 : 4);
    while (nw > 1 && small_lds(s, P, nw) > 64 * 1024) nw /= 2;
    return nw;
}

}  // namespace

// Parameters and one walker's scratch within 64 KB of LDS, and a batch of at most
// four rounds of the walkers that the chip holds at once (256 CUs of 160 KB): a
// round costs the same again, the layers' own kernels only their rows.  Measured
// here / layer by layer, us per log|psi|: 4500 parameters, 4096 walkers 31 / 85,
// 16384 (six rounds) 94 / 142; 7073 parameters (one walker per workgroup), 1024
// walkers 48 / 82, 2048 (four rounds) 92 / 95, 4096 181 / 116.
// Where results must not depend on the batch (grouped and served calls, "gemm_splitk"
// off) the network alone decides: four walkers of a workgroup have to fit.  Ten
// moves of such networks, group of 256 / 4096 / 65536: 4500 parameters 121 / 275 /
// 3554 here, 698 / 868 / 4020 layer by layer; 5484 parameters (about the
// most that fit) 164 / 415 / 6028 and 734 / 974 / 4595 (level at 16384).  Larger ones (one or two
// walkers) lose from about 2000 walkers on: 7073 parameters, 256 / 2048 / 16384:
// 210 / 834 / 6527 and 762 / 969 / 2872.
bool small_walk_supported(const Sys &s, const ParamLayout &P, int64_t B)
{
    if (s.N > SM_ELEC || s.w1 > SM_W1 || s.w2 > SM_W2 || s.K > SM_DET) return false;
    if (small_lds(s, P, 1) > 64 * 1024) return false;
    if (g_splitk_suppressed || !g_gemm_splitk) return small_lds(s, P, 4) <= 64 * 1024;
    const int nw = small_waves(s, P, B);
    return B <= 4 * 256 * (int64_t)(160 * 1024 / small_lds(s, P, nw)) * nw;
}

void launch_small_walk(const Sys &s, const ParamLayout &P, const double *theta, double *x, double *log_abs, int8_t *sign,
                       int64_t B, int n_steps, double sigma, const GroupTable &g, const double *z, const double *u,
                       int32_t *n_accept, hipStream_t st)
{
    const int nw = small_waves(s, P, B);
    hipLaunchKernelGGL(k_small_walk, dim3((unsigned)((B + nw - 1) / nw)), dim3(256), small_lds(s, P, nw), st, s, P, theta, x,
                       log_abs, sign, B, n_steps, sigma, g, z, u, n_accept, nw);
}

}  // namespace fn
