// fn_det.hip -- orbitals, envelope and determinants of one spin in one pass
// (Eq. 4 with the product rule; the record of k_orbdet in fn_net.hip), for
// spins of 3 to 10 electrons: one wave per determinant, one direction per lane.
//
//   A[i][j] = a_ij e_ij,  d_c A = (d_c a) e + a d_c e,
//   lap A = (lap a) e + a lap e + 2 grad_j a . grad_j e,  M_c = A^-1 d_c A,
//   d log|det| / dx_c = tr M_c,  lap log|det| = tr(A^-1 lap A) - sum_c tr(M_c M_c).
//
// What bounds it: FP64 arithmetic and the latency of its operands.  The
// wave-per-determinant kernel in fn_net.hip solves every column of every
// direction against LU factors in LDS, searches pivots in one lane, and its
// determinants of one walker land on all eight XCDs, so each XCD fetches the
// head's rows for 4 n of their 64 n bytes.  Here
//   - the inverse is formed once, by elimination with row pivoting on [A | I]
//     with a column per lane, the matrix in registers;
//   - a lane owns a direction: it forms two columns of d_c A at a time from the
//     head's rows (read row by row by consecutive lanes and turned in LDS),
//     multiplies them with the inverse (LDS, the same address for all lanes) and
//     accumulates tr M and tr M M from the columns and the entries below the
//     diagonal of earlier ones: nothing is exchanged between lanes;
//   - the Laplacian's trace needs one product per entry and is taken where the
//     entry's envelope is formed;
//   - a workgroup takes the same determinant of four walkers, which share its
//     envelope parameters in LDS, and all determinants of those walkers go to
//     one XCD.
// Determinant stage of a local energy, before -> after: 12 electrons, 4096
// walkers 1.29 -> 0.52 ms; 20 electrons, 8192 walkers 12.6 -> 9.7 ms; 7 electrons,
// 257 walkers 51 -> 24 us.
#include "fn_env.h"
#include "fn_internal.h"
#include "fn_kernels.h"
#include "fn_rules.h"

namespace fn {

namespace {

constexpr int DET_WAVES = 4;

// LDS written by some lanes of this wave is read by others: a wave's LDS
// operations execute in order, so only the compiler has to keep theirs
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ double read_lane(double v, int l)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, l), hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), l);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// A determinant's NS values of a row of the head's output, in vectors of V.
template <typename T, int NS>
struct DetRow {
    static constexpr int V = NS % 2 == 0 ? 2 : 1;                // values per load
    static constexpr int NL = NS / V;                            // loads per row, and per lane and 64 rows
    static constexpr int RS = (NL % 2 ? NL : NL + 1) * V;        // row stride in LDS: an odd number of vectors
};

// LDS bytes per wave: A then its inverse [n][n]; with the directions the
// envelope [n][n], a grad e [n][3][n] and 64 rows of the head's output
template <typename T, int NS, bool FL>
constexpr int det_wave_bytes()
{
    return ((FL ? 5 : 1) * NS * NS * 8 + 15) / 16 * 16 + (FL ? 64 * DetRow<T, NS>::RS * (int)sizeof(T) : 0);
}

inline int64_t det_params(const Sys &s, int n) { return ((int64_t)n * s.M * (s.iso ? 2 : 10) + n + 3) / 4 * 4; }

// ST: the determinant's envelope parameters and offsets in LDS (else read
// where they are); the values and the arithmetic are the same
template <typename T, int NS, bool FL, bool ST>
__global__ __launch_bounds__(64 * DET_WAVES) void k_orbdet_lanes(Sys s, const double *x, const T *theta, OrbSpins<T> S,
                                                                 int sp0, int64_t B, int TR, double *DR, int rec,
                                                                 int per, int nprm)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    constexpr int NN = NS * NS, NQ = (NN + 63) / 64;
    const int bid = (int)blockIdx.x % per, sp = sp0 + (int)blockIdx.x / per;
    int64_t gof = sp ? S.gof1 : S.gof0, piof = sp ? S.piof1 : S.piof0, sigof = sp ? S.sigof1 : S.sigof0;
    const int64_t ldo = sp ? S.ldo1 : S.ldo0;
    const T *O = sp ? S.O1 : S.O0;
    const int j0 = sp == 0 ? 0 : s.nu, n3 = 3 * s.N;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // four walkers' determinants k = 0 .. K - 1 follow each other on one XCD
    const int k = (bid >> 3) % s.K;
    const int64_t w = ((int64_t)((bid >> 3) / s.K) * 8 + (bid & 7)) * DET_WAVES + wave;
    const T *tp = theta;
    if constexpr (ST) {
        T *prm = (T *)smem_raw;
        const int64_t c0 = (int64_t)k * NS, npi = (int64_t)NS * s.M, sz = s.iso ? 1 : 9, nsg = npi * sz;
        for (int q = tid; q < npi + nsg + NS; q += 64 * DET_WAVES)
            prm[q] = q < npi ? theta[piof + c0 * s.M + q]
                             : (q < npi + nsg ? theta[sigof + c0 * s.M * sz + (q - npi)] : theta[gof + c0 + (q - npi - nsg)]);
        __syncthreads();
        // offsets such that column k NS + io lands on staged row io
        tp = prm;
        piof = -c0 * s.M;
        sigof = npi - c0 * s.M * sz;
        gof = npi + nsg - c0;
    }
    if (w >= B) return;
    double *AI = (double *)(smem_raw + (size_t)nprm * sizeof(T) + wave * det_wave_bytes<T, NS, FL>());
    double *EV = AI + NN, *U = EV + NN;

    // envelope and orbital value of every entry; its part of lap A stays in the lane
    double dl[NQ];
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        const int q = lane + 64 * u;
        dl[u] = 0.0;
        if (q < NN) {
            const int jj = q / NS, io = q - jj * NS, col = k * NS + io, j = j0 + jj;      // electron, orbital
            const double *xj = x + (w * s.N + j) * 3;
            const T *Oq = O + (w * NS + jj) * TR * ldo + col;
            double env = 0.0, ge[3] = {0.0, 0.0, 0.0}, le = 0.0;
            T ol = T(0), oa[3] = {T(0), T(0), T(0)};
            const T o0 = Oq[0];
            if constexpr (FL) {
                ol = Oq[(n3 + 1) * ldo];
#pragma unroll
                for (int a = 0; a < 3; ++a) oa[a] = Oq[(1 + 3 * j + a) * ldo];
            }
            for (int m = 0; m < s.M; ++m) env_add<T, FL>(s, tp, piof, sigof, col, m, xj, env, ge, le);
            const double a0 = (double)o0 + (double)tp[gof + col];
            AI[io * NS + jj] = a0 * env;
            if constexpr (FL) {
                EV[q] = env;
                double d = env * (double)ol + a0 * le;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    U[(3 * jj + a) * NS + io] = a0 * ge[a];
                    d += 2.0 * (double)oa[a] * ge[a];
                }
                dl[u] = d;
            }
        }
    }
    wave_order();
    // elimination with row pivoting (the first row of the largest magnitude):
    // lane c < NS holds column c of A, lane NS + c column c of the identity
    double v[NS];
#pragma unroll
    for (int r = 0; r < NS; ++r) v[r] = lane < NS ? AI[r * NS + (lane < NS ? lane : 0)] : (lane - NS == r ? 1.0 : 0.0);
    int sgn = 1;
    bool sing = false;
    double mypiv = 1.0;
#pragma unroll
    for (int c = 0; c < NS; ++c) {
        double f[NS];
#pragma unroll
        for (int r = 0; r < NS; ++r) f[r] = FL || r >= c ? read_lane(v[r], c) : 0.0;
        int p = c;
        double best = fabs(f[c]);
#pragma unroll
        for (int r = c + 1; r < NS; ++r) {
            const double a = fabs(f[r]);
            if (a > best) { best = a; p = r; }
        }
        sing = sing || best == 0.0;
#pragma unroll
        for (int r = c + 1; r < NS; ++r) {
            const bool sw = p == r;
            const double tv = v[c], tf = f[c];
            v[c] = sw ? v[r] : tv;
            v[r] = sw ? tv : v[r];
            f[c] = sw ? f[r] : tf;
            f[r] = sw ? tf : f[r];
        }
        if (p != c) sgn = -sgn;
        if (f[c] < 0.0) sgn = -sgn;
        mypiv = lane == c ? fabs(f[c]) : mypiv;
        const double ip = 1.0 / f[c];
        if constexpr (FL) {
            // multipliers first, as in the value form: pivots, sign and log|det| are then the
            // same bits there (with v[c] scaled first, equal columns can cancel to exact zeros
            // that the value form does not get: a node here and a finite log|psi| there)
#pragma unroll
            for (int r = 0; r < NS; ++r)
                if (r != c) v[r] -= (f[r] * ip) * v[c];
            v[c] *= ip;
        } else {
#pragma unroll
            for (int r = c + 1; r < NS; ++r) v[r] -= (f[r] * ip) * v[c];
        }
    }
    double *out = DR + (w * 2 + sp) * (int64_t)s.K * rec + (int64_t)k * rec;
    if (sing) {
        for (int q = lane; q < rec; q += 64) out[q] = q == 0 ? 0.0 : (q == 1 ? -INFINITY : NAN);
        return;
    }
    const double lg = wave_sum(lane < NS ? log(mypiv) : 0.0);
    if (lane == 0) {
        out[0] = (double)sgn;
        out[1] = lg;
    }
    if constexpr (FL) {
        // inverse [electron][orbital]
        if (lane >= NS && lane < 2 * NS)
#pragma unroll
            for (int r = 0; r < NS; ++r) AI[r * NS + lane - NS] = v[r];
        wave_order();
        double lap = 0.0;
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
            const int q = lane + 64 * u;
            if (q < NN) lap += dl[u] * AI[q];
        }
        typedef DetRow<T, NS> H;
        constexpr int V = H::V, NL = H::NL, RS = H::RS, CW = NS == 1 ? 1 : 2;
        typedef T vec __attribute__((ext_vector_type(V)));
        T *row = (T *)(smem_raw + (size_t)nprm * sizeof(T) + wave * det_wave_bytes<T, NS, FL>() + (5 * NN * 8 + 15) / 16 * 16);
        const T *Ow = O + w * NS * TR * ldo + k * NS;
        const int64_t estep = (int64_t)TR * ldo;
        for (int d0 = 0; d0 < n3; d0 += 64) {
            const int d = d0 + lane, nd = n3 - d0 < 64 ? n3 - d0 : 64;
            const bool act = lane < nd;
            const int je = d / 3 - j0, ax = d % 3;               // electron of the direction within the spin, axis
            // consecutive lanes read the determinant's values row by row, one
            // column ahead; LDS turns them to a row per lane
            int off[NL], put[NL];
#pragma unroll
            for (int l = 0; l < NL; ++l) {
                const int q = lane + 64 * l, rq = q / NL, pc = q - rq * NL;
                off[l] = (1 + d0 + (rq < nd ? rq : nd - 1)) * (int)ldo + V * pc;
                put[l] = rq * RS + V * pc;
            }
            vec nx[NL];
#pragma unroll
            for (int l = 0; l < NL; ++l) nx[l] = *(const vec *)(Ow + off[l]);
            double tr = 0.0, sq = 0.0, low[NS][NS];
#pragma unroll
            for (int c0 = 0; c0 < NS; c0 += CW) {
                double D[CW][NS], up = 0.0;       // up: M[c0][c0 + 1]
#pragma unroll
                for (int y = 0; y < CW; ++y) {
                    const int c = c0 + y;
                    if (c >= NS) continue;
                    wave_order();
#pragma unroll
                    for (int l = 0; l < NL; ++l) *(vec *)(row + put[l]) = nx[l];
                    wave_order();
                    if (c + 1 < NS)
#pragma unroll
                        for (int l = 0; l < NL; ++l) nx[l] = *(const vec *)(Ow + (c + 1) * estep + off[l]);
                    const bool own = je == c;
#pragma unroll
                    for (int l = 0; l < NL; ++l) {
                        const vec o = *(const vec *)(row + lane * RS + V * l);
#pragma unroll
                        for (int z = 0; z < V; ++z) {
                            const int i = V * l + z;
                            D[y][i] = EV[c * NS + i] * (double)o[z];
                        }
                    }
                    if (own)
#pragma unroll
                        for (int i = 0; i < NS; ++i) D[y][i] += U[(3 * c + ax) * NS + i];
                }
#pragma unroll
                for (int r = 0; r < NS; ++r) {
                    double m[CW];
#pragma unroll
                    for (int y = 0; y < CW; ++y) m[y] = 0.0;
#pragma unroll
                    for (int i = 0; i < NS; ++i) {
                        const double a = AI[r * NS + i];
#pragma unroll
                        for (int y = 0; y < CW; ++y)
                            if (c0 + y < NS) m[y] = fma(a, D[y][i], m[y]);
                    }
                    // M[r][c]: on the diagonal, above it (its mirror is there), or below it
#pragma unroll
                    for (int y = 0; y < CW; ++y) {
                        const int c = c0 + y;
                        if (c >= NS) continue;
                        if (r == c) {
                            tr += m[y];
                            sq = fma(m[y], m[y], sq);
                        } else if (r > c) {
                            low[r][c] = m[y];
                            if (r < c0 + CW) sq = fma(2.0 * m[y], up, sq);
                        } else if (r >= c0) {
                            up = m[y];
                        } else {
                            sq = fma(2.0 * m[y], low[c][r], sq);
                        }
                    }
                }
                // the sums are taken here (left to the compiler, they sink to
                // their last use and every M stays live until then)
                asm volatile("" : "+v"(tr), "+v"(sq));
            }
            if (act) {
                out[2 + d] = tr;
                lap -= sq;
            }
        }
        lap = wave_sum(lap);
        if (lane == 0) out[2 + n3] = lap;
    }
}

}  // namespace

template <typename T, int NS, bool FL>
static void launch_lanes(const Sys &s, const double *x, const T *theta, const OrbSpins<T> &S, int sp0, int nsp,
                         int64_t B, int TR, double *DR, int rec, hipStream_t st)
{
    const int64_t groups = (B + DET_WAVES - 1) / DET_WAVES;
    const int per = (int)((groups + 7) / 8 * 8 * s.K);
    const int64_t nprm = det_params(s, NS);
    const size_t base = (size_t)DET_WAVES * det_wave_bytes<T, NS, FL>();
    const dim3 grid((unsigned)(nsp * per)), block(64 * DET_WAVES);
    if (g_det_stage && base + nprm * sizeof(T) <= 64 * 1024)
        hipLaunchKernelGGL((k_orbdet_lanes<T, NS, FL, true>), grid, block, base + nprm * sizeof(T), st, s, x, theta, S, sp0,
                           B, TR, DR, rec, per, (int)nprm);
    else
        hipLaunchKernelGGL((k_orbdet_lanes<T, NS, FL, false>), grid, block, base, st, s, x, theta, S, sp0, B, TR, DR, rec,
                           per, 0);
}

template <typename T>
bool launch_orbdet_lanes(const Sys &s, const double *x, const T *theta, const OrbSpins<T> &S, int sp0, int nsp, int n,
                         int64_t B, int TR, bool fl, double *DR, int rec, hipStream_t st)
{
    if (B * s.K * nsp > (int64_t)1 << 31) return false;
    if (fl) {
        if (!det_lanes_fl(n, s.N, s.M, sizeof(T) == 8)) return false;
        switch (n) {
#define FN_LANES(NS)                                                                              \
    case NS: launch_lanes<T, NS, true>(s, x, theta, S, sp0, nsp, B, TR, DR, rec, st); return true;
            FN_LANES(3) FN_LANES(4) FN_LANES(5) FN_LANES(6) FN_LANES(7) FN_LANES(8) FN_LANES(9) FN_LANES(10)
#undef FN_LANES
        default: return false;
        }
    }
    switch (n) {
    case 9: launch_lanes<T, 9, false>(s, x, theta, S, sp0, nsp, B, TR, DR, rec, st); return true;
    case 10: launch_lanes<T, 10, false>(s, x, theta, S, sp0, nsp, B, TR, DR, rec, st); return true;
    default: return false;
    }
}

template bool launch_orbdet_lanes<float>(const Sys &, const double *, const float *, const OrbSpins<float> &, int, int,
                                         int, int64_t, int, bool, double *, int, hipStream_t);
template bool launch_orbdet_lanes<double>(const Sys &, const double *, const double *, const OrbSpins<double> &, int, int,
                                          int, int64_t, int, bool, double *, int, hipStream_t);

}  // namespace fn
