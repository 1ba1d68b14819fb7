// fn_walk.hip -- one one-electron stream layer in forward-Laplacian form (the
// layer of fn_layer.hip, bit for bit) for 5 to 20 electrons, by workgroups
// that walk over the electrons of whole walkers.
//
// What bounds it: HBM.  A layer reads and writes every row of h once (20
// electrons, 62 rows: 143 KB per electron with the pair means, 18.7k cycles of a
// CU's share of the rate of a copy; it takes about 21k).  The tiled kernel
// fetches its weights and splits its activations once per 128 x 128 tile and
// column half, and the spin means of the next layer need another pass over the
// rows it has written.  Here
//   - each of a workgroup's four waves keeps the weights of its 32 output
//     columns (16 with three weight parts) in registers for the whole launch;
//   - the electrons of a walker come one after the other: their rows are
//     requested two steps ahead (also across electrons and walkers), split once
//     for the workgroup's columns and put into LDS, double buffered, one barrier
//     per two steps (per step with four row blocks: LDS);
//   - a wave holds all 16-row blocks of an electron, so the value row, the
//     tangent rows and the Laplacian row of a column meet in one wave;
//   - the products are transposed (D^T = W X^T), so that a lane ends up with
//     four consecutive columns of a row: 16-byte loads and stores;
//   - the running spin means of h^{l+1} are kept in LDS and written when the
//     last electron of a spin is done, added in the order of the separate pass;
//   - two workgroups per CU, so that one's products run under the other's
//     epilogue (one workgroup of eight waves in step: 19k cycles per electron of
//     12-electron walkers against 15k).
// Stream layers and spin means of a local energy, tiled -> here: 12 electrons,
// 4096 walkers 9.5 -> 5.6 ms; 20 electrons, 8192 walkers 41.8 -> 26.6 ms.
#include "fn_internal.h"
#include "fn_kernels.h"
#include "fn_rules.h"

namespace fn {

namespace {

#pragma clang fp contract(off)

constexpr int WALK_WAVES = 4;

// LDS written by some lanes of this wave is read by others: a wave's LDS
// operations execute in order, so only the compiler has to keep theirs
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// workgroup barrier over LDS contents; global loads stay in flight
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int MODE, int LIVE, int KS>
struct WalkShape {
    static constexpr int NA = act_parts(MODE), NW = weight_parts(MODE);
    static constexpr int WJ = NW == 1 ? 2 : 1;                   // 16-column blocks of a wave
    static constexpr int NCG = 256 / (16 * WJ * WALK_WAVES);     // column groups
    static constexpr int D = KS == 10 ? 2 : KS;                  // steps requested ahead
    static constexpr int SP = LIVE == 4 ? 1 : 2;                 // steps per barrier
    static constexpr int SV = LIVE == 3 ? 2 : 4, SN = LIVE == 3 ? 3 : LIVE / 2;   // staging: SN vectors of SV inputs per thread
    static constexpr int PART = LIVE * 16 * 64;                  // bytes of one part of one step
    static constexpr int STEP = NA * PART;
    static constexpr int SST = 16 * 16 + 16;                     // scratch floats of one 16-row block (padded)
    static constexpr int SSZ = (LIVE * SST + 5 * 16 + 16 * WJ) * 4;   // per wave: tangents of 16 columns, tables, bias
    static constexpr int K1 = KS == 10 ? 256 : 32 * (KS - 1);    // inputs that are h (the rest: pair means)
    static constexpr int MSZ = WALK_WAVES * LIVE * WJ * 1024;    // running spin means
    static constexpr int OSCR = 2 * SP * STEP, OMEAN = OSCR + WALK_WAVES * SSZ, SMEM = OMEAN + MSZ;
    static constexpr int GI = 1;              // row blocks whose fragments are held together (more spill)
    static constexpr bool RESID = KS == 10;                      // 256 inputs: h^l is added to the output
};

// GOUT: the next layer's spin means are wanted
template <int MODE, int LIVE, int KS, bool GOUT>
__global__ __launch_bounds__(64 * WALK_WAVES, 2) void k_walk_layer(LayerArgs a, int TR, int64_t B)
{
    typedef WalkShape<MODE, LIVE, KS> S;
    constexpr int NA = S::NA, NW = S::NW, WJ = S::WJ, SST = S::SST, D = S::D;
    constexpr int LD = 256;                            // row length of h (in and out) and of the per-walker part
    __shared__ __attribute__((aligned(16))) unsigned char smem[S::SMEM];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // column groups of a walker 8 workgroups apart: same XCD, at the same time
    const int bid = blockIdx.x;
    const int cg = (bid >> 3) % S::NCG;
    const int blk = (bid & 7) + 8 * (bid / (8 * S::NCG)), nblk = gridDim.x / S::NCG;
    if (blk >= B) return;
    const int r = lane & 15, q = lane >> 4;
    const int n0 = (cg * WALK_WAVES + wave) * 16 * WJ;
    const int n3 = a.n3, tl = n3 + 1, N = a.N, nu = a.nu, nd = N - nu;

    bf16x8 hb[KS][NW][WJ];
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
        for (int p = 0; p < NW; ++p)
#pragma unroll
            for (int j = 0; j < WJ; ++j)
                hb[k][p][j] = *(const bf16x8 *)((const uint16_t *)a.W + (int64_t)p * a.wpart +
                                                (int64_t)(n0 + 16 * j + r) * a.ldw + 32 * k + 8 * q);

    // operand staging: vector v of a thread is SV consecutive inputs of row
    // srow + SROW v; rows past the Laplacian row take that row again (never stored)
    constexpr int SV = S::SV, SN = S::SN, SROW = 64 * WALK_WAVES * SV / 32;
    typedef typename std::conditional<SV == 4, float4, float2>::type svec;
    const int srow = tid / (32 / SV), sk = SV * (tid % (32 / SV));
    int s1[SN], s2[SN];
#pragma unroll
    for (int v = 0; v < SN; ++v) {
        const int t = srow + SROW * v < tl ? srow + SROW * v : tl;
        s1[v] = t * LD + sk;
        s2[v] = t * (int)a.lda2 + sk;
    }
    // (the chunk slot of a row repeats every 16 rows)
    const int swr = srow * 64 + 16 * lds_chunk(srow, sk >> 3) + 2 * (sk & 7);
    const int srd = r * 64 + 16 * lds_chunk(r, q);
    const int64_t e1 = (int64_t)TR * LD, e2 = (int64_t)TR * a.lda2;
    // the electron that follows electron (w, e) of this workgroup's walkers;
    // after the last one that one again
    struct Pos { int64_t w; int e; };
    auto next = [&](Pos p) {
        if (p.e + 1 < N) return Pos{p.w, p.e + 1};
        if (p.w + nblk < B) return Pos{p.w + nblk, 0};
        return p;
    };
    struct Step { svec v[SN]; };
    auto load = [&](Pos p, int k) {
        const int kb = 32 * k;
        const int64_t el = p.w * N + p.e;
        const float *s = kb < S::K1 ? a.A1 + el * e1 + kb : a.A2 + el * e2 + (kb - S::K1);
        Step x;
#pragma unroll
        for (int v = 0; v < SN; ++v) x.v[v] = *(const svec *)(s + (kb < S::K1 ? s1[v] : s2[v]));
        return x;
    };
    auto stage = [&](const Step &x, int slot) {
#pragma unroll
        for (int v = 0; v < SN; ++v) {
            unsigned char *d = smem + slot * S::STEP + swr + SROW * 64 * v;
            uint32_t a01[NA];
            split_bf16_pair<NA>(x.v[v].x, x.v[v].y, a01);
            if constexpr (SV == 4) {
                uint32_t a23[NA];
                split_bf16_pair<NA>(x.v[v].z, x.v[v].w, a23);
#pragma unroll
                for (int p = 0; p < NA; ++p) *(uint2 *)(d + p * S::PART) = make_uint2(a01[p], a23[p]);
            } else {
#pragma unroll
                for (int p = 0; p < NA; ++p) *(uint32_t *)(d + p * S::PART) = a01[p];
            }
        }
    };

    const int oo = r * LD + n0 + 4 * q;                // row r, this lane's columns (16 i rows further: block i)
    float *sz = (float *)(smem + S::OSCR + wave * S::SSZ), *tab = sz + LIVE * SST;
    f32x4 *mean = (f32x4 *)(smem + S::OMEAN + wave * LIVE * WJ * 1024) + lane;      // block (i, j) at 64 (i WJ + j)
    const int64_t ldg = 2 * (int64_t)a.W1p;
    const float iu = nu > 0 ? 1.f / nu : 0.f, id = nd > 0 ? 1.f / nd : 0.f;

    float *sb = tab + 80;
    if (lane < 16 * WJ) sb[lane] = a.bias[n0 + lane];
    if constexpr (GOUT)
#pragma unroll
        for (int i = 0; i < LIVE * WJ; ++i) mean[64 * i] = f32x4{0.f, 0.f, 0.f, 0.f};
    Pos p0{blk, 0}, p1 = next(p0), p2 = next(p1);
    Step pre[D];
#pragma unroll
    for (int k = 0; k < D; ++k) pre[k] = load(p0, k);
#pragma unroll
    for (int k = 0; k < S::SP; ++k) {
        stage(pre[k], k);
        pre[k] = D + k < KS ? load(p0, D + k) : load(p1, D + k - KS);
    }
    lds_barrier();
    int cur = 0;
    for (int64_t w = blk; w < B; w += nblk) {
        // the per-walker part; here and for the residual's rows, rows past the Laplacian
        // row (tl) hold whatever memory held: they stay in their own lane's rows, are masked
        // out of the Laplacian's source and never stored
        f32x4 pp[LIVE][WJ];
#pragma unroll
        for (int i = 0; i < LIVE; ++i)
#pragma unroll
            for (int j = 0; j < WJ; ++j) pp[i][j] = *(const f32x4 *)(a.Pw + w * e1 + oo + 16 * LD * i + 16 * j);
        for (int e = 0; e < N; ++e) {
            f32x4 acc[LIVE][WJ], rs[LIVE][WJ];
#pragma unroll
            for (int i = 0; i < LIVE; ++i)
#pragma unroll
                for (int j = 0; j < WJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            const int64_t el = w * N + e;
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                const int h = k % S::SP, n = k + S::SP;       // n: step staged now, n + D: step requested now
                const unsigned char *sa = smem + (S::SP * cur + h) * S::STEP;
                // the residual's rows, a block at a time (they have just been staged: L2)
                if constexpr (S::RESID)
                    if (k < LIVE * WJ)
                        rs[k / WJ][k % WJ] = *(const f32x4 *)(a.A1 + el * e1 + oo + 16 * LD * (k / WJ) + 16 * (k % WJ));
#pragma unroll
                for (int i0 = 0; i0 < LIVE; i0 += S::GI) {
                    bf16x8 ha[NA][S::GI];
#pragma unroll
                    for (int p = 0; p < NA; ++p)
#pragma unroll
                        for (int i = 0; i < S::GI; ++i) ha[p][i] = *(const bf16x8 *)(sa + srd + p * S::PART + (i0 + i) * 1024);
                    __builtin_amdgcn_s_setprio(1);
                    // products of an accumulator in the order of the tiled kernel, the accumulators in turn
#pragma unroll
                    for (int sum = NW == 1 ? 0 : NA - 1; sum >= 0; --sum)
#pragma unroll
                        for (int pa = 0; pa <= (NW == 1 ? NA - 1 : sum); ++pa)
#pragma unroll
                            for (int i = 0; i < S::GI; ++i)
#pragma unroll
                                for (int j = 0; j < WJ; ++j)
                                    acc[i0 + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                        hb[k][NW == 1 ? 0 : sum - pa][j], ha[pa][i], acc[i0 + i][j], 0, 0, 0);
                    __builtin_amdgcn_s_setprio(0);
                }
                stage(pre[n % D], S::SP * (cur ^ 1) + h);
                pre[n % D] = n + D < KS ? load(p0, n + D) : (n + D < 2 * KS ? load(p1, n + D - KS) : load(p2, n + D - 2 * KS));
                if (h == S::SP - 1) {
                    lds_barrier();
                    cur ^= 1;
                }
            }
            p0 = p1; p1 = p2; p2 = next(p2);
            // epilogue, 16 columns at a time: lane (r, q) holds columns 4 q .. 4 q + 3 of rows 16 i + r
            float *Ho = a.Hout + el * e1;
            const bool last = e == nu - 1 || e == N - 1;       // of its spin
            const int sp = e < nu ? 0 : 1;
            float *Gs = a.Gout + w * TR * ldg + sp * a.W1p + n0 + 4 * q;
            const float sc = sp ? id : iu;
#pragma unroll
            for (int j = 0; j < WJ; ++j) {
                const float4 b4 = *(const float4 *)(sb + 16 * j + 4 * q);
                f32x4 z[LIVE];
#pragma unroll
                for (int i = 0; i < LIVE; ++i) {
#pragma unroll
                    for (int x = 0; x < 4; ++x) z[i][x] = acc[i][j][x] + pp[i][j][x];
                    if (i == 0) {
                        const f32x4 zb = {z[0][0] + b4.x, z[0][1] + b4.y, z[0][2] + b4.z, z[0][3] + b4.w};
#pragma unroll
                        for (int x = 0; x < 4; ++x) z[0][x] = r == 0 ? zb[x] : z[0][x];
                    }
                    // (only the first block has the value row, only the last one rows past n3)
                    // tangent rows for the Laplacian's source; value and Laplacian rows for the column's derivatives
                    const int t = 16 * i + r;
                    f32x4 zt;
#pragma unroll
                    for (int x = 0; x < 4; ++x) zt[x] = (i > 0 || t > 0) && (i < LIVE - 1 || t < tl) ? z[i][x] : 0.f;
                    *(f32x4 *)(sz + i * SST + r * 16 + 4 * q) = zt;
                    if (i == 0 && t == 0) *(f32x4 *)(tab + 48 + 4 * q) = z[i];
                    if (i == LIVE - 1 && t == tl) *(f32x4 *)(tab + 64 + 4 * q) = z[i];
                }
                wave_lds_order();
                // lane (r, q): column r, the tangent rows of row block q summed in order
                const float *zc = sz + (q < LIVE ? q : 0) * SST + r;
                float src = 0.f;
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    const float v = zc[u * 16];
                    src = __builtin_fmaf(v, v, src);
                }
                float s = __shfl(src, r, 64);
#pragma unroll
                for (int i = 1; i < LIVE; ++i) s = s + __shfl(src, 16 * i + r, 64);
                const float z0 = tab[48 + r], zl = tab[64 + r];
                const float y0 = tanhf(z0);
                const float dd = __builtin_fmaf(-y0, y0, 1.f);
                const float lap = __builtin_fmaf(dd, zl, -(((2.f * y0) * dd) * s));
                tab[r] = y0;
                tab[16 + r] = dd;
                tab[32 + r] = lap;
                wave_lds_order();
                const f32x4 ty = *(const f32x4 *)(tab + 4 * q), td = *(const f32x4 *)(tab + 16 + 4 * q),
                            tp = *(const f32x4 *)(tab + 32 + 4 * q);
#pragma unroll
                for (int i = 0; i < LIVE; ++i) {
                    const int t = 16 * i + r;
                    f32x4 y;
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        float v = td[x] * z[i][x];
                        if (i == 0) v = t == 0 ? ty[x] : v;
                        if (i == LIVE - 1) v = t == tl ? tp[x] : v;
                        if constexpr (S::RESID) y[x] = v + rs[i][j][x];
                        else y[x] = v + 0.f;
                    }
                    if (i < LIVE - 1 || t <= tl) *(f32x4 *)(Ho + oo + 16 * LD * i + 16 * j) = y;
                    z[i] = y;
                }
                if constexpr (GOUT) {
                    f32x4 m[LIVE];
#pragma unroll
                    for (int i = 0; i < LIVE; ++i) {
                        m[i] = mean[64 * (i * WJ + j)];
#pragma unroll
                        for (int x = 0; x < 4; ++x) m[i][x] += z[i][x];
                    }
                    if (last) {
#pragma unroll
                        for (int i = 0; i < LIVE; ++i) {
                            const f32x4 g = {m[i][0] * sc, m[i][1] * sc, m[i][2] * sc, m[i][3] * sc};
                            if (i < LIVE - 1 || 16 * i + r <= tl) *(f32x4 *)(Gs + (16 * i + r) * ldg + 16 * j) = g;
                            m[i] = f32x4{0.f, 0.f, 0.f, 0.f};
                        }
                    }
#pragma unroll
                    for (int i = 0; i < LIVE; ++i) mean[64 * (i * WJ + j)] = m[i];
                }
                wave_lds_order();
            }
        }
        if (GOUT && (nu == 0 || nd == 0)) {          // the mean over no electrons is 0
            float *Gs = a.Gout + w * TR * ldg + (nu == 0 ? 0 : 1) * a.W1p + n0 + 4 * q;
#pragma unroll
            for (int i = 0; i < LIVE; ++i)
#pragma unroll
                for (int j = 0; j < WJ; ++j)
                    if (16 * i + r <= tl) *(float4 *)(Gs + (16 * i + r) * ldg + 16 * j) = make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
}

// The same layer on value rows only (no derivatives: log|psi| and Metropolis
// moves), flat rows of any number of electrons.  What bounds it: the vector ALUs
// (tanh of every output, the splits) about level with the matrix cores and the
// traffic of h.  As above weights stay in registers, rows are split once for a
// workgroup's columns, and the products are transposed; a tile is 32 rows, rows
// past the end repeat the last one (its outputs are stored again).
// Tiled -> here, a 256-wide layer: 12 electrons, 4096 walkers, three products 60
// -> 40 us (the features' layer 35 -> 21); 10 electrons, 2048 walkers, six
// products 38 -> 33 us.
template <int MODE, int KS>
struct ValueShape {
    static constexpr int NA = act_parts(MODE), NW = weight_parts(MODE);
    static constexpr int WJ = NW == 1 ? 2 : 1;
    static constexpr int NCG = 256 / (16 * WJ * WALK_WAVES);
    static constexpr int D = KS == 10 ? 5 : KS, SP = 2;
    static constexpr int PART = 2 * 16 * 64, STEP = NA * PART;
    static constexpr int K1 = KS == 10 ? 256 : 32 * (KS - 1);
    static constexpr bool RESID = KS == 10;
};

template <int MODE, int KS>
__global__ __launch_bounds__(64 * WALK_WAVES, 2) void k_walk_value(LayerArgs a)
{
    typedef ValueShape<MODE, KS> S;
    constexpr int NA = S::NA, NW = S::NW, WJ = S::WJ, D = S::D, LD = 256;
    __shared__ __attribute__((aligned(16))) unsigned char smem[2 * S::SP * S::STEP];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bid = blockIdx.x;
    const int cg = (bid >> 3) % S::NCG;
    const int64_t tiles = (a.rows + 31) / 32;
    const int blk = (bid & 7) + 8 * (bid / (8 * S::NCG)), nblk = gridDim.x / S::NCG;
    if (blk >= tiles) return;
    const int r = lane & 15, q = lane >> 4;
    const int n0 = (cg * WALK_WAVES + wave) * 16 * WJ;

    bf16x8 hb[KS][NW][WJ];
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
        for (int p = 0; p < NW; ++p)
#pragma unroll
            for (int j = 0; j < WJ; ++j)
                hb[k][p][j] = *(const bf16x8 *)((const uint16_t *)a.W + (int64_t)p * a.wpart +
                                                (int64_t)(n0 + 16 * j + r) * a.ldw + 32 * k + 8 * q);
    f32x4 bb[WJ];
#pragma unroll
    for (int j = 0; j < WJ; ++j) bb[j] = *(const f32x4 *)(a.bias + n0 + 16 * j + 4 * q);

    const int srow = tid >> 3, sk = 4 * (tid & 7);
    const int swr = srow * 64 + 16 * lds_chunk(srow, sk >> 3) + 2 * (sk & 7);
    const int srd = r * 64 + 16 * lds_chunk(r, q);
    auto clamp = [&](int64_t row) { return row < a.rows ? row : a.rows - 1; };
    auto load = [&](int64_t t, int k) {
        const int64_t row = clamp(32 * t + srow);
        return *(const float4 *)(32 * k < S::K1 ? a.A1 + row * LD + 32 * k + sk : a.A2 + row * a.lda2 + (32 * k - S::K1) + sk);
    };
    auto stage = [&](float4 x, int slot) {
        unsigned char *d = smem + slot * S::STEP + swr;
        uint32_t a01[NA], a23[NA];
        split_bf16_pair<NA>(x.x, x.y, a01);
        split_bf16_pair<NA>(x.z, x.w, a23);
#pragma unroll
        for (int p = 0; p < NA; ++p) *(uint2 *)(d + p * S::PART) = make_uint2(a01[p], a23[p]);
    };
    // the tile that follows tile t; after the last one that one again
    auto next = [&](int64_t t) { return t + nblk < tiles ? t + nblk : t; };
    int64_t t0 = blk, t1 = next(t0), t2 = next(t1);
    float4 pre[D];
#pragma unroll
    for (int k = 0; k < D; ++k) pre[k] = load(t0, k);
#pragma unroll
    for (int k = 0; k < S::SP; ++k) {
        stage(pre[k], k);
        pre[k] = D + k < KS ? load(t0, D + k) : load(t1, D + k - KS);
    }
    lds_barrier();
    int cur = 0;
    for (int64_t t = blk; t < tiles; t += nblk) {
        f32x4 acc[2][WJ], pw[2][WJ], rs[2][WJ];
        int64_t row[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            row[i] = clamp(32 * t + 16 * i + r);
            const int64_t w = row[i] / a.N;
#pragma unroll
            for (int j = 0; j < WJ; ++j) {
                acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                pw[i][j] = *(const f32x4 *)(a.Pw + w * LD + n0 + 16 * j + 4 * q);
                if constexpr (S::RESID) rs[i][j] = *(const f32x4 *)(a.A1 + row[i] * LD + n0 + 16 * j + 4 * q);
            }
        }
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const int h = k % S::SP, n = k + S::SP;       // n: step staged now, n + D: step requested now
            const unsigned char *sa = smem + (S::SP * cur + h) * S::STEP + srd;
            bf16x8 ha[NA][2];
#pragma unroll
            for (int p = 0; p < NA; ++p)
#pragma unroll
                for (int i = 0; i < 2; ++i) ha[p][i] = *(const bf16x8 *)(sa + p * S::PART + i * 1024);
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int sum = NW == 1 ? 0 : NA - 1; sum >= 0; --sum)
#pragma unroll
                for (int pa = 0; pa <= (NW == 1 ? NA - 1 : sum); ++pa)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < WJ; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hb[k][NW == 1 ? 0 : sum - pa][j], ha[pa][i],
                                                                                acc[i][j], 0, 0, 0);
            __builtin_amdgcn_s_setprio(0);
            stage(pre[n % D], S::SP * (cur ^ 1) + h);
            pre[n % D] = n + D < KS ? load(t0, n + D) : (n + D < 2 * KS ? load(t1, n + D - KS) : load(t2, n + D - 2 * KS));
            if (h == S::SP - 1) {
                lds_barrier();
                cur ^= 1;
            }
        }
        t0 = t1; t1 = t2; t2 = next(t2);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < WJ; ++j) {
                f32x4 y;
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const float v = tanhf((acc[i][j][x] + pw[i][j][x]) + bb[j][x]);
                    if constexpr (S::RESID) y[x] = v + rs[i][j][x];
                    else y[x] = v + 0.f;
                }
                *(f32x4 *)(a.Hout + row[i] * LD + n0 + 16 * j + 4 * q) = y;
            }
    }
}

}  // namespace

// Widths and reduction steps of walk_layer_supported; the spin means are left to
// their own pass, so not where the tiled kernels write them.  Below 4096 rows the
// reduction may be split over waves (other bits).  log|psi|, tiled -> here (us):
// 12 electrons, BF16 weights, 342 walkers (4104 rows) 170 -> 153, 1024 200 -> 188;
// 10 electrons, six products, 410 161 -> 148, 1024 189 -> 179.
bool walk_value_supported(int mode, const LayerArgs &a)
{
    const int ks = (a.K1 + a.K2) / 32;
    return (mode == GEMM_BF16W3 || mode == GEMM_BF16X6) && !a.Gout && a.w1 == 256 && a.W1p == 256 && a.lda1 == 256 &&
           a.ldh_out == 256 && a.nout == 256 && a.resid == (ks == 10) &&
           (ks == 10 ? a.K1 == 256 : (ks == 2 || ks == 4) && a.K2 == 32) && a.rows >= 4096;
}

template <int MODE>
static void launch_value_mode(const LayerArgs &a, hipStream_t st)
{
    const int64_t tiles = (a.rows + 31) / 32;
    auto go = [&](auto ks) {
        constexpr int KS = decltype(ks)::value, NCG = ValueShape<MODE, KS>::NCG;
        const int64_t nb = tiles < 512 / NCG ? (tiles + 7) / 8 * 8 : 512 / NCG;
        hipLaunchKernelGGL((k_walk_value<MODE, KS>), dim3((unsigned)(nb * NCG)), dim3(64 * WALK_WAVES), 0, st, a);
    };
    const int ks = (a.K1 + a.K2) / 32;
    if (ks == 2) go(std::integral_constant<int, 2>{});
    else if (ks == 4) go(std::integral_constant<int, 4>{});
    else go(std::integral_constant<int, 10>{});
}

void launch_walk_value(int mode, const LayerArgs &a, hipStream_t st)
{
    if (mode == GEMM_BF16W3) launch_value_mode<GEMM_BF16W3>(a, st);
    else launch_value_mode<GEMM_BF16X6>(a, st);
}

// Walkers whose workgroups run at the same time: two per CU (76 KB of LDS, 256
// registers), one per walker and column group.
static int walk_slots(int mode) { return mode == GEMM_BF16W3 ? 512 / WalkShape<GEMM_BF16W3, 2, 10>::NCG : 512 / WalkShape<GEMM_BF16X6, 3, 10>::NCG; }

// Shapes: 32 or 64 rows per electron, widths 256, a row's inputs in 2, 4 or 10
// steps of 32 (the features of up to 8 or of 17..24 nuclei with 4-wide pair
// rows; 256-wide layers with 32-wide pairs).
// Batches: walk_batch in fn_rules.h.
bool walk_layer_supported(int mode, const LayerArgs &a, int TR, int64_t B)
{
    const int ks = (a.K1 + a.K2) / 32, live = (a.n3 + 2 + 15) / 16;
    if (!(mode == GEMM_BF16W3 || mode == GEMM_BF16X6) || (TR != 32 && TR != 64) || a.w1 != 256 ||
        a.W1p != 256 || a.lda1 != 256 || a.ldh_out != 256 || a.nout != 256 || a.resid != (ks == 10) ||
        !(ks == 10 ? a.K1 == 256 : (ks == 2 || ks == 4) && a.K2 == 32))
        return false;
    return walk_batch(B, walk_slots(mode), live, mode == GEMM_BF16X6);
}

template <int MODE, int LIVE, int KS>
static void launch_walk(const LayerArgs &a, int TR, int64_t B, hipStream_t st)
{
    typedef WalkShape<MODE, LIVE, KS> S;
    const int64_t per = walk_slots(MODE);
    const int64_t nb = B < per ? (B + 7) / 8 * 8 : per;
    const dim3 grid((unsigned)(nb * S::NCG)), block(64 * WALK_WAVES);
    if (a.Gout) hipLaunchKernelGGL((k_walk_layer<MODE, LIVE, KS, true>), grid, block, 0, st, a, TR, B);
    else hipLaunchKernelGGL((k_walk_layer<MODE, LIVE, KS, false>), grid, block, 0, st, a, TR, B);
}

template <int MODE, int KS>
static void launch_walk_live(const LayerArgs &a, int TR, int64_t B, hipStream_t st)
{
    const int live = (a.n3 + 2 + 15) / 16;
    if constexpr (MODE == GEMM_BF16W3) {
        if (live <= 2) {
            launch_walk<MODE, 2, KS>(a, TR, B, st);
            return;
        }
    }
    if (live == 3) launch_walk<MODE, 3, KS>(a, TR, B, st);
    else launch_walk<MODE, 4, KS>(a, TR, B, st);
}

template <int MODE>
static void launch_walk_mode(const LayerArgs &a, int TR, int64_t B, hipStream_t st)
{
    const int ks = (a.K1 + a.K2) / 32;
    if (ks == 2) launch_walk_live<MODE, 2>(a, TR, B, st);
    else if (ks == 4) launch_walk_live<MODE, 4>(a, TR, B, st);
    else launch_walk_live<MODE, 10>(a, TR, B, st);
}

void launch_walk_layer(int mode, const LayerArgs &a, int TR, int64_t B, hipStream_t st)
{
    if (B <= 0) return;
    if (mode == GEMM_BF16W3) launch_walk_mode<GEMM_BF16W3>(a, TR, B, st);
    else launch_walk_mode<GEMM_BF16X6>(a, TR, B, st);
}

}  // namespace fn
