// fn_rules.h -- dispatch rules that need nothing but sizes, in plain C++ so that
// they can be checked without a GPU (constexpr functions also compile for the device).
#pragma once
#include <stdint.h>

namespace fn {

// Row splits of the column sums and, at most, of a weight-gradient product.
constexpr int MAX_SPLITS = 64;

constexpr int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Row splits of a weight-gradient product of R rows and `tiles` output tiles
// whose partial sums' buffer holds `cap` splits: three workgroups per CU where the rows
// give them, 32 rows per wave (a quarter of a split) or more; but chains of at
// most 512 rows per wave while MAX_SPLITS allows it.  (Layers wider than 256 fill the
// CUs with few splits: 1024 wide, 49152 rows, 4 splits, chains of 3072; the FP32
// weight gradient then was 1.6e-7 off, 1.1e-7 with chains of 512.)
constexpr int64_t tn_product_splits(int64_t R, int64_t tiles, int64_t cap)
{
    int64_t S = 768 / tiles + 1;
    if (S > R / 128) S = R / 128;
    if (S < ceil_div(R, 4 * 512)) S = ceil_div(R, 4 * 512);
    if (S > MAX_SPLITS) S = MAX_SPLITS;
    if (S > cap) S = cap;
    return S < 1 ? 1 : S;
}

// The split and output tile of workgroup `bid`.  Workgroups are dealt to the eight
// XCDs in turn; all tiles of a split follow each other on one XCD, so its rows come
// from HBM once.  Up to four splits of more tiles than an XCD has CUs would leave half of
// the XCDs or more idle: a split's tiles then go to 8, 4 or 2 of them.  (sp >= S or
// tile >= tiles: no work.)  Gradients, 1024 wide: 2 electrons, 16 walkers (one split) 913
// us with its tiles on one XCD, 753 on eight; 12 electrons, 1024 walkers (six, and two for
// the means) 3785 -> 3205.
struct TnBlock {
    int sp, tile;
};
constexpr int tn_xcd_bits(int S, int tiles)
{
    return tiles <= 32 || S > 4 ? 0 : (S == 1 ? 3 : (S == 2 ? 2 : 1));
}
constexpr TnBlock tn_block(int bid, int S, int tiles)
{
    const int b = tn_xcd_bits(S, tiles), xcd = bid & 7, idx = bid >> 3;
    if (b > 0) return TnBlock{xcd >> b, (idx << b) + (xcd & ((1 << b) - 1))};
    return TnBlock{(idx / tiles) * 8 + xcd, idx % tiles};
}
constexpr int64_t tn_grid(int S, int tiles)
{
    const int b = tn_xcd_bits(S, tiles);
    return b > 0 ? 8 * ceil_div(tiles, 1 << b) : 8 * ceil_div(S, 8) * tiles;
}

// Batches for which a stream layer walks over whole walkers (fn_walk.hip): it takes a
// round of `slots` walkers at a time, the tiled kernel spreads any number of rows, so
// the last round has to be full enough.  live: 16-row blocks of an electron; six: six
// products (else BF16 weights, three).  Whole local energies, tiled -> walking (us):
// 12 electrons, BF16 weights, 128 walkers (half a round) 501 -> 487, 257 914 -> 903, 300
// 1039 -> 930, 512 1681 -> 1224, but 100 427 -> 452; 20 electrons, 200 1836 -> 1632.
// 10 electrons (two blocks, where the epilogue weighs more) 256 535 -> 476, 1024 1871 ->
// 1556, but 300 619 -> 659; with six products it gains nothing there (7 electrons, 1024
// walkers: 1346 -> 1393) and is not used.  Six products otherwise, slots 128, times
// faster: 11 to 15 electrons 72 walkers 0.97 to 1.07, 82 1.01 to 1.09, 128 1.29 to 1.35, 143
// 1.07 to 1.09; 16 to 20 electrons 72 0.89 to 1.01, 82 0.95 to 1.11, 92 1.00 to 1.12, 128 1.14 to
// 1.25, 143 0.96 to 1.06, 154 1.01 to 1.15.
constexpr bool walk_batch(int64_t B, int64_t slots, int live, bool six)
{
    const int64_t rounds = ceil_div(B, slots);
    int full = live >= 3 ? 55 : 85;                  // percent of the rounds' walkers
    if (six && live == 3 && rounds == 1) full = 60;
    if (six && live == 4) full = rounds == 1 ? 70 : 58;
    return !(six && live < 3) && 100 * B >= full * rounds * slots;
}

// Forward-Laplacian determinants of n electrons of one spin (N in all, M nuclei) in
// the direction-per-lane kernel (else a wave per determinant with the matrices in
// LDS).  A lane per direction takes the same time for 20 electrons as for 8, the other
// kernel less for fewer, and its entries are formed at a higher occupancy; the line
// does not depend on the batch, so that the bits do not.  FP32, 16 determinants, 4096
// walkers, wave per determinant / here, us per local energy of a small network: (8, 0)
// and 2 nuclei 1321 / 1343, 20 nuclei 1770 / 2013; (8, 3) 20 nuclei 3449 / 3342; (9, 0)
// 1775 / 1967; (9, 2) 2445 / 2523; (9, 3) 2895 / 2725, 20 nuclei 4379 / 4453; (10, 0) 2299 /
// 2156, 20 nuclei 3071 / 3265; (10, 2) 20 nuclei 4355 / 4309.  Seven or fewer gain
// 1.06x or more at 32 nuclei, FP64 1.2x at any size.
constexpr bool det_lanes_fl(int n, int N, int M, bool f64)
{
    if (n < 3 || n > 10) return false;
    return f64 || n < 8 || N > (n == 9 ? 11 : 9) + M / 8;
}

}  // namespace fn
