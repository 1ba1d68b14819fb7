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
// from HBM once.  Up to four splits would leave half of the XCDs or more idle: a split's
// tiles then go to 8, 4 or 2 of them.  (sp >= S or tile >= tiles: no work.)  Gradients,
// 1024 wide: 2 electrons, 16 walkers (one split) 913 us with its tiles on one XCD, 753
// on eight; 12 electrons, 1024 walkers (six, and two for the means) 3785 -> 3205.
struct TnBlock {
    int sp, tile;
};
constexpr int tn_xcds(int S) { return S == 1 ? 8 : (S == 2 ? 4 : (S <= 4 ? 2 : 1)); }
constexpr TnBlock tn_block(int bid, int S, int tiles)
{
    const int g = tn_xcds(S), xcd = bid % 8, idx = bid / 8;
    if (g > 1) return TnBlock{xcd / g, idx * g + xcd % g};
    return TnBlock{(idx / tiles) * 8 + xcd, idx % tiles};
}
constexpr int64_t tn_grid(int S, int tiles)
{
    return tn_xcds(S) > 1 ? 8 * ceil_div(tiles, tn_xcds(S)) : 8 * ceil_div(S, 8) * tiles;
}

}  // namespace fn
