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

}  // namespace fn
