// Which output tile the projection on a prepared layer takes (kv_gemm_tile.hip; 256 x 256 is the kernel of
// kv_gemm_fold.hip).  Plain arithmetic, callable from the host alone, so that it can be checked without a GPU.
#pragma once
#include <stdint.h>

namespace hk {
namespace forms {

// A tile and the time per k block, in microseconds as measured: `first` for a compute unit with one tile, `more` for each
// further one, sharing the unit or after it.  Both grow with the tile's area, but `more` only from 64 x 64 on in
// proportion to it: small tiles move more bytes per product, large ones leave units idle.  All forms timed at 96 sizes,
// d = 768 to 9216, M = 8 to 3072, fp16 and bf16 (profiles/kv_gemm_tile_forms.txt): the choice is the fastest or within 5 %.
struct TileForm {
    int bm, bn;
    float first, more;
};
constexpr TileForm kForms[] = {
    {256, 256, 1.30f, 1.50f},
    {256, 128, 0.90f, 0.95f},
    {128, 256, 0.90f, 0.95f},
    {192, 128, 0.69f, 0.75f},
    {128, 128, 0.61f, 0.60f},
    {128, 64, 0.46f, 0.34f},
    {64, 128, 0.49f, 0.35f},
    {64, 64, 0.37f, 0.21f},
    {64, 32, 0.29f, 0.165f},
    {32, 64, 0.30f, 0.16f},
    {32, 32, 0.20f, 0.13f},
};
constexpr int kCount = sizeof(kForms) / sizeof(kForms[0]);

// Tiles of a form over M tokens and 2 d output features, and the estimated time for the compute unit with the most of them:
// first + more (n - 1) with n = tiles of the busiest of `cus` units.
inline int64_t row_tiles(const TileForm &f, int64_t M) { return (M + f.bm - 1) / f.bm; }
inline int64_t col_tiles(const TileForm &f, int d) { return (2 * d + f.bn - 1) / f.bn; }
inline double estimate(const TileForm &f, int64_t M, int d, int cus)
{
    return f.first + f.more * (double)((row_tiles(f, M) * col_tiles(f, d) + cus - 1) / cus - 1);
}

// Index of the form with the least estimated time, of those from `from` on.
inline int pick(int64_t M, int d, int cus, int from = 0)
{
    int best = from;
    double least = estimate(kForms[from], M, d, cus);
    for (int i = from + 1; i < kCount; ++i) {
        const double t = estimate(kForms[i], M, d, cus);
        if (t < least) {
            best = i;
            least = t;
        }
    }
    return best;
}

// One launch for all rows, or two: 256 x 256 tiles for as many rows as fill their rounds over the compute units, and the form
// that suits them for the rows whose tiles would have been a partly filled round.  A second launch adds its gap and its
// first loads, about 5 us; and the estimate has to gain a fifth of a round, because a round that few units take part in is
// faster than a full one (the clock is up, the memory idle): cut there too, 1551 rows of d = 7168 took 298 us against 281,
// 4000 of d = 9216 1067 against 1004.  Measured with the row statistics, one launch -> two, fp16: d = 4096, 2500 rows: 168 -> 138
// us, 12608: 642 -> 611; d = 5120, 1551 rows: 177 -> 138; d = 7168, 2500 rows: 444 -> 388; d = 9216, 12608 rows: 3358 -> 3181;
// from 20 rounds on it is level.  (First launches on smaller tiles never came out ahead.)
struct Plan {
    int form;
    int64_t rows;           // of the first launch; the others are the second's
    int rest_form;
};
constexpr double kSecondUs = 5., kSure = 0.2;
// cu_limit > 0: the caller keeps compute units free of the 256 x 256 tiles; rounds over all of them are not what that launch
// takes then (240 units, d = 4096, 2600 rows, beside the attention: 230 us in two launches, 200 in one).
inline Plan plan(int64_t M, int d, int cus, int cu_limit)
{
    const Plan one = {pick(M, d, cus), M, 0};
    if (cu_limit > 0) return one;
    const TileForm &f = kForms[0];
    const int64_t cols = col_tiles(f, d), tiles = row_tiles(f, M) * cols;
    if (tiles < cus) return one;
    const int64_t rows = tiles / cus * cus / cols * f.bm;                   // row tiles that fit the full rounds
    if (rows <= 0 || rows >= M) return one;
    const int rest = pick(M - rows, d, cus, 1);
    const double two = estimate(f, rows, d, cus) + estimate(kForms[rest], M - rows, d, cus) + kSecondUs * 64 / d + kSure * f.more;
    return two < estimate(kForms[one.form], M, d, cus) ? Plan{0, rows, rest} : one;
}

}  // namespace forms
}  // namespace hk
