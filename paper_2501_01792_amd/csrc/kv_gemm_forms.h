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

// Index of the form with the least estimated time for the compute unit with the most tiles, first + more (n - 1) with
// n = tiles of the busiest of `cus` units; M tokens, 2 d output features.
inline int pick(int64_t M, int d, int cus)
{
    int best = 0;
    double least = 0.;
    for (int i = 0; i < kCount; ++i) {
        const TileForm &f = kForms[i];
        const int64_t tiles = ((M + f.bm - 1) / f.bm) * ((2 * (int64_t)d + f.bn - 1) / f.bn);
        const double t = f.first + f.more * (double)((tiles + cus - 1) / cus - 1);
        if (i == 0 || t < least) {
            best = i;
            least = t;
        }
    }
    return best;
}

}  // namespace forms
}  // namespace hk
