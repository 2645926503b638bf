// Host check of the choice of the projection's tile (csrc/kv_gemm_forms.h).
//   usage: gemm_forms_check cus M_0 d_0 M_1 d_1 ...   prints the number of forms, then "<bm> <bn>" per pair (M, d)
#include "../../paper_2501_01792_amd/csrc/kv_gemm_forms.h"

#include <cstdio>
#include <cstdlib>

int main(int argc, char **argv)
{
    printf("%d\n", hk::forms::kCount);
    for (int i = 2; i + 1 < argc; i += 2) {
        const hk::forms::TileForm &f = hk::forms::kForms[hk::forms::pick(atoll(argv[i]), atoi(argv[i + 1]), atoi(argv[1]))];
        printf("%d %d\n", f.bm, f.bn);
    }
    return 0;
}
