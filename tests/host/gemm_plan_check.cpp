// Host check of the projection's launches on a prepared layer (csrc/kv_gemm_forms.h).
//   usage: gemm_plan_check cus M_0 d_0 M_1 d_1 ...   prints "<rows of the first launch> <bm> <bn of the second, 0 0 for none>"
//   per pair (M, d); then walks a range of sizes and fails where a plan is not one that the kernels take, or a caller
//   that keeps compute units free gets two launches.
#include "../../paper_2501_01792_amd/csrc/kv_gemm_forms.h"

#include <cstdio>
#include <cstdlib>

using namespace hk::forms;

int main(int argc, char **argv)
{
    const int cus = atoi(argv[1]);
    for (int i = 2; i + 1 < argc; i += 2) {
        const int64_t M = atoll(argv[i]);
        const Plan p = plan(M, atoi(argv[i + 1]), cus, 0);
        printf("%lld %d %d\n", (long long)p.rows, p.rows < M ? kForms[p.rest_form].bm : 0, p.rows < M ? kForms[p.rest_form].bn : 0);
    }
    for (int d = 128; d <= 16384; d += 64)
        for (int64_t M = 1; M < 300000; M += 1 + M / 7) {
            const Plan p = plan(M, d, cus, 0);
            const bool one = p.rows == M && p.form == pick(M, d, cus);
            const bool two = p.form == 0 && p.rows > 0 && p.rows < M && p.rows % 256 == 0 && p.rest_form > 0 && p.rest_form < kCount;
            if (!one && !two) {
                fprintf(stderr, "M %lld d %d: form %d rows %lld rest %d\n", (long long)M, d, p.form, (long long)p.rows, p.rest_form);
                return 1;
            }
            const Plan limited = plan(M, d, cus, cus - 16);
            if (limited.rows != M || limited.form != pick(M, d, cus)) {
                fprintf(stderr, "M %lld d %d: %lld rows in the first launch although units are kept free\n", (long long)M, d, (long long)limited.rows);
                return 1;
            }
        }
    return 0;
}
