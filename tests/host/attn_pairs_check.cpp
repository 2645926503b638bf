// Host check of the rules that choose between one workgroup per (sequence, head) and ranges with a merge (csrc/attn_pairs.h).
//   usage: attn_pairs_check c pairs L0 L1 head_dim   or   attn_pairs_check p requests heads room tokens head_dim, any number of
//   them; prints 1 (a workgroup per pair) or 0 (ranges) for each.
#include "../../paper_2501_01792_amd/csrc/attn_pairs.h"

#include <cstdio>
#include <cstdlib>

int main(int argc, char **argv)
{
    auto num = [&](int i) { return i < argc ? atoll(argv[i]) : 0; };
    for (int i = 1; i < argc;) {
        if (argv[i][0] == 'c') {
            printf("%d\n", hk::pairs::contiguous(num(i + 1), hk::pairs::steps((int)num(i + 2), (int)num(i + 3)), (int)num(i + 4)));
            i += 5;
        } else {
            printf("%d\n", hk::pairs::paged(num(i + 1), (int)num(i + 2), num(i + 3), num(i + 4), (int)num(i + 5)));
            i += 6;
        }
    }
    return 0;
}
