// Where the rows of the current tokens go in a paged cache: shared by the kernels that write them.
#pragma once
#include "hk_internal.h"

namespace hk {

// Where the current token of a request goes in a paged cache (QkvArgs): its table entry and its row in the block,
// or row < 0 when the request has no token, the table has no entry for it, or the caller's mask says that the
// token is not to be stored.
struct PagedDst {
    const int32_t *block_table, *seq_len;      // block_table == nullptr: contiguous stores
    const int32_t *store_mask;                 // optional: zero = the request's token is not stored
    int max_blocks, blk_log2, P_kv, P_act;
};
__device__ __forceinline__ void paged_slot(const PagedDst &p, int b, int32_t &entry, int &row)
{
    row = -1;
    entry = 0;
    if (p.store_mask && p.store_mask[b] == 0) return;
    const int t = p.seq_len[b] - 1;
    if (t < 0) return;
    const int bi = t >> p.blk_log2;
    if (bi >= p.max_blocks) return;
    entry = p.block_table[(int64_t)b * p.max_blocks + bi];
    row = t & ((1 << p.blk_log2) - 1);
}

inline PagedDst paged_dst(const QkvArgs &a)
{
    return PagedDst{a.block_table, a.seq_len, a.store_mask, a.max_blocks, a.blk_log2, a.P_kv, a.P_act};
}

}  // namespace hk
