// Single-query attention over a paged hybrid cache (Sec. 4.1, 4.2.1): every request's context is a
// list of logical blocks of `block_tokens` tokens, each either a KV block (its K/V rows sit in the KV
// pool) or an ACT block (its checkpoints sit in the activation pool; its K/V rows have just been
// regenerated into a pool of the same shape as the KV pool).  A per-request block table maps logical
// block -> (kind, physical block number).  Requests have their own lengths.  This is the role of the
// paper's attention kernel that reads both kinds of buffer (Sec. 5.1).
//
// Same organisation as the contiguous kernel (flash_decode.hip): the token positions of all
// (request, head) pairs form one line, pair-major, of H * sum(len) positions; it is cut into W equal
// ranges, one per resident wavefront; a wavefront emits one partial per pair it touches at index
// (wavefront + pair); a second kernel merges each pair's run of partials.  What differs is the address
// of a token: the block table is read with scalar loads, one entry for every 16 tokens of a step (steps are
// aligned to 64 tokens inside a pair, so that 16 tokens never straddle a block), during the step before.  Where a workgroup
// per pair keeps the chip as busy (attn_pairs.h), its wavefronts merge in LDS and there is no second kernel.
// Measured, the form taken (profiles/decode_attention_cached.txt, 16-token blocks in random order; in brackets ranges and merge
// where that is not the form taken, from another session): 411 MB of 32 ragged requests 64.8 us (72.8), 67 MB 10.5 (15.8), 33 MB of one
// request, ranges, 12.1.  Before, with ranges that ended inside a step, entries fetched when they were needed and a merge that
// walked the partials one by one: 411 MB 90.5, 7.6 GB 1212, one request 42.
#include "hk_internal.h"
#include "elem.h"
#include "attn_merge.h"
#include "attn_pairs.h"
#include "attn_ranges.h"
#include "attn_tile.h"

namespace hk {
namespace {

constexpr int kThreads = 256;
constexpr int kWavesPerBlock = 4;
using attn::kTile;
using merge::kNegBig;

using ranges::effective_waves;
using ranges::range_begin;

// Request that holds position p of the pair-major line: the last r with H * cu[r] <= p (cu has B + 1 entries).
__device__ __forceinline__ int request_of(const int64_t *__restrict__ cu, int B, int H, int64_t p)
{
    int lo = 0, hi = B;                  // invariant: H cu[lo] <= p < H cu[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((int64_t)H * cu[mid] <= p) lo = mid; else hi = mid;
    }
    return lo;
}

// Table entries of a step of 64 tokens: one for every 16 of them, which never straddle a block (block_tokens >= 16).
__device__ __forceinline__ void entries_of(const int32_t *__restrict__ tab, int tb, int last_block, int blk_log2, int32_t (&e)[4])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int bi = (tb + 16 * j) >> blk_log2;
        e[j] = tab[bi < last_block ? bi : last_block];
    }
}

// Asks for the K and V rows of a step: `rows` tokens from tb on, entries `ent`.
template <int DH, int DT>
__device__ __forceinline__ void load_step(
    const typename Elem<DT>::T *__restrict__ K_pool, const typename Elem<DT>::T *__restrict__ V_pool,
    const typename Elem<DT>::T *__restrict__ K_regen, const typename Elem<DT>::T *__restrict__ V_regen,
    const int32_t (&ent)[4], int P_kv, int P_act, int64_t blk_elems, int h, int blk, int tb, int rows, int lane,
    typename Elem<DT>::V8 (&kr)[attn::Tile<DH, DT>::NL], typename Elem<DT>::V8 (&vr)[attn::Tile<DH, DT>::NL])
{
    typedef typename Elem<DT>::V8 half8_t;
    constexpr int NL = attn::Tile<DH, DT>::NL, kPer = 16 / attn::Tile<DH, DT>::RPL;   // loads of 16 tokens
    __amdgpu_buffer_rsrc_t kb[4], vb[4];                       // 16 tokens each
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int32_t e = __builtin_amdgcn_readfirstlane(ent[j]);
        bool is_act = e < 0;
        int pb = is_act ? ~e : e;
        if ((is_act ? P_act : P_kv) <= 0) { is_act = !is_act; pb = 0; }   // a corrupt table cannot leave
        const int P = is_act ? P_act : P_kv;                              // the pools (one is not empty)
        pb = pb < P ? pb : P - 1;
        const int64_t at = (int64_t)pb * blk_elems + (int64_t)(h * blk + ((tb + 16 * j) & (blk - 1))) * DH;
        const int here = rows - 16 * j;
        const int n = here < 0 ? 0 : here < 16 ? here : 16;
        kb[j] = attn::step_rows((is_act ? K_regen : K_pool) + at, n, DH);
        vb[j] = attn::step_rows((is_act ? V_regen : V_pool) + at, n, DH);
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) kr[i] = attn::step_load<half8_t>(kb[i / kPer], i % kPer, lane);
#pragma unroll
    for (int i = 0; i < NL; ++i) vr[i] = attn::step_load<half8_t>(vb[i / kPer], i % kPer, lane);
}

template <int DH, int DT>
__global__ __launch_bounds__(kThreads, 3) void paged_decode_kernel(
    const typename Elem<DT>::T *__restrict__ q,
    const typename Elem<DT>::T *__restrict__ K_pool, const typename Elem<DT>::T *__restrict__ V_pool,      // KV blocks
    const typename Elem<DT>::T *__restrict__ K_regen, const typename Elem<DT>::T *__restrict__ V_regen,    // regenerated ACT blocks
    const int32_t *__restrict__ table, int max_blocks, int P_kv, int P_act,
    const int32_t *__restrict__ seq_len, const int64_t *__restrict__ cu,
    int B, int H, int blk_log2, int64_t total_host, const int64_t *__restrict__ total_dev, int W, float scale_log2e,
    float *__restrict__ partial)
{
    typedef typename Elem<DT>::V8 half8_t;
    typedef attn::Tile<DH, DT> tile_t;
    constexpr int LPR = tile_t::LPR, RPL = tile_t::RPL, NL = tile_t::NL;
    // positions of the line: known to the host, or (tables built on the device) H * total_dev[0] <= the host's bound
    const int64_t total = total_dev ? (int64_t)H * total_dev[0] : total_host;
    // The launch may be sized for more positions than the device finds (an upper bound on the host): then only
    // the first `total` wavefronts work, so that no range between two working wavefronts is empty and every
    // partial slot the merge reads has been written.  The merge derives the same number.
    W = effective_waves(W, total);

    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6));
    if (w >= W) return;                  // whole wavefronts leave; the kernel has no barrier
    const int g = lane / LPR, c = lane % LPR;
    const int blk = 1 << blk_log2;
    const int64_t blk_elems = (int64_t)H * blk * DH;       // elements of one pool block

    int64_t p = range_begin(w, total, W);
    const int64_t p_end = range_begin(w + 1, total, W);
    int r = request_of(cu, B, H, p);
    while (p < p_end) {
        // position p -> (request r, head h, token t_first); requests without tokens are stepped over
        int64_t base = (int64_t)H * cu[r];
        int len = seq_len[r];
        while (p >= base + (int64_t)H * len) { ++r; base = (int64_t)H * cu[r]; len = seq_len[r]; }
        const int h = (int)ranges::quot(p - base, len);
        const int t_begin = (int)(p - base - (int64_t)h * len);
        const int64_t pair_end = base + (int64_t)(h + 1) * len;
        const int t_end = (int)((p_end < pair_end ? p_end : pair_end) - (base + (int64_t)h * len));   // range: tokens [t_begin, t_end)
        // What the wavefront takes: whole steps of 64 tokens of the pair.  Both ends of a range are moved down to a
        // step (the pair's end stays), which keeps the ranges a partition; a range of 256 tokens then costs four steps
        // on average instead of five.  A range left empty still stores its (neutral) partial, which the merge reads.
        const int t_first = t_begin & ~(kTile - 1);
        const int t_last = t_end < len ? t_end & ~(kTile - 1) : len;
        const int pair = r * H + h;
        const int32_t *tab = table + (int64_t)r * max_blocks;
        int last_block = (t_last - 1) >> blk_log2;                 // used only when the range is not empty
        if (last_block >= max_blocks) last_block = max_blocks - 1;             // a corrupt length cannot leave the table's row

        const half8_t qv = *reinterpret_cast<const half8_t *>(q + (int64_t)pair * DH + c * 8);
        tile_t tile;
        tile.clear();

        int32_t ent[4] = {0, 0, 0, 0};
        if (t_first < t_last) entries_of(tab, t_first, last_block, blk_log2, ent);
        for (int tb = t_first; tb < t_last; tb += kTile) {
            half8_t kr[NL], vr[NL];
            const int rows = t_last - tb < kTile ? t_last - tb : kTile;
            load_step<DH, DT>(K_pool, V_pool, K_regen, V_regen, ent, P_kv, P_act, blk_elems, h, blk, tb, rows, lane, kr, vr);
            // the next step's entries (scalar loads) are on their way while this step's rows arrive
            if (tb + kTile < t_last) entries_of(tab, tb + kTile, last_block, blk_log2, ent);
            __builtin_amdgcn_sched_barrier(0);                     // every load of the step is on its way before the first use
            tile.consume(qv, kr, vr, lane, c * RPL + g < rows, scale_log2e);
        }
        tile.store(partial + ((int64_t)w + pair) * (DH + 2), lane);
        p = base + (int64_t)h * len + t_end;
    }
}

// One workgroup per (request, head): its wavefronts take the steps of the pair in turn and merge in LDS, so that one launch
// does what the ranges and their merge do in two (attn_pairs.h says when), and no wavefront looks for its request.
template <int DH, int DT>
__global__ __launch_bounds__(kThreads, 3) void paged_pair_kernel(
    const typename Elem<DT>::T *__restrict__ q,
    const typename Elem<DT>::T *__restrict__ K_pool, const typename Elem<DT>::T *__restrict__ V_pool,
    const typename Elem<DT>::T *__restrict__ K_regen, const typename Elem<DT>::T *__restrict__ V_regen,
    const int32_t *__restrict__ table, int max_blocks, int P_kv, int P_act, const int32_t *__restrict__ seq_len,
    int H, int blk_log2, float scale_log2e, typename Elem<DT>::T *__restrict__ out, float2 *__restrict__ lse)
{
    typedef typename Elem<DT>::V8 half8_t;
    typedef attn::Tile<DH, DT> tile_t;
    constexpr int LPR = tile_t::LPR, RPL = tile_t::RPL, NL = tile_t::NL, P = kWavesPerBlock;
    __shared__ __align__(16) float part[P][DH + 2];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int pair = blockIdx.x, r = pair / H, h = pair % H;
    const int g = lane / LPR, c = lane % LPR;
    const int blk = 1 << blk_log2;
    const int64_t blk_elems = (int64_t)H * blk * DH;
    const int64_t room = (int64_t)max_blocks << blk_log2;
    const int len = seq_len[r] < room ? seq_len[r] : (int)room;            // a corrupt length cannot leave the table's row
    const int last_block = (len - 1) >> blk_log2;              // used only when there are tokens
    const int32_t *tab = table + (int64_t)r * max_blocks;
    const half8_t qv = *reinterpret_cast<const half8_t *>(q + (int64_t)pair * DH + c * 8);
    tile_t tile;
    tile.clear();
    int32_t ent[4] = {0, 0, 0, 0};
    if (wave * kTile < len) entries_of(tab, wave * kTile, last_block, blk_log2, ent);
    for (int tb = wave * kTile; tb < len; tb += P * kTile) {
        half8_t kr[NL], vr[NL];
        const int rows = len - tb < kTile ? len - tb : kTile;
        load_step<DH, DT>(K_pool, V_pool, K_regen, V_regen, ent, P_kv, P_act, blk_elems, h, blk, tb, rows, lane, kr, vr);
        if (tb + P * kTile < len) entries_of(tab, tb + P * kTile, last_block, blk_log2, ent);   // while the rows arrive
        __builtin_amdgcn_sched_barrier(0);                     // every load of the step is on its way before the first use
        tile.consume(qv, kr, vr, lane, c * RPL + g < rows, scale_log2e);
    }
    tile.store(part[wave], lane);
    __syncthreads();
    if (wave != 0) return;
    const bool some = len > 0;
    merge::Shared<DH, 1> none;
    float m, l, o[DH / 64];
    merge::merge_run<DH, 1>(part[0], P, none, m, l, o);
    if (!some) {                         // no context: the softmax is over nothing; define the output as zero
#pragma unroll
        for (int e = 0; e < DH / 64; ++e) o[e] = 0.f;
    }
    merge::store_row<DH>(out + (int64_t)pair * DH, o, some ? l : 1.f);
    if (lse && lane == 0) lse[pair] = some ? make_float2(m, l) : make_float2(kNegBig, 0.f);
}

// Merge of the partials of every (request, head), P wavefronts each: positions [H cu[r] + h len, + len) of the line.
template <int DH, int DT, int P>
__global__ __launch_bounds__(merge::kThreads) void paged_merge_kernel(const float *__restrict__ partial,
                                                                      const int32_t *__restrict__ seq_len, const int64_t *__restrict__ cu,
                                                                      int pairs, int H, int64_t total_host,
                                                                      const int64_t *__restrict__ total_dev, int W,
                                                                      typename Elem<DT>::T *__restrict__ out, float2 *__restrict__ lse)
{
    __shared__ merge::Shared<DH, P> sh;
    const int64_t total = total_dev ? (int64_t)H * total_dev[0] : total_host;   // > 0 whenever a pair has tokens
    W = effective_waves(W, total);       // as in the streaming kernel: no empty range among the working wavefronts
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int pair = blockIdx.x * (kWavesPerBlock / P) + wave / P;
    const bool live = pair < pairs;
    if (!live) pair = pairs - 1;         // works on the last pair (the workgroup shares a barrier), stores nothing
    const int r = pair / H, h = pair % H;
    const int len = seq_len[r];
    const bool some = len > 0 && total > 0;
    int n = 0;
    const float *src = partial;
    if (some) {
        const int64_t lo = (int64_t)H * cu[r] + (int64_t)h * len, hi = lo + len - 1;
        const int w_first = ranges::owner(lo, total, W), w_last = ranges::owner(hi, total, W);
        src = partial + ((int64_t)w_first + pair) * (DH + 2);
        n = w_last - w_first + 1;
    }
    float m, l, o[DH / 64];
    merge::merge_run<DH, P>(src, n, sh, m, l, o);
    if (!live || wave % P != 0) return;
    if (!some) {                         // no context: the softmax is over nothing; define the output as zero
#pragma unroll
        for (int e = 0; e < DH / 64; ++e) o[e] = 0.f;
    }
    merge::store_row<DH>(out + (int64_t)pair * DH, o, some ? l : 1.f);
    if (lse && lane == 0) lse[pair] = some ? make_float2(m, l) : make_float2(kNegBig, 0.f);
}

template <int DH, int DT, int P>
void launch_merge(const PagedAttnArgs &a, int64_t total, hipStream_t s)
{
    constexpr int per_block = kWavesPerBlock / P;
    const int pairs = a.B * a.H;
    hipLaunchKernelGGL((paged_merge_kernel<DH, DT, P>), dim3((unsigned)((pairs + per_block - 1) / per_block)), dim3(merge::kThreads), 0, s,
                       a.partial, a.seq_len, a.cu_tokens, pairs, a.H, total > 0 ? total : 1, a.total_dev, a.n_waves > 0 ? a.n_waves : 1,
                       static_cast<typename Elem<DT>::T *>(a.out), a.lse);
}

template <int DH, int DT>
hipError_t launch_dh(const PagedAttnArgs &a, hipStream_t s)
{
    typedef typename Elem<DT>::T elem_t;
    const int64_t total = (int64_t)a.H * a.total_tokens;
    const float scale_log2e = a.scale * 1.4426950408889634f;
    int blk_log2 = 0;
    while ((1 << blk_log2) < a.block_tokens) ++blk_log2;
    if (total > 0 && pairs::paged(a.B, a.H, (int64_t)a.max_blocks * a.block_tokens, a.total_tokens - a.other_tokens, a.head_dim)) {
        hipLaunchKernelGGL((paged_pair_kernel<DH, DT>), dim3((unsigned)(a.B * a.H)), dim3(kThreads), 0, s,
                           static_cast<const elem_t *>(a.q),
                           static_cast<const elem_t *>(a.K_pool), static_cast<const elem_t *>(a.V_pool),
                           static_cast<const elem_t *>(a.K_regen), static_cast<const elem_t *>(a.V_regen),
                           a.block_table, a.max_blocks, a.P_kv, a.P_act, a.seq_len, a.H, blk_log2, scale_log2e,
                           static_cast<elem_t *>(a.out), a.lse);
        return hipGetLastError();
    }
    if (total > 0) {
        const unsigned blocks = (unsigned)((a.n_waves + kWavesPerBlock - 1) / kWavesPerBlock);
        hipLaunchKernelGGL((paged_decode_kernel<DH, DT>), dim3(blocks), dim3(kThreads), 0, s,
                           static_cast<const elem_t *>(a.q),
                           static_cast<const elem_t *>(a.K_pool), static_cast<const elem_t *>(a.V_pool),
                           static_cast<const elem_t *>(a.K_regen), static_cast<const elem_t *>(a.V_regen),
                           a.block_table, a.max_blocks, a.P_kv, a.P_act, a.seq_len, a.cu_tokens,
                           a.B, a.H, blk_log2, total, a.total_dev, a.n_waves, scale_log2e, a.partial);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (merge::waves_per_pair(a.n_waves, (int64_t)a.B * a.H) == 1) launch_merge<DH, DT, 1>(a, total, s);
    else launch_merge<DH, DT, 4>(a, total, s);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_paged_decode(const PagedAttnArgs &a, hipStream_t s)
{
    if (a.B <= 0) return hipSuccess;
    if (a.block_tokens < 16 || (a.block_tokens & (a.block_tokens - 1)) != 0) return hipErrorInvalidValue;
    if (a.total_tokens > 0 && (a.n_waves <= 0 || (int64_t)a.n_waves > (int64_t)a.H * a.total_tokens)) return hipErrorInvalidValue;
    if (a.head_dim == 128) return a.dtype == 1 ? launch_dh<128, 1>(a, s) : launch_dh<128, 0>(a, s);
    if (a.head_dim == 64) return a.dtype == 1 ? launch_dh<64, 1>(a, s) : launch_dh<64, 0>(a, s);
    return hipErrorInvalidValue;
}

}  // namespace hk
