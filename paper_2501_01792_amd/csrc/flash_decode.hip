// Single-query attention (Eq. 4) over cached ++ regenerated K/V (Eq. 3) for gfx950.
//
// The decode query of each (sequence, head) attends over every context token.  With one query
// per head the work is one pass over K and one over V: ~1 FLOP per byte, so the kernel is an HBM
// streaming kernel and is organised around the loads, not the arithmetic:
//   * The context of a (sequence, head) is two contiguous token segments (the cached rows and
//     the regenerated rows); they are never copied together.
//   * Work is split by bytes, not by (sequence, head): the tokens of all pairs form one line of
//     BH * L positions that is cut into W equal ranges, one per wavefront, with W chosen so that
//     all wavefronts are resident at once.  Every wavefront therefore streams the same number of
//     bytes and they all finish together; there is no partly filled last round of workgroups.
//     A range may cover the end of one pair and the start of the next; for every pair it touches
//     a wavefront emits one un-normalised partial (m, l, o[dh]) at index (wavefront + pair), which
//     is unique, and makes the partials of one pair a contiguous run.  A second small kernel
//     merges the run of every pair by log-sum-exp.  Wavefronts of this kernel never talk to each other:
//     no LDS, no barrier.  (Those of the merge may: attn_merge.h.)
//   * Where a workgroup per pair keeps the chip as busy (attn_pairs.h), its wavefronts merge in LDS and there is
//     neither a second kernel nor a partial in memory.
//   * A wavefront consumes 64 tokens at a time (attn_tile.h).  dh/8 lanes cover one row with 16-byte loads, so
//     every load instruction of a wavefront reads whole, consecutive rows (1 KiB contiguous), and all K and V
//     loads of the 64 tokens are issued before the first use: 128 registers of rows, 3 wavefronts per SIMD.  Left to
//     the compiler (4 per SIMD) the V rows were asked for behind the K rows' use, a second memory latency per step,
//     and in bf16 they were widened on arrival (246 registers, 2 per SIMD).
//   * Small problems that are cut into ranges have ranges of one step each, aligned to the pairs, so that they too fill the
//     chip and pay one latency (with at least 128 tokens per range, 64,000 positions ran on 125 of 256 compute units).
// Measured, the form taken (profiles/decode_attention_cached.txt; in brackets ranges and merge where that is not the form taken,
// from another session): 4.8 GB fp16 686 us, 7.04 TB/s (727), bf16 712 (747); 268 MB 39.5 (43.9); 67 MB 9.9 (15.0); 33 MB of one
// request, ranges, 9.7.  Before, with V asked for behind K, at least 128 tokens a range and a merge that walked the partials one
// by one: 4.8 GB fp16 737, bf16 771; 268 MB 47.5; one request 36.4.
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

using ranges::range_begin;

template <int DH, int DT>
__global__ __launch_bounds__(kThreads, 3) void flash_decode_kernel(
    const typename Elem<DT>::T *__restrict__ q,
    const typename Elem<DT>::T *__restrict__ K0, const typename Elem<DT>::T *__restrict__ V0,
    const typename Elem<DT>::T *__restrict__ K1, const typename Elem<DT>::T *__restrict__ V1,
    int L0, int L1, int64_t total, int W, float scale_log2e,
    float *__restrict__ partial)
{
    typedef typename Elem<DT>::T elem_t;
    typedef typename Elem<DT>::V8 half8_t;
    typedef attn::Tile<DH, DT> tile_t;
    constexpr int LPR = tile_t::LPR, RPL = tile_t::RPL, NL = tile_t::NL;

    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6));   // wavefront-uniform
    if (w >= W) return;                  // whole wavefronts leave; the kernel has no barrier
    const int g = lane / LPR, c = lane % LPR;
    const int L = L0 + L1;

    int64_t p = range_begin(w, total, W);
    const int64_t p_end = range_begin(w + 1, total, W);
    while (p < p_end) {
        const int bh = (int)ranges::quot(p, L);
        const int t_first = (int)(p - (int64_t)bh * L);
        const int64_t pair_end = (int64_t)(bh + 1) * L;
        const int t_last = (int)((p_end < pair_end ? p_end : pair_end) - (int64_t)bh * L);   // tokens [t_first, t_last) of pair bh

        const half8_t qv = *reinterpret_cast<const half8_t *>(q + (int64_t)bh * DH + c * 8);
        tile_t tile;
        tile.clear();

        // the part of [t_first, t_last) inside the first segment, then the part inside the second
#pragma unroll 1
        for (int seg = 0; seg < 2; ++seg) {
            const int s_lo = seg ? L0 : 0, s_hi = seg ? L : L0;
            const int a = t_first > s_lo ? t_first : s_lo, b = t_last < s_hi ? t_last : s_hi;
            if (a >= b) continue;
            const int Ls = seg ? L1 : L0;
            const elem_t *Kp = (seg ? K1 : K0) + (int64_t)bh * Ls * DH;
            const elem_t *Vp = (seg ? V1 : V0) + (int64_t)bh * Ls * DH;
            const int t_begin = a - s_lo, t_end = b - s_lo;        // token range inside the segment

            for (int tb = t_begin; tb < t_end; tb += kTile) {
                half8_t kr[NL], vr[NL];
                const int rows = t_end - tb < kTile ? t_end - tb : kTile;
                const __amdgpu_buffer_rsrc_t Kt = attn::step_rows(Kp + (int64_t)tb * DH, rows, DH);
                const __amdgpu_buffer_rsrc_t Vt = attn::step_rows(Vp + (int64_t)tb * DH, rows, DH);
#pragma unroll
                for (int i = 0; i < NL; ++i) kr[i] = attn::step_load<half8_t>(Kt, i, lane);
#pragma unroll
                for (int i = 0; i < NL; ++i) vr[i] = attn::step_load<half8_t>(Vt, i, lane);
                __builtin_amdgcn_sched_barrier(0);                 // every load of the step is on its way before the first use
                tile.consume(qv, kr, vr, lane, tb + c * RPL + g < t_end, scale_log2e);
            }
        }
        tile.store(partial + ((int64_t)w + bh) * (DH + 2), lane);
        p = (int64_t)bh * L + t_last;
    }
}

// One workgroup per pair: its P wavefronts take the steps of the two segments in turn and merge in LDS, so that one launch
// does what the ranges and their merge do in two (attn_pairs.h says when).  Bound by the latency of a step and of a
// launch for short contexts; for long ones by what one compute unit can ask for, 58 GB/s: 8 wavefronts of a pair were no
// faster than 4.  1 and 2 wavefronts a pair, several pairs a workgroup, for contexts of as many steps.
template <int DH, int DT, int P>
__global__ __launch_bounds__(kThreads, 3) void flash_pair_kernel(
    const typename Elem<DT>::T *__restrict__ q,
    const typename Elem<DT>::T *__restrict__ K0, const typename Elem<DT>::T *__restrict__ V0,
    const typename Elem<DT>::T *__restrict__ K1, const typename Elem<DT>::T *__restrict__ V1,
    int L0, int L1, int BH, float scale_log2e, typename Elem<DT>::T *__restrict__ out, float2 *__restrict__ lse)
{
    typedef typename Elem<DT>::V8 half8_t;
    typedef attn::Tile<DH, DT> tile_t;
    constexpr int LPR = tile_t::LPR, RPL = tile_t::RPL, NL = tile_t::NL;
    __shared__ __align__(16) float part[kWavesPerBlock][DH + 2];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int bh = blockIdx.x * (kWavesPerBlock / P) + wave / P;
    const bool live = bh < BH;
    if (!live) bh = BH - 1;              // works on the last pair (the workgroup shares a barrier), stores nothing
    const int g = lane / LPR, c = lane % LPR;
    const half8_t qv = *reinterpret_cast<const half8_t *>(q + (int64_t)bh * DH + c * 8);
    tile_t tile;
    tile.clear();
    const int n0 = (L0 + kTile - 1) / kTile, n = n0 + (L1 + kTile - 1) / kTile;     // steps of the two segments
    for (int s = wave % P; s < n; s += P) {
        const bool second = s >= n0;
        const int Ls = second ? L1 : L0, tb = (second ? s - n0 : s) * kTile;
        const int64_t at = ((int64_t)bh * Ls + tb) * DH;
        const int rows = Ls - tb < kTile ? Ls - tb : kTile;
        const __amdgpu_buffer_rsrc_t Kt = attn::step_rows((second ? K1 : K0) + at, rows, DH);
        const __amdgpu_buffer_rsrc_t Vt = attn::step_rows((second ? V1 : V0) + at, rows, DH);
        half8_t kr[NL], vr[NL];
#pragma unroll
        for (int i = 0; i < NL; ++i) kr[i] = attn::step_load<half8_t>(Kt, i, lane);
#pragma unroll
        for (int i = 0; i < NL; ++i) vr[i] = attn::step_load<half8_t>(Vt, i, lane);
        __builtin_amdgcn_sched_barrier(0);                     // every load of the step is on its way before the first use
        tile.consume(qv, kr, vr, lane, c * RPL + g < rows, scale_log2e);
    }
    tile.store(part[wave], lane);
    __syncthreads();
    if (!live || wave % P != 0) return;
    merge::Shared<DH, 1> none;
    float m, l, o[DH / 64];
    merge::merge_run<DH, 1>(part[wave], P, none, m, l, o);
    merge::store_row<DH>(out + (int64_t)bh * DH, o, l);
    if (lse && lane == 0) lse[bh] = make_float2(m, l);
}

// Log-sum-exp merge of the partials of every (sequence, head), P wavefronts each: those of the wavefronts whose range
// meets the pair's positions [bh L, (bh+1) L), at indices (wavefront + bh).
template <int DH, int DT, int P>
__global__ __launch_bounds__(merge::kThreads) void merge_partials_kernel(const float *__restrict__ partial, int L, int64_t total,
                                                                         int W, int BH, typename Elem<DT>::T *__restrict__ out,
                                                                         float2 *__restrict__ lse)
{
    __shared__ merge::Shared<DH, P> sh;
    const int wave = threadIdx.x >> 6;
    int bh = blockIdx.x * (kWavesPerBlock / P) + wave / P;
    const bool live = bh < BH;
    if (!live) bh = BH - 1;                                    // works on the last pair (the workgroup shares a barrier), stores nothing
    const int64_t lo = (int64_t)bh * L, hi = lo + L - 1;       // first and last position of the pair
    const int w_first = ranges::owner(lo, total, W), w_last = ranges::owner(hi, total, W);
    float m, l, o[DH / 64];
    merge::merge_run<DH, P>(partial + ((int64_t)w_first + bh) * (DH + 2), w_last - w_first + 1, sh, m, l, o);
    if (!live || wave % P != 0) return;
    merge::store_row<DH>(out + (int64_t)bh * DH, o, l);
    if (lse && (threadIdx.x & 63) == 0) lse[bh] = make_float2(m, l);
}

static_assert(pairs::kTile == kTile, "the rules count the kernel's steps");

template <int DH, int DT, int P>
void launch_merge(const AttnArgs &a, int L, int64_t total, hipStream_t s)
{
    constexpr int pairs = kWavesPerBlock / P;                  // of a workgroup
    hipLaunchKernelGGL((merge_partials_kernel<DH, DT, P>), dim3((unsigned)((a.BH + pairs - 1) / pairs)), dim3(merge::kThreads), 0, s,
                       a.partial, L, total, a.n_waves, a.BH, static_cast<typename Elem<DT>::T *>(a.out), a.lse);
}

template <int DH, int DT>
hipError_t launch_dh(const AttnArgs &a, hipStream_t s)
{
    typedef typename Elem<DT>::T elem_t;
    const int L = a.L0 + a.L1;
    const int64_t total = (int64_t)a.BH * L;
    const float scale_log2e = a.scale * 1.4426950408889634f;
    const int steps = pairs::steps(a.L0, a.L1);
    if (!a.ranges_given && pairs::contiguous(a.BH, steps, DH)) {
        auto launch = [&](auto kern, int per_block) {
            hipLaunchKernelGGL(kern, dim3((unsigned)((a.BH + per_block - 1) / per_block)), dim3(kThreads), 0, s,
                               static_cast<const elem_t *>(a.q),
                               static_cast<const elem_t *>(a.K0), static_cast<const elem_t *>(a.V0),
                               static_cast<const elem_t *>(a.K1), static_cast<const elem_t *>(a.V1),
                               a.L0, a.L1, a.BH, scale_log2e, static_cast<elem_t *>(a.out), a.lse);
        };
        if (steps == 1) launch(flash_pair_kernel<DH, DT, 1>, 4);
        else if (steps == 2) launch(flash_pair_kernel<DH, DT, 2>, 2);
        else launch(flash_pair_kernel<DH, DT, 4>, 1);
        const hipError_t e = hipGetLastError();
        return e == hipSuccess && a.after_main ? hipEventRecord(a.after_main, s) : e;
    }
    const unsigned blocks = (unsigned)((a.n_waves + kWavesPerBlock - 1) / kWavesPerBlock);
    hipLaunchKernelGGL((flash_decode_kernel<DH, DT>), dim3(blocks), dim3(kThreads), 0, s,
                       static_cast<const elem_t *>(a.q),
                       static_cast<const elem_t *>(a.K0), static_cast<const elem_t *>(a.V0),
                       static_cast<const elem_t *>(a.K1), static_cast<const elem_t *>(a.V1),
                       a.L0, a.L1, total, a.n_waves, scale_log2e, a.partial);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && a.after_main) e = hipEventRecord(a.after_main, s);
    if (e != hipSuccess) return e;
    if (merge::waves_per_pair(a.n_waves, a.BH) == 1) launch_merge<DH, DT, 1>(a, L, total, s);
    else launch_merge<DH, DT, 4>(a, L, total, s);
    return hipGetLastError();
}

// out = (w_a out_a + w_b out_b) / (w_a + w_b), w_x = l_x 2^(m_x - max(m_a, m_b)): the log-sum-exp join of two token
// segments.  A segment without tokens has denominator 0 and drops out.  4 elements per thread.
template <int DT>
__global__ __launch_bounds__(256) void segment_join_kernel(const typename Elem<DT>::T *__restrict__ out_a, const float2 *__restrict__ lse_a,
                                                           const typename Elem<DT>::T *__restrict__ out_b, const float2 *__restrict__ lse_b,
                                                           typename Elem<DT>::T *__restrict__ out, int64_t n4, int dh4)
{
    typedef typename Elem<DT>::T elem_t;
    typedef elem_t half4_t __attribute__((ext_vector_type(4)));
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n4) return;
    const int64_t bh = idx / dh4;
    const float2 sa = lse_a[bh], sb = lse_b[bh];
    const float m = fmaxf(sa.x, sb.x);
    const float wa = sa.y * __builtin_amdgcn_exp2f(sa.x - m), wb = sb.y * __builtin_amdgcn_exp2f(sb.x - m);
    const half4_t a = reinterpret_cast<const half4_t *>(out_a)[idx], b = reinterpret_cast<const half4_t *>(out_b)[idx];
    const float inv = wa + wb > 0.f ? 1.0f / (wa + wb) : 0.f;
    half4_t o;
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = (elem_t)((wa * (float)a[j] + wb * (float)b[j]) * inv);
    reinterpret_cast<half4_t *>(out)[idx] = o;
}

}  // namespace

hipError_t launch_segment_join(const void *out_a, const float2 *lse_a, const void *out_b, const float2 *lse_b, void *out,
                               int BH, int head_dim, int dtype, hipStream_t s)
{
    if (BH <= 0) return hipSuccess;
    if (head_dim % 4 != 0) return hipErrorInvalidValue;
    const int64_t n4 = (int64_t)BH * (head_dim / 4);
    const unsigned blocks = (unsigned)((n4 + 255) / 256);
    if (dtype == 1)
        hipLaunchKernelGGL(segment_join_kernel<1>, dim3(blocks), dim3(256), 0, s, static_cast<const __bf16 *>(out_a), lse_a,
                           static_cast<const __bf16 *>(out_b), lse_b, static_cast<__bf16 *>(out), n4, head_dim / 4);
    else
        hipLaunchKernelGGL(segment_join_kernel<0>, dim3(blocks), dim3(256), 0, s, static_cast<const _Float16 *>(out_a), lse_a,
                           static_cast<const _Float16 *>(out_b), lse_b, static_cast<_Float16 *>(out), n4, head_dim / 4);
    return hipGetLastError();
}

int attn_wavefronts(int64_t BH, int64_t L, int splits)
{
    const int64_t total = BH * L;
    if (total <= 0) return 0;
    int64_t W;
    if (splits > 0) {
        W = BH * splits;                                       // `splits` equal token ranges per pair
    } else {
        W = kAttnResidentWaves;                                // every wavefront resident: one round
        // Small problems: every pair cut into ranges of at most one step of 64 tokens, none across two pairs, so that
        // a wavefront asks for all of its bytes at once and pays one memory latency.
        const int64_t by_work = BH * ((L + kTile - 1) / kTile);
        if (W > by_work) W = by_work;
    }
    if (W > total) W = total;                                  // no empty range
    if (W > kAttnMaxWaves) W = kAttnMaxWaves;
    return (int)W;
}

hipError_t launch_flash_decode(const AttnArgs &a, hipStream_t s)
{
    if (a.BH <= 0) return hipSuccess;
    if (a.n_waves <= 0 || a.n_waves > kAttnMaxWaves || (int64_t)a.n_waves > (int64_t)a.BH * (a.L0 + a.L1))
        return hipErrorInvalidValue;
    if (a.head_dim == 128) return a.dtype == 1 ? launch_dh<128, 1>(a, s) : launch_dh<128, 0>(a, s);
    if (a.head_dim == 64) return a.dtype == 1 ? launch_dh<64, 1>(a, s) : launch_dh<64, 0>(a, s);
    return hipErrorInvalidValue;
}

}  // namespace hk
