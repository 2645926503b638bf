// One step of the single-query attention (Eq. 4) for one wavefront: 64 tokens of one (sequence, head), their K and V
// rows in registers, folded into the running softmax.  Shared by the contiguous and the paged kernel, which differ in
// where a token's rows are.
//
// DH / 8 lanes (LPR) cover one row with 16-byte loads, 64 / LPR rows (RPL) per load instruction, NL = LPR load
// instructions per operand and step: load i, lane group g (lane / LPR), lane c of the group (lane % LPR) holds elements
// 8 c .. 8 c + 7 of token i RPL + g.
//   * q.k: every lane forms the partial dot products of its 8 elements (v_dot2, fp32 sums); the LPR partials of the LPR
//     rows a group holds are combined by a reduce-scatter, after which lane (g, c) owns the complete score of token
//     c RPL + g: the softmax work (exp2, running maximum and sum) is done once per token, not per element.
//   * All exchanges inside a group are DPP moves on the vector ALU.  The butterfly's partners are lane ^ 8, ^ 7, ^ 2, ^ 1
//     (row rotate by 8, half-row mirror, quad permutes): these masks span a row of 16 lanes as 8, 4, 2, 1 do, and the
//     ownership is the same; a weight is spread over its group by a row broadcast.  Through the LDS permute network
//     (35 per step) they were a chain of LDS latencies.
//   * Online softmax per lane group in the log2 domain with a finite "-infinity".
//   * A step of fewer than 64 tokens reads zeros in the place of the missing rows (the bound of the buffer descriptor): a
//     repeated real row, masked by a weight of zero, would make 0 * inf = NaN of an infinite V element.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_merge.h"
#include "elem.h"

namespace hk {
namespace attn {

using merge::kNegBig;
constexpr int kTile = 64;               // tokens per wavefront step

template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
// The value of the exchange partner for the step of the butterfly that halves 2 H values (see above).
template <int H>
__device__ __forceinline__ float partner(float v)
{
    if constexpr (H == 8) return dpp<0x128>(v);            // row_ror:8          lane ^ 8
    else if constexpr (H == 4) return dpp<0x141>(v);       // row_half_mirror    lane ^ 7
    else if constexpr (H == 2) return dpp<0x4e>(v);        // quad_perm 2,3,0,1  lane ^ 2
    else return dpp<0xb1>(v);                              // quad_perm 1,0,3,2  lane ^ 1
}
// Value of lane I of the caller's row of 16 lanes.
template <int I>
__device__ __forceinline__ float row_bcast(float v) { return dpp<0x150 + I>(v); }

template <int DT>
__device__ __forceinline__ float dot8(typename Elem<DT>::V8 a, typename Elem<DT>::V8 b)
{
    typedef typename Elem<DT>::V2 half2_t;
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        half2_t x = {a[2 * j], a[2 * j + 1]};
        half2_t y = {b[2 * j], b[2 * j + 1]};
        s = Elem<DT>::dot2(x, y, s);
    }
    return s;
}

// Rows of one operand that lie in a row: `base` is the first, `rows` (0 .. 64) of them exist.  Both are wavefront-uniform;
// where the compiler cannot prove it, it would loop over the lanes' descriptors, so it is said.
template <typename elem_t>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t step_rows(const elem_t *base, int rows, int row_elems)
{
    const uint64_t at = reinterpret_cast<uintptr_t>(base);
    const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at);
    const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(at >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<elem_t *>(hi << 32 | lo), 0,
                                             __builtin_amdgcn_readfirstlane(rows) * row_elems * (int)sizeof(elem_t), 0x00020000);
}
// Load i of them: 64 lanes x 16 bytes, whole rows, non-temporal.
template <typename vec8_t>
__device__ __forceinline__ vec8_t step_load(__amdgpu_buffer_rsrc_t rows, int i, int lane)
{
    return __builtin_bit_cast(vec8_t, __builtin_amdgcn_raw_buffer_load_b128(rows, lane * 16 + i * 1024, 0, 2));
}

template <int DH, int DT>
struct Tile {
    typedef typename Elem<DT>::V8 vec8_t;
    static constexpr int LPR = DH / 8, RPL = 64 / LPR, NL = LPR;
    static_assert(LPR == 8 || LPR == 16, "the exchanges stay inside a row of 16 lanes");

    float m_run, l_run, acc[8];

    __device__ __forceinline__ void clear()
    {
        m_run = kNegBig;
        l_run = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = 0.f;
    }

    template <int H>
    static __device__ __forceinline__ void scatter(float (&pd)[NL], int c)
    {
        const bool up = (c & H) != 0;
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const float send = up ? pd[i] : pd[i + H];
            const float keep = up ? pd[i + H] : pd[i];
            pd[i] = keep + partner<H>(send);
        }
        if constexpr (H > 1) scatter<H / 2>(pd, c);
    }
    template <int H>
    static __device__ __forceinline__ float group_max(float v)
    {
        v = fmaxf(v, partner<H>(v));
        if constexpr (H > 1) return group_max<H / 2>(v);
        return v;
    }
    template <int I>
    __device__ __forceinline__ void add_rows(float pe, const vec8_t (&vr)[NL], bool high)
    {
        float w = row_bcast<I>(pe);                        // weight of token I RPL + g
        if constexpr (LPR == 8) w = high ? row_bcast<I + 8>(pe) : w;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = __builtin_fmaf(w, (float)vr[I][j], acc[j]);
        // a bf16 element is widened where it is used: ahead of time, the 64 registers of V rows become 128
        if constexpr (DT == 1) __builtin_amdgcn_sched_barrier(0);
        if constexpr (I + 1 < NL) add_rows<I + 1>(pe, vr, high);
    }

    // lane = (g, c); valid: the token this lane will own, c RPL + g of the step, takes part.
    __device__ __forceinline__ void consume(const vec8_t &qv, const vec8_t (&kr)[NL], const vec8_t (&vr)[NL], int lane, bool valid,
                                            float scale_log2e)
    {
        const int c = lane % LPR;
        float pd[NL];
#pragma unroll
        for (int i = 0; i < NL; ++i) pd[i] = dot8<DT>(qv, kr[i]);
        scatter<LPR / 2>(pd, c);
        const float s = valid ? pd[0] * scale_log2e : -INFINITY;
        const float m_new = fmaxf(m_run, group_max<LPR / 2>(s));
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        const float pe = __builtin_amdgcn_exp2f(s - m_new);
        m_run = m_new;
        l_run = l_run * alpha + pe;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] *= alpha;
        if constexpr (DT == 1) __builtin_amdgcn_sched_barrier(0);
        add_rows<0>(pe, vr, (lane & 8) != 0);
    }

    // Combines the lane groups: the denominator over the lanes of a group, then (m, l, o) over the groups; lanes of
    // group 0 store the un-normalised partial (m, l, o[DH]).
    __device__ __forceinline__ void store(float *__restrict__ dst, int lane)
    {
        l_run += partner<1>(l_run);
        l_run += partner<2>(l_run);
        l_run += partner<4>(l_run);
        if constexpr (LPR == 16) l_run += partner<8>(l_run);
#pragma unroll
        for (int off = LPR; off < 64; off <<= 1) {
            const float m_o = __shfl_xor(m_run, off, 64);
            const float l_o = __shfl_xor(l_run, off, 64);
            const float m_new = fmaxf(m_run, m_o);
            const float sa = __builtin_amdgcn_exp2f(m_run - m_new), sb = __builtin_amdgcn_exp2f(m_o - m_new);
            l_run = l_run * sa + l_o * sb;
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] = acc[j] * sa + __shfl_xor(acc[j], off, 64) * sb;
            m_run = m_new;
        }
        if (lane < LPR) {
#pragma unroll
            for (int j = 0; j < 4; ++j)                    // slots are 8-byte aligned
                *reinterpret_cast<float2 *>(dst + 2 + lane * 8 + 2 * j) = make_float2(acc[2 * j], acc[2 * j + 1]);
            if (lane == 0) *reinterpret_cast<float2 *>(dst) = make_float2(m_run, l_run);
        }
    }
};

}  // namespace attn
}  // namespace hk
