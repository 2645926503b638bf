// Log-sum-exp merge of the partials of one (sequence, head) pair, shared by the contiguous and the paged attention
// (Eq. 4 split over the token axis): `n` consecutive slots (m, l, o[DH]) in fp32, of which the caller knows the first.
//
// Bound by latency, not bytes (a pair has 1 .. a few dozen partials of 520 bytes): P wavefronts share a pair's run,
// each takes its part kBatch slots at a time with every load of a batch issued before the first use, and the P
// results meet in LDS.  With one thread per element walking the slots one after the other (two dependent passes, and
// 64-bit divisions in front) the merge of 4608 pairs of one or two partials took 15.9 us and that of 7168 pairs 22.8; now 6.8
// and 8.7 us (profiles/hybrid_step_opt66b.txt, hybrid_step_opt30b.txt).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hk {
namespace merge {

constexpr float kNegBig = -1.0e30f;      // finite stand-in for -inf in running maxima
constexpr int kBatch = 8;
constexpr int kThreads = 256;

// Wavefronts per pair for a launch of W wavefronts over `pairs` pairs: one while a pair's run fits a batch or so.
inline int waves_per_pair(int64_t W, int64_t pairs) { return pairs > 0 && W / pairs > 8 ? 4 : 1; }

template <int DH, int P>
struct Shared {
    float v[P > 1 ? kThreads / 64 : 1][DH + 2];
};

// All 256 threads of the workgroup call it (P > 1: one barrier).  Returns in every lane of the pair's first wavefront
// the merged (m, l) and in o[] its DH / 64 elements lane * DH / 64 + 0, 1 of the un-normalised output.
template <int DH, int P>
__device__ __forceinline__ void merge_run(const float *__restrict__ src, int n, Shared<DH, P> &sh, float &m, float &l, float (&o)[DH / 64])
{
    constexpr int E = DH / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int part = wave % P;
    const int per = (n + P - 1) / P;
    const int i_begin = part * per, i_end = i_begin + per < n ? i_begin + per : n;
    m = kNegBig;
    l = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) o[e] = 0.f;
    for (int i0 = i_begin; i0 < i_end; i0 += kBatch) {
        float mm[kBatch], ll[kBatch];
        float oo[kBatch][E];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const int i = i0 + j < i_end ? i0 + j : i_end - 1;                  // clamped: masked below
            const float *p = src + (int64_t)i * (DH + 2);
            mm[j] = p[0];
            ll[j] = p[1];
            if constexpr (E == 2) {
                const float2 v = *reinterpret_cast<const float2 *>(p + 2 + 2 * lane);   // slots are 8-byte aligned
                oo[j][0] = v.x;
                oo[j][1] = v.y;
            } else {
                oo[j][0] = p[2 + lane];
            }
        }
        float mx = m;
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            if (i0 + j >= i_end) {
                // neutral: weight 2^-inf = 0, and nothing for it to meet (the slot read in its place may hold an infinity)
                mm[j] = -INFINITY;
                ll[j] = 0.f;
#pragma unroll
                for (int e = 0; e < E; ++e) oo[j][e] = 0.f;
            }
            mx = fmaxf(mx, mm[j]);
        }
        const float a = __builtin_amdgcn_exp2f(m - mx);
        l *= a;
#pragma unroll
        for (int e = 0; e < E; ++e) o[e] *= a;
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const float w = __builtin_amdgcn_exp2f(mm[j] - mx);
            l = __builtin_fmaf(w, ll[j], l);
#pragma unroll
            for (int e = 0; e < E; ++e) o[e] = __builtin_fmaf(w, oo[j][e], o[e]);
        }
        m = mx;
    }
    if constexpr (P > 1) {
        sh.v[wave][0] = m;
        sh.v[wave][1] = l;
#pragma unroll
        for (int e = 0; e < E; ++e) sh.v[wave][2 + E * lane + e] = o[e];
        __syncthreads();
        if (part != 0) return;
        float mx = m;
#pragma unroll
        for (int q = 1; q < P; ++q) mx = fmaxf(mx, sh.v[wave + q][0]);
        const float a = __builtin_amdgcn_exp2f(m - mx);
        l *= a;
#pragma unroll
        for (int e = 0; e < E; ++e) o[e] *= a;
#pragma unroll
        for (int q = 1; q < P; ++q) {
            const float w = __builtin_amdgcn_exp2f(sh.v[wave + q][0] - mx);
            l = __builtin_fmaf(w, sh.v[wave + q][1], l);
#pragma unroll
            for (int e = 0; e < E; ++e) o[e] = __builtin_fmaf(w, sh.v[wave + q][2 + E * lane + e], o[e]);
        }
        m = mx;
    }
}

// o / l of the pair to its output row (DH elements of T), by the pair's first wavefront.
template <int DH, typename T>
__device__ __forceinline__ void store_row(T *__restrict__ out, const float (&o)[DH / 64], float l)
{
    constexpr int E = DH / 64;
    const int lane = threadIdx.x & 63;
    typedef T vec_t __attribute__((ext_vector_type(2)));
    if constexpr (E == 2) {
        const vec_t v = {(T)(o[0] / l), (T)(o[1] / l)};
        *reinterpret_cast<vec_t *>(out + 2 * lane) = v;
    } else {
        out[lane] = (T)(o[0] / l);
    }
}

}  // namespace merge
}  // namespace hk
