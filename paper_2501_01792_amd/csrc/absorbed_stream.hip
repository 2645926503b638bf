// The two passes over the checkpoint rows of the decode attention that does not regenerate their K/V (absorbed.hip):
//
//   scores  s_t(h) = sl [ f rstd_t (x_t - x_t[0]) . u_h + k_t c1_h + c2_h ],  k_t = -(mean_t - x_t[0]) rstd_t,  sl = scale log2(e),
//           c1 = q_h . c_K,h, c2 = q_h . b'_K,h, f the factor of the prepared layer's scaled weights; and from the same pass
//           the LayerNorm statistics of the rows and the softmax over a block of them:
//             e = ceil(max (s_t + log2 rstd_t)),  p_t = 2^(s_t - e),  w_t = fp16(2^14 rstd_t p_t) <= 2^14,
//             l = sum p_t,  mu = sum w_t mean_t
//   gather  Y_h = (sum_t w_t f_t x_t - sum f mu) / (2^14 sum f l),  f = 2^(e - max e) of the row's block
//
// e is a whole number, so f is a power of two and the weights of all blocks meet without a second rounding; the mean term
// is formed from the stored w_t, so that a row mean that is large against the row's spread cancels against what the product
// really adds.  Rows enter the score product minus their first element for the same reason.
//
// What bounds them: each is one pass over the rows (2 d bytes a row), and an L2 stream of the small operand beside it.
// The earlier forms moved rows through registers into LDS and had every wavefront fetch its share of the small operand: the
// loads retire in order, so the L2 loads queued behind the HBM loads, 4 waves a SIMD waited to issue, and both passes
// read 5.1 TB/s; a third kernel turned scores into weights.  Here:
//   * Rows go to LDS directly (16 bytes a lane, whole 128-byte lines, swizzled on the global side), a private ring per
//     wavefront, so that no barrier stands between a row's arrival and its use.
//   * One wavefront of the workgroup does nothing but fetch the small operand, with its own count of loads in flight.
//   * Rows that do not stay in the last-level cache for the second pass are asked for non-temporally (2.4 GB: 387 against 451
//     us; 134 MB, which stay: 25 against 22.5), and the results leave with non-temporal stores then: dirty lines that are
//     written back under a stream of reads cost it far more than their bytes (gather of 2.4 GB, 85 MB of results: 452
//     against 385 us).
// Measured on 64 x 2048 rows of d = 9216 (72 heads), before -> now (profiles/absorbed_step_opt66b_ratio0.5.txt, 42 calls on
// average, in brackets the least): scores and softmax 471 + 28 -> 385 us (376; 6.3 TB/s), gather 465 -> 412 (383); 32 x 512 rows of d =
// 4096 (32 heads, profiles/absorbed_step_opt6.7b.txt): 28.5 + 6.6 -> 27.0 (25.2), gather 31 -> 23.7 (23.1).  Error against 64 bits as
// before: 0.90 to 1.11 of it over 13 shapes, 0.99 in the middle (fp16 and bf16).
#include "hk_internal.h"
#include "kv_gemm_common.h"
#include "skinny_mma.h"

#include <type_traits>

namespace hk {
namespace {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void *lds_ptr_t;
typedef const __attribute__((address_space(1))) void *glb_ptr_t;

constexpr float kNegBig = -1.0e30f;
constexpr float kWeightScale = 16384.f;                    // of the stored weights: their largest is in (2^13, 2^14]
constexpr int kNt = 2;                                     // cache policy of a load: non-temporal

// Waits until at most N of the youngest vector memory operations of this wavefront are in flight.
template <int N>
__device__ __forceinline__ void wait_vm()
{
    static_assert(N <= 63, "vmcnt counts to 63");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

// A store that leaves no dirty line behind (NT), or one that the next kernel finds in cache.
template <bool NT, typename V>
__device__ __forceinline__ void store_as(V v, V *dst)
{
    if constexpr (NT) __builtin_nontemporal_store(v, dst);
    else *dst = v;
}

template <bool NT>
__device__ __forceinline__ void load_lds(const _Float16 *src, unsigned char *dst)
{
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_global_load_lds((glb_ptr_t)src, (lds_ptr_t)dst, 16, 0, NT ? kNt : 0);
#endif
}

struct ScoreArgs {
    const _Float16 *act, *U;                               // [B, L, d] or the pool; [H, B, d]
    const float2 *c12;                                     // [B, H]: (q . c_K, q . b'_K)
    const float *factor;                                   // of the scaled weights
    _Float16 *w;                                           // [B, H, Lp]
    float4 *part;                                          // [B, blocks, H]: (e, l, mu, -) of every block of rows
    int B, L, Lp, H, d, blocks;                            // L: rows of a sequence (the most, where n_rows says how many)
    float eps, sl;
    int nt;
    // rows in blocks scattered over a pool (PAGED): row r of sequence b is row r % 2^blk_log2 of pool block
    // list[b list_pitch + r / 2^blk_log2], n_rows[b] of them; cu_items: prefix sums over the sequences of ceil(n_rows / ROWS)
    const int32_t *list, *n_rows, *cu_items;
    int list_pitch, blk_log2;
};

template <bool PAGED>
__device__ __forceinline__ const _Float16 *row_ptr(const ScoreArgs &p, int64_t b, int t)
{
    if constexpr (PAGED) {
        const int64_t blk = p.list[b * p.list_pitch + (t >> p.blk_log2)];
        return p.act + ((blk << p.blk_log2) + (t & ((1 << p.blk_log2) - 1))) * p.d;
    } else {
        return p.act + (b * p.L + t) * p.d;
    }
}

// Sequence and block of an item of the ring form.
template <bool PAGED>
__device__ __forceinline__ void item_place(const ScoreArgs &p, int item, int64_t &b, int &k)
{
    if constexpr (PAGED) {
        const int lane = threadIdx.x & 63;
        int base = 0;
        for (;;) {                                         // sequences whose items all come before: cu_items[s + 1] <= item
            const int s = base + lane;
            const int n = __popcll(__ballot(s < p.B && p.cu_items[s < p.B ? s + 1 : p.B] <= item));
            base += n;
            if (n < 64) break;
        }
        b = __builtin_amdgcn_readfirstlane(base);
        k = item - __builtin_amdgcn_readfirstlane(p.cu_items[b]);
    } else {
        b = item / p.blocks;
        k = item % p.blocks;
    }
}

// LayerNorm statistics of a row from its moments about its first element.
struct RowStats {
    float rstd, kx, mean, lg;                              // kx = -(mean - first) rstd, lg = log2 rstd
};
__device__ __forceinline__ RowStats row_stats(float s1, float s2, float first, int d, float eps)
{
    const float inv_d = 1.0f / (float)d;
    const float dm = s1 * inv_d;                           // mean - first element
    const float var = fmaxf(__builtin_fmaf(-dm, dm, s2 * inv_d), 0.f);
    RowStats r;
    r.rstd = 1.0f / __builtin_sqrtf(var + eps);
    r.kx = -dm * r.rstd;
    r.mean = first + dm;
    r.lg = __builtin_amdgcn_logf(r.rstd);
    return r;
}

// Ring form: NW wavefronts of 16 RW rows each, and one that fetches U.  Items of ROWS = 16 RW NW rows of one sequence; a
// workgroup takes a run of them, and its loads run on from one item into the next, under the softmax of the first.
//   * Wavefront w's ring: XS stages of 16 RW rows x 64 elements.  U's ring: US stages of 16 HB heads x 64 elements.  One
//     barrier per 64 elements, behind which U's next stage is there and its stage before last is free.
//   * LDS row q = 16 i + m of a stage holds row 4 RW (m / 4) + 4 i + m % 4, so that a lane ends up with 4 RW consecutive
//     rows of one head: D of v_mfma_f32_16x16x32 has row 4 (lane / 16) + r of block i, head lane % 16.
//   * RW = 2, NW = 8 (256 rows, U read once for them) and RW = 4, NW = 4 were level (388 us; 128 rows: 431), as were 2 and 4
//     stages of rows and up to 8 of U; fragments of the next half read under the MFMAs of this one: 390.
//   * From six blocks of heads on the 256-row form keeps 25 to 64 registers in scratch, and is the best all the same: 96 heads, d =
//     12288, 65536 rows: 721 us the whole step, 742 with 128 rows (RW = 1, NW = 8, no scratch), 792 with 64; 128 heads, d =
//     16384: 1145 / 1152 / 1397.  Blocks of 16 heads one by one: 81 to 96 heads on the form of 128 took 781 us there, and in bf16
//     at 16384 rows of d = 6144 178, where six blocks take 163.
template <int HB, int RW, int NW, int XS, int US>
constexpr int ring_lds_bytes() { return NW * XS * RW * 2048 + US * HB * 2048 + NW * HB * 16 * 12; }

template <int HB, int RW, int NW, int XS, int US, int DT, bool PAGED, bool NT>
__global__ __launch_bounds__(64 * NW + 64) void absorbed_scores_ring_kernel(ScoreArgs p)
{
#if defined(__HIP_DEVICE_COMPILE__)                        // (the host pass drops the kernel's stub over a direct load in this body)
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int WR = 16 * RW, ROWS = WR * NW, XB = WR * 128, UB = HB * 2048, H16 = HB * 16;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int H = p.H, d = p.d;
    const int items = PAGED ? __builtin_amdgcn_readfirstlane(p.cu_items[p.B]) : p.blocks * p.B;
    const int run = gemm::xcd_regroup(blockIdx.x, gridDim.x);              // neighbouring runs share U in an XCD's L2
    const int i_begin = (int)((int64_t)run * items / gridDim.x), i_end = (int)((int64_t)(run + 1) * items / gridDim.x);
    if (i_begin >= i_end) return;                          // uniform over the workgroup, before any barrier
    const int steps = d / 64, total = (i_end - i_begin) * steps;
    unsigned char *uring = smem + NW * XS * XB;
    float *xmax = reinterpret_cast<float *>(uring + US * UB);              // [NW][H16]
    float *xlm = xmax + NW * H16;                                          // [NW][H16] (l, mu)
    const int g_row = lane >> 3;                           // of a load: 8 rows x 128 bytes, 8 lanes a row

    if (wave == NW) {                                      // ---- U
        const _Float16 *src[2 * HB];
        int item = i_begin, k = 0, slot = 0;
        auto set = [&] {
            int64_t b;
            int blk;
            item_place<PAGED>(p, item, b, blk);
#pragma unroll
            for (int i = 0; i < 2 * HB; ++i) {
                const int q = 8 * i + g_row, h = q < H ? q : H - 1;        // heads past the end: computed, never stored
                src[i] = p.U + ((int64_t)h * p.B + b) * d + 8 * ((lane & 7) ^ ((q >> 1) & 7));
            }
        };
        set();
        auto issue = [&] {
#pragma unroll
            for (int i = 0; i < 2 * HB; ++i) {
                load_lds<false>(src[i], uring + slot * UB + i * 1024);
                src[i] += 64;
            }
            slot = slot + 1 == US ? 0 : slot + 1;
            if (++k == steps) {
                k = 0;
                if (++item < i_end) set();
            }
        };
        for (int s = 0; s < US && s < total; ++s) issue();
        int left = steps;
        for (int s = 0; s < total; ++s) {
            // in front of barrier s, stages up to s + US - 2 (s = 0: US - 1) have been asked for
            if (s + US - 2 < total) wait_vm<2 * HB * (US - 2)>();
            else wait_vm<0>();
            asm volatile("s_barrier" ::: "memory");
            if (s > 0 && s - 1 + US < total) issue();
            if (--left == 0) {
                left = steps;
                asm volatile("s_barrier\n\ts_barrier" ::: "memory");       // the two of the softmax
            }
        }
        return;
    }

    // ---- rows
    unsigned char *my = smem + wave * XS * XB;
    const int fr = lane & 15, fc = lane >> 4;
    const _Float16 *src[2 * RW];
    int ask_item = i_begin, ask_k = 0, ask_slot = 0;
    auto set = [&] {
        int64_t b;
        int k;
        item_place<PAGED>(p, ask_item, b, k);
        const int n = PAGED ? p.n_rows[b] : p.L;
#pragma unroll
        for (int i = 0; i < 2 * RW; ++i) {
            const int q = 8 * i + g_row, m = q & 15;
            int t = k * ROWS + wave * WR + 4 * RW * (m >> 2) + 4 * (q >> 4) + (m & 3);
            if (t >= n) t = n - 1;                         // rows past the end: weight 0
            src[i] = row_ptr<PAGED>(p, b, t) + 8 * ((lane & 7) ^ ((q >> 1) & 7));
        }
    };
    set();
    auto issue = [&] {
#pragma unroll
        for (int i = 0; i < 2 * RW; ++i) {
            load_lds<NT>(src[i], my + ask_slot * XB + i * 1024);
            src[i] += 64;
        }
        ask_slot = ask_slot + 1 == XS ? 0 : ask_slot + 1;
        if (++ask_k == steps) {
            ask_k = 0;
            if (++ask_item < i_end) set();
        }
    };
    for (int s = 0; s < XS && s < total; ++s) issue();
    int foff[2];                                           // fragment: LDS row fr (+ 16 i), logical chunk 4 ks + fc
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) foff[ks] = fr * 128 + (((4 * ks + fc) ^ ((fr >> 1) & 7)) << 4);
    const float factor = *p.factor;
    int slot = 0, us = 0, done = 0;
    for (int item = i_begin; item < i_end; ++item) {
        int64_t b;
        int k;
        item_place<PAGED>(p, item, b, k);
        const int n = PAGED ? p.n_rows[b] : p.L;
        const int tw = k * ROWS + wave * WR;
        half2_t first[RW];
        float m1[RW], m2[RW];
        float4_t acc[RW][HB];
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            int t = tw + 4 * RW * (fr >> 2) + 4 * i + (fr & 3);
            if (t >= n) t = n - 1;
            const _Float16 f = skinny::stored_to_half<DT>(row_ptr<PAGED>(p, b, t));
            first[i] = half2_t{f, f};
            m1[i] = m2[i] = 0.f;
#pragma unroll
            for (int j = 0; j < HB; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
        }
        for (int s = 0; s < steps; ++s, ++done) {
            if (done + XS <= total) wait_vm<2 * RW * (XS - 1)>();          // this wavefront's stage is there
            else wait_vm<0>();
            asm volatile("s_barrier" ::: "memory");                        // and U's
            constexpr bool kAhead = HB <= 5;                               // registers for both halves' fragments
            half8_t xf[2][RW], uf[2][HB];
            auto fragments = [&](int ks) {
#pragma unroll
                for (int i = 0; i < RW; ++i) xf[ks][i] = *reinterpret_cast<const half8_t *>(my + slot * XB + i * 2048 + foff[ks]);
#pragma unroll
                for (int j = 0; j < HB; ++j) uf[ks][j] = *reinterpret_cast<const half8_t *>(uring + us * UB + j * 2048 + foff[ks]);
            };
            if constexpr (kAhead) {
                fragments(0);
                fragments(1);
            }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                if constexpr (!kAhead) {
                    __builtin_amdgcn_sched_barrier(0);
                    fragments(ks);
                }
#pragma unroll
                for (int i = 0; i < RW; ++i) {
                    half8_t v = skinny::to_half8<DT>(xf[ks][i]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const half2_t pr = half2_t{v[2 * e], v[2 * e + 1]} - first[i];
                        m1[i] = __builtin_amdgcn_fdot2(pr, half2_t{(_Float16)1.f, (_Float16)1.f}, m1[i], false);
                        m2[i] = __builtin_amdgcn_fdot2(pr, pr, m2[i], false);
                        v[2 * e] = pr[0];
                        v[2 * e + 1] = pr[1];
                    }
#pragma unroll
                    for (int j = 0; j < HB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(v, uf[ks][j], acc[i][j], 0, 0, 0);
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");             // every read of the stage has come back
            __builtin_amdgcn_sched_barrier(0);
            if (done + XS < total) issue();                                // into its slot
            slot = slot + 1 == XS ? 0 : slot + 1;
            us = us + 1 == US ? 0 : us + 1;
        }

        // ---- statistics, softmax over the item's rows, weights.  Lane: heads 16 j + fr, rows tl + 4 i + r.
        float2 cc[HB];
#pragma unroll
        for (int j = 0; j < HB; ++j) cc[j] = p.c12[b * H + (16 * j + fr < H ? 16 * j + fr : H - 1)];
        RowStats st[RW][4];
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            m1[i] += __shfl_xor(m1[i], 16, 64);
            m1[i] += __shfl_xor(m1[i], 32, 64);
            m2[i] += __shfl_xor(m2[i], 16, 64);
            m2[i] += __shfl_xor(m2[i], 32, 64);
            const RowStats own = row_stats(m1[i], m2[i], (float)first[i][0], d, p.eps);      // of LDS row 16 i + fr
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                st[i][r].rstd = __shfl(own.rstd, 4 * fc + r, 64);
                st[i][r].kx = __shfl(own.kx, 4 * fc + r, 64);
                st[i][r].mean = __shfl(own.mean, 4 * fc + r, 64);
                st[i][r].lg = __shfl(own.lg, 4 * fc + r, 64);
            }
        }
        const int tl = tw + 4 * RW * fc;
#pragma unroll
        for (int j = 0; j < HB; ++j) {
            float mx = kNegBig;
#pragma unroll
            for (int i = 0; i < RW; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float s = p.sl * __builtin_fmaf(st[i][r].rstd, acc[i][j][r] * factor, __builtin_fmaf(st[i][r].kx, cc[j].x, cc[j].y));
                    acc[i][j][r] = s;
                    if (tl + 4 * i + r < n) mx = fmaxf(mx, s + st[i][r].lg);
                }
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            if (fc == 0) xmax[wave * H16 + 16 * j + fr] = mx;
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        const int fill = (n + 63) & ~63;                   // weights are zero from n on to the next multiple of 64
#pragma unroll
        for (int j = 0; j < HB; ++j) {
            const int h = 16 * j + fr;
            float mx = kNegBig;
#pragma unroll
            for (int q = 0; q < NW; ++q) mx = fmaxf(mx, xmax[q * H16 + h]);
            const float e = __builtin_ceilf(mx);
            float l = 0.f, mu = 0.f;
            _Float16 o[4 * RW];
#pragma unroll
            for (int i = 0; i < RW; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const bool in = tl + 4 * i + r < n;
                    const float pt = in ? __builtin_amdgcn_exp2f(acc[i][j][r] - e) : 0.f;
                    const _Float16 wt = in ? (_Float16)(pt * st[i][r].rstd * kWeightScale) : (_Float16)0.f;
                    l += pt;
                    if (in) mu = __builtin_fmaf((float)wt, st[i][r].mean, mu);
                    o[4 * i + r] = wt;
                }
            if (h < H && tl < fill) {
                _Float16 *dst = p.w + (b * H + h) * p.Lp + tl;
                if constexpr (RW == 1) {
                    store_as<NT>(half4_t{o[0], o[1], o[2], o[3]}, reinterpret_cast<half4_t *>(dst));
                } else {
#pragma unroll
                    for (int q = 0; q < RW / 2; ++q) {
                        half8_t v;
#pragma unroll
                        for (int u = 0; u < 8; ++u) v[u] = o[8 * q + u];
                        store_as<NT>(v, reinterpret_cast<half8_t *>(dst + 8 * q));
                    }
                }
            }
            l += __shfl_xor(l, 16, 64);
            l += __shfl_xor(l, 32, 64);
            mu += __shfl_xor(mu, 16, 64);
            mu += __shfl_xor(mu, 32, 64);
            if (fc == 0) {
                xlm[2 * (wave * H16 + h)] = l;
                xlm[2 * (wave * H16 + h) + 1] = mu;
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        const int h = threadIdx.x;
        if (h < H) {
            float mx = kNegBig, l = 0.f, mu = 0.f;
#pragma unroll
            for (int q = 0; q < NW; ++q) {
                mx = fmaxf(mx, xmax[q * H16 + h]);
                l += xlm[2 * (q * H16 + h)];
                mu += xlm[2 * (q * H16 + h) + 1];
            }
            p.part[(b * p.blocks + k) * H + h] = make_float4(__builtin_ceilf(mx), l, mu, 0.f);
        }
    }
#endif
}

// Slab form, for few rows: 32 rows a workgroup, the reduction axis cut over its 4 wavefronts (skinny::slab_product), so that
// a small problem fills the chip and a workgroup's chain of steps is a quarter as long.
template <int RB, int DT, bool PAGED>
__global__ __launch_bounds__(256) void absorbed_scores_slab_kernel(ScoreArgs p)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int kSlab = skinny::kSlab;
    const int tid = threadIdx.x, H = p.H, d = p.d;
    const int item = gemm::xcd_regroup(blockIdx.x, p.blocks * p.B);
    const int64_t b = item / p.blocks;
    const int k = item % p.blocks, t0 = k * kSlab;
    const int n = PAGED ? p.n_rows[b] : p.L;
    if (t0 >= n) return;                                   // uniform over the workgroup, before any barrier
    const int rows = n - t0 < kSlab ? n - t0 : kSlab;
    auto row_of = [&](int r) { return row_ptr<PAGED>(p, b, t0 + r); };
    float (*red)[RB * 32][kSlab] = skinny::slab_product<RB, false, true, DT>(row_of, rows, p.U + b * d, H, (int64_t)p.B * d, d, smem);
    __shared__ RowStats st[kSlab];
    if (tid < kSlab) {
        float (*mom)[kSlab][2] = skinny::moments<RB>(smem);
        const float s1 = (mom[0][tid][0] + mom[1][tid][0]) + (mom[2][tid][0] + mom[3][tid][0]);
        const float s2 = (mom[0][tid][1] + mom[1][tid][1]) + (mom[2][tid][1] + mom[3][tid][1]);
        st[tid] = row_stats(s1, s2, (float)skinny::stored_to_half<DT>(row_of(tid < rows ? tid : rows - 1)), d, p.eps);
    }
    __syncthreads();
    const float factor = *p.factor;
    const int fill = (n + 63) & ~63;
    const int part = tid & 3, c0 = 8 * part;               // 4 lanes a head, 8 rows each
    for (int h = tid >> 2; h < H; h += 64) {
        const float2 cc = p.c12[b * H + h];
        float s[8], mx = kNegBig;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int c = c0 + u;
            const float a = (red[0][h][c] + red[1][h][c]) + (red[2][h][c] + red[3][h][c]);
            s[u] = p.sl * __builtin_fmaf(st[c].rstd, a * factor, __builtin_fmaf(st[c].kx, cc.x, cc.y));
            if (c < rows) mx = fmaxf(mx, s[u] + st[c].lg);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 1, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 2, 64));
        const float e = __builtin_ceilf(mx);
        float l = 0.f, mu = 0.f;
        half8_t o;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int c = c0 + u;
            const bool in = c < rows;
            const float pt = in ? __builtin_amdgcn_exp2f(s[u] - e) : 0.f;
            o[u] = in ? (_Float16)(pt * st[c].rstd * kWeightScale) : (_Float16)0.f;
            l += pt;
            if (in) mu = __builtin_fmaf((float)o[u], st[c].mean, mu);
        }
        _Float16 *dst = p.w + (b * H + h) * p.Lp + t0 + c0;
        *reinterpret_cast<half8_t *>(dst) = o;
        // the last slab also clears what the gather reads past it, up to the next multiple of 64 rows
        if (t0 + kSlab < fill && t0 + kSlab >= n) {
#pragma unroll
            for (int u = 0; u < 8; ++u) o[u] = (_Float16)0.f;
            *reinterpret_cast<half8_t *>(dst + kSlab) = o;
        }
        l += __shfl_xor(l, 1, 64);
        l += __shfl_xor(l, 2, 64);
        mu += __shfl_xor(mu, 1, 64);
        mu += __shfl_xor(mu, 2, 64);
        if (part == 0) p.part[(b * p.blocks + k) * H + h] = make_float4(e, l, mu, 0.f);
    }
}

// ---------------------------------------------------------------------------------------------------------
// gather: 4 wavefronts of 64 columns each, and one that fetches w.  A workgroup walks all rows of a sequence.
//   * Wavefront's ring: kXS stages of 32 rows x 128 bytes; w's ring: kWS tiles of 16 HB heads x 64 rows; one barrier a tile.
//   * The reduction runs over rows, so fragments leave LDS transposed (ds_read_b64_tr_b16): lane 16 g + i points at row
//     8 g + i / 4 (second read: 4 on) and 4 columns, and gets 4 rows of one column.  Column block nb takes columns
//     8 (i % 4) + 4 (nb % 2) + 32 (nb / 2) .. + 3, so that a lane ends up with two runs of 8 consecutive columns of a head
//     and stores them as they are.  The chunk swizzle keeps the two row pairs that a read pairs up on different banks.
//   * Two stages, two to three workgroups a compute unit: deeper rings were slower (3 stages 400 us against 385).
struct GatherArgs {
    const _Float16 *x, *w;                                 // rows or pool; [B, H, Lp]
    const float4 *part;                                    // [B, blocks, H]
    _Float16 *Y;                                           // [B, H, d]
    float4 *sums;                                          // [B, H]: (reference, denominator, -, -) of the sequence's checkpoint rows
    int B, L, Lp, H, d, blocks, rows_log2;                 // 2^rows_log2 rows a block of part
    int nt;
    const int32_t *list, *n_rows;
    int list_pitch, blk_log2;
};
constexpr int kGW = 4, kXS = 2, kWS = 3, kFT = 32;         // kFT: blocks of part whose factors are in LDS at a time

template <int HB>
constexpr int gather_lds_bytes()
{
    constexpr int H16 = 16 * HB, NSUB = 64 * kGW / H16;
    return kGW * kXS * 4096 + kWS * HB * 2048 + NSUB * H16 * 12 + H16 * 12 + kFT * H16 * 2;
}

// Swizzle of the 16-byte chunks of row q of a stage.
__device__ __forceinline__ int gather_swz(int q) { return 4 * (((q >> 1) ^ (q >> 3)) & 1); }

template <int HB, int DT, bool PAGED, bool NT>
__global__ __launch_bounds__(64 * kGW + 64) void absorbed_gather_kernel(GatherArgs p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int XB = 32 * 128, WB = HB * 2048, H16 = HB * 16, kThreads = 64 * kGW, NSUB = kThreads / H16;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int H = p.H, d = p.d;
    const int cols = (d + 64 * kGW - 1) / (64 * kGW);
    // The workgroups of a sequence share its w in one XCD's L2; sequences of different lengths go to all XCDs alike, so that
    // none gets the longer ones.
    const int item = PAGED ? (int)blockIdx.x : gemm::xcd_regroup(blockIdx.x, cols * p.B);
    const int64_t b = item / cols;
    const int cb = item % cols;
    const int n = PAGED ? __builtin_amdgcn_readfirstlane(p.n_rows[b]) : p.L;
    const int tiles = (n + 63) / 64, steps = (n + 31) / 32;
    const int nblk = (n + (1 << p.rows_log2) - 1) >> p.rows_log2;
    unsigned char *wring = smem + kGW * kXS * XB;
    float *lm = reinterpret_cast<float *>(wring + kWS * WB);               // [NSUB][H16] (l, mu)
    float *mxs = lm + 2 * NSUB * H16;                                      // [NSUB][H16]
    float *tab = mxs + NSUB * H16;                                         // [H16] (mu, 1 / (2^14 l))
    float *ref = tab + 2 * H16;                                            // [H16]
    _Float16 *ftab = reinterpret_cast<_Float16 *>(ref + H16);              // [kFT][H16]
    const int g_row = lane >> 3;
    const float4 *part = p.part + b * p.blocks * H;
    // Tile g begins a stretch of kFT blocks whose factors have to be worked out (the first stretch is part of the prologue).
    auto refill = [&](int g) {
        const int k = (64 * g) >> p.rows_log2;
        return g > 0 && k % kFT == 0 && (k << p.rows_log2) == 64 * g;
    };

    if (wave == kGW) {                                     // ---- w
        if (n <= 0) return;
        const _Float16 *src[2 * HB];
#pragma unroll
        for (int i = 0; i < 2 * HB; ++i) {
            const int q = 8 * i + g_row, h = q < H ? q : H - 1;
            src[i] = p.w + (b * H + h) * p.Lp + 8 * ((lane & 7) ^ ((q >> 1) & 7));
        }
        int slot = 0;
        auto issue = [&] {
#pragma unroll
            for (int i = 0; i < 2 * HB; ++i) {
                load_lds<false>(src[i], wring + slot * WB + i * 1024);
                src[i] += 64;
            }
            slot = slot + 1 == kWS ? 0 : slot + 1;
        };
        for (int g = 0; g < kWS && g < tiles; ++g) issue();
        asm volatile("s_barrier\n\ts_barrier" ::: "memory");               // the two of the prologue
        for (int g = 0; g < tiles; ++g) {
            if (refill(g)) asm volatile("s_barrier\n\ts_barrier" ::: "memory");
            if (g + kWS - 2 < tiles) wait_vm<2 * HB * (kWS - 2)>();
            else wait_vm<0>();
            asm volatile("s_barrier" ::: "memory");
            if (g > 0 && g - 1 + kWS < tiles) issue();
        }
        return;
    }

    // ---- rows
    int c = (cb * kGW + wave) * 64;
    const bool live = c < d;                               // a wavefront past the last columns works on those (it shares the
    if (!live) c = d - 64;                                 // barriers) and stores nothing
    const int fr = lane & 15, fc = lane >> 4;
    if (n <= 0) {                                          // no checkpoint rows
        half8_t zero;
#pragma unroll
        for (int e = 0; e < 8; ++e) zero[e] = (_Float16)0.f;
        if (live)
            for (int h = g_row; h < H; h += 8) *reinterpret_cast<half8_t *>(p.Y + (b * H + h) * d + c + 8 * (lane & 7)) = zero;
        if (cb == 0 && tid < H) p.sums[b * H + tid] = make_float4(kNegBig, 0.f, 0.f, 0.f);
        return;
    }
    unsigned char *my = smem + wave * kXS * XB;
    int lc[4], voff[4];                                    // load i of a step: rows 8 i + g_row
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        lc[i] = 8 * ((lane & 7) ^ gather_swz(8 * i + g_row));
        voff[i] = ((8 * (PAGED ? i & 1 : i) + g_row) * d + lc[i]) * 2;
    }
    int ask = 0, ask_slot = 0;
    // PAGED: the pool blocks of 64 consecutive blocks of the sequence, one a lane (a scalar load a step would be waited for
    // with the LDS reads: 645 us against 400)
    int32_t ids = 0;
    int ids_at = -64;
    auto block_id = [&](int k) {
        if (k >= ids_at + 64 || ids_at < 0) {
            ids_at = k & ~63;
            const int last = (n - 1) >> p.blk_log2;
            ids = p.list[b * p.list_pitch + (ids_at + lane < last ? ids_at + lane : last)];
            asm volatile("" : "+v"(ids));                  // waited for here, and not (with every row in flight) at each use
        }
        return (int64_t)__builtin_amdgcn_readlane(ids, k & 63);
    };
    auto issue = [&] {
        const int r0 = 32 * ask;
        __amdgpu_buffer_rsrc_t rs[2];
        const _Float16 *base = p.x + b * p.L * (int64_t)d + (int64_t)r0 * d + c;
        int first[2] = {0, 0};                             // row of the step that each half's buffer begins with
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            if constexpr (PAGED) {
                const bool in = r0 + 16 * hf < n;
                first[hf] = in ? 16 * hf : 0;
                base = p.x + ((block_id((r0 + first[hf]) >> p.blk_log2) << p.blk_log2) + ((r0 + first[hf]) & ((1 << p.blk_log2) - 1))) * d + c;
            }
            if (hf == 0 || PAGED) rs[hf] = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16 *>(base), 0, 0x7fffffff, 0x00020000);
            else rs[hf] = rs[0];
        }
        if (ask == steps - 1) {                            // rows past the end: the last one, under a weight of 0
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int f = PAGED ? first[i >> 1] : 0;
                int q = 8 * i + g_row;
                if (r0 + q >= n) q = n - 1 - r0;
                voff[i] = ((q - f < 0 ? 0 : q - f) * d + lc[i]) * 2;
            }
        }
        unsigned char *dst = my + ask_slot * XB;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs[i >> 1], (lds_ptr_t)(dst + i * 1024), 16, voff[i], 0, 0, NT ? kNt : 0);
        ++ask;
        ask_slot = ask_slot + 1 == kXS ? 0 : ask_slot + 1;
    };
    for (int s = 0; s < kXS && s < steps; ++s) issue();

    // ---- references of the blocks: thread -> head ph, every NSUB-th block from `sub` on
    const int ph = tid % H16, sub = tid / H16;
    const float4 *pp = part + (ph < H ? ph : H - 1);
    float E = kNegBig;
    constexpr int kAhead = 4;                              // blocks whose entries are on their way together (and kept, if that is all)
    float4 v[kAhead];
    auto entries = [&](int k0) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int k = k0 + u * NSUB;
            v[u] = pp[(int64_t)(k < nblk ? k : nblk - 1) * H];
        }
    };
    if (sub < NSUB) {
        for (int k0 = sub; k0 < nblk; k0 += kAhead * NSUB) {
            entries(k0);
#pragma unroll
            for (int u = 0; u < kAhead; ++u) E = fmaxf(E, v[u].x);         // (one past the end: the last one, again)
        }
        mxs[sub * H16 + ph] = E;
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (sub < NSUB) {
#pragma unroll
        for (int q = 0; q < NSUB; ++q) E = fmaxf(E, mxs[q * H16 + ph]);
        float l = 0.f, mu = 0.f;
        for (int k0 = sub; k0 < nblk; k0 += kAhead * NSUB) {
            if (nblk > kAhead * NSUB) entries(k0);
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int k = k0 + u * NSUB;
                if (k < nblk) {
                    const float f = __builtin_amdgcn_exp2f(v[u].x - E);
                    if (k < kFT) ftab[k * H16 + ph] = (_Float16)f;
                    l = __builtin_fmaf(v[u].y, f, l);
                    mu = __builtin_fmaf(v[u].z, (float)(_Float16)f, mu);   // of the weights as they are multiplied
                }
            }
        }
        lm[2 * (sub * H16 + ph)] = l;
        lm[2 * (sub * H16 + ph) + 1] = mu;
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (tid < H16) {
        float l = 0.f, mu = 0.f;
#pragma unroll
        for (int q = 0; q < NSUB; ++q) {
            l += lm[2 * (q * H16 + tid)];
            mu += lm[2 * (q * H16 + tid) + 1];
        }
        tab[2 * tid] = mu;
        tab[2 * tid + 1] = l > 0.f ? 1.f / (l * kWeightScale) : l;         // (a NaN stays one)
        ref[tid] = E;
        if (cb == 0 && tid < H) p.sums[b * H + tid] = make_float4(E, l, 0.f, 0.f);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                     // read behind the tiles' barriers

    int aoff[2], tro[4];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) aoff[ks] = fr * 128 + (((4 * ks + fc) ^ ((fr >> 1) & 7)) << 4);
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
        const int row = 8 * fc + (fr >> 2);
        tro[nb] = row * 128 + ((((fr & 3) + 4 * (nb >> 1)) ^ gather_swz(row)) << 4) + 8 * (nb & 1);
    }
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)my;
    float4_t acc[HB][4];
#pragma unroll
    for (int i = 0; i < HB; ++i)
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) acc[i][nb] = float4_t{0.f, 0.f, 0.f, 0.f};
    half2_t f2[HB];
    int slot = 0, ws = 0, kcur = -1;
    for (int g = 0; g < tiles; ++g) {
        if (refill(g)) {
            asm volatile("s_barrier" ::: "memory");                        // the factors of the stretch before are done with
            const int k0 = (64 * g) >> p.rows_log2;
            for (int idx = tid; idx < kFT * H16; idx += kThreads) {
                const int k = k0 + idx / H16, h = idx % H16;
                if (k < nblk) ftab[idx] = (_Float16)__builtin_amdgcn_exp2f(part[(int64_t)k * H + (h < H ? h : H - 1)].x - ref[h]);
            }
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        }
        asm volatile("s_barrier" ::: "memory");                            // tile g of w is there
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int s = 2 * g + ks;
            if (s < steps) {                                               // uniform
                if (s + kXS - 1 < steps) wait_vm<4 * (kXS - 1)>();
                else wait_vm<0>();
                __builtin_amdgcn_sched_barrier(0);
                const int k = (32 * s) >> p.rows_log2;
                if (k != kcur) {
                    kcur = k;
#pragma unroll
                    for (int i = 0; i < HB; ++i) {
                        const _Float16 f = ftab[(k % kFT) * H16 + 16 * i + fr];
                        f2[i] = half2_t{f, f};
                    }
                }
                half8_t xf[4], wf[HB];
#pragma unroll
                for (int i = 0; i < HB; ++i) wf[i] = *reinterpret_cast<const half8_t *>(wring + ws * WB + i * 2048 + aoff[ks]);
                {
                    // in one block with their wait: the compiler would put a wait for every load in flight before a
                    // transposing read, whose address it does not follow
                    short4_t lo[4], hi[4];
                    const unsigned base = lds0 + slot * XB;
                    asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:512\n\t"
                                 "ds_read_b64_tr_b16 %2, %9\n\tds_read_b64_tr_b16 %3, %9 offset:512\n\t"
                                 "ds_read_b64_tr_b16 %4, %10\n\tds_read_b64_tr_b16 %5, %10 offset:512\n\t"
                                 "ds_read_b64_tr_b16 %6, %11\n\tds_read_b64_tr_b16 %7, %11 offset:512\n\t"
                                 "s_waitcnt lgkmcnt(0)"
                                 : "=&v"(lo[0]), "=&v"(hi[0]), "=&v"(lo[1]), "=&v"(hi[1]), "=&v"(lo[2]), "=&v"(hi[2]), "=&v"(lo[3]), "=&v"(hi[3])
                                 : "v"(base + tro[0]), "v"(base + tro[1]), "v"(base + tro[2]), "v"(base + tro[3])
                                 : "memory");
#pragma unroll
                    for (int nb = 0; nb < 4; ++nb)
                        xf[nb] = skinny::to_half8<DT>(__builtin_bit_cast(half8_t, __builtin_shufflevector(lo[nb], hi[nb], 0, 1, 2, 3, 4, 5, 6, 7)));
                }
                __builtin_amdgcn_sched_barrier(0);
                if (ask < steps) issue();                                  // into the slot whose reads have come back
#pragma unroll
                for (int i = 0; i < HB; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const half2_t v = half2_t{wf[i][2 * e], wf[i][2 * e + 1]} * f2[i];
                        wf[i][2 * e] = v[0];
                        wf[i][2 * e + 1] = v[1];
                    }
#pragma unroll
                for (int i = 0; i < HB; ++i)
#pragma unroll
                    for (int nb = 0; nb < 4; ++nb) acc[i][nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xf[nb], wf[i], acc[i][nb], 0, 0, 0);
                slot = slot + 1 == kXS ? 0 : slot + 1;
            }
        }
        ws = ws + 1 == kWS ? 0 : ws + 1;
    }
    if (!live) return;
    // acc[i][nb][r]: head 16 i + fr, column 8 fc + 4 (nb % 2) + 32 (nb / 2) + r
#pragma unroll
    for (int i = 0; i < HB; ++i) {
        const int h = 16 * i + fr;
        const float mu = tab[2 * h], inv = tab[2 * h + 1];
        _Float16 *dst = p.Y + (b * H + h) * d + c + 8 * fc;
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            half8_t o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (_Float16)((acc[i][2 * hf + (e >> 2)][e & 3] - mu) * inv);
            if (h < H) store_as<NT>(o, reinterpret_cast<half8_t *>(dst + 32 * hf));
        }
    }
#endif
}

// ---------------------------------------------------------------------------------------------------------
template <int HB, int RW, int NW, int XS, int US, int DT, bool PAGED, bool NT>
hipError_t launch_ring(const ScoreArgs &p, int64_t items, int cus, hipStream_t s)
{
    auto kern = absorbed_scores_ring_kernel<HB, RW, NW, XS, US, DT, PAGED, NT>;
    constexpr int lds = ring_lds_bytes<HB, RW, NW, XS, US>();
    static_assert(lds <= 160 * 1024, "the workgroup must fit the LDS of a compute unit");
    static LdsOnce lds_once;
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds, lds_once);
    if (e != hipSuccess) return e;
    const int per_cu = NW * RW >= 16 ? 1 : 160 * 1024 / lds < 3 ? 160 * 1024 / lds : 3;
    const int64_t grid = items < (int64_t)cus * per_cu ? items : (int64_t)cus * per_cu;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * NW + 64), lds, s, p);
    return hipGetLastError();
}

template <int RB, int DT, bool PAGED>
hipError_t launch_slab(const ScoreArgs &p, int64_t items, hipStream_t s)
{
    auto kern = absorbed_scores_slab_kernel<RB, DT, PAGED>;
    constexpr int lds = skinny::lds_bytes<RB>() + skinny::kMomentBytes;
    static LdsOnce lds_once;
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds, lds_once);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)items), dim3(256), lds, s, p);
    return hipGetLastError();
}

template <int HB, int DT, bool PAGED>
hipError_t launch_ring_rows(const ScoreArgs &p, int rows_log2, int64_t items, int cus, hipStream_t s)
{
    if (rows_log2 == 8) return p.nt ? launch_ring<HB, 2, 8, 3, 3, DT, PAGED, true>(p, items, cus, s) : launch_ring<HB, 2, 8, 3, 3, DT, PAGED, false>(p, items, cus, s);
    return p.nt ? launch_ring<HB, 1, 4, 4, 3, DT, PAGED, true>(p, items, cus, s) : launch_ring<HB, 1, 4, 4, 3, DT, PAGED, false>(p, items, cus, s);
}

template <int DT, bool PAGED>
hipError_t launch_scores_form(const ScoreArgs &p, int rows_log2, int64_t items, int cus, hipStream_t s)
{
    if (rows_log2 == 5) {
        switch ((p.H + 31) / 32) {
        case 1: return launch_slab<1, DT, PAGED>(p, items, s);
        case 2: return launch_slab<2, DT, PAGED>(p, items, s);
        case 3: return launch_slab<3, DT, PAGED>(p, items, s);
        default: return launch_slab<4, DT, PAGED>(p, items, s);
        }
    }
    switch ((p.H + 15) / 16) {
    case 1: return launch_ring_rows<1, DT, PAGED>(p, rows_log2, items, cus, s);
    case 2: return launch_ring_rows<2, DT, PAGED>(p, rows_log2, items, cus, s);
    case 3: return launch_ring_rows<3, DT, PAGED>(p, rows_log2, items, cus, s);
    case 4: return launch_ring_rows<4, DT, PAGED>(p, rows_log2, items, cus, s);
    case 5: return launch_ring_rows<5, DT, PAGED>(p, rows_log2, items, cus, s);
    case 6: return launch_ring_rows<6, DT, PAGED>(p, rows_log2, items, cus, s);
    case 7: return launch_ring_rows<7, DT, PAGED>(p, rows_log2, items, cus, s);
    default: return launch_ring_rows<8, DT, PAGED>(p, rows_log2, items, cus, s);
    }
}

template <int HB, int DT, bool PAGED, bool NT>
hipError_t launch_gather_nt(const GatherArgs &p, hipStream_t s)
{
    auto kern = absorbed_gather_kernel<HB, DT, PAGED, NT>;
    constexpr int lds = gather_lds_bytes<HB>();
    static LdsOnce lds_once;
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds, lds_once);
    if (e != hipSuccess) return e;
    const int64_t grid = (int64_t)((p.d + 64 * kGW - 1) / (64 * kGW)) * p.B;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * kGW + 64), lds, s, p);
    return hipGetLastError();
}

template <int HB, int DT, bool PAGED>
hipError_t launch_gather_as(const GatherArgs &p, hipStream_t s)
{
    return p.nt ? launch_gather_nt<HB, DT, PAGED, true>(p, s) : launch_gather_nt<HB, DT, PAGED, false>(p, s);
}

template <int DT, bool PAGED>
hipError_t launch_gather(const GatherArgs &p, hipStream_t s)
{
    switch ((p.H + 15) / 16) {
    case 1: return launch_gather_as<1, DT, PAGED>(p, s);
    case 2: return launch_gather_as<2, DT, PAGED>(p, s);
    case 3: return launch_gather_as<3, DT, PAGED>(p, s);
    case 4: return launch_gather_as<4, DT, PAGED>(p, s);
    case 5: return launch_gather_as<5, DT, PAGED>(p, s);
    case 6: return launch_gather_as<6, DT, PAGED>(p, s);
    case 7: return launch_gather_as<7, DT, PAGED>(p, s);
    default: return launch_gather_as<8, DT, PAGED>(p, s);
    }
}

}  // namespace

// Rows that do not stay in the last-level cache (256 MB) until the second pass: loads and stores are non-temporal then.
bool absorbed_streams(int64_t rows, int d) { return rows * d * 2 > (192LL << 20); }

// Blocks of the fewest rows that the rule below takes for a layer.
int absorbed_finest_rows_log2(int d) { return d <= 2048 ? 6 : 5; }

// Rows of a block of the score pass, as a power of two: 2^5 the slab form, 2^6 and 2^8 the ring form.  Where the lines lie
// (whole step, no cached tokens, fp16, us with blocks of 32 / 64 / 256 rows):
//   a workgroup of the ring form walks the whole reduction axis (d / 64 stages, about 0.3 us each), of the slab form a
//   quarter of it: while few workgroups have work that chain is the time, and from some 8000 rows on the traffic is: d = 9216,
//   4000 rows 188 / 195 / 226, 5632 146 / 161 / 199, 9600 224 / 196 / 248; d = 4096, 5632 51 / 57 / 71, 9600 68 / 65 / 79.  Narrow
//   layers have short chains: d = 768, 64 rows 23.3 / 22.6 / 24.1, 4000 rows 64 / 58 / 61.
//   256 rows a workgroup read U a quarter as often as 64 and need 65536 rows for every compute unit to have some: d =
//   9216, 32768 rows 433 / 381 / 392, 65536 729 / 612 / 577; with up to 32 heads U is small: d = 4096, 65536 rows 249 / 239 / 246.
int absorbed_rows_log2(int64_t rows, int d, int H)
{
    if (rows >= 65536 && H > 32) return 8;
    return rows >= 8192 ? 6 : absorbed_finest_rows_log2(d);
}

hipError_t launch_absorbed_stream(const AbsorbedArgs &a, const AbsorbedRows *pr, int64_t rows, hipStream_t s)
{
    const int rows_log2 = absorbed_rows_log2(rows, a.d, a.H);
    const int Lp = absorbed_row_pitch(a.L_act);
    const int blocks = (a.L_act + (1 << rows_log2) - 1) >> rows_log2;
    const int64_t items = (int64_t)blocks * a.B;
    if (items > 0x7fffffffLL) return hipErrorInvalidValue;
    int dev = 0, cus = 0;
    hipError_t e = current_device_cus(&dev, &cus);
    if (e != hipSuccess) return e;
    ScoreArgs p;
    p.act = static_cast<const _Float16 *>(a.act); p.U = static_cast<const _Float16 *>(a.U); p.c12 = a.c12; p.factor = a.bvec + 2 * a.d;
    p.w = static_cast<_Float16 *>(a.w); p.part = a.part;
    p.B = a.B; p.L = a.L_act; p.Lp = Lp; p.H = a.H; p.d = a.d; p.blocks = blocks;
    p.eps = a.eps; p.sl = a.scale * 1.4426950408889634f; p.nt = absorbed_streams(rows, a.d);
    p.list = pr ? pr->list : nullptr; p.n_rows = pr ? pr->n_rows : nullptr; p.cu_items = pr ? pr->cu_items : nullptr;
    p.list_pitch = pr ? pr->list_pitch : 0; p.blk_log2 = pr ? pr->blk_log2 : 0;
    // a pool holds no more items than its rows allow, whatever the longest request could have
    int64_t ring_items = items;
    if (pr && ring_items > a.B + (rows >> rows_log2)) ring_items = a.B + (rows >> rows_log2);
    if (pr) e = a.dt == 1 ? launch_scores_form<1, true>(p, rows_log2, rows_log2 == 5 ? items : ring_items, cus, s)
                          : launch_scores_form<0, true>(p, rows_log2, rows_log2 == 5 ? items : ring_items, cus, s);
    else e = a.dt == 1 ? launch_scores_form<1, false>(p, rows_log2, items, cus, s) : launch_scores_form<0, false>(p, rows_log2, items, cus, s);
    if (e != hipSuccess) return e;
    GatherArgs g;
    g.x = p.act; g.w = p.w; g.part = a.part; g.Y = static_cast<_Float16 *>(a.Y); g.sums = a.sums;
    g.B = a.B; g.L = a.L_act; g.Lp = Lp; g.H = a.H; g.d = a.d; g.blocks = blocks; g.rows_log2 = rows_log2; g.nt = p.nt;
    g.list = p.list; g.n_rows = p.n_rows; g.list_pitch = p.list_pitch; g.blk_log2 = p.blk_log2;
    if (pr) return a.dt == 1 ? launch_gather<1, true>(g, s) : launch_gather<0, true>(g, s);
    return a.dt == 1 ? launch_gather<1, false>(g, s) : launch_gather<0, false>(g, s);
}

}  // namespace hk
