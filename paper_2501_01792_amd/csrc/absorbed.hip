// Decode attention over the activation checkpoints WITHOUT regenerating their K/V rows.
//
// The hybrid step (Sec. 4.2.2) turns every checkpoint row x_t into a K row and a V row (Eq. 7) and then runs
// the single-query attention (Eq. 4) over them.  For one query per head the two linear maps can be moved to
// the other side of the sums, which gives the same result (up to rounding) for ~head_dim times fewer FLOP:
// with the folded LayerNorm  K_t = rstd_t (x_t W'_K^T) + nmr_t c_K + b'_K  (likewise V),
//
//   score_t(h) = scale [ rstd_t (x_t . u_h - mean_t sum_k u_h[k]) + q_h . b'_K,h ],     u_h = q_h W'_K,h   [d]
//   o_h        = W'_V,h y_h + b'_V,h,            y_h = sum_t w_t (x_t - mean_t),         w_t = p_t rstd_t / l
//
// so the checkpoints are streamed twice (scores, weighted row sum) and the weights once; nothing of size
// [tokens, 2 d] is ever written.  u_h, w_t and y_h are kept in fp16; the two mean terms are formed from the
// ROUNDED values (sum_k of the stored u_h, sum_t of the stored w_t) and subtracted in fp32 before anything is
// rounded again, so that a row mean that is large against the row's spread cancels exactly as it does in
// the LayerNorm, instead of leaving the rounding error of u_h or w_t multiplied by it.  The cached K/V segment goes through the ordinary decode kernel and the two
// segments are joined by their softmax maxima and denominators.  Tensors stored as bfloat16 (q, the checkpoints, the
// prepared weights, the cached segment's output, out) are converted to fp16 where they are loaded, so the
// arithmetic, and with it the cancellation argument above, is the same for both storage types; u, w, y are fp16
// either way.  This is a comparison variant beyond the
// paper's design (which regenerates K/V with a GEMM); the paper's Eq. 3/4/7 define the result.
//
// Kernels (B sequences, H heads, L_act checkpoint rows per sequence):
//   carry   U[h,b,:]  = q[b,h,:] W'_K,h          rows of W' reduced       column_product (MFMA)
//   scores  w[b,h,t], from x[b,t,:] . U[h,b,:]   rows of x streamed       absorbed_stream.hip (MFMA); also the LayerNorm
//                                                                         statistics of the rows and their softmax
//   gather  Y[b,h,:]  = sum_t w[b,h,t] (x[b,t,:] - mean_t)   rows of x reduced   absorbed_stream.hip (MFMA)
//   project o[b,h,:]  = W'_V,h Y[b,h,:] + b'_V   rows of W' streamed      skinny::slab_product (MFMA), joins the cached part;
//                                                                         layers of 5120 features or more: block_product
//                                                                         with the reduction axis cut over workgroups, then
//                                                                         a join kernel
#include "hk_internal.h"
#include "kv_gemm_common.h"
#include "skinny_mma.h"

namespace hk {
namespace {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4_t *lds_short4_ptr;

// ---------------------------------------------------------------------------------------------------------
// column_product: Out[z][m][c] = sum_r A[z][m][r] * S[z][r][c]   (m < a_rows <= 32 RB, r < R, c < n_cols)
//
// The streamed operand S is row-major and the reduction runs over its ROWS, so it reaches the matrix cores
// transposed.  Every wavefront owns a block of 64 columns and walks all R rows in steps of 16: whole 128-byte
// pieces of 16 rows go from HBM to registers (kDepth - 1 steps in flight) and row-wise into the wavefront's
// private LDS block, from which every lane takes the 8 values of its column with two transposing reads
// (ds_read_b64_tr_b16; rows 192 bytes apart, so that the four rows one such read touches fall on disjoint banks).  The small operand A (few rows, reduction axis contiguous, zero
// beyond R up to the next multiple of 64) is the same for the four wavefronts of a workgroup: it is fetched
// once per 64 reduction elements with whole-line loads, two tiles ahead, and shared through a double-buffered
// LDS tile (one barrier per 64 reduction elements).  The result leaves through the private LDS block so that it is
// stored as whole 128-byte rows.  A last workgroup of every z takes the two dot products of the rows of A with
// per-row-of-S constants (cvec, bvec).
struct ColArgs {
    const _Float16 *S; int64_t s_batch, ld_s; int R, n_cols;
    const _Float16 *A; int64_t a_batch, ld_a; int a_rows;
    _Float16 *Out; int64_t o_batch, ld_out;
    const float *cvec, *bvec; float2 *c12; int c12_stride;     // c12[m c12_stride + z] = (A[z][m] . cvec[z R ..], A[z][m] . bvec[z R ..])
    int s_dt, a_dt;                                        // storage types of S and of A (Out is fp16)
    int nt;                                                // Out is stored non-temporally
};

constexpr int kColBlock = 64;                              // columns of one wavefront
constexpr int kColPitch = 2 * kColBlock + 64;               // bytes between rows of a wavefront's private LDS block
constexpr int kColStage = 32 * kColPitch;                  // bytes of private LDS per wavefront
constexpr int kTileBytes = 32 * 128;                       // 32 operand rows x 64 reduction elements

template <int RB>
constexpr int col_lds_bytes() { return 4 * kColStage + 2 * RB * kTileBytes; }

template <int RB, int SDT, int ADT, bool NT>
__global__ __launch_bounds__(256) void column_product_kernel(ColArgs p)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int NB = kColBlock / 32;
    constexpr int XS = kColPitch;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (blockIdx.x == gridDim.x - 1) {                     // 4 threads a row of A
        const int64_t zc = blockIdx.y;
        for (int m = tid >> 2; m < p.a_rows; m += 64) {
            float c1 = 0.f, c2 = 0.f;
            for (int r = tid & 3; r < p.R; r += 4) {
                const float a = skinny::stored_to_float<ADT>(p.A + zc * p.a_batch + (int64_t)m * p.ld_a + r);
                c1 = __builtin_fmaf(a, p.cvec[zc * p.R + r], c1);
                c2 = __builtin_fmaf(a, p.bvec[zc * p.R + r], c2);
            }
            c1 += __shfl_xor(c1, 1, 64);
            c1 += __shfl_xor(c1, 2, 64);
            c2 += __shfl_xor(c2, 1, 64);
            c2 += __shfl_xor(c2, 2, 64);
            if ((tid & 3) == 0) p.c12[(int64_t)m * p.c12_stride + zc] = make_float2(c1, c2);
        }
        return;
    }
    int c0 = (blockIdx.x * 4 + wave) * kColBlock;
    const bool live = c0 < p.n_cols;                       // a wavefront past the last column block works on the
    if (!live) c0 = p.n_cols - kColBlock;                  // last one (it shares the barriers) and stores nothing
    const int64_t z = blockIdx.y;
    const _Float16 *S = p.S + z * p.s_batch + c0;
    const _Float16 *A = p.A + z * p.a_batch;
    const int R = p.R;
    const int steps = (R + 15) / 16;
    const int tiles = (steps + 3) / 4;

    // one load instruction: 8 rows x 128 bytes, 8 lanes per row
    const int g_row = lane >> 3, g_chunk = lane & 7;
    const int ln = lane & 31, lh = lane >> 5;
    // the A tile: thread -> (row tid / 8 of every 32-row block, 16-byte chunk tid % 8)
    const int t_row = tid >> 3, t_chunk = tid & 7;
    const _Float16 *ap[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        int m = rb * 32 + t_row;
        if (m >= p.a_rows) m = p.a_rows - 1;               // clamp: rows past the end are computed, never stored
        ap[rb] = A + (int64_t)m * p.ld_a + 8 * t_chunk;
    }
    // tile layout: row-major 128-byte rows, chunk index XOR-ed with (row / 2) % 8 (conflict-free both ways)
    const int t_wr = t_row * 128 + ((t_chunk ^ ((t_row >> 1) & 7)) << 4);
    int t_rd[4];                                           // operand fragment of step s % 4: chunks 2 (s % 4) + lane / 32
#pragma unroll
    for (int q = 0; q < 4; ++q) t_rd[q] = ln * 128 + (((2 * q + lh) ^ ((ln >> 1) & 7)) << 4);
    unsigned char *my = smem + wave * kColStage;
    unsigned char *tile = smem + 4 * kColStage;
    // source address of this lane in the transposing reads of the private block: lane 16 g + t points at row
    // 8 (g / 2) + t / 4, columns 16 (g % 2) + 4 (t % 4) .. + 3 (of column block nb: + 32 nb; second read: 4 rows on)
    const int tr_off = (8 * (lane >> 5) + ((lane & 15) >> 2)) * XS + 2 * (16 * ((lane >> 4) & 1) + 4 * (lane & 3));

    float16_t acc[RB][NB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[rb][nb][r] = 0.f;

    constexpr int kDepth = 8;                              // streamed steps in registers; two tiles per pass of the loop
    half8_t sv[kDepth][2];
    half8_t av[2][RB];
    const int last = steps - 1, last_tile = tiles - 1;
    auto clamp = [&](int sc) { return sc < last ? sc : last; };
    auto load_s = [&](int slot, int sc) {
        const int r0 = 16 * sc;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            int rr = 8 * j + g_row;
            if (r0 + rr >= R) rr = R - 1 - r0;             // rows past the end meet zeros of A; r0 < R for every step asked for
            sv[slot][j] = *reinterpret_cast<const half8_t *>(S + (int64_t)(r0 + rr) * p.ld_s + 8 * g_chunk);
        }
    };
    auto load_a = [&](int slot, int g) {
        if (g > last_tile) g = last_tile;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) av[slot][rb] = *reinterpret_cast<const half8_t *>(ap[rb] + 64 * g);
    };
    auto put_a = [&](int slot, int buf) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
            *reinterpret_cast<half8_t *>(tile + (buf * RB + rb) * kTileBytes + t_wr) = skinny::to_half8<ADT>(av[slot][rb]);
    };
    // Every load of the loop is unconditional (steps and tiles past the end re-read the last one), so that
    // the number of loads in flight at each wait is a compile-time fact.
    load_a(0, 0);
    load_a(1, 1);
#pragma unroll
    for (int u = 0; u < kDepth - 1; ++u) load_s(u, clamp(u));
    put_a(0, 0);
    __syncthreads();
    for (int g0 = 0; g0 < tiles; g0 += 2) {
#pragma unroll
        for (int gg = 0; gg < 2; ++gg) {
            const int g = g0 + gg;
            if (g < tiles) {                               // uniform over the workgroup
                put_a((gg + 1) & 1, (gg + 1) & 1);         // tile g + 1 (fetched one pass ago) for the next pass
                load_a(gg, g + 2);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int u = 4 * gg + q, sc = 4 * g + q;
                    load_s((u + kDepth - 1) % kDepth, clamp(sc + kDepth - 1));
                    if (sc < steps) {
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            *reinterpret_cast<half8_t *>(my + (8 * j + g_row) * XS + 16 * g_chunk) = skinny::to_half8<SDT>(sv[u][j]);
                        // bf[nb][i] = element (row 8 lh + i, column 32 nb + ln) of the block, by two transposing reads:
                        // ds_read_b64_tr_b16 hands lane t of a 16-lane group the four rows that the group's lanes
                        // 4 j + t / 4 .. point at, at column 4 (source lane % 4) + ... = t of the group's 16 columns
                        half8_t bf[NB];
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) {
                            const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(my + tr_off + 64 * nb));
                            const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(my + tr_off + 64 * nb + 4 * XS));
                            bf[nb] = __builtin_bit_cast(half8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                        }
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb) {
                            const half8_t af = *reinterpret_cast<const half8_t *>(tile + (gg * RB + rb) * kTileBytes + t_rd[q]);
#pragma unroll
                            for (int nb = 0; nb < NB; ++nb)
                                acc[rb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af, bf[nb], acc[rb][nb], 0, 0, 0);
                        }
                    }
                }
                __syncthreads();                           // tile g + 1 is complete; tile g is free for g + 2
            }
        }
    }
    if (!live) return;                                     // no barrier below

    // ---- fp16, through the private LDS block, out as whole rows.
    // acc[rb][nb][r]: row 32 rb + 8 (r/4) + 4 (lane/32) + r%4, column 32 nb + lane%32.
    _Float16 *Out = p.Out + z * p.o_batch + c0;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                *reinterpret_cast<_Float16 *>(my + (8 * (r >> 2) + 4 * lh + (r & 3)) * XS + 2 * (32 * nb + ln)) =
                    (_Float16)acc[rb][nb][r];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int m = 32 * rb + 8 * j + g_row;
            const half8_t o = *reinterpret_cast<const half8_t *>(my + (8 * j + g_row) * XS + 16 * g_chunk);
            half8_t *dst = reinterpret_cast<half8_t *>(Out + (int64_t)m * p.ld_out + 8 * g_chunk);
            if (m < p.a_rows) {
                if constexpr (NT) __builtin_nontemporal_store(o, dst);
                else *dst = o;
            }
        }
    }
}

template <int RB, int SDT, int ADT, bool NT>
hipError_t launch_col_as(const ColArgs &p, int batches, hipStream_t s)
{
    auto kern = column_product_kernel<RB, SDT, ADT, NT>;
    constexpr int lds = col_lds_bytes<RB>();
    static LdsOnce lds_once;
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds, lds_once);
    if (e != hipSuccess) return e;
    const int blocks_x = (p.n_cols / kColBlock + 3) / 4 + 1;      // and the one of the dot products
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks_x, (unsigned)batches), dim3(256), lds, s, p);
    return hipGetLastError();
}

template <int RB>
hipError_t launch_col(const ColArgs &p, int batches, hipStream_t s)
{
    if (p.s_dt == 0 && p.a_dt == 0) return p.nt ? launch_col_as<RB, 0, 0, true>(p, batches, s) : launch_col_as<RB, 0, 0, false>(p, batches, s);
    if (p.s_dt == 1 && p.a_dt == 1) return p.nt ? launch_col_as<RB, 1, 1, true>(p, batches, s) : launch_col_as<RB, 1, 1, false>(p, batches, s);
    return hipErrorInvalidValue;
}

// A must be readable (and zero beyond R) up to the next multiple of 64 reduction elements.
hipError_t launch_column_product(const ColArgs &p, int batches, hipStream_t s)
{
    if (p.a_rows <= 0 || p.a_rows > 128 || p.R <= 0 || p.n_cols % kColBlock != 0 || batches <= 0 || batches > 65535)
        return hipErrorInvalidValue;
    switch ((p.a_rows + 31) / 32) {
    case 1: return launch_col<1>(p, batches, s);
    case 2: return launch_col<2>(p, batches, s);
    case 3: return launch_col<3>(p, batches, s);
    default: return launch_col<4>(p, batches, s);
    }
}

// ---------------------------------------------------------------------------------------------------------
// project: o_a[b,h,e] = W'_V[h dh + e, :] . Y[b,h,:] + b'_V for a slab of 32 output features of one head, then
// the join with the cached segment's (maximum, denominator, output).  Workgroup ids are regrouped so that the
// slabs of one head, which share that head's Y rows, run on one XCD.
template <int RB, int DT>
__global__ __launch_bounds__(256) void absorbed_project_kernel(const _Float16 *__restrict__ Wv, const _Float16 *__restrict__ Y,
                                                               const float *__restrict__ bv,
                                                               const float4 *__restrict__ sums,
                                                               const _Float16 *__restrict__ out_c, const float2 *__restrict__ lse_c,
                                                               _Float16 *__restrict__ out, int Bc, int H, int head_dim, int d)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const int per_head = head_dim / skinny::kSlab;
    const int item = gemm::xcd_regroup(blockIdx.x, per_head * H);
    const int h = item / per_head;
    const int n0 = h * head_dim + (item % per_head) * skinny::kSlab;   // first V feature of the slab
    float (*red)[RB * 32][skinny::kSlab] = skinny::slab_product<RB, true, false, DT>(
        [=](int r) { return Wv + ((int64_t)n0 + r) * d; }, skinny::kSlab, Y + (int64_t)h * d, Bc, (int64_t)H * d, d, smem);
    for (int idx = tid; idx < Bc * skinny::kSlab; idx += 256) {
        const int b = idx / skinny::kSlab, c = idx % skinny::kSlab;
        const int n = n0 + c;
        const int64_t bh = (int64_t)b * H + h;
        const float4 sa = sums[bh];
        float o = (red[0][b][c] + red[1][b][c]) + (red[2][b][c] + red[3][b][c]);
        o = __builtin_fmaf(o, bv[d], bv[n]);               // bv[d]: the factor of the scaled weights
        // join of the two segments; a segment without tokens has denominator 0 and drops out, both empty: zero
        float m = sa.x, wc = 0.f, oc = 0.f;
        if (lse_c) {
            const float2 sc = lse_c[bh];
            m = fmaxf(sc.x, sa.x);
            wc = sc.y * __builtin_amdgcn_exp2f(sc.x - m);
            oc = skinny::stored_to_float<DT>(out_c + bh * head_dim + (n - h * head_dim));
        }
        const float wa = sa.y * __builtin_amdgcn_exp2f(sa.x - m);
        o = wc + wa > 0.f ? (wc * oc + wa * o) / (wc + wa) : 0.f;
        skinny::float_to_stored<DT>(out + bh * head_dim + (n - h * head_dim), o);
    }
}

// project, form for large layers: a workgroup per (head, part of the reduction axis) streams the head's rows of
// W'_V (head_dim <= 128 of them) once and shares the Y tile of the step through LDS (skinny::block_product),
// where the slab form above re-reads Y from L2 once per 32 features.  fp32 partial sums part[ks][b][n].
template <int RB, int DT>
__global__ __launch_bounds__(256) void absorbed_project_block_kernel(const _Float16 *__restrict__ Wv, const _Float16 *__restrict__ Y,
                                                                     float *__restrict__ part, int Bc, int H, int head_dim, int d,
                                                                     int steps_per_part)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = blockIdx.x, ks = blockIdx.y;
    const int steps = d / 64;
    const int k_begin = ks * steps_per_part;                               // < steps: the launcher leaves no part empty
    const int k_steps = steps - k_begin < steps_per_part ? steps - k_begin : steps_per_part;
    float16_t acc[RB];
    skinny::block_product<RB, true, DT>(Wv + (int64_t)h * head_dim * d, head_dim, d, Y + (int64_t)h * d, Bc, (int64_t)H * d,
                                        k_begin, k_steps, smem, acc);
    // acc[rb][r]: sequence 32 rb + 8 (r/4) + 4 (lane/32) + r%4, feature 32 wave + lane%32 of the head
    const int ln = lane & 31, lh = lane >> 5;
    const int c = 32 * wave + ln;
    if (c < head_dim) {
        float *dst = part + (int64_t)ks * Bc * d + h * head_dim + c;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = 32 * rb + 8 * (r >> 2) + 4 * lh + (r & 3);
                if (m < Bc) dst[(int64_t)m * d] = acc[rb][r];
            }
    }
}

// Sum of the parts, bias, and the join with the cached segment (as in absorbed_project_kernel); 4 features per thread.
template <int DT>
__global__ __launch_bounds__(256) void absorbed_join_kernel(const float *__restrict__ part, int parts, const float *__restrict__ bv,
                                                            const float4 *__restrict__ sums,
                                                            const _Float16 *__restrict__ out_c, const float2 *__restrict__ lse_c,
                                                            _Float16 *__restrict__ out, int Bc, int H, int head_dim, int d)
{
    typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
    const int per_row = d / 4;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)Bc * per_row) return;
    const int b = (int)(idx / per_row), n = (int)(idx % per_row) * 4;     // 4 | head_dim: one head
    const int64_t stride = (int64_t)Bc * d;
    const float *src = part + (int64_t)b * d + n;
    float4_t o = *reinterpret_cast<const float4_t *>(src);
    for (int ks = 1; ks < parts; ++ks) o += *reinterpret_cast<const float4_t *>(src + ks * stride);
    const int h = n / head_dim;
    const int64_t bh = (int64_t)b * H + h;
    const float4 sa = sums[bh];
    float m = sa.x, wc = 0.f;
    half4_t oc = {0, 0, 0, 0};                             // 4 stored elements, whatever their type
    if (lse_c) {
        const float2 sc = lse_c[bh];
        m = fmaxf(sc.x, sa.x);
        wc = sc.y * __builtin_amdgcn_exp2f(sc.x - m);
        oc = *reinterpret_cast<const half4_t *>(out_c + (int64_t)b * d + n);
    }
    const float wa = sa.y * __builtin_amdgcn_exp2f(sa.x - m);
    half4_t res;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float oa = __builtin_fmaf(o[j], bv[d], bv[n + j]);
        const float ocj = skinny::stored_to_float<DT>(reinterpret_cast<const _Float16 *>(&oc) + j);
        skinny::float_to_stored<DT>(reinterpret_cast<_Float16 *>(&res) + j, wc + wa > 0.f ? (wc * ocj + wa * oa) / (wc + wa) : 0.f);
    }
    *reinterpret_cast<half4_t *>(out + (int64_t)b * d + n) = res;
}

// Below, the slab form of the projection is used (measured: 15.4 against 12.5 + 4.4 us at d = 4096, B = 32;
// 37 against 21 + 5 us at d = 5120, B = 64; 97 against 49 + 5 us at d = 9216, B = 64).
constexpr int kProjectBlockMinD = 5120;

template <int RB, int DT>
hipError_t launch_project_as(const AbsorbedArgs &a, int b0, int Bc, hipStream_t s)
{
    auto kern = absorbed_project_kernel<RB, DT>;
    constexpr int lds = skinny::lds_bytes<RB>();
    static LdsOnce lds_once;
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds, lds_once);
    if (e != hipSuccess) return e;
    const int64_t bh0 = (int64_t)b0 * a.H;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.head_dim / skinny::kSlab * a.H)), dim3(256), lds, s,
                       static_cast<const _Float16 *>(a.Wp) + (int64_t)a.d * a.d, static_cast<const _Float16 *>(a.Y) + bh0 * a.d,
                       a.bvec + a.d, a.sums + bh0,
                       a.L_kv > 0 ? static_cast<const _Float16 *>(a.out_c) + bh0 * a.head_dim : nullptr,
                       a.L_kv > 0 ? a.lse_c + bh0 : nullptr,
                       static_cast<_Float16 *>(a.out) + bh0 * a.head_dim, Bc, a.H, a.head_dim, a.d);
    return hipGetLastError();
}

template <int RB>
hipError_t launch_project(const AbsorbedArgs &a, int b0, int Bc, hipStream_t s)
{
    return a.dt == 1 ? launch_project_as<RB, 1>(a, b0, Bc, s) : launch_project_as<RB, 0>(a, b0, Bc, s);
}

template <int RB, int DT>
hipError_t launch_project_block_as(const AbsorbedArgs &a, int b0, int Bc, hipStream_t s)
{
    int parts, steps_per_part;
    absorbed_project_parts(a.d, a.H, &parts, &steps_per_part);
    if ((size_t)parts * Bc * a.d > a.proj_part_floats) return hipErrorInvalidValue;
    auto kern = absorbed_project_block_kernel<RB, DT>;
    constexpr int lds = skinny::block_lds_bytes<RB>();
    static LdsOnce lds_once;
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds, lds_once);
    if (e != hipSuccess) return e;
    const int64_t bh0 = (int64_t)b0 * a.H;
    hipLaunchKernelGGL(kern, dim3((unsigned)a.H, (unsigned)parts), dim3(256), lds, s,
                       static_cast<const _Float16 *>(a.Wp) + (int64_t)a.d * a.d, static_cast<const _Float16 *>(a.Y) + bh0 * a.d,
                       a.proj_part, Bc, a.H, a.head_dim, a.d, steps_per_part);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int64_t threads = (int64_t)Bc * (a.d / 4);
    hipLaunchKernelGGL(absorbed_join_kernel<DT>, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s,
                       a.proj_part, parts, a.bvec + a.d, a.sums + bh0,
                       a.L_kv > 0 ? static_cast<const _Float16 *>(a.out_c) + bh0 * a.head_dim : nullptr,
                       a.L_kv > 0 ? a.lse_c + bh0 : nullptr,
                       static_cast<_Float16 *>(a.out) + bh0 * a.head_dim, Bc, a.H, a.head_dim, a.d);
    return hipGetLastError();
}

template <int RB>
hipError_t launch_project_block(const AbsorbedArgs &a, int b0, int Bc, hipStream_t s)
{
    return a.dt == 1 ? launch_project_block_as<RB, 1>(a, b0, Bc, s) : launch_project_block_as<RB, 0>(a, b0, Bc, s);
}

}  // namespace

int absorbed_row_pitch(int L_act) { return (L_act + 63) / 64 * 64; }

// Parts of the reduction axis of the output projection: at most one workgroup per compute unit over the H heads
// (measured on d = 7168 and 9216: more parts cost more in partial sums than they gain), at least 4 steps of 64
// per part, no empty part.
void absorbed_project_parts(int d, int H, int *parts, int *steps_per_part)
{
    const int steps = d / 64;
    int want = 256 / (H > 0 ? H : 1);
    if (want > steps / 4) want = steps / 4;
    if (want < 1) want = 1;
    if (want > 8) want = 8;
    *steps_per_part = (steps + want - 1) / want;
    *parts = (steps + *steps_per_part - 1) / *steps_per_part;
}

namespace {

// rows: checkpoint rows in all.  Where they outgrow the last-level cache U is stored non-temporally: left dirty in the cache
// it was written back under the score pass (85 MB, 2.4 GB of rows: 437 against 381 us for that pass, 50 for this one either way).
hipError_t launch_carry(const AbsorbedArgs &a, int64_t rows, hipStream_t s)
{
    const int64_t d = a.d;
    // the queries through the key weights, at most kAbsorbMaxBatch sequences per launch
    for (int b0 = 0; b0 < a.B; b0 += kAbsorbMaxBatch) {
        const int Bc = a.B - b0 < kAbsorbMaxBatch ? a.B - b0 : kAbsorbMaxBatch;
        ColArgs c;
        c.S = static_cast<const _Float16 *>(a.Wp); c.s_batch = (int64_t)a.head_dim * d; c.ld_s = d; c.R = a.head_dim; c.n_cols = a.d;
        c.A = static_cast<const _Float16 *>(a.q) + b0 * d; c.a_batch = a.head_dim; c.ld_a = d; c.a_rows = Bc;
        c.Out = static_cast<_Float16 *>(a.U) + b0 * d; c.o_batch = a.B * d; c.ld_out = d;
        c.cvec = a.cvec; c.bvec = a.bvec; c.c12 = a.c12 + (int64_t)b0 * a.H; c.c12_stride = a.H;
        c.s_dt = a.dt; c.a_dt = a.dt;                      // prepared weights and queries as stored
        c.nt = absorbed_streams(rows, a.d);
        const hipError_t e = launch_column_product(c, a.H, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// output projection and join
hipError_t launch_output(const AbsorbedArgs &a, hipStream_t s)
{
    hipError_t e;
    for (int b0 = 0; b0 < a.B; b0 += kAbsorbMaxBatch) {
        const int Bc = a.B - b0 < kAbsorbMaxBatch ? a.B - b0 : kAbsorbMaxBatch;
        const bool block_mode = a.proj_part != nullptr && a.d >= kProjectBlockMinD;
        switch ((Bc + 31) / 32) {
        case 1: e = block_mode ? launch_project_block<1>(a, b0, Bc, s) : launch_project<1>(a, b0, Bc, s); break;
        case 2: e = block_mode ? launch_project_block<2>(a, b0, Bc, s) : launch_project<2>(a, b0, Bc, s); break;
        case 3: e = block_mode ? launch_project_block<3>(a, b0, Bc, s) : launch_project<3>(a, b0, Bc, s); break;
        default: e = block_mode ? launch_project_block<4>(a, b0, Bc, s) : launch_project<4>(a, b0, Bc, s); break;
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------------------------------------
// Paged cache (Sec. 4.1, 4.2.1): the checkpoint rows of a request sit in blocks of the activation pool named by
// its row of the block table (entries < 0: checkpoint block ~entry).
//
// index: one wavefront per request walks its table row and leaves (a) the request's checkpoint blocks in logical
// order (list) and the request's number of checkpoint rows (only its final block can be partly filled); (b) the same view of its KV blocks: a table row that holds only them,
// in order, and the request's number of cached tokens, i.e. what the block-table attention kernel needs to walk
// the cached tokens alone.  Checkpoint blocks outside the pool prefix in use are left out.
__global__ __launch_bounds__(256) void paged_index_kernel(const int32_t *__restrict__ table, int max_blocks,
                                                          const int32_t *__restrict__ seq_len, int blk_log2, int n_act_used, int B,
                                                          int32_t *__restrict__ list, int32_t *__restrict__ n_rows,
                                                          int32_t *__restrict__ kv_table, int32_t *__restrict__ kv_len)
{
    const int lane = threadIdx.x & 63;
    const int b = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (b >= B) return;                                    // whole wavefront leaves together; no barrier in this kernel
    const int bt = 1 << blk_log2;
    const int len = seq_len[b];
    int nb = len > 0 ? (len + bt - 1) >> blk_log2 : 0;
    if (nb > max_blocks) nb = max_blocks;
    int k0 = 0, last_i = -1, c0 = 0, last_c = -1;
    for (int base = 0; base < nb; base += 64) {
        const int i = base + lane;
        const int32_t e = i < nb ? table[(int64_t)b * max_blocks + i] : 0;
        const bool is = i < nb && e < 0 && ~e < n_act_used;
        const bool kv = i < nb && e >= 0;
        const unsigned long long below = (1ull << lane) - 1ull;
        const unsigned long long mask = __ballot(is), cmask = __ballot(kv);
        if (is) list[(int64_t)b * max_blocks + k0 + __popcll(mask & below)] = ~e;
        if (kv) kv_table[(int64_t)b * max_blocks + c0 + __popcll(cmask & below)] = e;
        k0 += __popcll(mask);
        c0 += __popcll(cmask);
        if (mask) last_i = base + 63 - __builtin_clzll(mask);
        if (cmask) last_c = base + 63 - __builtin_clzll(cmask);
    }
    if (lane == 0) {
        auto rows_of = [&](int n_blocks, int last) {       // rows of n_blocks blocks whose last one is logical block `last`
            if (n_blocks <= 0) return 0;
            const int rest = len - (last << blk_log2);
            return ((n_blocks - 1) << blk_log2) + (rest < bt ? rest : bt);
        };
        n_rows[b] = rows_of(k0, last_i);
        kv_len[b] = rows_of(c0, last_c);
    }
}

// cu[0] = 0, cu[b + 1] = cu[b] + len[b], and the same of the requests' blocks of 2^rows_log2 checkpoint rows: one wavefront,
// 64 requests per step.
__global__ __launch_bounds__(64) void paged_prefix_kernel(const int32_t *__restrict__ len, const int32_t *__restrict__ n_rows, int rows_log2,
                                                          int B, int64_t *__restrict__ cu, int32_t *__restrict__ cu_items)
{
    const int lane = threadIdx.x;
    int64_t carry = 0;
    int32_t carry_i = 0;
    if (lane == 0) {
        cu[0] = 0;
        cu_items[0] = 0;
    }
    for (int base = 0; base < B; base += 64) {
        const int i = base + lane;
        int64_t v = i < B ? len[i] : 0;
        int32_t n = i < B ? (n_rows[i] + (1 << rows_log2) - 1) >> rows_log2 : 0;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int64_t up = __shfl_up(v, off, 64);
            const int32_t up_i = __shfl_up(n, off, 64);
            if (lane >= off) {
                v += up;
                n += up_i;
            }
        }
        if (i < B) {
            cu[i + 1] = carry + v;
            cu_items[i + 1] = carry_i + n;
        }
        carry += __shfl(v, 63, 64);
        carry_i += __shfl(n, 63, 64);
    }
}

}  // namespace

hipError_t launch_absorbed(const AbsorbedArgs &a, hipStream_t s)
{
    if (a.B <= 0 || a.L_act <= 0) return hipSuccess;
    if (a.H > kAbsorbMaxHeads || a.d % 64 != 0 || a.B > 65535 || (int64_t)a.H * a.head_dim != a.d || (a.dt != 0 && a.dt != 1))
        return hipErrorInvalidValue;
    const int64_t rows = (int64_t)a.B * a.L_act;
    hipError_t e = launch_carry(a, rows, s);
    if (e == hipSuccess) e = launch_absorbed_stream(a, nullptr, rows, s);
    return e == hipSuccess ? launch_output(a, s) : e;
}

// The two views of the block table that the paged step without regeneration works on (see paged_index_kernel).
hipError_t launch_paged_index(const PagedAbsorbedArgs &p, hipStream_t s)
{
    const AbsorbedArgs &a = p.abs;
    if (a.B <= 0) return hipSuccess;
    if (p.block_tokens < 16 || (p.block_tokens & (p.block_tokens - 1)) != 0 || p.max_blocks <= 0) return hipErrorInvalidValue;
    int blk_log2 = 0;
    while ((1 << blk_log2) < p.block_tokens) ++blk_log2;
    hipLaunchKernelGGL(paged_index_kernel, dim3((unsigned)((a.B + 3) / 4)), dim3(256), 0, s,
                       p.block_table, p.max_blocks, p.seq_len, blk_log2, p.n_act_used, a.B, p.list, p.n_rows,
                       p.kv_table, p.kv_len);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(paged_prefix_kernel, dim3(1), dim3(64), 0, s, p.kv_len, p.n_rows,
                       absorbed_rows_log2((int64_t)p.n_act_used * p.block_tokens, a.d, a.H), a.B, p.kv_cu, p.cu_items);
    return hipGetLastError();
}

// After launch_paged_index (and the attention over the KV view).  a.abs: act = the activation pool, L_act =
// max_blocks * block_tokens (the most rows a request can have), L_kv != 0 iff out_c / lse_c hold the attention
// over the KV blocks; w has pitch absorbed_row_pitch(L_act).
hipError_t launch_paged_absorbed(const PagedAbsorbedArgs &p, hipStream_t s)
{
    const AbsorbedArgs &a = p.abs;
    if (a.B <= 0) return hipSuccess;
    if (a.H > kAbsorbMaxHeads || a.d % 64 != 0 || a.B > 65535 || (int64_t)a.H * a.head_dim != a.d || (a.dt != 0 && a.dt != 1))
        return hipErrorInvalidValue;
    if (p.block_tokens < 16 || (p.block_tokens & (p.block_tokens - 1)) != 0 || p.max_blocks <= 0 || a.L_act != p.max_blocks * p.block_tokens)
        return hipErrorInvalidValue;
    int blk_log2 = 0;
    while ((1 << blk_log2) < p.block_tokens) ++blk_log2;
    const int64_t rows = (int64_t)p.n_act_used * p.block_tokens;
    hipError_t e = launch_carry(a, rows, s);
    AbsorbedRows pr;
    pr.list = p.list; pr.n_rows = p.n_rows; pr.cu_items = p.cu_items; pr.list_pitch = p.max_blocks; pr.blk_log2 = blk_log2;
    if (e == hipSuccess) e = launch_absorbed_stream(a, &pr, rows, s);
    return e == hipSuccess ? launch_output(a, s) : e;
}

}  // namespace hk
