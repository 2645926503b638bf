// QKV generation for the current input tokens (qkv_current.hip), form for many rows and for wide layers (qkv_stream_takes
// says which), in three launches:
//   norm   xhat = LayerNorm(x) [B, d] in the storage type (fp32 statistics, one rounding), and the checkpoint copy
//   stream parts of xhat [Wq; Wkv]^T, fp32, from a fixed number of persistent workgroups
//   finish sum of the parts, bias, rounding, store of q and of the K / V rows (in the stream kernel where the parts are large)
//
// What bounds it: one pass over the weights (6 d^2 bytes).  The one-launch kernel builds the normalised tile, the two
// correction sums and the operand layout on the vector ALU and in LDS beside the products, in every workgroup: with 64 to
// 128 rows that, and not the weights, set its time, and its workgroups (128 features each) left a third of the compute
// units idle at d = 7168.  Here:
//   * 128 features x 64 reduction elements of the weights are a unit of work (64 features where d is no multiple of 128).
//     The units of all feature tiles, in order, are cut into equal runs, one per workgroup, so that every compute unit has
//     the same work whatever the number of tiles; a run leaves one fp32 part per tile that it meets, and the order in
//     which parts are added is fixed by the sizes.  The cut is that of Q, K and V also where only Q is asked for: q must
//     not depend on whether K / V rows are produced.
//   * xhat and the weights have wavefronts and LDS rings of their own: loads of one wavefront land in order, and the rows (L2)
//     behind weights (HBM) came as late as those.  A fifth wavefront asks for the rows, a block of 64 reduction elements per
//     stage, shared by the four that multiply (one barrier per stage, with the next stage's fragments read behind it); each
//     of the four asks for the weights of its own features and needs nobody to tell it that they are there.  Against one
//     ring for both: B = 128, d = 7168: 90.5 -> 87.8 us, 9216: 139 -> 132; B <= 32 level.
//   * Weights straight to registers in the operand layout, 64 bytes of a row per load, ran at 4.5 TB/s: whole lines through LDS.
//   * The weights are asked for non-temporally: xhat (up to 2.4 MB), which every workgroup reads once per tile, stays in
//     L2 (d = 7168, B = 32: 70 -> 61 us).
//   * Q alone is a third of the units: two workgroups share a run then, 64 features each (d = 4096, B = 64 / 128: 24.1 / 30.9 ->
//     20.0 / 24.2 us; d = 7168: 50.3 / 66 -> 39.6 / 48.7; with up to 32 rows it was so before: 35.8 -> 34.7).
//   * Where the parts are large (kFusedParts) there is no finishing kernel: a wavefront that has part of a tile stores it and
//     counts itself; the last of those that share the 32 features reads the other parts and finishes, in the same order of
//     addition.  The last one's own part is never read, and the launch and its pass over all parts go (d = 7168, B = 128: 87.8 ->
//     84 us, 9216: 132 -> 125); with small parts the chain store, count, read at the end of the last run is the longer one
//     (d = 4096, B = 128: 37.4 -> 40.4; 7168, B = 32: 61.6 -> 63.4).
//   * Non-temporal stores of the parts were slower (B = 64, d = 7168: 74 us against 72): the finishing kernel finds them in cache.
// Measured, fp16, Q + K + V, new weights in every call, in brackets the one-launch kernel
// (profiles/qkv_single_kernel_vs_three_launches.txt): d = 7168, B = 32 / 64 / 128: 63 / 71 / 84 us (83 / 111 / 120; 308 MB of
// weights); d = 4096, B = 128: 38 (70); d = 9216, B = 128: 128 (157).  Error against 64 bits
// 2.9e-4 (3.6e-4: two roundings on the way into the product); bf16 2.35e-3 (2.8e-3).
#include "hk_internal.h"
#include "elem.h"
#include "mma_ring.h"
#include "qkv_dst.h"

#include <type_traits>

namespace hk {
namespace {

constexpr int kUnitK = 64;                                  // reduction elements of a unit: 128-byte LDS rows
constexpr int kStreamed = 2;                                // cache policy of the weight loads: non-temporal, the rows stay in L2
constexpr int kCoherent = 16;                               // cache policy (sc1) of parts that another XCD reads in the same launch
constexpr int64_t kFusedParts = 2400000;                    // rows (a multiple of 32) x features from which the last wavefront finishes
constexpr int kMinRun = 4;                                  // fewest units of a run worth a part of its own

// Runs: workgroup w of n takes units [w u / n, (w + 1) u / n).  A tile's parts come from consecutive workgroups; the part
// of (workgroup w, tile t) is number t + w, so that there are fewer than tiles + n.
__host__ __device__ inline int run_begin(int w, int units, int n) { return (int)((int64_t)w * units / n); }
__host__ __device__ inline int run_of(int unit, int units, int n) { return (int)((((int64_t)unit + 1) * n - 1) / units); }

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}
// Sum over the 256 threads; `buf` holds 4 floats and is used once per call.
__device__ __forceinline__ float block_sum(float v, float *buf)
{
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) buf[threadIdx.x >> 6] = v;
    __syncthreads();
    return (buf[0] + buf[1]) + (buf[2] + buf[3]);
}

// norm: a workgroup per row, the row in registers.  Mean, then centred sum of squares, in fp32.
constexpr int kMaxD = 9216;                                 // widest layer that comes here (qkv_stream_takes)
constexpr int kKeep = (kMaxD / 8 + 255) / 256;              // 16-byte chunks of a thread
template <int DT>
__global__ __launch_bounds__(256) void qkv_norm_kernel(const typename Elem<DT>::T *__restrict__ x,
                                                       const typename Elem<DT>::T *__restrict__ gamma,
                                                       const typename Elem<DT>::T *__restrict__ beta,
                                                       typename Elem<DT>::T *__restrict__ xhat,
                                                       typename Elem<DT>::T *__restrict__ act_dst, int64_t act_row_stride,
                                                       int d, float eps, PagedDst pd, int32_t *__restrict__ arrived, int n_arrived)
{
    typedef typename Elem<DT>::T elem_t;
    typedef typename Elem<DT>::V8 vec8_t;
    __shared__ float buf[2][4];
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n_arrived; i += gridDim.x * 256) arrived[i] = 0;
    const int m = blockIdx.x, tid = threadIdx.x, nvec = d >> 3;
    const vec8_t *row = reinterpret_cast<const vec8_t *>(x + (int64_t)m * d);
    vec8_t *ckpt = nullptr;
    if (act_dst) {
        if (pd.block_table) {
            int32_t entry;
            int r;
            paged_slot(pd, m, entry, r);
            if (r >= 0 && entry < 0 && ~entry < pd.P_act)
                ckpt = reinterpret_cast<vec8_t *>(act_dst + ((((int64_t)~entry) << pd.blk_log2) + r) * d);
        } else {
            ckpt = reinterpret_cast<vec8_t *>(act_dst + (int64_t)m * act_row_stride);
        }
    }
    vec8_t v[kKeep];
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
        const int c = tid + 256 * i;
        v[i] = row[c < nvec ? c : nvec - 1];
    }
    float s = 0.f;
    auto add = [&](const vec8_t &e8) {
#pragma unroll
        for (int e = 0; e < 8; ++e) s += (float)e8[e];
    };
#pragma unroll
    for (int i = 0; i < kKeep; ++i)
        if (tid + 256 * i < nvec) add(v[i]);
    const float mean = block_sum(s, buf[0]) / (float)d;
    s = 0.f;
    auto add_sq = [&](const vec8_t &e8) {
#pragma unroll
        for (int e = 0; e < 8; ++e) { const float df = (float)e8[e] - mean; s = __builtin_fmaf(df, df, s); }
    };
#pragma unroll
    for (int i = 0; i < kKeep; ++i)
        if (tid + 256 * i < nvec) add_sq(v[i]);
    const float rstd = 1.0f / __builtin_sqrtf(block_sum(s, buf[1]) / (float)d + eps);
    vec8_t *out = reinterpret_cast<vec8_t *>(xhat + (int64_t)m * d);
    auto put = [&](const vec8_t &e8, int c) {
        const vec8_t g = reinterpret_cast<const vec8_t *>(gamma)[c], b = reinterpret_cast<const vec8_t *>(beta)[c];
        vec8_t o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (elem_t)__builtin_fmaf(((float)e8[e] - mean) * rstd, (float)g[e], (float)b[e]);
        out[c] = o;
        if (ckpt) ckpt[c] = e8;
    };
#pragma unroll
    for (int i = 0; i < kKeep; ++i)
        if (tid + 256 * i < nvec) put(v[i], tid + 256 * i);
}

struct StreamArgs {
    const void *xhat, *Wq, *Wkv, *bq, *bkv;
    void *q_out, *K_dst, *V_dst;
    float *part;
    int32_t *arrived;
    int B, d, n_heads, head_dim, L_cap, tok_pos, q_tiles, nks, units, runs, live;   // live: units that are asked for (the first ones)
    int split;                                                 // workgroups that share a run: each takes 64 TN features of its tiles
    PagedDst pd;
};

// Feature n of Q (is_q) or of K, V in the row that a store begins with, and where row m lies from there (-1: it is not stored).
template <int DT>
__device__ __forceinline__ typename Elem<DT>::T *feature_dst(const StreamArgs &p, bool is_q, int n)
{
    typedef typename Elem<DT>::T elem_t;
    const int f = n < p.d ? n : n - p.d;
    const int head_stride = p.pd.block_table ? (p.head_dim << p.pd.blk_log2) : p.L_cap * p.head_dim;
    return is_q ? static_cast<elem_t *>(p.q_out) + n
                : static_cast<elem_t *>(n < p.d ? p.K_dst : p.V_dst) + (int64_t)(f / p.head_dim) * head_stride + f % p.head_dim;
}
__device__ __forceinline__ int64_t row_offset(const StreamArgs &p, bool is_q, int m)
{
    int64_t base = -1;
    if (is_q) {
        base = (int64_t)m * p.d;
    } else if (p.pd.block_table) {
        int32_t entry;
        int row;
        paged_slot(p.pd, m, entry, row);
        if (row >= 0 && entry >= 0 && entry < p.pd.P_kv) base = ((((int64_t)entry * p.n_heads) << p.pd.blk_log2) + row) * p.head_dim;
    } else {
        base = ((int64_t)m * p.n_heads * p.L_cap + p.tok_pos) * p.head_dim;
    }
    return base;
}

// Store of 4 TN consecutive features from feature n of Q (is_q) or of K, V, bias added and rounded.
template <int TN, int DT>
struct Output {
    typedef typename Elem<DT>::T elem_t;
    typedef elem_t out_t __attribute__((ext_vector_type(4 * TN)));
    const StreamArgs &p;
    const bool is_q;
    elem_t *dst;
    out_t bias;

    __device__ __forceinline__ Output(const StreamArgs &args, bool is_q_, int n) : p(args), is_q(is_q_)
    {
        bias = *reinterpret_cast<const out_t *>(static_cast<const elem_t *>(is_q ? p.bq : p.bkv) + n);
        dst = feature_dst<DT>(p, is_q, n);
    }
    __device__ __forceinline__ void store(int m, const float4_t (&sum)[TN]) const
    {
        if (m >= p.B) return;
        const int64_t base = row_offset(p, is_q, m);
        if (base < 0) return;
        out_t o;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) o[4 * j + r] = (elem_t)(sum[j][r] + (float)bias[4 * j + r]);
        *reinterpret_cast<out_t *>(dst + base) = o;
    }
};

template <int N>
__device__ __forceinline__ void wait_vm()
{
    static_assert(N <= 63, "vmcnt counts to 63");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

template <int MT, int TN, int NA, int NB>
constexpr int stream_lds_bytes() { return (NA * MT * 16 + NB * 64 * TN) * kUnitK * 2; }

// MT: blocks of 16 rows; TN: blocks of 16 features of a wavefront; NA, NB: stages of the rings of the rows and of a wavefront's
// weights; FUSED: no finishing kernel follows.
template <int MT, int TN, int NA, int NB, bool FUSED, int DT>
__global__ __launch_bounds__(320) void qkv_stream_kernel(StreamArgs p)
{
#if defined(__HIP_DEVICE_COMPILE__)                            // (the host pass drops the kernel's stub over a direct load in this body)
    typedef typename Elem<DT>::T elem_t;
    typedef typename Elem<DT>::V8 vec8_t;
    typedef __attribute__((address_space(3))) void *lds_ptr_t;
    typedef unsigned u4_t __attribute__((ext_vector_type(4)));
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int kStage = MT * 16 * kUnitK * 2, BN = 64 * TN;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int d = p.d, nks = p.nks;
    const int run = (int)blockIdx.x / p.split, part = (int)blockIdx.x % p.split;
    const int u_begin = run_begin(run, p.units, p.runs);
    const int u_end = run_begin(run + 1, p.units, p.runs);
    const int n = (u_end < p.live ? u_end : p.live) - u_begin; // >= 1: no more runs than units, none past the live ones
    const int tile0 = u_begin / nks, k0 = u_begin - tile0 * nks;

    if (wave == 4) {                                           // ---- the rows: 8 of them a load, chunks swizzled by row / 2
        constexpr int LA = 2 * MT;
        int voff[LA];
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const int q = 8 * i + (lane >> 3);
            voff[i] = ((q < p.B ? q : p.B - 1) * d + 8 * ((lane & 7) ^ ((q >> 1) & 7))) * 2;       // rows past the end: never stored
        }
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<elem_t *>(static_cast<const elem_t *>(p.xhat)), 0, p.B * d * 2, 0x00020000);
        int slot = 0, k = k0;
        auto issue = [&] {
#pragma unroll
            for (int i = 0; i < LA; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(smem + slot * kStage + i * 1024), 16, voff[i], k * (kUnitK * 2), 0, 0);
            slot = slot + 1 == NA ? 0 : slot + 1;
            k = k + 1 == nks ? 0 : k + 1;
        };
        for (int s = 0; s < NA && s < n; ++s) issue();
        for (int s = -1; s + 1 < n; ++s) {                     // stage s + 1 is there
            if (s + NA - 1 < n) wait_vm<LA * (NA - 2)>();
            else wait_vm<0>();
            asm volatile("s_barrier" ::: "memory");            // and that of s is free
            if (s >= 0 && s + NA < n) issue();
        }
        return;
    }

    // ---- the weights: each wavefront its own, in a ring of its own
    constexpr int LB = 2 * TN, kMine = TN * 16 * kUnitK * 2;
    unsigned char *mine = smem + NA * kStage + wave * (NB * kMine);
    const int c = lane & 15, g = lane >> 4;
    int voff[LB];
#pragma unroll
    for (int i = 0; i < LB; ++i) {                             // LDS row 16 j + c: so that a lane ends up with 4 TN consecutive features
        const int row = 8 * i + (lane >> 3), cc = row & 15, j = row >> 4;
        voff[i] = ((16 * TN * wave + 4 * TN * (cc >> 2) + 4 * j + (cc & 3)) * d + 8 * ((lane & 7) ^ ((row >> 1) & 7))) * 2;
    }
    auto tile_rsrc = [&](int tile) {
        const elem_t *W = tile < p.q_tiles ? static_cast<const elem_t *>(p.Wq) + (int64_t)(tile * p.split + part) * BN * d
                                           : static_cast<const elem_t *>(p.Wkv) + (int64_t)((tile - p.q_tiles) * p.split + part) * BN * d;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<elem_t *>(W), 0, BN * d * 2, 0x00020000);
    };
    int ask_tile = tile0, ask_k = k0, ask_slot = 0, asked = 0;
    __amdgpu_buffer_rsrc_t rs = tile_rsrc(ask_tile);
    auto ask = [&] {
#pragma unroll
        for (int i = 0; i < LB; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(mine + ask_slot * kMine + i * 1024), 16, voff[i], ask_k * (kUnitK * 2), 0, kStreamed);
        ask_slot = ask_slot + 1 == NB ? 0 : ask_slot + 1;
        ++asked;
        if (++ask_k == nks) {
            ask_k = 0;
            ++ask_tile;
            if (asked < n) rs = tile_rsrc(ask_tile);
        }
    };
    int foff[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) foff[ks] = c * 128 + (((4 * ks + g) ^ ((c >> 1) & 7)) << 4);
    vec8_t fa[2][MT], fb[2][TN];
    auto read = [&](int ks, int slot, int own) {
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[ks][j] = *reinterpret_cast<const vec8_t *>(mine + own * kMine + j * 2048 + foff[ks]);
#pragma unroll
        for (int i = 0; i < MT; ++i) fa[ks][i] = *reinterpret_cast<const vec8_t *>(smem + slot * kStage + i * 2048 + foff[ks]);
    };
    float4_t acc[MT][TN];
    auto clear = [&] {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
    };
    auto multiply = [&](int ks) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < MT; ++i) acc[i][j] = Elem<DT>::mfma_16x16x32(fb[ks][j], fa[ks][i], acc[i][j]);
    };
    for (int s = 0; s < NB && s < n; ++s) ask();
    clear();
    if (n >= NB) wait_vm<LB * (NB - 1)>();
    else wait_vm<0>();
    asm volatile("s_barrier" ::: "memory");
    read(0, 0, 0);
    int tile = tile0, k = k0, cur = 0, own = 0;
    constexpr int kPart = MT * TN * 256 * 16;                  // bytes of a part, thread for thread: a block of 16 x 16 is 1 KB of each wavefront
    const __amdgpu_buffer_rsrc_t parts = __builtin_amdgcn_make_buffer_rsrc(p.part, 0, 0x7ffffff0, 0x00020000);
    const int lane_at = (int)threadIdx.x * 16;
    auto finish = [&] {
        const bool is_q = tile < p.q_tiles;
        const Output<TN, DT> out(p, is_q, ((is_q ? tile : tile - p.q_tiles) * p.split + part) * BN + 16 * TN * wave + 4 * TN * g);
#pragma unroll
        for (int i = 0; i < MT; ++i) out.store(16 * i + c, acc[i]);
    };
    // acc = the sum of the parts w0 .. w1 of the tile, acc itself in the place of this run's
    auto add_others = [&](int w0, int w1) {
        constexpr int IB = MT > 4 ? MT / 2 : MT;               // as many blocks at a time as there are registers for
#pragma unroll
        for (int i0 = 0; i0 < MT; i0 += IB) {
            float4_t v[IB][TN], sum[IB][TN];
            auto load = [&](int w) {
                const int from = ((tile + w) * p.split + part) * kPart + i0 * TN * 4096;
#pragma unroll
                for (int i = 0; i < IB; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        v[i][j] = __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(parts, lane_at, from + (i * TN + j) * 4096, kCoherent));
            };
            auto add = [&](bool first) {
#pragma unroll
                for (int i = 0; i < IB; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) sum[i][j] = first ? v[i][j] : sum[i][j] + v[i][j];
            };
            for (int w = w0; w < run; ++w) {
                load(w);
                add(w == w0);
            }
#pragma unroll
            for (int i = 0; i < IB; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) sum[i][j] = run > w0 ? sum[i][j] + acc[i0 + i][j] : acc[i0 + i][j];
            for (int w = run + 1; w <= w1; ++w) {
                load(w);
                add(false);
            }
#pragma unroll
            for (int i = 0; i < IB; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i0 + i][j] = sum[i][j];
        }
    };
    auto leave = [&] {                                         // the tile ends here for this run
        bool last = FUSED;
        const int w0 = FUSED ? run_of(tile * nks, p.units, p.runs) : 0, w1 = FUSED ? run_of(tile * nks + nks - 1, p.units, p.runs) : 1;
        if (w0 != w1) {
            const int slot = (tile + run) * p.split + part;
            if constexpr (!FUSED) {
                float4_t *dst = reinterpret_cast<float4_t *>(p.part) + (int64_t)slot * (kPart / 16) + threadIdx.x;
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) dst[(i * TN + j) * 256] = acc[i][j];
            } else {
                // The accumulators are not touched before these stores have completed, below: behind a raw buffer store with
                // a scalar offset the compiler leaves no wait state, and cleared at once its last lanes could store zeros.
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4_t, acc[i][j]), parts, lane_at, slot * kPart + (i * TN + j) * 4096, kCoherent);
            }
            if constexpr (FUSED) {
                // The wavefronts of the runs that share these features count themselves.  Parts are written and read as
                // device-scope atomics are (sc1), and each has arrived (vmcnt) before its wavefront counts; nobody waits.
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                int before = 0;
                if (lane == 0)
                    before = __hip_atomic_fetch_add(p.arrived + (tile * p.split + part) * 4 + wave, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                last = __builtin_amdgcn_readfirstlane(before) == w1 - w0;
                asm volatile("" ::: "memory");
                if (last) add_others(w0, w1);
            }
        }
        if constexpr (FUSED) {
            if (last) finish();
        }
        clear();
        k = 0;
        ++tile;
    };
    for (int s = 0; s + 1 < n; ++s) {
        read(1, cur, own);
        __builtin_amdgcn_sched_barrier(0);
        multiply(0);
        __builtin_amdgcn_sched_barrier(0);
        cur = cur + 1 == NA ? 0 : cur + 1;
        own = own + 1 == NB ? 0 : own + 1;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the slots of this unit are free
        if (s + NB < n) {
            ask();
            wait_vm<LB * (NB - 1)>();
        } else {
            wait_vm<0>();
        }
        asm volatile("s_barrier" ::: "memory");
        read(0, cur, own);
        __builtin_amdgcn_sched_barrier(0);
        multiply(1);
        __builtin_amdgcn_sched_barrier(0);
        if (++k == nks) leave();
    }
    read(1, cur, own);
    multiply(0);
    multiply(1);
    leave();
#endif
}

// finish: a workgroup per (tile or part of it, block of 16 rows); thread for thread the layout of the parts.
template <int MT, int TN, int DT>
__global__ __launch_bounds__(256) void qkv_finish_kernel(StreamArgs p)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tile = (int)blockIdx.x / p.split, part = (int)blockIdx.x % p.split, i = blockIdx.y;
    const int m = 16 * i + (lane & 15);
    if (m >= p.B) return;                                                   // no barrier in this kernel
    const int w0 = run_of(tile * p.nks, p.units, p.runs), w1 = run_of(tile * p.nks + p.nks - 1, p.units, p.runs);
    const float4_t *src = reinterpret_cast<const float4_t *>(p.part) + (int64_t)((tile + w0) * p.split + part) * (MT * TN * 256) + i * TN * 256 + tid;
    float4_t sum[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) sum[j] = src[256 * j];
    for (int w = w0 + 1; w <= w1; ++w) {
        src += p.split * (MT * TN * 256);
#pragma unroll
        for (int j = 0; j < TN; ++j) sum[j] += src[256 * j];
    }
    const bool is_q = tile < p.q_tiles;
    const Output<TN, DT> out(p, is_q, ((is_q ? tile : tile - p.q_tiles) * p.split + part) * (64 * TN) + 16 * TN * wave + 4 * TN * (lane >> 4));
    out.store(m, sum);
}

// ---- layers that 128 does not divide: units of 64 features, both operands in one ring, two workgroups a compute unit and twice as
// many runs, so that Q alone, a third of them, fills the chip (d = 8128, B = 64: 47 us; with rings of their own and one workgroup
// a unit 69, where Q, K and V gain 1 to 3 %).
// Workgroups of a compute unit: two where the LDS of one allows it.
template <int BM, int BN, int NS>
constexpr int ring_per_cu() { return ring::lds_bytes<BM, BN, NS>() <= 80 * 1024 ? 2 : 1; }

template <int BM, int BN, int NS, int DT>
__global__ __launch_bounds__(256, (ring_per_cu<BM, BN, NS>())) void qkv_ring_kernel(StreamArgs p)
{
#if defined(__HIP_DEVICE_COMPILE__)                            // (the host pass drops the kernel's stub over a direct load in this body)
    typedef typename Elem<DT>::T elem_t;
    typedef ring::Ring<BM, BN, NS, DT> ring_t;
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int LA = ring_t::kLoadsA, LB = ring_t::kLoadsB, TM = ring_t::TM, TN = ring_t::TN;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int d = p.d, nks = p.nks;
    const int run = (int)blockIdx.x / p.split, part = (int)blockIdx.x % p.split;
    const int u_begin = run_begin(run, p.units, p.runs);
    const int u_end = run_begin(run + 1, p.units, p.runs);
    const int n = (u_end < p.live ? u_end : p.live) - u_begin; // >= 1: no more runs than units, none past the live ones

    ring_t r(smem, tid, wave);
    const __amdgpu_buffer_rsrc_t a_rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<elem_t *>(static_cast<const elem_t *>(p.xhat)), 0, p.B * d * 2, 0x00020000);
    int a_voff[LA], b_voff[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i)                               // rows past the end: the last row, never stored
        a_voff[i] = ((r.a_row(i) < p.B ? r.a_row(i) : p.B - 1) * d + r.lane_chunk * 8) * 2;
#pragma unroll
    for (int i = 0; i < LB; ++i) b_voff[i] = (r.b_row(i) * d + r.lane_chunk * 8) * 2;
    // the unit to ask for next: its tile's rows and its place on the reduction axis
    int ask_tile = u_begin / nks, ask_k = u_begin % nks;
    auto tile_rsrc = [&](int tile) {
        const elem_t *W = tile < p.q_tiles ? static_cast<const elem_t *>(p.Wq) + (int64_t)(tile * p.split + part) * BN * d
                                           : static_cast<const elem_t *>(p.Wkv) + (int64_t)((tile - p.q_tiles) * p.split + part) * BN * d;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<elem_t *>(W), 0, BN * d * 2, 0x00020000);
    };
    __amdgpu_buffer_rsrc_t b_rsrc = tile_rsrc(ask_tile);
    auto issue = [&](int slot, int i) {
        // weights first: they come from HBM, the rows from L2
        if (i < LB)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(b_rsrc, r.b_dst(slot, i), 16, b_voff[i], ask_k * ring::kRowBytes, 0, kStreamed);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, r.a_dst(slot, i - LB), 16, a_voff[i - LB], ask_k * ring::kRowBytes, 0, 0);
    };
    auto asked = [&](bool more) {                              // more: another unit of this run will be asked for
        if (++ask_k == nks) {
            ask_k = 0;
            ++ask_tile;
            if (more) b_rsrc = tile_rsrc(ask_tile);
        }
    };

    r.clear();
    for (int s = 0; s < NS; ++s) {
        if (s < n) {
#pragma unroll
            for (int i = 0; i < ring_t::kLoads; ++i) issue(s, i);
            asked(s + 1 < n);
        }
    }
    r.start(n);

    int tile = u_begin / nks, k = u_begin % nks;
    // One unit (kind as in Ring::block), and the part of a tile that ends with it.
    auto unit = [&](auto kind, int i) {
        constexpr int KIND = decltype(kind)::value;
        r.template block<KIND>(issue, n - 2 - i);
        if constexpr (KIND == 2) asked(i + NS + 1 < n);
        if (++k == nks || KIND == 0) {                         // the tile ends here for this run: its part leaves
            float4_t *dst = reinterpret_cast<float4_t *>(p.part + (int64_t)((tile + run) * p.split + part) * (BM * BN));
#pragma unroll
            for (int ii = 0; ii < TM; ++ii)
#pragma unroll
                for (int j = 0; j < TN; ++j) dst[(ii * TN + j) * 256 + tid] = r.acc[ii][j];
            r.clear();
            k = 0;
            ++tile;
        }
    };
    int i = 0;
    for (; i + NS < n; ++i) unit(std::integral_constant<int, 2>{}, i);
    for (; i + 1 < n; ++i) unit(std::integral_constant<int, 1>{}, i);
    unit(std::integral_constant<int, 0>{}, i);
#endif
}

// Its parts: thread for thread the layout of the ring's accumulators; a workgroup per (tile, 16-row blocks i of the wavefront rows).
template <int BM, int BN, int DT>
__global__ __launch_bounds__(256) void qkv_ring_finish_kernel(StreamArgs p)
{
    typedef typename Elem<DT>::T elem_t;
    typedef elem_t out_t __attribute__((ext_vector_type(BN / 32)));
    constexpr int TN = BN / 32;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tile = (int)blockIdx.x / p.split, part = (int)blockIdx.x % p.split, i = blockIdx.y;
    const int m0 = (wave >> 1) * (BM / 2) + 16 * i + 4 * (lane >> 4);       // first of this thread's 4 rows
    if (m0 >= p.B) return;                                                  // no barrier in this kernel
    const int w0 = run_of(tile * p.nks, p.units, p.runs), w1 = run_of(tile * p.nks + p.nks - 1, p.units, p.runs);
    const float4_t *src = reinterpret_cast<const float4_t *>(p.part + (int64_t)((tile + w0) * p.split + part) * (BM * BN)) + i * TN * 256 + tid;
    float4_t sum[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) sum[j] = src[256 * j];
    for (int w = w0 + 1; w <= w1; ++w) {
        src += p.split * (BM * BN / 4);
#pragma unroll
        for (int j = 0; j < TN; ++j) sum[j] += src[256 * j];
    }
    const bool is_q = tile < p.q_tiles;
    const int n = ((is_q ? tile : tile - p.q_tiles) * p.split + part) * BN + (BN / 2) * (wave & 1) + TN * (lane & 15);   // first of TN features
    const out_t bias = *reinterpret_cast<const out_t *>(static_cast<const elem_t *>(is_q ? p.bq : p.bkv) + n);
    elem_t *dst = feature_dst<DT>(p, is_q, n);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int m = m0 + r;
        if (m >= p.B) break;
        const int64_t base = row_offset(p, is_q, m);
        if (base >= 0) {
            out_t o;
#pragma unroll
            for (int j = 0; j < TN; ++j) o[j] = (elem_t)(sum[j][r] + (float)bias[j]);
            *reinterpret_cast<out_t *>(dst + base) = o;
        }
    }
}

size_t align256(size_t n) { return (n + 255) / 256 * 256; }

int stream_runs(int units, int workgroups)
{
    const int most = units / kMinRun > 0 ? units / kMinRun : 1;
    return workgroups < most ? workgroups : most;
}

template <int MT, int TN, int NA, int NB, int SPLIT, bool FUSED, int DT>
hipError_t launch_dt(const QkvArgs &a, int cus, hipStream_t s)
{
    typedef typename Elem<DT>::T elem_t;
    const PagedDst pd = paged_dst(a);
    elem_t *xhat = static_cast<elem_t *>(a.scratch);
    float *part = reinterpret_cast<float *>(static_cast<char *>(a.scratch) + align256((size_t)a.B * a.d * 2));
    StreamArgs t;
    t.xhat = xhat; t.Wq = a.Wq; t.Wkv = a.Wkv; t.bq = a.bq; t.bkv = a.bkv; t.part = part;
    t.q_out = a.q_out; t.K_dst = a.K_dst; t.V_dst = a.V_dst; t.pd = pd;
    t.n_heads = a.n_heads; t.head_dim = a.head_dim; t.L_cap = a.L_cap; t.tok_pos = a.tok_pos;
    t.B = a.B; t.d = a.d; t.q_tiles = a.d / (64 * TN * SPLIT); t.nks = a.d / kUnitK; t.split = SPLIT;
    const int tiles = a.K_dst ? 3 * t.q_tiles : t.q_tiles;
    t.units = 3 * t.q_tiles * t.nks;
    t.live = tiles * t.nks;
    t.runs = stream_runs(t.units, cus);
    // the counters lie behind the last part, where qkv_stream_scratch_bytes has room for one more
    t.arrived = reinterpret_cast<int32_t *>(part + (int64_t)(3 * t.q_tiles + t.runs - 1) * SPLIT * (MT * TN * 1024));
    hipLaunchKernelGGL(qkv_norm_kernel<DT>, dim3((unsigned)a.B), dim3(256), 0, s, static_cast<const elem_t *>(a.x),
                       static_cast<const elem_t *>(a.ln_w), static_cast<const elem_t *>(a.ln_b), xhat,
                       static_cast<elem_t *>(a.act_dst), a.act_row_stride, a.d, a.eps, pd, t.arrived, FUSED ? tiles * SPLIT * 4 : 0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    auto kern = qkv_stream_kernel<MT, TN, NA, NB, FUSED, DT>;
    constexpr int lds = stream_lds_bytes<MT, TN, NA, NB>();
    static_assert(lds <= 160 * 1024, "the workgroup must fit the LDS of a compute unit");
    static LdsOnce lds_once;
    e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds, lds_once);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(SPLIT * (run_of(t.live - 1, t.units, t.runs) + 1))), dim3(320), lds, s, t);
    if ((e = hipGetLastError()) != hipSuccess || FUSED) return e;
    hipLaunchKernelGGL((qkv_finish_kernel<MT, TN, DT>), dim3((unsigned)(SPLIT * tiles), (unsigned)((a.B + 15) / 16)), dim3(256), 0, s, t);
    return hipGetLastError();
}

template <int BM, int NS, int DT>
hipError_t launch_ring_dt(const QkvArgs &a, int cus, hipStream_t s)
{
    constexpr int BN = 64;
    typedef typename Elem<DT>::T elem_t;
    elem_t *xhat = static_cast<elem_t *>(a.scratch);
    StreamArgs t;
    t.xhat = xhat; t.Wq = a.Wq; t.Wkv = a.Wkv; t.bq = a.bq; t.bkv = a.bkv;
    t.part = reinterpret_cast<float *>(static_cast<char *>(a.scratch) + align256((size_t)a.B * a.d * 2));
    t.arrived = nullptr;
    t.q_out = a.q_out; t.K_dst = a.K_dst; t.V_dst = a.V_dst; t.pd = paged_dst(a);
    t.n_heads = a.n_heads; t.head_dim = a.head_dim; t.L_cap = a.L_cap; t.tok_pos = a.tok_pos;
    t.B = a.B; t.d = a.d; t.q_tiles = a.d / BN; t.nks = a.d / kUnitK; t.split = 1;
    const int tiles = a.K_dst ? 3 * t.q_tiles : t.q_tiles;
    t.units = 3 * t.q_tiles * t.nks;
    t.live = tiles * t.nks;
    t.runs = stream_runs(t.units, ring_per_cu<BM, BN, NS>() * cus);
    hipLaunchKernelGGL(qkv_norm_kernel<DT>, dim3((unsigned)a.B), dim3(256), 0, s, static_cast<const elem_t *>(a.x),
                       static_cast<const elem_t *>(a.ln_w), static_cast<const elem_t *>(a.ln_b), xhat,
                       static_cast<elem_t *>(a.act_dst), a.act_row_stride, a.d, a.eps, t.pd, t.arrived, 0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    auto kern = qkv_ring_kernel<BM, BN, NS, DT>;
    constexpr int lds = ring::lds_bytes<BM, BN, NS>();
    static_assert(lds <= 160 * 1024, "the workgroup must fit the LDS of a compute unit");
    static LdsOnce lds_once;
    e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds, lds_once);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(run_of(t.live - 1, t.units, t.runs) + 1)), dim3(256), lds, s, t);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL((qkv_ring_finish_kernel<BM, BN, DT>), dim3((unsigned)tiles, BM / 32), dim3(256), 0, s, t);
    return hipGetLastError();
}

template <int BM, int NS>
hipError_t launch_ring(const QkvArgs &a, int cus, hipStream_t s)
{
    return a.dtype == 1 ? launch_ring_dt<BM, NS, 1>(a, cus, s) : launch_ring_dt<BM, NS, 0>(a, cus, s);
}

template <int MT, int TN, int NA, int NB, int SPLIT, bool FUSED = false>
hipError_t launch_types(const QkvArgs &a, int cus, hipStream_t s)
{
    return a.dtype == 1 ? launch_dt<MT, TN, NA, NB, SPLIT, FUSED, 1>(a, cus, s) : launch_dt<MT, TN, NA, NB, SPLIT, FUSED, 0>(a, cus, s);
}

// Rings as deep as the LDS of a compute unit and the counter of loads (63) allow.
template <int TN, int SPLIT>
hipError_t launch_any(const QkvArgs &a, int cus, hipStream_t s)
{
    constexpr int W = 2 / TN;                                  // a stage of weights is 8 KB x TN
    const int rows = (a.B + 31) / 32 * 32;
    if constexpr (TN == 2) {
        if ((int64_t)rows * 3 * a.d >= kFusedParts) {
            if (rows == 128) return launch_types<8, TN, 5, 5, SPLIT, true>(a, cus, s);
            if (rows == 96) return launch_types<6, TN, 5, 6, SPLIT, true>(a, cus, s);
        }
    }
    switch (rows / 32) {
    case 1: return launch_types<2, TN, 10, 7 * W, SPLIT>(a, cus, s);
    case 2: return launch_types<4, TN, 6, 7 * W, SPLIT>(a, cus, s);
    case 3: return launch_types<6, TN, 5, 6 * W, SPLIT>(a, cus, s);
    default: return launch_types<8, TN, 5, 5 * W, SPLIT>(a, cus, s);
    }
}

}  // namespace

// Where the lines lie (new weights in every call, replayed from a graph, us a call, one-launch kernel against this one, fp16 /
// bf16 where they differ).  The sizes that come here: profiles/qkv_single_kernel_vs_three_launches.txt, 306 of them, none slower
// than 0.96 of the one-launch kernel.  The sizes that stay there (marked *) were measured with rings that both operands shared, 0
// to 3 % slower than now, and not since.  Three launches cost 12 to 14 us however small the layer, so many rows and wide
// layers come here.
//   97 rows and more: every layer from d = 768 on: 25.1 / 28.0 against 13.9 / 13.7 (B = 128); 4096: 70 / 84 against 38; 7168:
//     120 / 143 against 84; 9216: 157 / 194 against 128; 9152 (units of 64 features): 160 / 194 against 150
//   65 to 96 rows: from d = 768 on: 18.7 / 20.8 against 12.5 (B = 65).  fp16 below 8448: 8192, B = 96: 118 against 104;
//     8256, B = 65: 118 against 110; 8448, B = 96: 111.7 against 116.6*; 9216, B = 96: 118 against 127*; 9152: 118 against
//     137*.  bf16 everywhere: 9216, B = 96: 154 against 121
//   33 to 64 rows: from d = 2048 on: 21.2 / 24.2 against 17.8 (B = 33).  fp16 below 8192, where the one-launch kernel
//     changes to workgroups of 128 features: 8128, B = 64: 135 against 96; 8192, B = 33: 91 against 95 and 101 against 98
//     (two sessions)*; 8704: level*.  bf16 below 8448: 8256, B = 64: 111 against 103; 8448: 101 against 103*; 9152: 109
//     against 123*; 9216: level*
//   up to 32 rows: while the one-launch kernel's workgroups (64 features) fit 256 units at once it is level within 8 % or
//     faster: 4096, B = 32: 29.7 against 27.4*; from 5504 on 60 against 41 (B = 1); 9216: 99 against 94 (B = 1), 111
//     against 97 (B = 32)
// Wider layers than 9216 stay with one launch.  A build without the limit gained on Q + K + V (10240: 0.81 to 1.10 of the
// one-launch kernel's time; 11264 and 12288, where that kernel's workgroups need a second round: 0.47 to 0.87; 16384: 0.60 to
// 0.97), but lost on Q alone from 11264 on (up to 1.07 there, 1.14 at 12288, 1.27 at 14336), and q must come from the same
// form in both.  That was with a third of the workgroups for Q alone; they fill the chip since two share a run, and the
// widths beyond 9216 have not been measured again.
bool qkv_stream_takes(int B, int d, int dtype)
{
    if (B <= 0 || B > kQkvMaxRows || d % kUnitK != 0 || d > kMaxD) return false;
    if (B > 96) return d >= 768;
    if (B > 64) return d >= 768 && (dtype == 1 || d < 8448);
    if (B > 32) return d >= 2048 && d < (dtype == 1 ? 8448 : 8192);
    return 3 * (d / 64) > 256;
}

// Scratch of one launch of B rows: xhat and the parts (fewer than tiles + runs of them).  The number of runs follows the
// device; the bound is for kQkvStreamCus compute units, and a device with more gets as many runs as for that number.
size_t qkv_stream_scratch_bytes(int B, int d)
{
    const size_t rows = (B + 31) / 32 * 32;
    const size_t parts = d % 128 == 0 ? (size_t)(3 * (d / 128) + kQkvStreamCus) * 128 : (size_t)(3 * (d / 64) + 2 * kQkvStreamCus) * 64;
    return align256((size_t)B * d * 2) + rows * parts * 4;
}

hipError_t launch_qkv_stream(const QkvArgs &a, hipStream_t s)
{
    if (a.B <= 0 || a.B > kQkvMaxRows || a.d % kUnitK != 0 || a.d > kMaxD ||
        a.scratch_bytes < qkv_stream_scratch_bytes(a.B, a.d)) return hipErrorInvalidValue;
    int dev = 0, cus = 0;
    const hipError_t e = current_device_cus(&dev, &cus);
    if (e != hipSuccess) return e;
    if (cus > kQkvStreamCus) cus = kQkvStreamCus;
    if (a.d % 128 != 0) {
        switch ((a.B + 31) / 32) {
        case 1: return launch_ring<32, 6>(a, cus, s);
        case 2: return launch_ring<64, 5>(a, cus, s);
        case 3: return launch_ring<96, 4>(a, cus, s);
        default: return launch_ring<128, 3>(a, cus, s);
        }
    }
    // Q alone: two workgroups a run, each with the same units along the reduction of 64 features, so the bits are the same
    return a.K_dst ? launch_any<2, 1>(a, cus, s) : launch_any<1, 2>(a, cus, s);
}

}  // namespace hk
