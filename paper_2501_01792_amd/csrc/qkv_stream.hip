// QKV generation for the current input tokens (qkv_current.hip), form for many rows and for wide layers (qkv_stream_takes
// says which), in three launches:
//   norm   xhat = LayerNorm(x) [B, d] in the storage type (fp32 statistics, one rounding), and the checkpoint copy
//   stream parts of xhat [Wq; Wkv]^T, fp32, from a fixed number of persistent workgroups
//   finish sum of the parts, bias, rounding, store of q and of the K / V rows
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
//   * Both operands of a unit are one stage of the LDS ring of mma_ring.h, which runs on across tiles, so the loads never
//     drain.
//   * The weights are asked for non-temporally: xhat (up to 2.4 MB), which every workgroup reads once per tile, stays in
//     L2 (d = 7168, B = 32: 70 -> 61 us).  64-feature units read xhat twice as often (B = 128: 95 us against 87).
//   * One workgroup with a ring as deep as the LDS allows beat two with half of it each (B = 64: 69 us against 71).
//   * Non-temporal stores of the parts were slower (B = 64, d = 7168: 74 us): the finishing kernel finds them in cache.
// Measured, fp16, Q + K + V, new weights in every call, in brackets the one-launch kernel
// (profiles/qkv_single_kernel_vs_three_launches.txt): d = 7168, B = 32 / 64 / 128: 64 / 72 / 90 us (83 / 113 / 120; 308 MB of
// weights); d = 4096, B = 128: 39 (69); d = 9216, B = 128: 136 to 140 (148 to 169, two sessions).  Error against 64 bits
// 2.9e-4 (3.6e-4: two roundings on the way into the product); bf16 2.35e-3 (2.8e-3).
#include "hk_internal.h"
#include "elem.h"
#include "mma_ring.h"
#include "qkv_dst.h"

#include <type_traits>

namespace hk {
namespace {

constexpr int kUnitK = ring::kBlockK;                       // reduction elements of a unit: a block of the ring
constexpr int kStreamed = 2;                                // cache policy of the weight loads: non-temporal, the rows stay in L2
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
                                                       int d, float eps, PagedDst pd)
{
    typedef typename Elem<DT>::T elem_t;
    typedef typename Elem<DT>::V8 vec8_t;
    __shared__ float buf[2][4];
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
    const void *xhat, *Wq, *Wkv;
    float *part;
    int B, d, q_tiles, nks, units, runs, live;                 // live: units that are asked for (the first ones)
    int split;                                                 // workgroups that share a run: each takes BN features of its tiles
};

// Workgroups of a compute unit: two where the LDS of one allows it.
template <int BM, int BN, int NS>
constexpr int stream_per_cu() { return ring::lds_bytes<BM, BN, NS>() <= 80 * 1024 ? 2 : 1; }

template <int BM, int BN, int NS, int DT>
__global__ __launch_bounds__(256, (stream_per_cu<BM, BN, NS>())) void qkv_stream_kernel(StreamArgs p)
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

// finish: a workgroup per (tile or part of it, 16-row blocks i of the wavefront rows); thread for thread the layout of the parts.
struct FinishArgs {
    const float *part;
    const void *bq, *bkv;
    void *q_out, *K_dst, *V_dst;
    int B, d, n_heads, head_dim, L_cap, tok_pos, q_tiles, nks, units, runs, split;
    PagedDst pd;
};

template <int BM, int BN, int DT>
__global__ __launch_bounds__(256) void qkv_finish_kernel(FinishArgs p)
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
    const int f = n < p.d ? n : n - p.d;
    const int h = f / p.head_dim, e = f % p.head_dim;
    const int head_stride = p.pd.block_table ? (p.head_dim << p.pd.blk_log2) : p.L_cap * p.head_dim;
    elem_t *dst = is_q ? static_cast<elem_t *>(p.q_out) + n
                       : static_cast<elem_t *>(n < p.d ? p.K_dst : p.V_dst) + (int64_t)h * head_stride + e;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int m = m0 + r;
        if (m >= p.B) break;
        int64_t base = -1;                                                  // or the row is not stored
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

template <int BM, int BN, int NS, int SPLIT, int DT>
hipError_t launch_dt(const QkvArgs &a, int cus, hipStream_t s)
{
    typedef typename Elem<DT>::T elem_t;
    const PagedDst pd = paged_dst(a);
    elem_t *xhat = static_cast<elem_t *>(a.scratch);
    float *part = reinterpret_cast<float *>(static_cast<char *>(a.scratch) + align256((size_t)a.B * a.d * 2));
    hipLaunchKernelGGL(qkv_norm_kernel<DT>, dim3((unsigned)a.B), dim3(256), 0, s, static_cast<const elem_t *>(a.x),
                       static_cast<const elem_t *>(a.ln_w), static_cast<const elem_t *>(a.ln_b), xhat,
                       static_cast<elem_t *>(a.act_dst), a.act_row_stride, a.d, a.eps, pd);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    StreamArgs t;
    t.xhat = xhat; t.Wq = a.Wq; t.Wkv = a.Wkv; t.part = part;
    t.B = a.B; t.d = a.d; t.q_tiles = a.d / (BN * SPLIT); t.nks = a.d / kUnitK; t.split = SPLIT;
    const int tiles = a.K_dst ? 3 * t.q_tiles : t.q_tiles;
    t.units = 3 * t.q_tiles * t.nks;
    t.live = tiles * t.nks;
    t.runs = stream_runs(t.units, stream_per_cu<BM, BN, NS>() * cus);
    auto kern = qkv_stream_kernel<BM, BN, NS, DT>;
    constexpr int lds = ring::lds_bytes<BM, BN, NS>();
    static_assert(lds <= 160 * 1024, "the workgroup must fit the LDS of a compute unit");
    static LdsOnce lds_once;
    e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds, lds_once);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(SPLIT * (run_of(t.live - 1, t.units, t.runs) + 1))), dim3(256), lds, s, t);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    FinishArgs f;
    f.part = part; f.bq = a.bq; f.bkv = a.bkv; f.q_out = a.q_out; f.K_dst = a.K_dst; f.V_dst = a.V_dst;
    f.B = a.B; f.d = a.d; f.n_heads = a.n_heads; f.head_dim = a.head_dim; f.L_cap = a.L_cap; f.tok_pos = a.tok_pos;
    f.q_tiles = t.q_tiles; f.nks = t.nks; f.units = t.units; f.runs = t.runs; f.split = SPLIT; f.pd = pd;
    hipLaunchKernelGGL((qkv_finish_kernel<BM, BN, DT>), dim3((unsigned)(SPLIT * tiles), BM / 32), dim3(256), 0, s, f);
    return hipGetLastError();
}

template <int BM, int BN, int NS, int SPLIT = 1>
hipError_t launch_any(const QkvArgs &a, int cus, hipStream_t s)
{
    return a.dtype == 1 ? launch_dt<BM, BN, NS, SPLIT, 1>(a, cus, s) : launch_dt<BM, BN, NS, SPLIT, 0>(a, cus, s);
}

}  // namespace

// Where the lines lie (measured, new weights in every call, replayed from a graph, us a call, one-launch kernel against
// this one, fp16 / bf16 where they differ).  Three launches cost 12 to 14 us however small the layer, so many rows and wide
// layers come here.
//   97 rows and more: every layer from d = 768 on: 25.0 / 28.1 against 15.1 (B = 128); 4096: 69 / 84 against 39; 7168:
//     116 / 141 against 91; 9216: 148 / 179 against 136; 9152 (units of 64 features): 148 against 149 / 181 against 150
//   65 to 96 rows: from d = 768 on: 18.8 / 20.9 against 13.5 (B = 65).  fp16 below 8448: 8192, B = 96: 118 against 108;
//     8256, B = 65: 114 against 107; 8448, B = 96: 111.7 against 116.6; 9216, B = 96: 118 against 127; 9152: 118 against
//     137.  bf16 everywhere: 9216, B = 96: 145 against 128
//   33 to 64 rows: from d = 2048 on: 20.6 / 23.7 against 18.0 (B = 33).  fp16 below 8192, where the one-launch kernel
//     changes to workgroups of 128 features: 8128, B = 64: 132 against 97; 8192, B = 33: 91 against 95 and 101 against 98
//     (two sessions); 8704: level.  bf16 below 8448: 8256, B = 64: 111 against 104; 8448: 101 against 103; 9152: 109
//     against 123; 9216: level
//   up to 32 rows: while the one-launch kernel's workgroups (64 features) fit 256 units at once it is level within 8 % or
//     faster: 4096, B = 32: 29.7 against 27.4; from 5504 on 60 against 39 (B = 1); 9216: 98 against 93 (B = 1), 105
//     against 94 (B = 32)
// Wider layers than 9216 stay with one launch.  A build without the limit gained on Q + K + V (10240: 0.81 to 1.10 of the
// one-launch kernel's time; 11264 and 12288, where that kernel's workgroups need a second round: 0.47 to 0.87; 16384: 0.60 to
// 0.97), but lost on Q alone from 11264 on (up to 1.07 there, 1.14 at 12288, 1.27 at 14336), and q must come from the same
// form in both: a rule for them needs the cut of Q alone to fill the chip first.
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
        case 1: return launch_any<32, 64, 6>(a, cus, s);
        case 2: return launch_any<64, 64, 5>(a, cus, s);
        case 3: return launch_any<96, 64, 4>(a, cus, s);
        default: return launch_any<128, 64, 3>(a, cus, s);
        }
    }
    switch ((a.B + 31) / 32) {
    case 1: {
        // Q alone occupies a third of the compute units, each of which waits for its own units: two workgroups a run then,
        // 64 features each, with a ring of more units.  The cut along the reduction, and with it the bits, is the same.
        // Q alone, B = 1 / 32, fp16: d = 7168: 40.8 / 44.3 -> 29.6 / 35.0 us (one-launch kernel: 36.6 / 41.0), 9216: 60.3 /
        // 65.7 -> 40.5 / 48.9 (46.5 / 53.8).  With more rows one workgroup a run is faster than the one-launch kernel too.
        static_assert(stream_per_cu<32, 128, 7>() == stream_per_cu<32, 64, 12>(), "the cut follows the workgroups of a compute unit");
        return a.K_dst ? launch_any<32, 128, 7>(a, cus, s) : launch_any<32, 64, 12, 2>(a, cus, s);
    }
    case 2: return launch_any<64, 128, 6>(a, cus, s);
    case 3: return launch_any<96, 128, 5>(a, cus, s);
    default: return launch_any<128, 128, 4>(a, cus, s);
    }
}

}  // namespace hk
