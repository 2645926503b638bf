// "KV Gen" (Sec. 4.2.2; Eq. 7) for gfx950 on a prepared layer, for problems with too few 256 x 256 output tiles to
// keep every compute unit busy with one (kv_gemm_fold.hip): the same folded LayerNorm,
//     [K V][m, n] = rstd_m (x_m . W'[n,:]) + nmr_m c[n] + b'[n],
// with the same products in the same order (the results are the same bits whatever the tile), on smaller tiles.
//
// What bounds it: with a few hundred tokens the weights (4 d^2 bytes) and the matrix cores would allow 10 to 50 us at
// d = 4096, but a 256 x 256 tile has only 2 k blocks in flight per compute unit and takes 1.2 us for each of them
// however many of its rows are real, and 32 to 128 of such tiles leave most of the chip idle.  So: smaller tiles until
// every compute unit has one, and a ring of k blocks as deep as the LDS allows.
//   * 4 wavefronts, 2 x 2, (BM/2) x (BN/2) accumulators each in 16 x 16 x 32 MFMA blocks; one workgroup per tile.
//   * A k block (64 reduction elements) of both operands is one stage of an LDS ring of NS stages, filled by direct
//     loads (16 bytes per lane, 8 lanes per 128-byte line, XOR swizzle of the chunk index applied on the global side).
//     All NS stages are asked for before the first is used.
//   * Fragments are double-buffered in registers: the reads of a half k block run under the MFMAs of the half before.
//     One barrier per k block, in its middle, where the next block must have landed and the slot of the current one,
//     whose last fragments are in registers, is free for block kb + NS.
//   * Tiles are walked column panel by column panel over up to 8 row tiles inside an XCD: a weight panel leaves HBM once.
// Measured with its row statistics (ln_stats, 4 to 6 us of it), fp16, against the 128 x 128 kernel with the LayerNorm
// prologue / the 256 x 256 kernel: d = 4096, M = 64: 24.6 us (93.6 / 75.3); M = 512: 45.6 (93.9 / 79.1); M = 1024: 67.5
// (112 / 86.2); d = 9216, M = 8: 77 (201 / 156); M = 256: 144 (214 / 168); d = 768, M = 512: 9.4 (22.8 / 23.0).
#include "hk_internal.h"
#include "elem.h"
#include "kv_gemm_common.h"
#include "kv_gemm_forms.h"

#include <type_traits>

namespace hk {
namespace {

using namespace gemm;

constexpr int kTileBK = 64;                                 // reduction elements of a k block: 128-byte LDS rows
constexpr int kTileRow = kTileBK * 2;

typedef __attribute__((address_space(3))) void *lds_ptr_t;

template <int BM, int BN, int NS>
constexpr int tile_lds_bytes() { return NS * (BM + BN) * kTileRow + BM * (int)sizeof(RowDst); }

// Waits until at most r (<= R) of the youngest k blocks this wavefront has asked for, LPS loads each, are in flight.
template <int R, int LPS>
__device__ __forceinline__ void wait_blocks(int r)
{
    if constexpr (R > 0) {
        if (r < R) return wait_blocks<R - 1, LPS>(r);
    }
    static_assert(R * LPS <= 63, "vmcnt counts to 63");
    __builtin_amdgcn_s_waitcnt((R * LPS & 15) | ((R * LPS >> 4) << 14) | 0x0F70);   // vmcnt(R * LPS)
}

template <int BM, int BN, int NS, int DT>
__global__ __launch_bounds__(256, BM * BN <= 128 * 128 ? 2 : 1) void kv_gemm_tile_kernel(
    const typename Elem<DT>::T *__restrict__ act, const float2 *__restrict__ stats,
    const typename Elem<DT>::T *__restrict__ Wp, const float *__restrict__ cvec, const float *__restrict__ bvec,
    typename Elem<DT>::T *__restrict__ K_out, typename Elem<DT>::T *__restrict__ V_out,
    int64_t M, int d, int n_heads, int head_dim, int L_act, int L_cap, int tok_off, int tiles_m, int tiles_n)
{
#if defined(__HIP_DEVICE_COMPILE__)                            // (the host pass drops the kernel's stub over a direct load in this body)
    typedef typename Elem<DT>::T elem_t;
    typedef typename Elem<DT>::V8 vec8_t;
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int LA = BM / 32, LB = BN / 32, LPS = LA + LB;   // direct loads of a lane per k block
    constexpr int TM = BM / 32, TN = BN / 32;                  // 16 x 16 MFMA blocks of a wavefront (2 x 2 wavefronts)
    constexpr int kStage = (BM + BN) * kTileRow;
    const int N = 2 * d;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int nks = d / kTileBK;

    int tm, tn;
    tile_coords<8>((int)blockIdx.x, tiles_m, tiles_n, tm, tn);
    const int64_t m0 = (int64_t)tm * BM;
    const int n0 = tn * BN;

    // ---- what the epilogue needs from memory, asked for first
    RowDst my_row;
    {
        const int64_t m = m0 + tid < M ? m0 + tid : M - 1;     // rows past the end: see the epilogue
        if (tid < BM) my_row = row_dst(m, M, n_heads, head_dim, L_act, L_cap, tok_off, stats);
    }
    const int nb = n0 + wn * (BN / 2) + TN * (lane & 15);      // first of this lane's TN output features
    float cn[TN], bn[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        cn[j] = nb < N ? cvec[nb + j] : 0.f;
        bn[j] = nb < N ? bvec[nb + j] : 0.f;
    }

    // ---- direct loads: load i of wavefront w fills LDS rows 8 (w + 4 i) .. + 7 of a unit; lane l writes row l / 8,
    // physical chunk l % 8, and fetches logical chunk (l % 8) ^ ((row / 2) % 8), so 8 lanes fetch one 128-byte line
    const int l_row = 8 * wave + (lane >> 3);
    const int l_chunk = (lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7);
    int64_t a_bytes = (M - m0) * (int64_t)d * 2, b_bytes = ((int64_t)N - n0) * d * 2;
    if (a_bytes > 0x7fffffff) a_bytes = 0x7fffffff;            // a tile spans < 2^30 bytes
    if (b_bytes > 0x7fffffff) b_bytes = 0x7fffffff;
    const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<elem_t *>(act + m0 * (int64_t)d), 0, (int)a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t b_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<elem_t *>(Wp + (int64_t)n0 * d), 0, (int)b_bytes, 0x00020000);
    const int ra = M - m0 < BM ? (int)(M - m0) - 1 : BM - 1;
    const int rb = N - n0 < BN ? N - n0 - 1 : BN - 1;
    int a_voff[LA], b_voff[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int r = l_row + 32 * i;
        a_voff[i] = ((r < ra ? r : ra) * d + l_chunk * 8) * 2;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        // LDS row rho of the weight unit: wavefront column rho / (BN/2), MFMA block j, block column c; it holds weight
        // row (BN/2) (rho / (BN/2)) + TN c + j, so that a lane ends up with TN consecutive features
        const int rho = l_row + 32 * i;
        const int w = rho / (BN / 2), in = rho % (BN / 2);
        const int r = w * (BN / 2) + TN * (in & 15) + (in >> 4);
        b_voff[i] = ((r < rb ? r : rb) * d + l_chunk * 8) * 2;
    }
    auto issue = [&](int slot, int kb, int i) {
        unsigned char *dst = smem + slot * kStage + wave * 1024;
        // weights first: they come from HBM, the activations mostly from L2
        if (i < LB)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(b_rsrc, (lds_ptr_t)(dst + BM * kTileRow + i * 4096), 16, b_voff[i], kb * kTileRow, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_ptr_t)(dst + (i - LB) * 4096), 16, a_voff[i - LB], kb * kTileRow, 0, 0);
    };

    // ---- fragment reads: row lane % 16 (+ 16 i) of the wavefront's part, logical chunk 4 ks + lane / 16
    const int fr = lane & 15, fc = lane >> 4;
    int frag_off[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) frag_off[ks] = fr * kTileRow + (((4 * ks + fc) ^ ((fr >> 1) & 7)) << 4);
    const int a_rd = wm * (BM / 2) * kTileRow, b_rd = BM * kTileRow + wn * (BN / 2) * kTileRow;
    vec8_t fa[2][TM], fb[2][TN];
    auto read_frag = [&](int ks, int slot, int which) {        // in the order the MFMAs need them: a[0], b[..], a[1..]
        const unsigned char *src = smem + slot * kStage + frag_off[ks];
        if (which == 0 || which > TN) {
            const int i = which == 0 ? 0 : which - TN;
            fa[ks][i] = *reinterpret_cast<const vec8_t *>(src + a_rd + i * (16 * kTileRow));
        } else {
            fb[ks][which - 1] = *reinterpret_cast<const vec8_t *>(src + b_rd + (which - 1) * (16 * kTileRow));
        }
    };

    float4_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};

    for (int s = 0; s < NS; ++s) {
        if (s < nks) {
#pragma unroll
            for (int i = 0; i < LPS; ++i) issue(s, s, i);
        }
    }
    wait_blocks<NS - 1, LPS>(nks < NS ? nks - 1 : NS - 1);
    asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int q = 0; q < TM + TN; ++q) read_frag(0, 0, q);

    constexpr int kMma = TM * TN, kFrags = TM + TN;
    constexpr int kSlotsA = kMma > kFrags ? kMma : kFrags;
    constexpr int kSlotsB = kSlotsA > LPS ? kSlotsA : LPS;
    int cur = 0;
    // One k block (kind 0: last; 1: a next block exists; 2: and block kb + NS exists).  Its first half multiplies
    // fragments that are in registers already and reads those of the second half; then this wavefront waits for its
    // loads of block kb + 1 and meets the others, after which block kb + 1 is complete in LDS and block kb's slot
    // (every read of it has come back) takes block kb + NS; the second half reads the first fragments of block kb + 1.
    auto block = [&](auto kind, int kb) {
        constexpr int KIND = decltype(kind)::value;
        const int nxt = cur + 1 == NS ? 0 : cur + 1;
#pragma unroll
        for (int q = 0; q < kSlotsA; ++q) {
            if (q < kMma) acc[q / TN][q % TN] = Elem<DT>::mfma_16x16x32(fa[0][q / TN], fb[0][q % TN], acc[q / TN][q % TN]);
            if (q < kFrags) read_frag(1, cur, q);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (KIND == 2) wait_blocks<NS - 2, LPS>(NS - 2);
        if constexpr (KIND == 1) wait_blocks<NS - 2, LPS>(nks - 2 - kb);
        if constexpr (KIND > 0) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < kSlotsB; ++q) {
            if (q < kMma) acc[q / TN][q % TN] = Elem<DT>::mfma_16x16x32(fa[1][q / TN], fb[1][q % TN], acc[q / TN][q % TN]);
            if (KIND > 0 && q < kFrags) read_frag(0, nxt, q);
            if (KIND == 2 && q < LPS) issue(cur, kb + NS, q);
            __builtin_amdgcn_sched_barrier(0);
        }
        cur = nxt;
    };
    int kb = 0;
    for (; kb + NS < nks; ++kb) block(std::integral_constant<int, 2>{}, kb);
    for (; kb + 1 < nks; ++kb) block(std::integral_constant<int, 1>{}, kb);
    block(std::integral_constant<int, 0>{}, kb);

    // ---- statistics, constants of the layer, 16-bit rounding, head split.  Rows past the last token stand for it (their
    // operand loads were clamped to its row): they store the same bytes to the same place.
    RowDst *tab = reinterpret_cast<RowDst *>(smem + NS * kStage);
    if (tid < BM) tab[tid] = my_row;
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (nb >= N) return;
    const bool is_v = nb >= d;
    const int nn = is_v ? nb - d : nb;
    const int h = nn / head_dim, e = nn % head_dim;
    elem_t *dst_base = (is_v ? V_out : K_out) + ((int64_t)h * L_cap * head_dim + e);
    const RowDst *my = tab + wm * (BM / 2) + 4 * (lane >> 4);
    typedef unsigned short out_t __attribute__((ext_vector_type(TN)));     // the TN stored elements, whatever their type
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const RowDst row = my[16 * i + r];
            out_t v;
#pragma unroll
            for (int j = 0; j < TN; ++j)
                v[j] = __builtin_bit_cast(unsigned short, (elem_t)__builtin_fmaf(acc[i][j][r], row.rstd, __builtin_fmaf(row.nmr, cn[j], bn[j])));
            __builtin_nontemporal_store(v, reinterpret_cast<out_t *>(dst_base + row.base));
        }
#endif
}

template <int BM, int BN, int NS, int DT>
hipError_t launch_tile_dt(const KvGemmArgs &a, hipStream_t s)
{
    typedef typename Elem<DT>::T elem_t;
    const int64_t tiles_m = (a.M + BM - 1) / BM;
    const int tiles_n = (2 * a.d + BN - 1) / BN;
    if (tiles_m * tiles_n > 0x7fffffffLL) return hipErrorInvalidValue;
    auto kern = kv_gemm_tile_kernel<BM, BN, NS, DT>;
    constexpr int lds = tile_lds_bytes<BM, BN, NS>();
    static_assert(lds <= 160 * 1024, "the workgroup must fit the LDS of a compute unit");
    static LdsOnce lds_once;
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds, lds_once);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n)), dim3(256), lds, s,
                       static_cast<const elem_t *>(a.act), a.stats, static_cast<const elem_t *>(a.Wp), a.cvec, a.bvec,
                       static_cast<elem_t *>(a.K_out), static_cast<elem_t *>(a.V_out),
                       a.M, a.d, a.n_heads, a.head_dim, a.L_act, a.L_cap, a.tok_off, (int)tiles_m, tiles_n);
    return hipGetLastError();
}

template <int BM, int BN, int NS>
hipError_t launch_tile_any(const KvGemmArgs &a, hipStream_t s)
{
    return a.dtype == 1 ? launch_tile_dt<BM, BN, NS, 1>(a, s) : launch_tile_dt<BM, BN, NS, 0>(a, s);
}

// The kernels of forms::kForms, in its order.
hipError_t (*const kLaunch[])(const KvGemmArgs &, hipStream_t) = {
    launch_kv_gemm_fold,
    launch_tile_any<256, 128, 3>,
    launch_tile_any<128, 256, 3>,
    launch_tile_any<192, 128, 3>,
    launch_tile_any<128, 128, 4>,
    launch_tile_any<128, 64, 3>,
    launch_tile_any<64, 128, 3>,
    launch_tile_any<64, 64, 4>,
    launch_tile_any<64, 32, 6>,
    launch_tile_any<32, 64, 6>,
    launch_tile_any<32, 32, 9>,
};
static_assert(sizeof(kLaunch) / sizeof(kLaunch[0]) == forms::kCount, "one kernel per form");

}  // namespace

hipError_t launch_kv_gemm_form(const KvGemmArgs &a, int form, hipStream_t s)
{
    if (a.M <= 0 || a.d % kTileBK != 0 || form < 0 || form >= forms::kCount) return hipErrorInvalidValue;
    return kLaunch[form](a, s);
}

hipError_t launch_kv_gemm_prepared(const KvGemmArgs &a, hipStream_t s)
{
    int dev = 0, cus = 0;
    const hipError_t e = current_device_cus(&dev, &cus);
    if (e != hipSuccess) return e;
    return launch_kv_gemm_form(a, forms::pick(a.M, a.d, cus), s);
}

}  // namespace hk
