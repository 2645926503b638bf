// "KV Gen" (Sec. 4.2.2; Eq. 7) for gfx950 on a prepared layer, for problems with too few 256 x 256 output tiles to
// keep every compute unit busy with one (kv_gemm_fold.hip): the same folded LayerNorm,
//     [K V][m, n] = rstd_m (x_m . W'[n,:]) + nmr_m c[n] + b'[n],
// with the same products in the same order (the results are the same bits whatever the tile), on smaller tiles.
//
// What bounds it: with a few hundred tokens the weights (4 d^2 bytes) and the matrix cores would allow 10 to 50 us at
// d = 4096, but a 256 x 256 tile has only 2 k blocks in flight per compute unit and takes 1.2 us for each of them
// however many of its rows are real, and 32 to 128 of such tiles leave most of the chip idle.  So: smaller tiles until
// every compute unit has one, and a ring of k blocks as deep as the LDS allows.
//   * The main loop is that of mma_ring.h: a k block (64 reduction elements) of both operands is one stage of an LDS ring
//     of NS stages filled by direct loads, all NS asked for before the first is used.
//   * Tiles are walked column panel by column panel over up to 8 row tiles inside an XCD: a weight panel leaves HBM once.
// Measured with its row statistics, fp16 (profiles/kv_gemm_tile_forms.txt; in brackets the 128 x 128 kernel with the LayerNorm
// prologue / the 256 x 256 kernel): d = 4096, M = 64: 18.6 us (73 / 71); M = 512: 42 (76 / 73); M = 1024: 67 (102 / 74);
// d = 9216, M = 8: 72 (201 / 154); M = 256: 147 (210 / 163); d = 768, M = 512: 8.8 (21 / 22).
#include "hk_internal.h"
#include "elem.h"
#include "kv_gemm_common.h"
#include "kv_gemm_forms.h"
#include "mma_ring.h"

namespace hk {
namespace {

using namespace gemm;

template <int BM, int BN, int NS>
constexpr int tile_lds_bytes() { return ring::lds_bytes<BM, BN, NS>() + BM * (int)sizeof(RowDst); }

// REST: rows from m_begin on, the second launch of a problem.  The first has code of its own: with the begin as a plain argument
// the way to its first load was some hundred nanoseconds longer (d = 768, 8 rows with their statistics: 7.54 -> 7.75 us, d = 4096, 100
// rows: 18.6 -> 19.25).
template <int BM, int BN, int NS, int DT, bool REST>
__global__ __launch_bounds__(256, BM * BN <= 128 * 128 ? 2 : 1) void kv_gemm_tile_kernel(
    const typename Elem<DT>::T *__restrict__ act, const float2 *__restrict__ stats,
    const typename Elem<DT>::T *__restrict__ Wp, const float *__restrict__ cvec, const float *__restrict__ bvec,
    typename Elem<DT>::T *__restrict__ K_out, typename Elem<DT>::T *__restrict__ V_out,
    int64_t M, int d, int n_heads, int head_dim, int L_act, int L_cap, int tok_off, int tiles_m, int tiles_n, int64_t m_begin)
{
#if defined(__HIP_DEVICE_COMPILE__)                            // (the host pass drops the kernel's stub over a direct load in this body)
    typedef typename Elem<DT>::T elem_t;
    typedef ring::Ring<BM, BN, NS, DT> ring_t;
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int LA = ring_t::kLoadsA, LB = ring_t::kLoadsB, TM = ring_t::TM, TN = ring_t::TN;
    const int N = 2 * d;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int nks = d / ring::kBlockK;

    int tm, tn;
    tile_coords<8>((int)blockIdx.x, tiles_m, tiles_n, tm, tn);
    const int64_t m0 = (REST ? m_begin : 0) + (int64_t)tm * BM;
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

    // ---- direct loads; rows past the end are clamped to the last one
    ring_t r(smem, tid, wave);
    int64_t a_bytes = (M - m0) * (int64_t)d * 2, b_bytes = ((int64_t)N - n0) * d * 2;
    if (a_bytes > 0x7fffffff) a_bytes = 0x7fffffff;            // a tile spans < 2^30 bytes
    if (b_bytes > 0x7fffffff) b_bytes = 0x7fffffff;
    const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<elem_t *>(act + m0 * (int64_t)d), 0, (int)a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t b_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<elem_t *>(Wp + (int64_t)n0 * d), 0, (int)b_bytes, 0x00020000);
    const int ra = M - m0 < BM ? (int)(M - m0) - 1 : BM - 1;
    const int rb = N - n0 < BN ? N - n0 - 1 : BN - 1;
    int a_voff[LA], b_voff[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i) a_voff[i] = ((r.a_row(i) < ra ? r.a_row(i) : ra) * d + r.lane_chunk * 8) * 2;
#pragma unroll
    for (int i = 0; i < LB; ++i) b_voff[i] = ((r.b_row(i) < rb ? r.b_row(i) : rb) * d + r.lane_chunk * 8) * 2;
    auto issue = [&](int slot, int kb, int i) {
        // weights first: they come from HBM, the activations mostly from L2
        if (i < LB)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(b_rsrc, r.b_dst(slot, i), 16, b_voff[i], kb * ring::kRowBytes, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, r.a_dst(slot, i - LB), 16, a_voff[i - LB], kb * ring::kRowBytes, 0, 0);
    };

    r.clear();
    for (int s = 0; s < NS; ++s) {
        if (s < nks) {
#pragma unroll
            for (int i = 0; i < ring_t::kLoads; ++i) issue(s, s, i);
        }
    }
    r.start(nks);
    int kb = 0;
    auto next = [&](int slot, int i) { issue(slot, kb + NS, i); };
    for (; kb + NS < nks; ++kb) r.template block<2>(next, 0);
    for (; kb + 1 < nks; ++kb) r.template block<1>(next, nks - 2 - kb);
    r.template block<0>(next, 0);

    // ---- statistics, constants of the layer, 16-bit rounding, head split.  Rows past the last token stand for it (their
    // operand loads were clamped to its row): they store the same bytes to the same place.
    RowDst *tab = reinterpret_cast<RowDst *>(smem + NS * ring_t::kStage);
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
        for (int e4 = 0; e4 < 4; ++e4) {
            const RowDst row = my[16 * i + e4];
            out_t v;
#pragma unroll
            for (int j = 0; j < TN; ++j)
                v[j] = __builtin_bit_cast(unsigned short, (elem_t)__builtin_fmaf(r.acc[i][j][e4], row.rstd, __builtin_fmaf(row.nmr, cn[j], bn[j])));
            __builtin_nontemporal_store(v, reinterpret_cast<out_t *>(dst_base + row.base));
        }
#endif
}

template <int BM, int BN, int NS, int DT, bool REST>
hipError_t launch_tile_dt(const KvGemmArgs &a, hipStream_t s)
{
    typedef typename Elem<DT>::T elem_t;
    const int64_t tiles_m = (a.M - a.m_begin + BM - 1) / BM;
    const int tiles_n = (2 * a.d + BN - 1) / BN;
    if (tiles_m * tiles_n > 0x7fffffffLL) return hipErrorInvalidValue;
    auto kern = kv_gemm_tile_kernel<BM, BN, NS, DT, REST>;
    constexpr int lds = tile_lds_bytes<BM, BN, NS>();
    static_assert(lds <= 160 * 1024, "the workgroup must fit the LDS of a compute unit");
    static LdsOnce lds_once;
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds, lds_once);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n)), dim3(256), lds, s,
                       static_cast<const elem_t *>(a.act), a.stats, static_cast<const elem_t *>(a.Wp), a.cvec, a.bvec,
                       static_cast<elem_t *>(a.K_out), static_cast<elem_t *>(a.V_out),
                       a.M, a.d, a.n_heads, a.head_dim, a.L_act, a.L_cap, a.tok_off, (int)tiles_m, tiles_n, a.m_begin);
    return hipGetLastError();
}

template <int BM, int BN, int NS>
hipError_t launch_tile_any(const KvGemmArgs &a, hipStream_t s)
{
    if (a.m_begin > 0) return a.dtype == 1 ? launch_tile_dt<BM, BN, NS, 1, true>(a, s) : launch_tile_dt<BM, BN, NS, 0, true>(a, s);
    return a.dtype == 1 ? launch_tile_dt<BM, BN, NS, 1, false>(a, s) : launch_tile_dt<BM, BN, NS, 0, false>(a, s);
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
    if (a.m_begin < 0 || a.M <= a.m_begin || (form == 0 && a.m_begin != 0) || a.d % ring::kBlockK != 0 || form < 0 || form >= forms::kCount)
        return hipErrorInvalidValue;
    return kLaunch[form](a, s);
}

hipError_t launch_kv_gemm_prepared(const KvGemmArgs &a, hipStream_t s)
{
    int dev = 0, cus = 0;
    const hipError_t e = current_device_cus(&dev, &cus);
    if (e != hipSuccess) return e;
    const forms::Plan p = forms::plan(a.M, a.d, cus, a.cu_limit);
    KvGemmArgs part = a;
    part.M = p.rows;
    const hipError_t first = launch_kv_gemm_form(part, p.form, s);
    if (first != hipSuccess || p.rows == a.M) return first;
    part.m_begin = p.rows;
    part.M = a.M;
    return launch_kv_gemm_form(part, p.rest_form, s);
}

}  // namespace hk
