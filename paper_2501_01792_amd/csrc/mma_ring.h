// The main loop of the products whose two operands both stream through LDS (kv_gemm_tile.hip, qkv_stream.hip): a BM x BN
// output tile, 4 wavefronts, 2 x 2, (BM/2) x (BN/2) accumulators each in 16 x 16 x 32 MFMA blocks, and a ring of NS stages
// in LDS, each a "block" of 64 reduction elements of both operands.
//   * Loads go to LDS directly, 16 bytes per lane.  Load i of wavefront w fills LDS rows 8 (w + 4 i) .. + 7 of an operand;
//     lane l writes row l / 8, physical chunk l % 8, and fetches logical chunk (l % 8) ^ ((row / 2) % 8), so 8 lanes fetch
//     one 128-byte line and the fragment reads are free of bank conflicts.
//   * LDS row rho of the second operand (the weights) holds weight row (BN/2) (rho / (BN/2)) + TN c + j, with MFMA block j
//     and block column c of wavefront column rho / (BN/2), so that a lane ends up with TN consecutive features.
//   * Fragments are double-buffered in registers: the reads of a half block run under the MFMAs of the half before.  One
//     barrier per block, in its middle, where the next block must have landed and the slot of the current one, whose last
//     fragments are in registers, is free for block i + NS.
// Where the rows come from (buffers, clamping, cache policy) is the caller's business: it hands in `issue(slot, i)`, load i
// (0 .. kLoads - 1, weights first) of the block that is asked for next.
#pragma once
#include <hip/hip_runtime.h>

#include "elem.h"

namespace hk {
namespace ring {

constexpr int kBlockK = 64;                                 // reduction elements of a block: 128-byte LDS rows
constexpr int kRowBytes = kBlockK * 2;

typedef __attribute__((address_space(3))) void *lds_ptr_t;

template <int BM, int BN, int NS>
constexpr int lds_bytes() { return NS * (BM + BN) * kRowBytes; }

// Waits until at most r (<= R) of the youngest blocks this wavefront has asked for, LOADS loads each, are in flight (stores
// count too: the wait is then for more than it needs).
template <int R, int LOADS>
__device__ __forceinline__ void wait_blocks(int r)
{
    if constexpr (R > 0) {
        if (r < R) return wait_blocks<R - 1, LOADS>(r);
    }
    static_assert(R * LOADS <= 63, "vmcnt counts to 63");
    __builtin_amdgcn_s_waitcnt((R * LOADS & 15) | ((R * LOADS >> 4) << 14) | 0x0F70);   // vmcnt(R * LOADS)
}

template <int BM, int BN, int NS, int DT>
struct Ring {
    typedef typename Elem<DT>::V8 vec8_t;
    static constexpr int kLoadsA = BM / 32, kLoadsB = BN / 32, kLoads = kLoadsA + kLoadsB;   // direct loads of a lane per block
    static constexpr int TM = BM / 32, TN = BN / 32;        // MFMA blocks of a wavefront
    static constexpr int kStage = (BM + BN) * kRowBytes;

    unsigned char *smem;
    int wave, lane_row, lane_chunk, a_rd, b_rd, frag_off[2], cur;
    vec8_t fa[2][TM], fb[2][TN];
    float4_t acc[TM][TN];

    __device__ __forceinline__ Ring(unsigned char *lds, int tid, int wave_) : smem(lds), wave(wave_), cur(0)
    {
        const int lane = tid & 63;
        lane_row = 8 * wave + (lane >> 3);
        lane_chunk = (lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7);
        // fragment reads: row lane % 16 (+ 16 i) of the wavefront's part, logical chunk 4 ks + lane / 16
        const int fr = lane & 15, fc = lane >> 4;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) frag_off[ks] = fr * kRowBytes + (((4 * ks + fc) ^ ((fr >> 1) & 7)) << 4);
        a_rd = (wave >> 1) * (BM / 2) * kRowBytes;
        b_rd = BM * kRowBytes + (wave & 1) * (BN / 2) * kRowBytes;
    }
    // Row of the operand that this lane fetches with load i.
    __device__ __forceinline__ int a_row(int i) const { return lane_row + 32 * i; }
    __device__ __forceinline__ int b_row(int i) const
    {
        const int rho = lane_row + 32 * i, w = rho / (BN / 2), in = rho % (BN / 2);
        return w * (BN / 2) + TN * (in & 15) + (in >> 4);
    }
    // Where load i of an operand goes.
    __device__ __forceinline__ lds_ptr_t a_dst(int slot, int i) const { return (lds_ptr_t)(smem + slot * kStage + wave * 1024 + i * 4096); }
    __device__ __forceinline__ lds_ptr_t b_dst(int slot, int i) const
    {
        return (lds_ptr_t)(smem + slot * kStage + wave * 1024 + BM * kRowBytes + i * 4096);
    }
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void read_frag(int ks, int slot, int which)      // in the order the MFMAs need them: a[0], b[..], a[1..]
    {
        const unsigned char *src = smem + slot * kStage + frag_off[ks];
        if (which == 0 || which > TN) {
            const int i = which == 0 ? 0 : which - TN;
            fa[ks][i] = *reinterpret_cast<const vec8_t *>(src + a_rd + i * (16 * kRowBytes));
        } else {
            fb[ks][which - 1] = *reinterpret_cast<const vec8_t *>(src + b_rd + (which - 1) * (16 * kRowBytes));
        }
    }
    // The first n (all that there are, or NS) blocks have been asked for; the first lands and its first fragments are read.
    __device__ __forceinline__ void start(int n)
    {
        wait_blocks<NS - 1, kLoads>(n < NS ? n - 1 : NS - 1);
        asm volatile("s_barrier" ::: "memory");
#pragma unroll
        for (int q = 0; q < TM + TN; ++q) read_frag(0, 0, q);
    }
    // One block (KIND 0: the last; 1: a next one exists, and `younger` blocks behind that have been asked for; 2: NS - 2 have,
    // and issue() asks for one more).  Its first half multiplies fragments that are in registers already and reads those of
    // the second half; then this wavefront waits for its loads of the next block and meets the others, after which that
    // block is complete in LDS and the slot of the current one (every read of it has come back) is free; the second half
    // reads the first fragments of the next block.
    template <int KIND, typename Issue>
    __device__ __forceinline__ void block(Issue &&issue, int younger)
    {
        constexpr int kMma = TM * TN, kFrags = TM + TN;
        constexpr int kSlotsA = kMma > kFrags ? kMma : kFrags;
        constexpr int kSlotsB = kSlotsA > kLoads ? kSlotsA : kLoads;
        const int nxt = cur + 1 == NS ? 0 : cur + 1;
#pragma unroll
        for (int q = 0; q < kSlotsA; ++q) {
            if (q < kMma) acc[q / TN][q % TN] = Elem<DT>::mfma_16x16x32(fa[0][q / TN], fb[0][q % TN], acc[q / TN][q % TN]);
            if (q < kFrags) read_frag(1, cur, q);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (KIND == 2) wait_blocks<NS - 2, kLoads>(NS - 2);
        if constexpr (KIND == 1) wait_blocks<NS - 2, kLoads>(younger);
        if constexpr (KIND > 0) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < kSlotsB; ++q) {
            if (q < kMma) acc[q / TN][q % TN] = Elem<DT>::mfma_16x16x32(fa[1][q / TN], fb[1][q % TN], acc[q / TN][q % TN]);
            if (KIND > 0 && q < kFrags) read_frag(0, nxt, q);
            if (KIND == 2 && q < kLoads) issue(cur, q);
            __builtin_amdgcn_sched_barrier(0);
        }
        cur = nxt;
    }
};

}  // namespace ring
}  // namespace hk
