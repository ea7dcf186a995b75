// Grouped GEMM tile over a ring of 128-byte K slices in LDS, for either element size: a K slice
// is 128 bytes of every row of the tile (64 bf16 / float16 values or 32 float32 ones), fetched by
// global -> LDS loads that each cover 8 whole 128-byte rows, NS slices in the ring, one barrier
// per slice. LDS rows are 128 bytes with the 16-byte chunk c of row r at position
// c ^ ((r >> 1) & 7), which keeps the fragment reads (16 rows x 4 chunks) free of bank conflicts.
// Four such chunks of a row (64 bytes) feed one v_mfma_f32_16x16x32 (bf16, float16) or four
// v_mfma_f32_16x16x4 (float32: step j multiplies component j of each lane's chunk), K ascending
// over the chunks. Addresses are 64-bit per lane, so no operand size is out of reach.
#pragma once
#include "gemm_common.h"

namespace pcm {
namespace {

template <int BM_, int BN_, int WM_, int WN_, int NS_>
struct RCfg {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, NS = NS_;
    static constexpr int NW = WM * WN, NT = NW * 64;
    static constexpr int WTM = BM / WM, WTN = BN / WN, MB = WTM / 16, NBK = WTN / 16;
    static constexpr int QA = BM / 8 / NW, LPW = QA + BN / 8 / NW;   // loads per wave and slice
    static constexpr int SA = BM * 128, SLICE = SA + BN * 128, LDS_BYTES = NS * SLICE;
    static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "every wave issues the same loads");
    static_assert(WTM % 16 == 0 && WTN % 16 == 0, "whole MFMA blocks");
    static_assert(NS >= 2 && (NS - 2) * LPW <= 62 && LDS_BYTES <= 160 * 1024, "vmcnt range, LDS");
};

// A workgroup barrier that neither the compiler's nor its scheduler's reordering crosses.
__device__ __forceinline__ void ring_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// The accumulators of one wave over KT slices (waves 0 .. C::NW - 1 of the workgroup). src[q]: this
// lane's address of load q (A rows for q < QA, then B rows) in the first slice: row
// (q' * NW + wave) * 8 + lane / 8 of its part, chunk (lane % 8) ^ ((row >> 1) & 7). KT barriers.
// E: the element type (SIZE bytes, NJ MFMA steps per chunk, fragment reads, step).
// FOLD: the sums of every `fold` (>= 1) slices are added to a total instead of running on.
template <class E, class C, bool NT = false, bool FOLD = false>
__device__ __forceinline__ void ring_loop(const char* (&src)[C::LPW], int KT, char* lds,
                                          floatx4 (&acc)[C::NBK][C::MB], int fold = 0) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / C::WN, wn = wave % C::WN;
    auto issue = [&](int slot) {
#pragma unroll
        for (int q = 0; q < C::LPW; ++q) {
            const int blk = (q < C::QA ? q : q - C::QA) * C::NW + wave;
            if (q < C::QA)
                __builtin_amdgcn_global_load_lds((const PCM_GLOBAL void*)src[q],
                                                 (PCM_LDS void*)(lds + slot * C::SLICE + blk * 1024), 16, 0, 0);
            else
                __builtin_amdgcn_global_load_lds((const PCM_GLOBAL void*)src[q],
                                                 (PCM_LDS void*)(lds + slot * C::SLICE + C::SA + blk * 1024), 16, 0,
                                                 weight_policy(NT));
            src[q] += 128;
        }
    };
#pragma unroll
    for (int nb = 0; nb < C::NBK; ++nb)
#pragma unroll
        for (int mb = 0; mb < C::MB; ++mb) acc[nb][mb] = floatx4{0.f, 0.f, 0.f, 0.f};
    floatx4 total[C::NBK][C::MB];
    int left = fold;
    if constexpr (FOLD)
#pragma unroll
        for (int nb = 0; nb < C::NBK; ++nb)
#pragma unroll
            for (int mb = 0; mb < C::MB; ++mb) total[nb][mb] = acc[nb][mb];
    const int r16 = lane & 15, kg = lane >> 4;
#pragma unroll
    for (int s = 0; s < C::NS - 1; ++s)
        if (s < KT) issue(s);
    for (int base = 0; base < KT; base += C::NS) {
#pragma unroll
        for (int j = 0; j < C::NS; ++j) {
            const int kt = base + j;
            if (kt >= KT) break;
            // slice kt has landed (this wave's loads of it; the barrier covers the others'), and
            // every wave is done with slice kt - 1, whose slot takes slice kt + NS - 1
            if (kt + C::NS - 2 < KT) __builtin_amdgcn_s_waitcnt(waitcnt_imm((C::NS - 2) * C::LPW, 0));
            else __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
            ring_barrier();
            if (kt + C::NS - 1 < KT) issue((j + C::NS - 1) % C::NS);
            const char* S = lds + j * C::SLICE;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int off = r16 * 128 + (((4 * s + kg) ^ ((r16 >> 1) & 7)) * 16);
                typename E::T bf[C::NBK], af[C::MB];
#pragma unroll
                for (int nb = 0; nb < C::NBK; ++nb)
                    bf[nb] = E::weights(S + C::SA + (wn * C::WTN + nb * 16) * 128 + off);
#pragma unroll
                for (int mb = 0; mb < C::MB; ++mb) af[mb] = E::acts(S + (wm * C::WTM + mb * 16) * 128 + off);
#pragma unroll
                for (int st = 0; st < E::NJ; ++st)
#pragma unroll
                    for (int nb = 0; nb < C::NBK; ++nb)
#pragma unroll
                        for (int mb = 0; mb < C::MB; ++mb) acc[nb][mb] = E::step(st, bf[nb], af[mb], acc[nb][mb]);
            }
            if constexpr (FOLD)
                if (--left == 0) {   // uniform
                    left = fold;
#pragma unroll
                    for (int nb = 0; nb < C::NBK; ++nb)
#pragma unroll
                        for (int mb = 0; mb < C::MB; ++mb) {
                            total[nb][mb] += acc[nb][mb];
                            acc[nb][mb] = floatx4{0.f, 0.f, 0.f, 0.f};
                        }
                }
        }
    }
    if constexpr (FOLD)
#pragma unroll
        for (int nb = 0; nb < C::NBK; ++nb)
#pragma unroll
            for (int mb = 0; mb < C::MB; ++mb) acc[nb][mb] += total[nb][mb];
}

// One tile: rows [row0, row1) of group e, N tile ntile, K slice kslice of g.ksplit.
template <class E, class C, int MODE, bool NT>
__device__ __forceinline__ void ring_tile(const GemmArgs& g, char* lds, int e, int row0, int row1,
                                          int ntile, int kslice) {
    static_assert(C::WTN % 32 == 0, "gate/up halves");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = g.N;
    const int64_t rowb = (int64_t)g.K * E::SIZE;   // bytes of a row of either operand
    constexpr int kOutCols = (MODE == kExpand) ? C::BN / 2 : C::BN;
    const int KT = g.K / g.ksplit * E::SIZE / 128;
    const char* src[C::LPW];
    int64_t srow[C::QA];   // every row index is loaded before any is used
#pragma unroll
    for (int q = 0; q < C::QA; ++q)
        srow[q] = a_source_row(g, row0 + (q * C::NW + wave) * 8 + (lane >> 3), row1);
#pragma unroll
    for (int q = 0; q < C::LPW; ++q) {
        const int lr = ((q < C::QA ? q : q - C::QA) * C::NW + wave) * 8 + (lane >> 3);
        const int chunk = (lane & 7) ^ ((lr >> 1) & 7);
        const char* base;
        if (q < C::QA) {
            base = (const char*)g.a + srow[q < C::QA ? q : 0] * rowb;
        } else if (MODE == kExpand) {   // a wave's weight rows: half gate, half up of its columns
            const int grp = lr / C::WTN, jj = lr % C::WTN, half = jj / (C::WTN / 2);
            const int f = min(ntile * kOutCols + grp * (C::WTN / 2) + jj % (C::WTN / 2), N - 1);
            base = (const char*)(half ? g.b1 : g.b0) + ((int64_t)e * N + f) * rowb;
        } else {
            base = (const char*)g.b0 + ((int64_t)e * N + min(ntile * kOutCols + lr, N - 1)) * rowb;
        }
        src[q] = base + (int64_t)kslice * KT * 128 + chunk * 16;
    }
    floatx4 acc[C::NBK][C::MB];
    ring_loop<E, C, NT>(src, KT, lds, acc);
    GemmArgs gs = g;
    if (kslice) gs.out = (float*)g.out + (int64_t)kslice * g.rows_total * N;
    epilogue<MODE, C::MB, C::NBK, C::WTM, C::WTN, kOutCols, typename E::Silu>(gs, acc, row0, row1, ntile, wave / C::WN,
                                                                              wave % C::WN, lane);
}

// Workgroups walk the expert-major order of em_item with the window `window`. A group's last tile with
// at most CT::BM rows runs as the smaller tile CT (the same columns), sparing the loads of padding
// rows (bf16, one group of 150 rows, H 2048, F 5632: three kernels 47.2 -> 38.5 us; CT = C: none).
// once: weights_once.
template <class E, class C, class CT, int MODE>
__global__ __launch_bounds__(C::NT) void gemm_ring_kernel(GemmArgs g, int nt, int window, bool once) {
    static_assert(CT::NT == C::NT && CT::BN == C::BN && CT::BM <= C::BM && CT::LDS_BYTES <= C::LDS_BYTES, "tail tile");
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    int* const s_item = (int*)lds;   // read into registers before the first loads overwrite it
    if (!em_item<C::BM, C::BM>(g, nt, window, false, s_item)) return;   // workgroup-uniform
    const int e = s_item[0], row0 = s_item[1], row1 = s_item[2], ntile = s_item[3], kslice = s_item[4];
    __syncthreads();
    // the group's only row tile: its weights are read once (bf16 layers; float32 ones are small)
    const bool single = E::SIZE == 2 && once && g.offsets[e + 1] - g.offsets[e] <= C::BM;
    if (CT::BM < C::BM && row1 - row0 <= CT::BM) {
        if (single) ring_tile<E, CT, MODE, E::SIZE == 2>(g, lds, e, row0, row1, ntile, kslice);
        else ring_tile<E, CT, MODE, false>(g, lds, e, row0, row1, ntile, kslice);
    } else {
        if (single) ring_tile<E, C, MODE, E::SIZE == 2>(g, lds, e, row0, row1, ntile, kslice);
        else ring_tile<E, C, MODE, false>(g, lds, e, row0, row1, ntile, kslice);
    }
}

template <class E, class C, class CT, int MODE>
hipError_t launch_ring(const GemmArgs& g, int64_t R, hipStream_t s, int window) {
    const int64_t mt_upper = most_tiles(g, R, C::BM);
    const int nt = (int)ceil_div(g.N, MODE == kExpand ? C::BN / 2 : C::BN);
    const int64_t grid = ceil_div(mt_upper * nt * g.ksplit, 8) * 8;
    if (grid <= 0) return hipSuccess;
    // em_item counts in 32 bits, up to 8 times the items. (No call that fits the card comes near: as many
    // tiles of at least 32 x 32 outputs are 550 GB of output, or, as tails, 2 TB of weights.)
    if (grid >= int64_t(1) << 27) return hipErrorInvalidValue;
    // set on every launch (idempotent, and the library keeps no state between calls)
    const hipError_t err = hipFuncSetAttribute((const void*)gemm_ring_kernel<E, C, CT, MODE>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES);
    if (err != hipSuccess) return err;
    gemm_ring_kernel<E, C, CT, MODE><<<dim3((unsigned)grid), dim3(C::NT), C::LDS_BYTES, s>>>(g, nt, window,
        weights_once(g, R, MODE));
    return hipGetLastError();
}

}  // namespace
}  // namespace pcm
