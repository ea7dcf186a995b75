// Grouped bf16 GEMMs on the gfx950 matrix cores (v_mfma_f32_16x16x32_bf16, float32
// accumulate) for the two sides of a SwiGLU expert (Section 4.1):
//   expand:  U[r, f] = SiLU(x[tok(r)] . W_gate[e][f]) * (x[tok(r)] . W_up[e][f])
//            one row per (token, source) pair, rows of expert e contiguous (Section 4.3),
//            x rows gathered through row_token; SwiGLU fused into the epilogue; U kept in
//            float32. bf16 x bf16 MFMA (v_mfma_f32_16x16x32_bf16).
//   down:    O[r, h] = row_scale[r'] * (Z[r'] . W_down[e][h]), r' = gather[r] or r
//                                                  (store, or accumulate into y
//                                                  for a dense FFN whose rows are tokens)
//            Z arrives as row-scaled float16; each bf16 W_down fragment is widened to
//            float16 in registers after its LDS read (exact in float16's normal range), and
//            the product runs on v_mfma_f32_16x16x32_f16 at the same rate.
// Both operands are K-contiguous (x rows and W rows run along H; Z rows and W_down rows
// along F), so a lane's 8 consecutive K values of a row are one 16-byte load.
//
// Four kernel shapes share the epilogue and the work decomposition (pick_tile, pick_shape):
//  * "interleaved" (large tiles, 256 x 256): four waves, one per SIMD, each owning a 128 x 128
//    block of C in 256 accumulation registers, or eight waves, two per SIMD, each owning a
//    128 x 64 block in 128 (the expansion's default: while one wave of a SIMD waits, the other
//    can issue MFMAs; same loads, same bits). Global -> LDS direct buffer loads
//    (buffer_load_dwordx4 ... lds, no register staging: one 32-bit offset per lane for the
//    whole tile, the stage's K offset in a scalar register) of 64-wide K stages, two stages
//    of A and three of B (the weights, mostly fetched from HBM, get two stages of latency
//    budget, the activations one), each load covering 8 whole 128-byte rows; one workgroup
//    barrier per 32-wide substep,
//    within which each wave issues its 64 MFMAs interleaved with the fragment reads of the
//    next substep (and, once per stage, the loads of A two stages and of B three stages
//    ahead). LDS rows are
//    128 bytes; the 16-byte chunk c of row r sits at position c ^ ((r >> 1) & 7), which
//    keeps the fragment reads (16 rows x 4 chunks per instruction) free of bank conflicts.
//    A group's last tile with at most 128 rows runs as a 128 x 256 tile (64 x 128 per wave)
//    in the same launch.
//  * "staged" (medium tiles): loads through registers into two LDS stages of 64-wide K
//    steps; rows of 128 bytes with chunk c of row r at position c ^ ((r >> 1) & 7). Runs
//    only where the large tiles' 32-bit buffer offsets would not reach.
//  * "stream" (fewer than 16 rows per group, decode): each wave streams its 32 weight rows
//    and its activation block through a ring of its own in LDS (no barrier), every direct
//    load covering whole 128-byte lines; the weights are the traffic. A register-ring
//    variant (fragments loaded straight into registers several k-steps ahead) runs where
//    the ring's 32-bit offsets would not reach. Where K is long, the four waves of a workgroup
//    share its slices over the same weight rows (LStream).
//  * "ring" (gemm_ring.h: 64 x 128 and 64 x 64 tiles, several workgroups on a compute unit): few
//    rows per group, and products whose large tiles would leave most of the chip idle.
// The MFMA takes the weight fragment as its first operand, so each lane's four
// accumulators are four consecutive output columns of one row (16-byte stores). For the
// expansion, a wave's weight rows are half gate and half up for the same columns, so the
// gate and up values of an output element sit in the same lane and register slot.
//
// Work decomposition: the grid is (upper bound of M tiles) x (N tiles) (x K slices). Each
// workgroup finds its group (expert) and row range from the group offsets with one wave-wide
// scan of per-group tile counts; workgroups past the last tile exit. Every order is
// XCD-aware (workgroup ids are dispatched round-robin over the 8 XCDs). Grouped rows of the
// large tiles walk an expert-major order (em_item: all row blocks of one expert for a few
// N tiles at a time, so a weight tile is fetched while every row block that needs it runs);
// a K-split projection lists each XCD's full-height tiles before its 128-row tail tiles
// (il_item); one group of rows (the dense shared expert) and the medium tiles use the
// grouped order of tile_of.
#include <type_traits>

#include "gemm_ring.h"

namespace pcm {
namespace {

// Find this workgroup's group and row range (s_tile: group, row0, row1, rows of the group). Returns
// false past the last tile.
template <int BM>
__device__ bool find_tile(const int32_t* __restrict__ offsets, int n, int64_t a_rows, int64_t mt,
                          int* s_tile) {
    if (offsets == nullptr) {  // one group: rows [0, a_rows)
        if (mt * BM >= a_rows) return false;
        s_tile[0] = 0;
        s_tile[1] = (int)(mt * BM);
        s_tile[2] = (int)min<int64_t>(a_rows, (mt + 1) * BM);
        s_tile[3] = (int)a_rows;
        return true;
    }
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        if (lane == 0) s_tile[0] = -1;
        int lo[4], rows[4], cnt[4], local = 0;
        group_bounds(offsets, n, a_rows, lane, lo, rows);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            cnt[j] = (rows[j] + BM - 1) / BM;
            local += cnt[j];
        }
        const int incl = wave_incl_scan_i32(local);
        int start = incl - local;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (mt >= start && mt < start + cnt[j]) {
                const int x = lane * 4 + j;
                const int r0 = lo[j] + (int)(mt - start) * BM;
                s_tile[0] = x;
                s_tile[1] = r0;
                s_tile[2] = min(lo[j] + rows[j], r0 + BM);
                s_tile[3] = rows[j];
            }
            start += cnt[j];
        }
    }
    __syncthreads();
    return s_tile[0] >= 0;
}

// Tile of workgroup `bid` in a grid of `grid` (a multiple of 8) workgroups.
// Workgroups are dispatched round-robin over the 8 XCDs (bid % 8), so ids are first
// remapped to make each XCD's share a contiguous run. That run is walked in groups of GN
// N-tiles: inside a group the M-tile varies slowest, so the workgroups resident on one XCD
// at a time share a few weight tiles (same expert, neighbouring M-tiles) and a few
// activation tiles (same M-tile, neighbouring N-tiles) through that XCD's L2.
__device__ inline void tile_from_id(int64_t id, int64_t mt_count, int nt, int GN, int64_t* mt,
                                    int* ntile) {
    const int64_t gsize = (int64_t)GN * mt_count;
    const int64_t grp = id / gsize, in = id % gsize;
    const int64_t gn = min<int64_t>(GN, nt - grp * GN);
    *mt = in / gn;
    *ntile = (int)(grp * GN + in % gn);
}
__device__ inline bool tile_of(int64_t bid, int64_t grid, int64_t mt_upper, int nt, int GN,
                               int64_t* mt, int* ntile) {
    const int64_t id = (bid % 8) * (grid / 8) + bid / 8;
    if (id >= mt_upper * nt) return false;
    tile_from_id(id, mt_upper, nt, GN, mt, ntile);
    return true;
}

// Weight row (element offset of its K = 0) of B row j of the tile; rows past N repeat row
// N - 1 (their outputs are never stored).
template <int MODE, int WTN, int OUT_COLS>
__device__ inline const uint16_t* b_source_row(const GemmArgs& g, int e, int ntile, int j) {
    if (MODE == kExpand) {
        const int grp = j / WTN, jj = j % WTN, half = jj / (WTN / 2);
        int f = ntile * OUT_COLS + grp * (WTN / 2) + jj % (WTN / 2);
        f = f < g.N ? f : g.N - 1;
        return (const uint16_t*)(half ? g.b1 : g.b0) + ((int64_t)e * g.N + f) * g.K;
    }
    int h = ntile * OUT_COLS + j;
    h = h < g.N ? h : g.N - 1;
    return (const uint16_t*)g.b0 + ((int64_t)e * g.N + h) * g.K;
}

// Weight row (within its expert) of B row j of the tile, and whether it is an up row (the
// expansion's second half); rows past N repeat row N - 1 (their outputs are never stored).
// `up` is uniform over a load of 8 rows.
template <int MODE, int WTN, int OUT_COLS>
__device__ inline int b_source_col(const GemmArgs& g, int ntile, int j, bool* up) {
    if (MODE == kExpand) {
        const int grp = j / WTN, jj = j % WTN, half = jj / (WTN / 2);
        const int f = ntile * OUT_COLS + grp * (WTN / 2) + jj % (WTN / 2);
        *up = half != 0;
        return f < g.N ? f : g.N - 1;
    }
    const int h = ntile * OUT_COLS + j;
    *up = false;
    return h < g.N ? h : g.N - 1;
}

// Raw buffer resource over `bytes` bytes at `base` (loads past the end read zero).
__device__ inline __amdgpu_buffer_rsrc_t buffer_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

// bfloat16 -> float16, 8 lanes of a fragment (exact for |w| in float16's normal range)
__device__ inline halfx8 widen_to_f16(bf16x8 v) {
    const uint4 q = __builtin_bit_cast(uint4, v);
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
    halfx8 h;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        h[2 * i] = (_Float16)__uint_as_float(w[i] << 16);
        h[2 * i + 1] = (_Float16)__uint_as_float(w[i] & 0xFFFF0000u);
    }
    return h;
}

// Fragment types and loads of a mode: bf16 x bf16 for the expansion; for the projection
// the weight fragment is widened to float16 as it is read (outside the MFMA stream).
template <int MODE>
struct Frag {
    using T = typename std::conditional<MODE == kExpand, bf16x8, halfx8>::type;
    // a weight fragment as loaded (8 bf16 values, or 8 float16 values for half_weights)
    __device__ static T wide(bf16x8 v) {
        if constexpr (MODE == kExpand) return v;
        else if constexpr (half_weights(MODE)) return __builtin_bit_cast(halfx8, v);
        else return widen_to_f16(v);
    }
    __device__ static T weights(const char* p) {
        const bf16x8 v = *(const bf16x8*)p;
        return wide(v);
    }
    __device__ static T acts(const char* p) { return *(const T*)p; }
};
__device__ inline floatx4 mfma_step(const bf16x8& w, const bf16x8& a, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, a, c, 0, 0, 0);
}
__device__ inline floatx4 mfma_step(const halfx8& w, const halfx8& a, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(w, a, c, 0, 0, 0);
}

// ---------------------------------------------------------- interleaved kernel
// One wave per SIMD, each owning a 128 x 128 block of C (256 accumulator registers). K runs
// in 64-wide stages; LDS holds two stages of A and three of B (160 KB for 256 x 256 tiles,
// the whole of it: the kernel has no static LDS, and the work item is broadcast through the
// first bytes of the first A stage before its loads are issued). A stage is two 32-wide
// MFMA substeps, and every substep starts at a workgroup barrier. Between two barriers a
// wave issues the 64 MFMAs of one substep from registers, interleaved with the LDS fragment
// reads of the next substep (into the other register set); the first substep of stage kt
// also issues the global->LDS loads of A for stage kt + 2 and of B for stage kt + 3 (into
// the stage slots just freed). A third B stage (weights, mostly fetched from HBM) took the
// Mixtral-shaped expansion from 1583 to 1527 us and its projection from 1162 to 1089 us.
// A load covers 8 whole 128-byte rows, so each fetched cache line is used in full.
template <int BM_, int BNB_, int WM_, int WN_>
struct ICfg {
    static constexpr int BM = BM_, BNB = BNB_, WM = WM_, WN = WN_;
    static constexpr int NW = WM * WN, NT = NW * 64;
    static constexpr int WTM = BM / WM, WTN = BNB / WN, MB = WTM / 16, NBK = WTN / 16;
    static constexpr int A_ROWS = BM;
    static constexpr int A_INSTR = A_ROWS / 8, B_INSTR = BNB / 8;
    static constexpr int QA = A_INSTR / NW, QB = B_INSTR / NW, LPW = QA + QB;
    static constexpr int SA = A_ROWS * 128, SB = BNB * 128;   // one stage of A, of B
    static constexpr int LDS_BYTES = 2 * SA + 3 * SB;          // A: 2 stages, B: 3 stages
    // schedule of a substep: MFMA i is followed by fragment read i / R_EVERY (weights
    // first), load i / L_EVERY and, from slot W_FROM on, WPS dwords of weight widening
    static constexpr int NM = NBK * MB, NR = NBK + MB;
    static constexpr int R_EVERY = 3 * (NR - 1) < NM ? 3 : (2 * (NR - 1) < NM ? 2 : 1);
    static constexpr int L_EVERY = NM / LPW;
    static constexpr int W_FROM = R_EVERY * NBK + 2;
    static constexpr int WPS = (4 * NBK + (NM - W_FROM) - 1) / (NM - W_FROM);
    static_assert(A_INSTR % NW == 0 && B_INSTR % NW == 0, "every wave issues the same loads");
    static_assert(WTM % 16 == 0 && WTN % 32 == 0, "whole MFMA blocks, gate/up halves");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget (the kernel has no static LDS)");
    static_assert(LPW <= 63, "vmcnt range");
    static_assert(R_EVERY * (NR - 1) < NM && L_EVERY >= 1 && L_EVERY * (LPW - 1) + 1 < NM, "slots");
    static_assert(W_FROM < NM && (NM - W_FROM) * WPS >= 4 * NBK, "widen slots");
};

// 256 x 256 tiles; an expert's last tile with at most 128 rows runs as a 128 x 256 tile
// (each wave 64 x 128), which halves the MFMA work spent on padding rows.
using LargeIl = ICfg<256, 256, 2, 2>;
using LargeIlTail = ICfg<128, 256, 2, 2>;
// The same tiles on eight waves, two per SIMD (each 128 x 64, 128 accumulators): while one
// wave of a SIMD waits at a barrier or for its fragment reads, the other can issue MFMAs.
using WideIl = ICfg<256, 256, 2, 4>;
using WideIlTail = ICfg<128, 256, 2, 4>;

// MFMA through inline assembly with the accumulator pinned to AGPRs ("a" constraint):
// 256 accumulators per lane exceed what the compiler keeps in AGPRs across a loop without
// copies. FIRST starts from a zero accumulator (srcC = 0).
template <bool FIRST>
__device__ inline void mfma_agpr(floatx4& c, const bf16x8& w, const bf16x8& a) {
    if constexpr (FIRST)
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(c) : "v"(w), "v"(a));
    else
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(w), "v"(a));
}
template <bool FIRST>
__device__ inline void mfma_agpr(floatx4& c, const halfx8& w, const halfx8& a) {
    if constexpr (FIRST)
        asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, 0" : "=a"(c) : "v"(w), "v"(a));
    else
        asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(w), "v"(a));
}

// One dword of a bf16 weight fragment (two values) widened to two float16 values, in
// inline assembly so that it keeps its place in the interleaved instruction stream.
__device__ inline uint32_t widen_pair_asm(uint32_t w) {
    uint32_t out, lo, hi;
    asm volatile(
        "v_lshlrev_b32 %1, 16, %3\n\t"
        "v_and_b32 %2, 0xffff0000, %3\n\t"
        "v_cvt_pk_f16_f32 %0, %1, %2"
        : "=v"(out), "=&v"(lo), "=&v"(hi)
        : "v"(w));
    return out;
}

// bf16 -> float16 of a weight array (count values) by the same instructions as the widening
// of each fragment in the projection kernels, so that projecting with the widened copy gives
// the bits the bf16 weights give: 8 values per thread and step, then the count % 8 last ones.
__global__ __launch_bounds__(256) void widen_kernel(const uint16_t* __restrict__ src, int64_t count,
                                                    uint16_t* __restrict__ dst) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t n8 = count / 8, first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = first; i < n8; i += stride) {
        const uint4 v = ((const uint4*)src)[i];
        uint4 o;
        o.x = widen_pair_asm(v.x);
        o.y = widen_pair_asm(v.y);
        o.z = widen_pair_asm(v.z);
        o.w = widen_pair_asm(v.w);
        ((uint4*)dst)[i] = o;
    }
    const int64_t i = n8 * 8 + first;
    if (i < count) dst[i] = (uint16_t)widen_pair_asm((uint32_t)src[i]);
}

// One tile of configuration C: rows [row0, row1) of group e, N tile ntile, K slice kslice.
template <class C, int MODE, bool NT>
__device__ __forceinline__ void il_tile(const GemmArgs& g, char* lds, int e, int row0, int row1,
                                        int ntile, int kslice) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int K = g.K / g.ksplit;
    const int64_t k_byte0 = (int64_t)kslice * K * 2;
    constexpr int kOutCols = (MODE == kExpand) ? C::BNB / 2 : C::BNB;

    // load q of a lane: LDS row blk * 8 + lane / 8 of the A or B region, 16-byte position
    // lane % 8, holding chunk (lane % 8) ^ ((row >> 1) & 7) of that row. Loads are buffer
    // loads: a 32-bit byte offset per lane (fixed for the tile) and the stage's K offset as
    // the uniform scalar offset, against resources for `a` and for expert e's weights.
    uint32_t voff[C::LPW];
    int dst[C::LPW];
    const int lrow = lane >> 3;
    const int64_t wbytes = (int64_t)g.N * g.K * 2;   // one expert's weights
    const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(g.a, (uint32_t)((int64_t)g.a_rows * g.K * 2));
    const __amdgpu_buffer_rsrc_t rb0 = buffer_rsrc((const char*)g.b0 + e * wbytes, (uint32_t)wbytes);
    const __amdgpu_buffer_rsrc_t rb1 =
        MODE == kExpand ? buffer_rsrc((const char*)g.b1 + e * wbytes, (uint32_t)wbytes) : rb0;
    bool up[C::LPW];
    // source rows of this lane's A loads: with a gather, every index is loaded before any is
    // used (one wait instead of one per load)
    int srows[C::QA];
#pragma unroll
    for (int q = 0; q < C::QA; ++q) srows[q] = min(row0 + (q * C::NW + wave) * 8 + lrow, row1 - 1);
    if (g.gather) {
#pragma unroll
        for (int q = 0; q < C::QA; ++q) srows[q] = g.gather[srows[q]];
#pragma unroll
        for (int q = 0; q < C::QA; ++q)
            srows[q] = srows[q] < 0 ? 0 : (srows[q] >= g.a_rows ? (int)(g.a_rows - 1) : srows[q]);
    }
#pragma unroll
    for (int q = 0; q < C::LPW; ++q) {
        up[q] = false;
        if (q < C::QA) {
            const int blk = q * C::NW + wave, lr = blk * 8 + lrow;
            const int chunk = (lane & 7) ^ ((lr >> 1) & 7);
            const int64_t srow = srows[q];
            voff[q] = (uint32_t)(srow * (int64_t)g.K * 2 + k_byte0 + chunk * 16);
            dst[q] = blk * 1024;
        } else {
            const int blk = (q - C::QA) * C::NW + wave, lb = blk * 8 + lrow;
            const int chunk = (lane & 7) ^ ((lb >> 1) & 7);
            const int f = b_source_col<MODE, C::WTN, kOutCols>(g, ntile, lb, &up[q]);
            voff[q] = (uint32_t)((int64_t)f * g.K * 2 + k_byte0 + chunk * 16);
            dst[q] = blk * 1024;
        }
    }
    // A stage i at lds + i * SA (i < 2), B stage i at lds + 2 * SA + i * SB (i < 3)
    auto load = [&](int q, int ksa, int ksb, char* abase, char* bbase) {
        if (q < C::QA)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (PCM_LDS void*)(abase + dst[q]), 16, voff[q], ksa * 128, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(up[q] ? rb1 : rb0, (PCM_LDS void*)(bbase + dst[q]), 16, voff[q],
                                                     ksb * 128, 0, weight_policy(NT));
    };
    char* const A0 = lds;
    char* const B0 = lds + 2 * C::SA;

    floatx4 acc[C::NBK][C::MB];
    const int KT2 = K / 64;
    // fragment of row (lane & 15), chunk 4 * sub + (lane >> 4) of a 16-row block
    const int fr = lane & 15;
    const int foff0 = fr * 128 + (((lane >> 4) ^ (fr >> 1)) * 16);
    const int foff1 = fr * 128 + (((4 + (lane >> 4)) ^ (fr >> 1)) * 16);
    using FT = typename Frag<MODE>::T;
    FT af[2][C::MB], bf[2][C::NBK];
    bf16x8 braw[C::NBK];
    uint32_t bw[C::NBK][4];
    auto b_at = [&](const char* S, int nb, int fo) { return S + (wn * C::WTN + nb * 16) * 128 + fo; };
    auto a_at = [&](const char* S, int mb, int fo) { return S + (wm * C::WTM + mb * 16) * 128 + fo; };
    auto barrier = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int NM = C::NM, NR = C::NR, R_EVERY = C::R_EVERY, L_EVERY = C::L_EVERY;
    constexpr int W_FROM = C::W_FROM, WPS = C::WPS;
    // One 32-wide substep: the MFMAs of (ca, cb), the fragment reads of the next substep
    // from the A and B stages SAr, SBr at chunk offset fo, and (LOADS, the first substep of a
    // stage) every load of A stage ksa into slot la and of B stage ksb into slot lb. It
    // starts with this wave's fragment reads complete and a barrier; a LOADS substep first
    // waits until only the newest B loads (the next B stage, issued after the A loads of the
    // stage its reads need) may be in flight, so that stage has landed, and the barrier
    // makes the slots it loads free (read by every wave).
    // The barrier also keeps VALU writes of fragment registers (the prologue's widening)
    // at least two wait states ahead of the MFMAs that read them: the MFMAs are inline
    // assembly, which the compiler's hazard checks do not see.
    auto sub = [&](auto first, auto loads, FT (&ca)[C::MB], FT (&cb)[C::NBK],
                   FT (&na)[C::MB], FT (&nb_)[C::NBK], const char* SAr, const char* SBr, int fo, int ksa, int ksb,
                   char* la, char* lb) {
        // a LOADS substep waits for the stage its reads need; only the B loads issued after
        // that stage's A loads (the next B stage) may stay in flight
        __builtin_amdgcn_s_waitcnt(waitcnt_imm(decltype(loads)::value ? C::QB : kNoVm, 0));
        barrier();
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            mfma_agpr<decltype(first)::value>(acc[i / C::MB][i % C::MB], cb[i / C::MB], ca[i % C::MB]);
            if (i % R_EVERY == 0 && i / R_EVERY < NR) {
                const int j = i / R_EVERY;
                if (j < C::NBK) {
                    if constexpr (MODE == kExpand || half_weights(MODE)) nb_[j] = *(const FT*)b_at(SBr, j, fo);
                    else braw[j] = *(const bf16x8*)b_at(SBr, j, fo);
                } else {
                    na[j - C::NBK] = Frag<MODE>::acts(a_at(SAr, j - C::NBK, fo));
                }
            }
            if constexpr (decltype(loads)::value)
                if (i % L_EVERY == 1 && i / L_EVERY < C::LPW) load(i / L_EVERY, ksa, ksb, la, lb);
            if constexpr (MODE != kExpand && !half_weights(MODE)) {
#pragma unroll
                for (int w = 0; w < WPS; ++w) {
                    const int d = (i - W_FROM) * WPS + w;
                    if (i >= W_FROM && d < 4 * C::NBK) {
                        const uint4 q4 = __builtin_bit_cast(uint4, braw[d / 4]);
                        const uint32_t wv = (d % 4 == 0) ? q4.x : (d % 4 == 1) ? q4.y : (d % 4 == 2) ? q4.z : q4.w;
                        bw[d / 4][d % 4] = widen_pair_asm(wv);
                        if (d % 4 == 3)
                            nb_[d / 4] = __builtin_bit_cast(FT, uint4{bw[d / 4][0], bw[d / 4][1], bw[d / 4][2], bw[d / 4][3]});
                    }
                }
            }
        }
    };
    using T_ = std::true_type;
    using F_ = std::false_type;

    // prologue: stages 0 and 1 in flight, stage 0 landed, the fragments of substep 0 read
    // stages 0 and 1 of A and stages 0-2 of B in flight (in that order: A0 B0 A1 B1 B2),
    // stage 0 landed, the fragments of substep 0 read
    const int s1 = KT2 > 1 ? 1 : 0, s2 = KT2 > 2 ? 2 : KT2 - 1;
#pragma unroll
    for (int q = 0; q < C::LPW; ++q) load(q, 0, 0, A0, B0);
#pragma unroll
    for (int q = 0; q < C::LPW; ++q) load(q, s1, s1, A0 + C::SA, B0 + C::SB);
#pragma unroll
    for (int q = C::QA; q < C::LPW; ++q) load(q, s2, s2, A0, B0 + 2 * C::SB);
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(C::QA + 2 * C::QB, kNoLgkm));
    barrier();
#pragma unroll
    for (int nb = 0; nb < C::NBK; ++nb) bf[0][nb] = Frag<MODE>::weights(b_at(B0, nb, foff0));
#pragma unroll
    for (int mb = 0; mb < C::MB; ++mb) af[0][mb] = Frag<MODE>::acts(a_at(A0, mb, foff0));
    // substep 0: stage 0, first half; reads its second half
    sub(T_{}, F_{}, af[0], bf[0], af[1], bf[1], A0, B0, foff1, 0, 0, A0, B0);
    int bi = 0;                                          // kt % 3
    for (int kt = 0; kt + 1 < KT2; ++kt) {
        const int bn = bi == 2 ? 0 : bi + 1;
        char* ca = A0 + (kt & 1) * C::SA;               // stage kt: free after the barrier
        char* cb = B0 + bi * C::SB;
        const char* na = A0 + ((kt + 1) & 1) * C::SA;
        const char* nbp = B0 + bn * C::SB;
        // past the end: re-read, never used
        const int ksa = kt + 2 < KT2 ? kt + 2 : KT2 - 1, ksb = kt + 3 < KT2 ? kt + 3 : KT2 - 1;
        // second half of stage kt; reads the first half of stage kt+1; loads A kt+2, B kt+3
        sub(F_{}, T_{}, af[1], bf[1], af[0], bf[0], na, nbp, foff0, ksa, ksb, ca, cb);
        // first half of stage kt+1; reads its second half
        sub(F_{}, F_{}, af[0], bf[0], af[1], bf[1], na, nbp, foff1, ksa, ksb, ca, cb);
        bi = bn;
    }
    // second half of the last stage: MFMAs only (after the two wait states its fragments'
    // last VALU writes need)
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 1" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NM; ++i) mfma_agpr<false>(acc[i / C::MB][i % C::MB], bf[1][i / C::MB], af[1][i % C::MB]);
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    GemmArgs gs = g;
    if (kslice) gs.out = (float*)g.out + (int64_t)kslice * g.rows_total * g.N;
    // the expansion, and a projection that adds into its output: the shared epilogue
    if (MODE == kExpand || (base_mode(MODE) == kDownAccum && g.accumulate)) {
        epilogue<MODE, C::MB, C::NBK, C::WTM, C::WTN, kOutCols>(gs, acc, row0, row1, ntile, wm, wn, lane);
        return;
    }
    // The projection's epilogue through LDS: each wave writes its outputs (the row scale
    // applied) in the MFMA layout (16 rows x 16 columns per block) into a private LDS area,
    // 64 rows at a time, and reads them back in row order, so that each store covers whole
    // rows with lanes in address order (2 rows of the wave's 128 columns) instead of half
    // lines of 16 rows: OLMoE-shaped projection-and-combine -4.3%, fine-grained -2.5%, the
    // 256 KB of float32 per tile being a quarter of the tile's time there (the expansion,
    // with half the output bytes per tile, was not faster this way). LDS row ro holds
    // 16-byte chunk c at position c ^ (ro & FM) (conflict-free writes of 16 rows x 1 chunk
    // and reads of 1 row x 16 chunks).
    constexpr int OUTW = C::WTN;                                     // output columns per wave
    constexpr int LPR = OUTW / 4;                                    // 16-byte chunks per row
    constexpr int RPI = 64 / LPR;                                     // rows per store
    constexpr int PM = C::MB < 4 ? C::MB : 4;                        // 16-row blocks per pass
    constexpr int RS = OUTW * 4;                                      // LDS row stride, bytes
    constexpr int FM = (LPR - 1) < 15 ? (LPR - 1) : 15;
    static_assert(C::MB % PM == 0 && 64 % LPR == 0 && C::NW * PM * 16 * RS <= C::LDS_BYTES, "LDS epilogue");
    float scs[C::MB];   // row scales, loaded first and waited for once
#pragma unroll
    for (int mb = 0; mb < C::MB; ++mb) {
        const int r = min(row0 + wm * C::WTM + mb * 16 + (lane & 15), row1 - 1);
        scs[mb] = g.row_scale ? g.row_scale[scale_row(g, r)] : 1.0f;
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, kNoLgkm));
    barrier();   // every wave's fragment reads of the last stage are done
    char* wl = lds + wave * (PM * 16 * RS);
    const int c0 = ntile * kOutCols + wn * OUTW;
    float* O = (float*)gs.out;
    const int N = g.N;
#pragma unroll
    for (int ps = 0; ps < C::MB / PM; ++ps) {
#pragma unroll
        for (int ml = 0; ml < PM; ++ml) {
            const int mb = ps * PM + ml, ro = ml * 16 + (lane & 15);
            const float sc = scs[mb];
#pragma unroll
            for (int nb = 0; nb < C::NBK; ++nb) {
                const float4 v = make_float4(acc[nb][mb][0] * sc, acc[nb][mb][1] * sc,
                                             acc[nb][mb][2] * sc, acc[nb][mb][3] * sc);
                const int c = nb * 4 + (lane >> 4);
                *(float4*)(wl + ro * RS + 16 * (c ^ (ro & FM))) = v;
            }
        }
#pragma unroll
        for (int i = 0; i < PM * 16 / RPI; ++i) {
            const int ro = i * RPI + lane / LPR, c = lane % LPR;
            const float4 v = *(const float4*)(wl + ro * RS + 16 * (c ^ (ro & FM)));
            const int r = row0 + wm * C::WTM + ps * PM * 16 + ro, col = c0 + c * 4;
            if (r < row1 && col < N) *(float4*)(O + (int64_t)r * N + col) = v;
        }
    }
}

// Work item of workgroup bid for the large-tile kernel, longest first. A group of c rows has
// c / BM full tiles and, if rows remain, one remainder tile: a long item when more than TBM
// rows remain, a short (tail-shape) item otherwise. Workgroups are dispatched round-robin over
// the 8 XCDs (bid % 8) and in bid order within each; each XCD's run of ids holds its eighth of
// the long items (every K slice) and then its eighth of the short items, so the short tiles
// fill the last round instead of lengthening it. Within each list the order is the grouped
// one of tile_from_id. Wave 0 counts and searches; the result is broadcast through LDS
// (s_item: group, row0, row1, ntile, kslice, valid). Returns false past the last item.
template <int BM, int TBM>
__device__ bool il_item(const GemmArgs& g, int nt, int GN, int* s_item) {
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        int lo[4], cnt[4], hi[4], full[4], nl[4], ns[4], suml = 0, sums = 0;
        group_bounds(g.offsets, g.n, g.a_rows, lane, lo, cnt);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int rem = cnt[j] % BM;
            hi[j] = lo[j] + cnt[j];
            full[j] = cnt[j] / BM;
            nl[j] = full[j] + (rem > TBM ? 1 : 0);
            ns[j] = (rem > 0 && rem <= TBM) ? 1 : 0;
            suml += nl[j];
            sums += ns[j];
        }
        const int incl = wave_incl_scan_i32(suml), incs = wave_incl_scan_i32(sums);
        // 32-bit arithmetic throughout: the host keeps item counts (times 8) within range
        // the short list in halves: 2 * nt N-tiles of half width
        const int Lt = __builtin_amdgcn_readlane(incl, 63), St = __builtin_amdgcn_readlane(incs, 63);
        const int LT = Lt * nt * g.ksplit, ST = St * 2 * nt * g.ksplit;
        const int x8 = (int)(blockIdx.x % 8), j8 = (int)(blockIdx.x / 8);
        const int l0 = x8 * LT / 8, l1 = (x8 + 1) * LT / 8;
        const int s0 = x8 * ST / 8, s1 = (x8 + 1) * ST / 8;
        bool valid = true, is_long = true;
        int item = 0, count = Lt;
        if (j8 < l1 - l0) {
            item = l0 + j8;
        } else if (j8 - (l1 - l0) < s1 - s0) {
            item = s0 + j8 - (l1 - l0);
            is_long = false;
            count = St;
        } else {
            valid = false;
        }
        if (lane == 0) {
            s_item[5] = valid ? 1 : 0;
            s_item[6] = is_long ? 0 : 1;
        }
        if (valid) {
            const int ntl = is_long ? nt : 2 * nt, gnl = is_long ? GN : 2 * GN;
            const int per_slice = count * ntl;
            const int kslice = item / per_slice;
            // grouped order within the list (as tile_from_id)
            const int id = item - kslice * per_slice;
            const int gsize = gnl * count;
            const int grp = id / gsize, in = id - grp * gsize;
            const int gn = min(gnl, ntl - grp * gnl);
            const int m = in / gn;
            const int ntile = grp * gnl + (in - m * gn);
            // group holding list entry m: this lane's groups start at the exclusive prefix
            int start = is_long ? incl - suml : incs - sums;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int cnt = is_long ? nl[j] : ns[j];
                if (m >= start && m < start + cnt) {
                    const int r0 = lo[j] + (is_long ? (m - start) * BM : full[j] * BM);
                    s_item[0] = lane * 4 + j;
                    s_item[1] = r0;
                    s_item[2] = min(hi[j], r0 + BM);
                    s_item[3] = ntile;
                    s_item[4] = kslice;
                }
                start += cnt;
            }
        }
    }
    __syncthreads();
    return s_item[5] != 0;
}

// Work orders of the large-tile kernel.
enum IlOrder { kGrouped = 0, kLongestFirst = 1, kExpertMajor = 2 };

// order (an IlOrder): kLongestFirst is the order of il_item, kGrouped the grouped order of
// tile_of, kExpertMajor the order of em_item (group_n is then the window).
// once: weights_once.
template <class C, class CT, int MODE>
__global__ __launch_bounds__(C::NT) void gemm_il_kernel(GemmArgs g, int64_t mt_upper, int nt,
                                                         int group_n, int order, bool once) {
    // half of a tail tile (128 x 128 for the large tiles, each wave 64 x 64): the longest-first
    // order runs each tail item as two of these, so that shorter items fill the last round
    using CH = ICfg<CT::BM, C::BNB / 2, CT::WM, CT::WN>;
    static_assert(CT::NT == C::NT && CT::BNB == C::BNB && CT::BM <= C::BM && CT::WTN == C::WTN,
                  "the tail tile runs on the same workgroup and N tiling");
    static_assert(CH::NT == C::NT && CH::LDS_BYTES <= C::LDS_BYTES, "the half tail tile fits");
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    int* const s_item = (int*)lds;   // read into registers before the stage loads overwrite it
    int e, row0, row1, ntile, kslice;
    if (order == kLongestFirst) {          // workgroup-uniform branches and returns
        if (!il_item<C::BM, CT::BM>(g, nt, group_n, s_item)) return;
        e = s_item[0], row0 = s_item[1], row1 = s_item[2], ntile = s_item[3], kslice = s_item[4];
        const int half = s_item[6];
        __syncthreads();
        if (half) {                        // half of a tail item: N-tile of half width
            il_tile<CH, MODE, false>(g, lds, e, row0, row1, ntile, kslice);
            return;
        }
    } else if (order == kExpertMajor) {
        if (!em_item<C::BM, CT::BM>(g, nt, group_n, true, s_item)) return;
        e = s_item[0], row0 = s_item[1], row1 = s_item[2], ntile = s_item[3], kslice = s_item[4];
        __syncthreads();
    } else {
        int64_t mt;
        const int64_t per_slice = gridDim.x / g.ksplit;
        kslice = (int)(blockIdx.x / per_slice);
        if (!tile_of(blockIdx.x % per_slice, per_slice, mt_upper, nt, group_n, &mt, &ntile)) return;
        if (!find_tile<C::BM>(g.offsets, g.n, g.a_rows, mt, s_item)) return;
        e = s_item[0], row0 = s_item[1], row1 = s_item[2];
        __syncthreads();
    }
    // the group's only row tile: its weights are read once (an accumulating projection has one group,
    // and the two more tile bodies made it spill)
    constexpr bool kOnce = base_mode(MODE) != kDownAccum;
    const bool single = kOnce && once && g.offsets[e + 1] - g.offsets[e] <= C::BM;
    if (row1 - row0 <= CT::BM) {
        if (single) il_tile<CT, MODE, kOnce>(g, lds, e, row0, row1, ntile, kslice);
        else il_tile<CT, MODE, false>(g, lds, e, row0, row1, ntile, kslice);
    } else {
        if (single) il_tile<C, MODE, kOnce>(g, lds, e, row0, row1, ntile, kslice);
        else il_tile<C, MODE, false>(g, lds, e, row0, row1, ntile, kslice);
    }
}

// --------------------------------------------------------------- staged kernel
template <int BM_, int BNB_, int WM_, int WN_>
struct SCfg {
    static constexpr int BM = BM_, BNB = BNB_, WM = WM_, WN = WN_;
    static constexpr int NT = WM * WN * 64;
    static constexpr int WTM = BM / WM, WTN = BNB / WN, MB = WTM / 16, NBK = WTN / 16;
    static constexpr int A_ROWS = BM;                      // 128-byte LDS rows: 64 K values
    static constexpr int A_CHUNKS = A_ROWS * 8, B_CHUNKS = BNB * 8;
    static constexpr int A_PER_T = (A_CHUNKS + NT - 1) / NT, B_PER_T = (B_CHUNKS + NT - 1) / NT;
    static constexpr int STAGE = (A_ROWS + BNB) * 128;
    static constexpr int LDS_BYTES = 2 * STAGE;
    static_assert(WTM % 16 == 0 && WTN % 32 == 0, "whole MFMA blocks, gate/up halves");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
    static_assert(A_CHUNKS % NT == 0 && B_CHUNKS % NT == 0, "every thread owns whole chunks");
};

using MediumStaged = SCfg<128, 128, 2, 2>;

template <class C, int MODE>
__global__ __launch_bounds__(C::NT) void gemm_staged_kernel(GemmArgs g, int64_t mt_upper, int nt,
                                                            int group_n) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    __shared__ int s_tile[4];
    int64_t mt;
    int ntile;
    if (!tile_of(blockIdx.x, gridDim.x, mt_upper, nt, group_n, &mt, &ntile)) return;
    if (!find_tile<C::BM>(g.offsets, g.n, g.a_rows, mt, s_tile)) return;
    const int e = s_tile[0], row0 = s_tile[1], row1 = s_tile[2];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int K = g.K;
    constexpr int kOutCols = (MODE == kExpand) ? C::BNB / 2 : C::BNB;

    // chunk i of a stage: LDS row i / 8, logical chunk i % 8 (16 bytes), stored at position
    // (i % 8) ^ ((row >> 1) & 7); every thread owns A_PER_T + B_PER_T chunks
    const char* aptr[C::A_PER_T];
    const char* bptr[C::B_PER_T];
    int aoff[C::A_PER_T], boff[C::B_PER_T];
#pragma unroll
    for (int i = 0; i < C::A_PER_T; ++i) {
        const int c = tid + i * C::NT, lr = c / 8, kc = c % 8;
        const int64_t srow = a_source_row(g, row0 + lr, row1);
        aptr[i] = (const char*)g.a + srow * (int64_t)K * 2 + kc * 16;
        aoff[i] = lr * 128 + ((kc ^ ((lr >> 1) & 7)) * 16);
    }
#pragma unroll
    for (int i = 0; i < C::B_PER_T; ++i) {
        const int c = tid + i * C::NT, j = c / 8, kc = c % 8;
        bptr[i] = (const char*)b_source_row<MODE, C::WTN, kOutCols>(g, e, ntile, j) + kc * 16;
        boff[i] = (C::A_ROWS + j) * 128 + ((kc ^ ((j >> 1) & 7)) * 16);
    }

    uint4 ra[C::A_PER_T], rb[C::B_PER_T];
#define PCM_STAGED_GLOAD(kt)                                                              \
    do {                                                                                  \
        _Pragma("unroll") for (int i = 0; i < C::A_PER_T; ++i)                            \
            ra[i] = *(const uint4*)(aptr[i] + (int64_t)(kt) * 128);                       \
        _Pragma("unroll") for (int i = 0; i < C::B_PER_T; ++i)                            \
            rb[i] = *(const uint4*)(bptr[i] + (int64_t)(kt) * 128);                       \
    } while (0)
#define PCM_STAGED_LSTORE(buf)                                                            \
    do {                                                                                  \
        char* S_ = lds + (buf) * C::STAGE;                                                \
        _Pragma("unroll") for (int i = 0; i < C::A_PER_T; ++i) *(uint4*)(S_ + aoff[i]) = ra[i]; \
        _Pragma("unroll") for (int i = 0; i < C::B_PER_T; ++i) *(uint4*)(S_ + boff[i]) = rb[i]; \
    } while (0)

    floatx4 acc[C::NBK][C::MB];
#pragma unroll
    for (int nb = 0; nb < C::NBK; ++nb)
#pragma unroll
        for (int mb = 0; mb < C::MB; ++mb) acc[nb][mb] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int KT = K / 64;
    PCM_STAGED_GLOAD(0);
    PCM_STAGED_LSTORE(0);
    __syncthreads();
    for (int kt = 0; kt < KT; ++kt) {
        const int cur = kt & 1;
        // unconditional (the last step re-reads itself into the idle stage): a conditional
        // load keeps the staging registers out of SROA and in scratch memory
        PCM_STAGED_GLOAD(kt + 1 < KT ? kt + 1 : kt);
        const char* S = lds + cur * C::STAGE;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int ck = ks * 4 + (lane >> 4);
            const int off = (lane & 15) * 128 + ((ck ^ (((lane & 15) >> 1) & 7)) * 16);
            typename Frag<MODE>::T bfr[C::NBK], afr[C::MB];
#pragma unroll
            for (int nb = 0; nb < C::NBK; ++nb)
                bfr[nb] = Frag<MODE>::weights(S + (C::A_ROWS + wn * C::WTN + nb * 16) * 128 + off);
#pragma unroll
            for (int mb = 0; mb < C::MB; ++mb)
                afr[mb] = Frag<MODE>::acts(S + (wm * C::WTM + mb * 16) * 128 + off);
#pragma unroll
            for (int nb = 0; nb < C::NBK; ++nb)
#pragma unroll
                for (int mb = 0; mb < C::MB; ++mb) acc[nb][mb] = mfma_step(bfr[nb], afr[mb], acc[nb][mb]);
        }
        PCM_STAGED_LSTORE(cur ^ 1);
        __syncthreads();
    }
#undef PCM_STAGED_GLOAD
#undef PCM_STAGED_LSTORE
    epilogue<MODE, C::MB, C::NBK, C::WTM, C::WTN, kOutCols>(g, acc, row0, row1, ntile, wm, wn, lane);
}


// --------------------------------------------------------------- stream kernel
// Few rows per group (decode): the weights are the traffic. Each wave owns NB 16-row weight
// blocks (for the expansion, gate rows of NB / 2 blocks of 16 columns and the up rows of the
// same columns; for the projection, NB * 16 output columns) and one 16-row block of
// activation rows, and loads MFMA fragments straight from global memory into a ring of SDP
// register sets, SDP k-steps ahead of the MFMAs (no LDS). A lane reads 16 bytes of one row
// per k-step (row lane & 15, K offset 8 * (lane >> 4)), the same mapping for weights and
// activations; the activation fragment is shared by the wave's NB weight blocks.
constexpr int SROWS = 16;      // activation rows per tile
constexpr int SWAVES = 4;

template <int MODE, int NB, int SDP>
__global__ __launch_bounds__(SWAVES * 64) void gemm_stream_kernel(GemmArgs g, int64_t mt_upper,
                                                                 int nt, int n_fastest) {
    static_assert(NB % 2 == 0 && (NB + 1) * (SDP - 1) <= 63, "gate/up halves; vmcnt range");
    __shared__ int s_tile[4];
    const int64_t mt = n_fastest ? blockIdx.x / nt : blockIdx.x % mt_upper;
    const int ntile = n_fastest ? (int)(blockIdx.x % nt) : (int)(blockIdx.x / mt_upper);
    if (!find_tile<SROWS>(g.offsets, g.n, g.a_rows, mt, s_tile)) return;
    const int e = s_tile[0], row0 = s_tile[1], row1 = s_tile[2];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int K = g.K, N = g.N;
    // output columns of this wave: expansion NB * 8 (gate + up rows), projection NB * 16
    constexpr int kWaveCols = (MODE == kExpand) ? NB * 8 : NB * 16;
    const int col0 = (ntile * SWAVES + wave) * kWaveCols;
    if (col0 >= N) return;  // wave-uniform; no barrier follows
    const int r16 = lane & 15, kg = lane >> 4;
    // weight row of block b for this lane
    const uint16_t* wp[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        int wr;
        const uint16_t* base;
        if (MODE == kExpand) {
            wr = col0 + (b % (NB / 2)) * 16 + r16;
            base = (const uint16_t*)(b >= NB / 2 ? g.b1 : g.b0);
        } else {
            wr = col0 + b * 16 + r16;
            base = (const uint16_t*)g.b0;
        }
        wr = wr < N ? wr : N - 1;
        wp[b] = base + ((int64_t)e * N + wr) * K + kg * 8;
    }
    const uint16_t* ap = (const uint16_t*)g.a + a_source_row(g, row0 + r16, row1) * (int64_t)K + kg * 8;

    floatx4 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = floatx4{0.f, 0.f, 0.f, 0.f};
    bf16x8 wbuf[SDP][NB], abuf[SDP];
    const int KT = K / 32;
    auto load = [&](int slot, int kt) {
#pragma unroll
        for (int b = 0; b < NB; ++b) wbuf[slot][b] = *(const bf16x8*)(wp[b] + kt * 32);
        abuf[slot] = *(const bf16x8*)(ap + kt * 32);
    };
#pragma unroll
    for (int j = 0; j < SDP; ++j)
        if (j < KT) load(j, j);
    for (int base = 0; base < KT; base += SDP) {
#pragma unroll
        for (int j = 0; j < SDP; ++j) {
            const int kt = base + j;
            if (kt >= KT) break;
            // this step's NB + 1 loads have landed (the newer steps may still be in flight)
            if (kt + SDP - 1 < KT) __builtin_amdgcn_s_waitcnt(waitcnt_imm((NB + 1) * (SDP - 1), kNoLgkm));
            else __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, kNoLgkm));
            if constexpr (MODE == kExpand) {
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[b] = mfma_step(wbuf[j][b], abuf[j], acc[b]);
            } else {
                const halfx8 a16 = __builtin_bit_cast(halfx8, abuf[j]);
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[b] = mfma_step(Frag<MODE>::wide(wbuf[j][b]), a16, acc[b]);
            }
            if (kt + SDP < KT) load(j, kt + SDP);
        }
    }
    // epilogue: lane holds output columns c..c+3 (c = 4 * (lane >> 4)) of activation row r16
    // in each block
    const int r = row0 + r16;
    if (r >= row1) return;
    if (MODE == kExpand) {
#pragma unroll
        for (int b = 0; b < NB / 2; ++b) {
            const int f = col0 + b * 16 + 4 * kg;
            if (f >= N) continue;
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = silu(acc[b][i]) * acc[b + NB / 2][i];
            *(float4*)((float*)g.out + (int64_t)r * N + f) = make_float4(v[0], v[1], v[2], v[3]);
        }
    } else {
        const float sc = g.row_scale ? g.row_scale[scale_row(g, r)] : 1.0f;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int h = col0 + b * 16 + 4 * kg;
            if (h >= N) continue;
            float4 v = make_float4(acc[b][0] * sc, acc[b][1] * sc, acc[b][2] * sc, acc[b][3] * sc);
            float4* dst = (float4*)((float*)g.out + (int64_t)r * N + h);
            if (base_mode(MODE) == kDownAccum && g.accumulate) {
                const float4 o = *dst;
                v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
            }
            *dst = v;
        }
    }
}

// LDS-ring streaming kernel: the streaming kernel with its operands staged through a per-wave
// LDS ring. A weight load of the register-ring kernel covers 16 rows x 64 bytes (the MFMA operand
// layout puts four lanes on a row), half a cache line per row, and the weight stream then ran
// at 5.4 TB/s; here each direct buffer -> LDS load covers 8 rows x 128 bytes (the 64 K values
// of two MFMA steps, whole lines) and the MFMA fragments are read back from LDS. Ring slot j of
// a wave holds NB blocks of 16 weight rows and MB blocks of 16 activation rows, each row
// 128 bytes with chunk c of row r at position c ^ ((r >> 1) & 7) (conflict-free fragment
// reads); D slots, D - 1 slices in flight. No barrier in the loop: each wave owns its ring, and a
// slot is reloaded only after the MFMAs that used its fragments. With the activations in the ring
// as well, the loop holds no load into registers, whose waits the compiler would place itself
// (it drained every load in flight at the loop head). K is a multiple of 64 (as the layer
// entry points require of H and F), and `a` and one group's weights are below 4 GiB (32-bit
// buffer offsets); otherwise the register-ring kernel runs.
//
// KW = 1: the four waves own NB * 16 weight rows each. KW = 4: the workgroup owns NB * 16 rows; each
// wave loads every fourth slice of K into its own slots and runs some of the output blocks over all
// slices, in ascending order, so the sums are those of every other kernel, bit for bit. Four times
// the workgroups, where the weight rows alone would leave compute units idle or too little in
// flight. One barrier per G slices: it says that their loads have landed and that the slots of the G
// before them, which are then reloaded, have been read; 4 D - G slices are in flight between two.
// (The body is a device function: the buffer resources and LDS-destination loads it uses have
// no host form, and the host pass does not emit a kernel whose own body uses them.)
template <int MODE, int NB, int MB, int D, int KW, int G>
struct LStream {
    static constexpr int kWaveCols = (MODE == kExpand) ? NB * 8 : NB * 16;   // output columns
    static constexpr int kWgCols = kWaveCols * (KW == 1 ? SWAVES : 1);
    static constexpr int kSlot = (NB + MB) * 2048;   // NB weight blocks, then MB activation blocks
    static constexpr int kLds = SWAVES * D * kSlot;
    static constexpr int kLoads = 2 * (NB + MB);     // loads of a slice
    static constexpr int kUnits = (MODE == kExpand ? NB / 2 : NB) * MB;   // blocks of 16 x 16 outputs
    static constexpr int U = KW == 1 ? kUnits : (kUnits + SWAVES - 1) / SWAVES;   // of them in a wave
    static constexpr int kSteady = G == SWAVES ? D - 2 : D - 1;   // KW = 4: slices that may be in flight behind the one waited for
    static_assert(KW == 1 || (KW == SWAVES && (G == 2 || (G == SWAVES && D > 2))), "the waves share their rows or their slices");
    static_assert((MODE != kExpand || NB % 2 == 0) && D >= 2 && (D - 1) * kLoads <= 62, "gate/up halves; vmcnt range");
};

// Waits until at most n * LOADS of the wave's loads are in flight, for n = 0 .. MOST (no wait otherwise).
template <int LOADS, int MOST>
__device__ __forceinline__ void wait_last(int n) {
    if (n == MOST) __builtin_amdgcn_s_waitcnt(waitcnt_imm(MOST * LOADS, kNoLgkm));
    if constexpr (MOST > 0) wait_last<LOADS, MOST - 1>(n);
}

// One output row r and 4 columns from c on: the projection's store or accumulation.
template <int MODE>
__device__ inline void store_down4(const GemmArgs& g, int r, int c, const floatx4& acc, float sc) {
    float4 v = make_float4(acc[0] * sc, acc[1] * sc, acc[2] * sc, acc[3] * sc);
    float4* dst = (float4*)((float*)g.out + (int64_t)r * g.N + c);
    if (base_mode(MODE) == kDownAccum && g.accumulate) {
        const float4 o = *dst;
        v.x = __fadd_rn(o.x, v.x); v.y = __fadd_rn(o.y, v.y);
        v.z = __fadd_rn(o.z, v.z); v.w = __fadd_rn(o.w, v.w);
    }
    *dst = v;
}
__device__ inline void store_swiglu4(const GemmArgs& g, int r, int c, const floatx4& gate, const floatx4& up) {
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = silu(gate[i]) * up[i];
    *(float4*)((float*)g.out + (int64_t)r * g.N + c) = make_float4(v[0], v[1], v[2], v[3]);
}

// Rows [row0, row1) of group e (at most 16 * MB), N tile ntile.
template <int MODE, int NB, int MB, int D, int KW, int G, bool NT>
__device__ __forceinline__ void lstream_tile(const GemmArgs& g, char* lds, int e, int row0, int row1,
                                             int ntile) {
    using C = LStream<MODE, NB, MB, D, KW, G>;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int K = g.K, N = g.N;
    const int col0 = KW == 1 ? (ntile * SWAVES + wave) * C::kWaveCols : ntile * C::kWaveCols;
    if (KW == 1 && col0 >= N) return;  // wave-uniform; no barrier follows
    char* ring = lds + wave * (D * C::kSlot);
    const int r16 = lane & 15, kg = lane >> 4;
    // source rows of the activation loads, (the projection) the row scales: loaded first, and used
    // only once the first weights are on their way too
    int arow[MB][2];
    constexpr int kScales = KW == 1 ? MB : C::U;
    float sc[kScales];   // of row block m, or (KW = 4) of the row block of this wave's block u
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            arow[m][h] = min(row0 + m * 16 + h * 8 + (lane >> 3), row1 - 1);
            if (g.gather) arow[m][h] = g.gather[arow[m][h]];
        }
#pragma unroll
    for (int u = 0; u < kScales; ++u) {
        sc[u] = 1.0f;
        const int m = KW == 1 ? u : (u * SWAVES + wave) % MB;
        if constexpr (MODE != kExpand)
            if (g.row_scale) sc[u] = g.row_scale[scale_row(g, min(row0 + m * 16 + r16, row1 - 1))];
    }
    // weight row (within expert e) behind row R of block b; rows past N repeat row N - 1
    auto wrow = [&](int b, int R) {
        const int wr = (MODE == kExpand) ? col0 + (b % (NB / 2)) * 16 + R : col0 + b * 16 + R;
        return wr < N ? wr : N - 1;
    };
    const int64_t wbytes = (int64_t)N * K * 2;
    const __amdgpu_buffer_rsrc_t rb0 = buffer_rsrc((const char*)g.b0 + e * wbytes, (uint32_t)wbytes);
    const __amdgpu_buffer_rsrc_t rb1 =
        MODE == kExpand ? buffer_rsrc((const char*)g.b1 + e * wbytes, (uint32_t)wbytes) : rb0;
    const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(g.a, (uint32_t)((int64_t)g.a_rows * K * 2));
    // load (b, h) of a slice: rows h * 8 + lane / 8 of block b, position lane % 8
    uint32_t voff[NB][2], aoff[MB][2];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int R = h * 8 + (lane >> 3);
            voff[b][h] = (uint32_t)(wrow(b, R) * (int64_t)K * 2 + ((lane & 7) ^ ((R >> 1) & 7)) * 16);
        }
    // this wave loads slices wave, wave + KW, ... (KW = 1: all) of 64 K values
    const int slices = K / 64, first = KW == 1 ? 0 : wave;
    const int KP = (slices - first + KW - 1) / KW;   // at least 2 with KW = 4 (K >= 512)
    // (past the end, in the first slots only: the last slice again, never used)
    auto issue_w = [&](int j, int p) {
        char* slot = ring + j * C::kSlot;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                __builtin_amdgcn_raw_ptr_buffer_load_lds((MODE == kExpand && b >= NB / 2) ? rb1 : rb0,
                                                         (PCM_LDS void*)(slot + b * 2048 + h * 1024), 16,
                                                         voff[b][h], (first + min(p, KP - 1) * KW) * 128, 0, weight_policy(NT));
    };
    auto issue_a = [&](int j, int p) {
        char* slot = ring + j * C::kSlot;
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (PCM_LDS void*)(slot + (NB + m) * 2048 + h * 1024), 16,
                                                         aoff[m][h], (first + min(p, KP - 1) * KW) * 128, 0, 0);
    };
    // Issued before the loop: D - 1 slices (KW = 1) or D, every weight load before every activation
    // load, whose row indices are still on their way, with the rings that grouped rows take
    constexpr int kAhead = KW == 1 ? D - 1 : D;
    constexpr bool kWeightsFirst = KW == 1 || D == 2;
    if constexpr (kWeightsFirst)
#pragma unroll
        for (int j = 0; j < kAhead; ++j) issue_w(j, j);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int R = h * 8 + (lane >> 3);
            int64_t src = arow[m][h];
            src = src < 0 ? 0 : (src >= g.a_rows ? g.a_rows - 1 : src);
            aoff[m][h] = (uint32_t)(src * K * 2 + ((lane & 7) ^ ((R >> 1) & 7)) * 16);
        }
    // the scales have landed here (a load into a register still in flight across the loop makes
    // the compiler wait for every load in it)
    if constexpr (MODE != kExpand)
#pragma unroll
        for (int u = 0; u < kScales; ++u) asm volatile("" : "+v"(sc[u])::"memory");
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
        if constexpr (!kWeightsFirst) issue_w(j, j);
        issue_a(j, j);
    }
    // fragment of row r16, chunk 4 * step + kg
    const int fo0 = r16 * 128 + ((kg ^ ((r16 >> 1) & 7)) * 16);
    const int fo1 = r16 * 128 + (((4 + kg) ^ ((r16 >> 1) & 7)) * 16);

    // lane holds output columns c..c+3 (c = 4 * (lane >> 4)) of activation row r16 in each block
    if constexpr (KW == 1) {
        floatx4 acc[NB][MB];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int m = 0; m < MB; ++m) acc[b][m] = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int base = 0; base < KP; base += D) {
#pragma unroll
            for (int j = 0; j < D; ++j) {
                const int p = base + j;
                if (p >= KP) break;
                // slot (j + D - 1) % D held slice p - 1, whose fragments the previous MFMAs used
                if (p + D - 1 < KP) {
                    issue_w((j + D - 1) % D, p + D - 1);
                    issue_a((j + D - 1) % D, p + D - 1);
                }
                // slice p has landed: only loads issued after it may still be in flight (of the first
                // D - 1 slices every weight load came before every activation load)
                if (p + D - 1 >= KP) __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, kNoLgkm));
                else if (j < D - 2 && base == 0) __builtin_amdgcn_s_waitcnt(waitcnt_imm((D - 2) * 2 * MB + C::kLoads, kNoLgkm));
                else __builtin_amdgcn_s_waitcnt(waitcnt_imm((D - 1) * C::kLoads, kNoLgkm));
                const char* slot = ring + j * C::kSlot;
#pragma unroll
                for (int st = 0; st < 2; ++st) {
                    const int fo = st ? fo1 : fo0;
                    typename Frag<MODE>::T av[MB];
#pragma unroll
                    for (int m = 0; m < MB; ++m) av[m] = Frag<MODE>::acts(slot + (NB + m) * 2048 + fo);
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const typename Frag<MODE>::T wv = Frag<MODE>::weights(slot + b * 2048 + fo);
#pragma unroll
                        for (int m = 0; m < MB; ++m) acc[b][m] = mfma_step(wv, av[m], acc[b][m]);
                    }
                }
            }
        }
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            const int r = row0 + m * 16 + r16;
            if (r >= row1) continue;
            if constexpr (MODE == kExpand) {
#pragma unroll
                for (int b = 0; b < NB / 2; ++b) {
                    const int f = col0 + b * 16 + 4 * kg;
                    if (f < N) store_swiglu4(g, r, f, acc[b][m], acc[b + NB / 2][m]);
                }
            } else {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const int h = col0 + b * 16 + 4 * kg;
                    if (h < N) store_down4<MODE>(g, r, h, acc[b][m], sc[m]);
                }
            }
        }
    } else {
        constexpr int U = C::U, P = MODE == kExpand ? 2 : 1;
        floatx4 acc[U][P];   // block i = u * 4 + wave: weight block i / MB (and its up half), row block i % MB
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int h = 0; h < P; ++h) acc[u][h] = floatx4{0.f, 0.f, 0.f, 0.f};
        auto has = [&](int u) { return (u + 1) * SWAVES <= C::kUnits || u * SWAVES + wave < C::kUnits; };
        // the blocks of this wave over n slices, ascending: slots 0, D, 2 D .. of the waves' rings from `slots` on
        auto run = [&](const char* slots, auto n) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (!has(u)) continue;   // wave-uniform
                const int b = (u * SWAVES + wave) / MB, m = (u * SWAVES + wave) % MB;
                // every fragment is read before the first MFMA (a wave has few blocks, and their MFMAs are a
                // chain: with reads two or three ahead, as the compiler orders them, the chain waited for each)
                constexpr int N = decltype(n)::value;
                typename Frag<MODE>::T av[N][2];
                bf16x8 wv[N][2][P];
#pragma unroll
                for (int q = 0; q < N; ++q)
#pragma unroll
                    for (int st = 0; st < 2; ++st) {
                        const char* slot = slots + q * D * C::kSlot + (st ? fo1 : fo0);
                        av[q][st] = Frag<MODE>::acts(slot + (NB + m) * 2048);
#pragma unroll
                        for (int h = 0; h < P; ++h) wv[q][st][h] = *(const bf16x8*)(slot + (b + h * (NB / 2)) * 2048);
                    }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = 0; q < N; ++q)
#pragma unroll
                    for (int st = 0; st < 2; ++st)
#pragma unroll
                        for (int h = 0; h < P; ++h)
                            acc[u][h] = mfma_step(Frag<MODE>::wide(wv[q][st][h]), av[q][st], acc[u][h]);
            }
        };
        // a round: one slice of every wave; slice r of this wave is in slot j = r % D
        for (int r = 0, j = 0; r * SWAVES < slices; ++r, j = j + 1 == D ? 0 : j + 1) {
#pragma unroll
            for (int h = 0; h < SWAVES / G; ++h) {   // slices h * G .. h * G + G - 1 of the round
                // They have landed: of each wave that owns one, only loads issued after it are in flight,
                // kSteady slices while there are any left to issue (a wave that owns none of them has no more
                // than that in flight). Slice 0 with the weights first: the activations of slice 1.
                if (kWeightsFirst && r == 0) {
                    __builtin_amdgcn_s_waitcnt(waitcnt_imm((D - 1) * 2 * MB, 0));
                } else if (r + C::kSteady < KP) {
                    __builtin_amdgcn_s_waitcnt(waitcnt_imm(C::kSteady * C::kLoads, 0));
                } else {
                    __builtin_amdgcn_s_waitcnt(waitcnt_imm(kNoVm, 0));
                    wait_last<C::kLoads, C::kSteady - 1>(KP - 1 - r);
                }
                ring_barrier();
                // the G slices before these have been read: their waves reload the slots
                const int done = h ? r : r - 1;
                if ((G == SWAVES || wave / G != h) && done >= 0 && done + D < KP) {
                    const int slot = h ? j : (j ? j : D) - 1;
                    issue_w(slot, done + D);
                    issue_a(slot, done + D);
                }
                const int p = r * SWAVES + h * G;
                const char* const slots = lds + (h * G * D + j) * C::kSlot;
                if (p + G <= slices) run(slots, std::integral_constant<int, G>());
                else
                    for (int q = 0; p + q < slices; ++q) run(slots + q * D * C::kSlot, std::integral_constant<int, 1>());
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int b = (u * SWAVES + wave) / MB, m = (u * SWAVES + wave) % MB;
            const int r = row0 + m * 16 + r16, c = col0 + b * 16 + 4 * kg;
            if (!has(u) || r >= row1 || c >= N) continue;
            if constexpr (MODE == kExpand) store_swiglu4(g, r, c, acc[u][0], acc[u][1]);
            else store_down4<MODE>(g, r, c, acc[u][0], sc[u]);
        }
    }
}

// once: weights_once.
template <int MODE, int NB, int MB, int D, int KW, int G>
__global__ __launch_bounds__(SWAVES * 64) void gemm_lstream_kernel(GemmArgs g, int64_t mt_upper, int nt,
                                                                  bool once) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    __shared__ int s_tile[4];
    // the expansion runs a group's N tiles back to back (its gathered activation rows are then
    // shared through L2: 6% faster on the decode-shaped layer); the projection interleaves
    // the groups (4% faster than N tiles back to back there)
    const int64_t mt = MODE == kExpand ? blockIdx.x / nt : blockIdx.x % mt_upper;
    const int ntile = MODE == kExpand ? (int)(blockIdx.x % nt) : (int)(blockIdx.x / mt_upper);
    if (!find_tile<16 * MB>(g.offsets, g.n, g.a_rows, mt, s_tile)) return;
    if (once && s_tile[3] <= 16 * MB)   // the group's only row tile
        lstream_tile<MODE, NB, MB, D, KW, G, true>(g, lds, s_tile[0], s_tile[1], s_tile[2], ntile);
    else
        lstream_tile<MODE, NB, MB, D, KW, G, false>(g, lds, s_tile[0], s_tile[1], s_tile[2], ntile);
}

template <int MODE, int NB, int MB, int D, int KW = 1, int G = 1>
hipError_t launch_lstream_cfg(const GemmArgs& g, int64_t R, hipStream_t s) {
    using C = LStream<MODE, NB, MB, D, KW, G>;
    const int64_t mt_upper = most_tiles(g, R, 16 * MB);
    const int nt = (int)ceil_div(g.N, C::kWgCols);
    const int64_t grid = mt_upper * nt;
    if (grid <= 0) return hipSuccess;
    // set on every launch (idempotent, and the library keeps no state between calls)
    const hipError_t err = hipFuncSetAttribute((const void*)gemm_lstream_kernel<MODE, NB, MB, D, KW, G>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, C::kLds);
    if (err != hipSuccess) return err;
    gemm_lstream_kernel<MODE, NB, MB, D, KW, G><<<dim3((unsigned)grid), dim3(SWAVES * 64), C::kLds, s>>>(
        g, mt_upper, nt, weights_once(g, R, MODE));
    return hipGetLastError();
}

template <int MODE, int NB, int SDP>
hipError_t launch_stream_cfg(const GemmArgs& g, int64_t R, hipStream_t s) {
    const int64_t mt_upper = most_tiles(g, R, SROWS);
    constexpr int kWgCols = SWAVES * ((MODE == kExpand) ? NB * 8 : NB * 16);
    const int nt = (int)ceil_div(g.N, kWgCols);
    const int64_t grid = mt_upper * nt;
    if (grid <= 0) return hipSuccess;
    // the expansion runs a group's N tiles back to back (its gathered activation rows are then
    // shared through L2: 6% faster on the decode-shaped layer); the projection interleaves
    // the groups (4% faster than N tiles back to back there)
    const int n_fastest = MODE == kExpand ? 1 : 0;
    gemm_stream_kernel<MODE, NB, SDP><<<dim3((unsigned)grid), dim3(SWAVES * 64), 0, s>>>(g, mt_upper, nt, n_fastest);
    return hipGetLastError();
}

// 32-bit buffer offsets reach every row of `a` and of one group's weights.
inline bool offsets_reach(const GemmArgs& g) {
    return g.a_rows * g.K * 2 < (int64_t(1) << 32) && (int64_t)g.N * g.K * 2 < (int64_t(1) << 32);
}

// The streaming kernels whose waves share the slices of K (KW = 4). One group of rows: every
// output column block has few workgroups (2048 columns: 64 of 32), so each takes up to 64 rows at
// once, and the projection 16 columns per workgroup. Shared expert, H 2048, F 5632, the layer's three
// kernels: 1 row 55.9 -> 22.1 us, 48 rows 69.6 -> 25.4, 64 rows 87.3 -> 25.7 (the large tiles from 16
// rows on before, 8 to 44 workgroups). With every wave's own sums over its slices, added at the end,
// they took 18.9, 23.6 and 23.9, but u and y then differed in their last bits from every other kernel's.
//
// 16-column blocks per workgroup: one, or two where one makes more workgroups than there are compute
// units (the activations are then fetched half as often: 48 rows, H 2048, F 5632, the three kernels
// 33.8 -> 30.6 us).
inline int one_group_blocks(const GemmArgs& g, int64_t R) {
    return ceil_div(R, 64) * ceil_div(g.N, 16) > 256 ? 2 : 1;
}
// 16-row blocks per workgroup: with two column blocks all rows, up to 64; with one the fewest that
// leave no more workgroups than compute units. A workgroup fetches its rows' activations whole, at most 54 GB/s to
// a compute unit, so where columns alone leave units idle the rows are split over them too (H 2048,
// F 5632, the three kernels, cold weights: 32 rows 26.3 -> 23.4 us, 64 rows 33.3 -> 27.5; past 256
// workgroups, H 3072 and F 8192, the split loses: 64 rows 49.0 -> 53.1).
inline int one_group_row_blocks(const GemmArgs& g, int64_t R) {
    for (int m = 1; m < 4 && one_group_blocks(g, R) == 1; ++m)
        if (ceil_div(R, 16 * m) * ceil_div(g.N, 16) <= 256) return m;
    return (int)std::min<int64_t>(4, ceil_div(R, 16));
}
// One group of rows: rings of 64 to 80 KB (two workgroups fit a compute unit where there are that many),
// two slices of each wave where a slice is more than that allows; deeper rings measured slower (up to 144
// KB: 48 rows, three kernels 26.8 us). A barrier per four slices, per two where two slices of each wave are
// all the ring holds (H 2048, F 5632, 1 row, projection 21.8 us with a barrier per two slices, 17.8 with
// one per four).
template <int MODE, int NB, int MB>
hipError_t launch_stream_group(const GemmArgs& g, int64_t R, hipStream_t s) {
    constexpr int D = NB + MB == 2 ? 4 : (NB + MB == 3 ? 3 : 2);
    return launch_lstream_cfg<MODE, NB, MB, D, SWAVES, (D > 2 ? SWAVES : 2)>(g, R, s);
}
template <int MODE>
hipError_t launch_stream_shared(const GemmArgs& g, int64_t R, hipStream_t s) {
    if (!g.offsets) {
        constexpr int E = MODE == kExpand ? 2 : 1;   // weight blocks of 16 output columns
        const int mb = one_group_row_blocks(g, R);
        if (one_group_blocks(g, R) == 2) {
            switch (mb) {
                case 1: return launch_stream_group<MODE, 2 * E, 1>(g, R, s);
                case 2: return launch_stream_group<MODE, 2 * E, 2>(g, R, s);
                case 3: return launch_stream_group<MODE, 2 * E, 3>(g, R, s);
                default: return launch_stream_group<MODE, 2 * E, 4>(g, R, s);
            }
        }
        switch (mb) {
            case 1: return launch_stream_group<MODE, E, 1>(g, R, s);
            case 2: return launch_stream_group<MODE, E, 2>(g, R, s);
            case 3: return launch_stream_group<MODE, E, 3>(g, R, s);
            default: return launch_stream_group<MODE, E, 4>(g, R, s);
        }
    }
    // 32 rows per tile from a mean of 4 rows on, where groups of more than 16 become common (40
    // tokens on the Mixtral shape: expansion 339 -> 311 us, projection 210 -> 188; below, 0-2% slower).
    // Two slices of each wave in the ring and a barrier per two slices, so that three workgroups (two of
    // the 32-row ones) run on a compute unit: decode shape, 32 tokens, layer 2054 us, 2140 with three
    // slices and a barrier per four; 40 tokens on the Mixtral shape 474 and 539.
    return R >= 4 * (int64_t)g.n ? launch_lstream_cfg<MODE, 2, 2, 2, SWAVES, 2>(g, R, s)
                                 : launch_lstream_cfg<MODE, 2, 1, 2, SWAVES, 2>(g, R, s);
}

// The default of the streaming kernels. Sharing the slices pays from long sums on: expansions from H =
// 4096 (Mixtral shape, 3 tokens 206 -> 188 us, 60 tokens 360 -> 316; decode shape 1409 and 1413; H 2048,
// 64 experts, 24 tokens 75 -> 97), projections from F = 2048 (Mixtral shape, 3 tokens 110 -> 96 us, 60
// tokens 224 -> 189; F 2048 and H 1024, 16 experts, 8 tokens 14.3 -> 11.2; at F = 1408 34.7 -> 37.6), one
// group of rows from K = 512; with 16 rows per group and more (only when forced) there are workgroups
// enough.
// A forced depth of 2-6 runs the four waves side by side with that ring, 0 the register ring.
template <int MODE>
hipError_t launch_stream(const GemmArgs& g, int64_t R, hipStream_t s, int depth) {
    if (g.K % 64 == 0 && offsets_reach(g)) {
        const bool few = !g.offsets || R < 16 * (int64_t)g.n;
        if (depth < 0 && few && g.K >= (g.offsets ? (MODE == kExpand ? 4096 : 2048) : 512))
            return launch_stream_shared<MODE>(g, R, s);
        // ring depth 3 for the expansion and 2 for the projection (decode-shaped layer: 2-6 within
        // 0.5% for the expansion; the projection 3% slower at 3)
        const int dv = depth >= 0 ? depth : (MODE == kExpand ? 3 : 2);
        if (dv == 2) return launch_lstream_cfg<MODE, 2, 1, 2>(g, R, s);
        if (dv == 4) return launch_lstream_cfg<MODE, 2, 1, 4>(g, R, s);
        if (dv == 6) return launch_lstream_cfg<MODE, 2, 1, 6>(g, R, s);
        if (dv != 0) return launch_lstream_cfg<MODE, 2, 1, 3>(g, R, s);
    }
    // register-ring kernel: two 16-row blocks per wave, eight k-steps in flight (four or six
    // blocks, or six steps, measured 1-3% slower on the decode-shaped layer)
    return launch_stream_cfg<MODE, 2, 8>(g, R, s);
}

// ---------------------------------------------------------------------- launch
template <class C, int MODE, bool IL, class CT = LargeIlTail>
hipError_t launch_cfg(const GemmArgs& g, int64_t R, hipStream_t s, const GemmTune& t) {
    // set on every launch (idempotent, and the library keeps no state between calls)
    const void* fn;
    if constexpr (IL)
        fn = (const void*)gemm_il_kernel<C, CT, MODE>;
    else
        fn = (const void*)gemm_staged_kernel<C, MODE>;
    const hipError_t err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES);
    if (err != hipSuccess) return err;
    const int64_t mt_upper = most_tiles(g, R, C::BM);
    constexpr int kOutCols = (MODE == kExpand) ? C::BNB / 2 : C::BNB;
    const int nt = (int)ceil_div(g.N, kOutCols);
    if (mt_upper * nt <= 0) return hipSuccess;
    const int group_n = t.group_n > 0 ? t.group_n : 4;
    if constexpr (IL) {
        // default: one group of rows the orders tuned for it; grouped rows the expert-major order,
        // except for
        //  - an expansion of at least 16 N tiles with a mean below 256 rows, few of whose row tiles
        //    share a weight tile: the grouped order, which has every XCD walk all groups over N tiles
        //    of its own (Mixtral shape: 203 tokens 380 -> 351 us, 400 tokens 415 -> 387, 768 tokens
        //    500 -> 492; equal at 1024 tokens);
        //  - a projection whose tiles fill fewer than 4 rounds of the chip (or that splits K): the
        //    longest-first order, whose short items fill the last round (the expert-major order was 17%
        //    slower on the Mixtral-shaped projection without a K split), unless most row tiles are
        //    tails (203 tokens there: longest first 216 us, expert-major 202; 512 tokens 271 and 302)
        int order = t.order;
        if (order < 0 || order > 2) {
            if (g.offsets == nullptr) order = MODE == kExpand ? kGrouped : kLongestFirst;
            else if (MODE == kExpand) order = nt >= 16 && R < 256 * (int64_t)g.n ? kGrouped : kExpertMajor;
            else order = !mostly_tails(g, R) && (g.ksplit > 1 || mt_upper * nt < 4 * 256) ? kLongestFirst : kExpertMajor;
        }
        // the searches of il_item and em_item run in 32-bit integers (item counts times 8)
        if ((mt_upper + g.n + 1) * nt * g.ksplit >= (int64_t(1) << 27)) order = kGrouped;
        int64_t grid;
        int gparam = group_n;
        if (order == kLongestFirst) {
            // each XCD's run holds at most ceil(long / 8) + ceil(2 * short / 8) items, where
            // long + short <= mt_upper * nt * ksplit and short <= groups * nt * ksplit
            const int64_t groups = g.offsets ? g.n : 1;
            grid = (ceil_div((mt_upper + groups) * nt * g.ksplit, 8) + 2) * 8;
        } else if (order == kExpertMajor) {
            // each XCD's run holds at most ceil(items / 8) <= ceil(mt_upper * nt * ksplit / 8)
            // window 8: with three weight stages 0.2-1.1% ahead of 12, 16 and 24 on the three
            // grouped workloads (12 was best with two)
            grid = ceil_div(mt_upper * nt * g.ksplit, 8) * 8;
            gparam = t.window > 0 ? t.window : 8;
        } else {
            grid = ceil_div(mt_upper * nt, 8) * 8 * g.ksplit;
        }
        gemm_il_kernel<C, CT, MODE><<<dim3((unsigned)grid), dim3(C::NT), C::LDS_BYTES, s>>>(
            g, mt_upper, nt, gparam, order, weights_once(g, R, MODE));
    } else {
        const int64_t grid = ceil_div(mt_upper * nt, 8) * 8 * g.ksplit;
        gemm_staged_kernel<C, MODE><<<dim3((unsigned)grid), dim3(C::NT), C::LDS_BYTES, s>>>(g, mt_upper, nt, group_n);
    }
    return hipGetLastError();
}

// Tile family: a forced choice (tile = 'S', 'M', 'L' or 'W', for tests and tuning), otherwise by the
// mean rows per group (below 16 the streaming kernel, else the large tiles, in whose place pick_shape
// may then take smaller ones). The large tiles
// address `a` and one group's weights through 32-bit buffer offsets, so both must stay below
// 4 GiB (a_bytes: all rows of `a`; w_bytes: one group's weights).
char pick_tile(int64_t R, int groups, int64_t a_bytes, int64_t w_bytes, char tile) {
    const bool large_ok = a_bytes < (int64_t(1) << 32) && w_bytes < (int64_t(1) << 32);
    if (tile == 'S' || tile == 'M' || tile == 'L' || tile == 'W')
        return (tile == 'L' || tile == 'W') && !large_ok ? 'M' : tile;
    // below 16 rows per group the streaming kernel (weights streamed once, little MFMA work
    // wasted on padding); from 16 on the large tiles, which were faster than the medium ones
    // at every size measured (Mixtral-shaped, 1024 tokens: 2.6 -> 0.87 ms for the two GEMMs
    // and the combine) and, of grouped rows, than the streaming kernel; the medium tiles only
    // where the large tiles' 32-bit offsets would not reach
    const int64_t mean = R / (groups > 0 ? groups : 1);
    if (mean < 16) return 'S';
    return large_ok ? 'L' : 'M';
}

}  // namespace

int down_ksplit(int64_t R, int n, int H, int F, char tile) {
    // only the large-tile kernel slices K; its grid is (R/256 + n) x (H/256) tiles. Below one
    // round of the chip the K split doubles the workgroups; from one round on the longest-first
    // order (tail items as halves) fills the last round as well without the second o slice
    // (Mixtral-shaped projection and combine 922 -> 902 us, with 268 MB less o traffic)
    const char t = pick_tile(R, n, R * F * 2, (int64_t)H * F * 2, tile);
    if (t != 'L' && t != 'W') return 1;
    const int64_t tiles = (ceil_div(R, 256) + n) * ceil_div(H, 256);
    return (tiles < 256 && (F / 2) % 64 == 0 && F / 32 >= 128) ? 2 : 1;
}

namespace {
// The element types of the ring tiles (gemm_ring.h): the fragments and MFMAs of the other kernels.
template <int MODE>
struct ElemB16 {
    static constexpr int SIZE = 2, NJ = 1;
    using T = typename Frag<MODE>::T;
    using Silu = FastSilu;
    __device__ static T weights(const char* p) { return Frag<MODE>::weights(p); }
    __device__ static T acts(const char* p) { return Frag<MODE>::acts(p); }
    __device__ static floatx4 step(int, const T& w, const T& a, floatx4 c) { return mfma_step(w, a, c); }
};

// Ring tiles: 64 rows x 128 or 64 weight rows, two or three workgroups on a compute unit.
using RingWide = RCfg<64, 128, 2, 2, 3>;
using RingNarrow = RCfg<64, 64, 2, 2, 3>;
using RingWideTail = RCfg<32, 128, 2, 2, 3>;
using RingNarrowTail = RCfg<32, 64, 2, 2, 4>;

// The shape that the large tiles' work runs in when no kernel is forced: 'L', or smaller tiles where
// the large ones would leave most of the chip idle: 'R' RingWide, 'N' RingNarrow, 'S' the streaming
// kernel with shared slices (one group of rows). Every kernel here is bound by the bytes a compute
// unit loads, 54 KB per us whatever the tile (large tiles 64 KB per 64-wide K stage and 1.18 us,
// RingWide 24 KB and 0.42-0.48 us, RingNarrow 16 KB and 0.26-0.37 us, streaming 10-12 KB and
// 0.12-0.3 us), so smaller tiles move more bytes per output but spread over more compute units. The
// times below are those rates over 256 compute units (shared expert, H 2048, F 5632, expansion and
// projection in us, L / R / N / S: 64 rows 29 49 / 19 45 / 16 34 / 15 13; 256 rows 43 106 / 29 44 /
// 28 34 / 35 22; 1000 rows 52 102 / 73 45 / 82 48 / 129 83; 4096 rows 147 107 / 271 159 / 398 220 /
// 451 307). The smaller tiles are taken where they come out a fifth faster. Groups of fewer than 40
// rows on average are bound by their weights, and one 64-row tile wastes least (OLMoE shape, 256
// tokens: expansion 116 -> 108 us, projection with mix and combine 87 -> 78; where the projection
// splits K the large tiles are faster, Mixtral shape, 128 tokens 187 against 208 us). Each shape sums K in
// the large tiles' order.
char pick_shape(const GemmArgs& g, int64_t R, bool expand) {
    const double KT = (double)(g.K / g.ksplit) / 64, ne = g.offsets ? (double)(R < g.n ? R : g.n) : 1;
    if (g.offsets && g.ksplit == 1 && R < 40 * ne) return 'R';
    auto tiles = [&](int BM, int cols) {
        const double rows = g.offsets ? ((double)R / BM + ne / 2 > ne ? (double)R / BM + ne / 2 : ne) : (double)ceil_div(R, BM);
        return rows * (double)(ceil_div(g.N, cols) * g.ksplit) / 256;
    };
    auto most = [](double a, double b) { return a > b ? a : b; };
    auto up = [](double v) { return (double)(int64_t)(v + 0.999); };
    const int half = expand ? 2 : 1;   // gate and up rows of each output column
    const double large = KT * up(tiles(256, 256 / half)) * (R <= 128 * ne ? 0.89 : 1.18) + 6;
    const double wide = KT * most(0.48, 0.42 * tiles(64, 128 / half)) + 4;
    const double narrow = KT * most(0.37, 0.26 * tiles(64, 64 / half)) + 4;
    double best = 0.8 * large;
    char t = 'L';
    if (wide < best) { best = wide; t = 'R'; }
    if (narrow < best) { best = narrow; t = 'N'; }
    if (!g.offsets && g.K >= 512) {
        // the blocks that launch_stream_shared takes; a slice takes its bytes' time, or 0.12 us
        const int nb = one_group_blocks(g, R), mb = one_group_row_blocks(g, R);
        const double stream = KT * up(tiles(16 * mb, 16 * nb)) * most(0.12, 2.0 * (half * nb + mb) / 54) + 3.5;
        if (stream < best) t = 'S';
    }
    return t;
}

template <int MODE>
hipError_t launch_mode(const GemmArgs& g, int64_t R, hipStream_t s, const GemmTune& tune, char t) {
    if (t == 'S') return launch_stream<MODE>(g, R, s, tune.stream_depth);
    if (t == 'R') return launch_ring<ElemB16<MODE>, RingWide, RingWideTail, MODE>(g, R, s, 1);
    if (t == 'N') return launch_ring<ElemB16<MODE>, RingNarrow, RingNarrowTail, MODE>(g, R, s, 1);
    if (t == 'M') return launch_cfg<MediumStaged, MODE, false>(g, R, s, tune);
    // the large tiles: eight waves for the expansion, four for the projections (interleaved
    // A/B, bit-identical: expansion -2.7% / -2.4% / -0.3% on the Mixtral-, OLMoE- and
    // fine-grained-shaped layers, projections +1% to +1.7%), and for projections of mostly tail
    // tiles (the same shapes as the expert-major order below: Mixtral shape, 203 tokens 205 -> 202 us)
    if (t == 'W' || (t == 'L' && tune.tile != 'L' && (MODE == kExpand || mostly_tails(g, R))))
        return launch_cfg<WideIl, MODE, true, WideIlTail>(g, R, s, tune);
    return launch_cfg<LargeIl, MODE, true>(g, R, s, tune);
}
}  // namespace

hipError_t launch_gemm_bf16(GemmMode mode, const GemmArgs& g0, int64_t R, hipStream_t s,
                            const GemmTune& tune) {
    GemmArgs g = g0;
    if (g.ksplit < 1) g.ksplit = 1;
    char t = pick_tile(R, g.offsets ? g.n : 1, g.a_rows * g.K * 2, (int64_t)g.N * g.K * 2, tune.tile);
    if (g.ksplit > 1 && (mode != kDownStore || (t != 'L' && t != 'W'))) return hipErrorInvalidValue;
    if (tune.tile == 0 && t == 'L') t = pick_shape(g, R, mode == kExpand);
    switch (mode) {
        case kExpand: return launch_mode<kExpand>(g, R, s, tune, t);
        case kDownStore:
            return g.b_f16 ? launch_mode<kDownStore | kHalfW>(g, R, s, tune, t)
                           : launch_mode<kDownStore>(g, R, s, tune, t);
        default:
            return g.b_f16 ? launch_mode<kDownAccum | kHalfW>(g, R, s, tune, t)
                           : launch_mode<kDownAccum>(g, R, s, tune, t);
    }
}

hipError_t launch_widen_f16(const uint16_t* src, int64_t count, uint16_t* dst, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    const int64_t n8 = count / 8;
    const int64_t blocks = n8 > 0 ? (ceil_div(n8, 256) < 8192 ? ceil_div(n8, 256) : 8192) : 1;
    widen_kernel<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(src, count, dst);
    return hipGetLastError();
}

}  // namespace pcm
