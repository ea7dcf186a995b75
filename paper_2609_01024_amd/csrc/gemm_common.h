// Device code shared by the grouped GEMM kernels (gemm_bf16.hip, gemm_f32.hip): row and work-item
// lookup, the s_waitcnt encoding and the epilogue.
#pragma once
#include "internal.h"

#define PCM_LDS __attribute__((address_space(3)))
#define PCM_GLOBAL __attribute__((address_space(1)))

namespace pcm {
namespace {

// s_waitcnt immediates (gfx9 encoding: vmcnt[3:0]+[15:14], expcnt[6:4], lgkmcnt[11:8])
constexpr int waitcnt_imm(int vm, int lgkm) {
    return (vm & 0xF) | (7 << 4) | ((lgkm & 0xF) << 8) | (((vm >> 4) & 3) << 14);
}
constexpr int kNoVm = 63, kNoLgkm = 15;

// Most row tiles of BM rows that R rows make in the groups of g: a group with c rows has
// ceil(c / BM) <= (c + BM - 1) / BM tiles, and at most min(n, R) groups have rows.
inline int64_t most_tiles(const GemmArgs& g, int64_t R, int BM) {
    if (!g.offsets) return ceil_div(R, BM);
    return (R + (BM - 1) * (R < g.n ? R : g.n)) / BM;
}

// Cache policy of a weight load: non-temporal where every weight is read once (weights_once).
constexpr int weight_policy(bool nt) { return nt ? 2 : 0; }

// Whether a grouped product's weights are worth reading non-temporally by the groups of a single row
// tile, which read each of them once (the kernels check that): together they are more than half of the
// 256 MB MALL, so that little of them is left there from the call before. A plain stream of 8 GB then reads at 7.1 TB/s instead of 6.2,
// whatever the pattern (128 to 1024 bytes of a row, rows 2 to 28 KB apart). Decode shape, 32 tokens:
// expansion 1548 -> 1376 us, projection 797 -> 717; Mixtral shape, 3 tokens 136 -> 126 and 87 -> 77; 40
// tokens 312 -> 286 and 190 -> 173. Weights that stay in the MALL between calls are slower that way
// (shared expert of 69 MB 31.1 -> 33.2 us, OLMoE shape, 1 token, projection 21.0 -> 22.6), as is a
// second row tile (OLMoE shape, 100 tokens on 16-row tiles without that check, 73 -> 79 us).
inline bool weights_once(const GemmArgs& g, int64_t R, int mode) {
    const int64_t groups = R < g.n ? R : g.n;
    // (from a mean of 512 rows on few groups are that small, and the check costs 0.3% of the fine-grained
    // prefill)
    return g.offsets && R < 512 * (int64_t)g.n && groups * g.N * g.K * (mode == kExpand ? 4 : 2) >= (int64_t(128) << 20);
}

// A mean of fewer than 96 rows per group: most row tiles are tail tiles of at most 128 rows.
inline bool mostly_tails(const GemmArgs& g, int64_t R) { return g.offsets && R < 96 * (int64_t)g.n; }

// First row and row count of groups 4 * lane .. 4 * lane + 3 (0 rows past n; without offsets one group
// of a_rows rows). The five offsets are loaded without branches and waited for once: behind the bounds
// check of each group they were four loads one after another, 1.5 us of every workgroup's start.
__device__ __forceinline__ void group_bounds(const int32_t* __restrict__ offsets, int n, int64_t a_rows, int lane,
                                             int (&lo)[4], int (&cnt)[4]) {
    if (offsets == nullptr) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            lo[j] = 0;
            cnt[j] = lane == 0 && j == 0 ? (int)a_rows : 0;
        }
        return;
    }
    int o[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) o[j] = offsets[min(lane * 4 + j, n)];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        lo[j] = o[j];
        cnt[j] = o[j + 1] - o[j];   // past n both are offsets[n]
    }
}

// Source row of A row r of the tile (rows past row1 repeat a valid row; their outputs are
// never stored).
__device__ inline int64_t a_source_row(const GemmArgs& g, int r, int row1) {
    if (r >= row1) r = row1 - 1;
    int64_t src = r;
    if (g.gather) {
        src = g.gather[r];
        src = src < 0 ? 0 : (src >= g.a_rows ? g.a_rows - 1 : src);
    }
    return src;
}

// Row of `a` (and of row_scale) behind output row r.
__device__ inline int64_t scale_row(const GemmArgs& g, int r) {
    if (!g.gather) return r;
    const int64_t s = g.gather[r];
    return s < 0 ? 0 : (s >= g.a_rows ? g.a_rows - 1 : s);
}

// SiLU(g) = g / (1 + e^-g) with the hardware reciprocal (about 1 ulp) instead of an IEEE
// division; for g below about -88, e^-g is +inf and the result is -0.
__device__ inline float silu(float g) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }
struct FastSilu {
    __device__ static float silu(float g) { return pcm::silu(g); }
};

// Shared epilogue: acc[nb][mb] holds C[row = .. + (lane & 15)][cols c0 .. c0+3].
template <int MODE, int MB, int NBK, int WTM, int WTN, int OUT_COLS, class SILU = FastSilu>
__device__ inline void epilogue(const GemmArgs& g, const floatx4 (&acc)[NBK][MB], int row0,
                                int row1, int ntile, int wm, int wn, int lane) {
    const int N = g.N;
    // The row scales of all of this lane's rows are loaded first, without branches, and
    // waited for once, in code that every store follows. A scale load that is still in
    // flight where the stores' branches (row and column bounds) merge makes the compiler
    // wait for all outstanding memory operations before each store, the earlier stores
    // included: the 64 stores of a wave then ran one after another (13 us of a 256 x 256
    // projection tile).
    float scs[MB];
    if constexpr (MODE != kExpand) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int r = min(row0 + wm * WTM + mb * 16 + (lane & 15), row1 - 1);
            scs[mb] = g.row_scale ? g.row_scale[scale_row(g, r)] : 1.0f;
        }
        __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, kNoLgkm));
    }
    if constexpr (MODE == kExpand) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int r = row0 + wm * WTM + mb * 16 + (lane & 15);
            if (r >= row1) continue;
#pragma unroll
            for (int nb = 0; nb < NBK / 2; ++nb) {
                const int f = ntile * OUT_COLS + wn * (WTN / 2) + nb * 16 + (lane >> 4) * 4;
                if (f >= N) continue;
                const floatx4 gt = acc[nb][mb], up = acc[nb + NBK / 2][mb];
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = SILU::silu(gt[i]) * up[i];
                *(float4*)((float*)g.out + (int64_t)r * N + f) = make_float4(v[0], v[1], v[2], v[3]);
            }
        }
    } else if (base_mode(MODE) == kDownAccum && g.accumulate) {
        // read-modify-write: each row block's values are loaded before its stores
        float* O = (float*)g.out;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int r = row0 + wm * WTM + mb * 16 + (lane & 15);
            if (r >= row1) continue;
            float4 prev[NBK];
#pragma unroll
            for (int nb = 0; nb < NBK; ++nb) {
                const int h = min(ntile * OUT_COLS + wn * WTN + nb * 16 + (lane >> 4) * 4, N - 4);
                prev[nb] = *(const float4*)(O + (int64_t)r * N + h);
            }
            const float sc = scs[mb];
#pragma unroll
            for (int nb = 0; nb < NBK; ++nb) {
                const int h = ntile * OUT_COLS + wn * WTN + nb * 16 + (lane >> 4) * 4;
                if (h >= N) continue;
                // the stored value plus the scaled product, each rounded (no fused multiply-add),
                // so that accumulating adds exactly what the store path writes
                *(float4*)(O + (int64_t)r * N + h) = make_float4(
                    __fadd_rn(prev[nb].x, __fmul_rn(acc[nb][mb][0], sc)), __fadd_rn(prev[nb].y, __fmul_rn(acc[nb][mb][1], sc)),
                    __fadd_rn(prev[nb].z, __fmul_rn(acc[nb][mb][2], sc)), __fadd_rn(prev[nb].w, __fmul_rn(acc[nb][mb][3], sc)));
            }
        }
    } else {
        float* O = (float*)g.out;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int r = row0 + wm * WTM + mb * 16 + (lane & 15);
            if (r >= row1) continue;
            const float sc = scs[mb];
#pragma unroll
            for (int nb = 0; nb < NBK; ++nb) {
                const int h = ntile * OUT_COLS + wn * WTN + nb * 16 + (lane >> 4) * 4;
                if (h >= N) continue;
                *(float4*)(O + (int64_t)r * N + h) = make_float4(acc[nb][mb][0] * sc, acc[nb][mb][1] * sc,
                                                                 acc[nb][mb][2] * sc, acc[nb][mb][3] * sc);
            }
        }
    }
}

// Work item of workgroup bid in the expert-major order. Group x has m_x = ceil(rows / BM)
// M-tiles; its m_x * nt items are walked in blocks of gn_x N-tiles (gn_x = window / m_x,
// at least 1), the M-tile varying slowest within a block, so that the `window` workgroups
// an XCD runs at once cover all of a group's rows for a few N-tiles: each weight tile is
// fetched while every row block that needs it runs, each activation tile once per block.
// Each XCD (bid % 8) takes a contiguous eighth of the list (every K slice, slice-major), or, with
// `interleave`, for groups of at least 16 N tiles in multiples of 8, every eighth window (below). A last
// row block of at most TBM rows runs as the shorter tail tile.
// Wave 0 counts and searches; the result is broadcast through LDS (s_item: group, row0, row1,
// ntile, kslice, valid). Returns false past the last item.
template <int BM, int TBM>
__device__ bool em_item(const GemmArgs& g, int nt, int window, bool interleave, int* s_item) {
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        int lo[4], cnt[4], m[4], local = 0;
        group_bounds(g.offsets, g.n, g.a_rows, lane, lo, cnt);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            m[j] = (cnt[j] + BM - 1) / BM;
            local += m[j] * nt;
        }
        const int x8 = (int)(blockIdx.x % 8), j8 = (int)(blockIdx.x / 8);
        if (interleave && g.ksplit == 1 && nt % 8 == 0 && nt >= 16) {
            // Window-interleaved assignment: a group's N tiles are cut into windows of gw tiles,
            // gw the largest divisor of nt / 8 not above window / m (so that every window has
            // the same width and their number is a multiple of 8), and window i runs on XCD
            // i % 8. Every XCD then holds exactly an eighth of every group's items and works
            // through the groups in step with the others (the same mix of tile shapes at the
            // same time), instead of the XCDs holding different groups whose tiles take
            // different times (Mixtral-shaped expansion -1.9%); within a window the M-tile
            // varies slowest. With fewer than 16 N tiles a group's activation rows would be
            // fetched by every XCD for one N tile each (OLMoE-shaped projection +5%), so the
            // contiguous eighths below stay.
            // A group whose last row block takes the tail tile walks its windows over the full
            // row blocks first and then that row block over the same N tiles. Within an XCD the
            // hardware deals workgroups to its four shader arrays in strict rotation, one
            // array's turn waiting for a free compute unit there; with the tail row inside every
            // window the tail tiles repeat with the window's period and, where that period is
            // even, fall on the same one or two arrays, whose turns then come round faster than
            // the others' (Mixtral-shaped expansion: per-workgroup timelines, all 70 tail tiles
            // of an XCD on two of its arrays, 13% more work on the other two). A run of one
            // group's tail tiles gives every array the same mix: the mean gap between two tiles
            // on a compute unit fell from 4.8 to 1.1 us, the expansion 0.7% faster (its tiles
            // run slower with the compute units fuller, the clock falling under the load).
            const int n8 = nt / 8;
            int xl = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) xl += m[j] * n8;
            const int xincl = wave_incl_scan_i32(xl);
            const bool valid = j8 < __builtin_amdgcn_readlane(xincl, 63);
            if (lane == 0) s_item[5] = valid ? 1 : 0;
            if (valid) {
                // this lane's group that holds item j8 (at most one lane has one); the divisions are
                // then done once, by that lane
                int start = xincl - xl, hit = -1, q = 0, mm_ = 0, lo_ = 0, cnt_ = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool in = j8 >= start && j8 < start + m[j] * n8;
                    hit = in ? j : hit;
                    q = in ? j8 - start : q;
                    mm_ = in ? m[j] : mm_;
                    lo_ = in ? lo[j] : lo_;
                    cnt_ = in ? cnt[j] : cnt_;
                    start += m[j] * n8;
                }
                if (hit >= 0) {
                    const int last = cnt_ - (mm_ - 1) * BM;   // rows of the last row block
                    const int mf = last <= TBM ? mm_ - 1 : mm_;
                    const int lim = window / (mf > 0 ? mf : 1);
                    int gw = lim < 1 ? 1 : (lim > n8 ? n8 : lim);
                    while (n8 % gw != 0) --gw;
                    int mm, col;
                    if (q < mf * n8) {              // the full row blocks, window by window
                        const int gsize = gw * mf;
                        const int kw = q / gsize, in = q - kw * gsize;
                        mm = in / gw;
                        col = (kw * 8 + x8) * gw + (in - mm * gw);   // window kw * 8 + x8
                    } else {                        // the tail row block, same N tiles
                        const int t = q - mf * n8;
                        mm = mm_ - 1;
                        col = ((t / gw) * 8 + x8) * gw + t % gw;
                    }
                    const int r0 = lo_ + mm * BM;
                    s_item[0] = lane * 4 + hit;
                    s_item[1] = r0;
                    s_item[2] = min(lo_ + cnt_, r0 + BM);
                    s_item[3] = col;
                    s_item[4] = 0;
                }
            }
        } else {
            const int incl = wave_incl_scan_i32(local);
            // 32-bit arithmetic throughout: the host keeps item counts (times 8) within range
            const int Tt = __builtin_amdgcn_readlane(incl, 63), TT = Tt * g.ksplit;
            const int l0 = x8 * TT / 8, l1 = (x8 + 1) * TT / 8;
            const bool valid = j8 < l1 - l0;
            if (lane == 0) s_item[5] = valid ? 1 : 0;
            if (valid) {
                const int item = l0 + j8;
                const int kslice = item / Tt;
                const int id = item - kslice * Tt;
                int start = incl - local, hit = -1, l = 0, mm_ = 1, lo_ = 0, cnt_ = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool in = id >= start && id < start + m[j] * nt;
                    hit = in ? j : hit;
                    l = in ? id - start : l;
                    mm_ = in ? m[j] : mm_;
                    lo_ = in ? lo[j] : lo_;
                    cnt_ = in ? cnt[j] : cnt_;
                    start += m[j] * nt;
                }
                if (hit >= 0) {
                    int gn = window / mm_;
                    gn = gn < 1 ? 1 : (gn > nt ? nt : gn);
                    const int gsize = gn * mm_;
                    const int grp = l / gsize, in = l - grp * gsize;
                    const int gcols = min(gn, nt - grp * gn);
                    const int mm = in / gcols;
                    const int r0 = lo_ + mm * BM;
                    s_item[0] = lane * 4 + hit;
                    s_item[1] = r0;
                    s_item[2] = min(lo_ + cnt_, r0 + BM);
                    s_item[3] = grp * gn + (in - mm * gcols);
                    s_item[4] = kslice;
                }
            }
        }
    }
    __syncthreads();
    return s_item[5] != 0;
}

}  // namespace
}  // namespace pcm
