// Path table and grouped dispatch layout (Section 4.2: inactive paths are masked out
// before weighting, with m_ii = 1; Section 4.3: dispatch metadata grouped by expansion
// source so that each (token, source) expansion runs once).
//
// Per token (one thread each): the active paths Pi = {(a,b): a == b or m[e_a][e_b]}, their
// weights beta, and the token's k rows. Rows are ordered by (expert, token); the rank of a
// row inside its expert is found without atomics whose order matters:
//   - each wave of 64 tokens ORs its lane bit into words[wave][e] for each selected e
//     (OR is order-independent, so the words are deterministic);
//   - rows of e before token (wave, lane) = rows of e in earlier blocks (a scan over
//     block counts) + in earlier waves of this block (popcounts) + popcount(words[wave][e]
//     & lanes below this one).
// T <= 256 runs as one launch (paths_small_kernel); larger T as count / scan / scatter launches.
#include "internal.h"

namespace pcm {

namespace {

constexpr int kWaves = kPathBlock / 64;

enum Phase { kFused = 0, kCount = 1, kScatter = 2 };

struct PathSmem {
    unsigned long long words[kWaves][kMaxN];
    int prefix[kWaves][kMaxN];
    int scan[kMaxN];
};

// Exclusive scan of smem.scan[0..n) in place; returns the total to every thread.
__device__ int block_exclusive_scan(int* scan, int n) {
    const int tid = threadIdx.x;
    int own = (tid < n) ? scan[tid] : 0;
    for (int d = 1; d < kMaxN; d <<= 1) {
        int v = (tid < kMaxN && tid >= d) ? scan[tid - d] : 0;
        __syncthreads();
        if (tid < kMaxN) scan[tid] += v;
        __syncthreads();
    }
    const int total = scan[kMaxN - 1];
    __syncthreads();
    if (tid < kMaxN) scan[tid] -= own;
    __syncthreads();
    return total;
}

template <int PH>
__global__ __launch_bounds__(kPathBlock) void paths_kernel(
    const int32_t* __restrict__ ids, const float* __restrict__ w, const uint8_t* __restrict__ mask,
    int64_t T, int n, int k, int beta_mode, uint64_t* __restrict__ bits_out,
    float* __restrict__ beta_out, int32_t* __restrict__ row_token, int32_t* __restrict__ row_slot,
    int32_t* __restrict__ row_of, int32_t* __restrict__ block_counts) {
    __shared__ PathSmem sm;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    for (int i = tid; i < kWaves * kMaxN; i += kPathBlock) (&sm.words[0][0])[i] = 0ull;
    __syncthreads();

    const int64_t t = (int64_t)blockIdx.x * kPathBlock + tid;
    const bool valid = t < T;
    int e[kMaxK];
#pragma unroll
    for (int a = 0; a < kMaxK; ++a) {
        int v = (valid && a < k) ? ids[t * k + a] : 0;
        e[a] = v < 0 ? 0 : (v >= n ? n - 1 : v);
    }
    if (valid) {
        if (PH != kScatter) {
            float p[kMaxK];
#pragma unroll
            for (int a = 0; a < kMaxK; ++a) p[a] = a < k ? w[t * k + a] : 0.0f;
            // every (a, b) entry is loaded (e[] is always a valid id), so the 64 loads are
            // issued together instead of one dependent load per branch
            uint8_t mv[kMaxK][kMaxK];
#pragma unroll
            for (int a = 0; a < kMaxK; ++a)
#pragma unroll
                for (int b = 0; b < kMaxK; ++b) mv[a][b] = mask[(int64_t)e[a] * n + e[b]];
            uint64_t bits = 0;
#pragma unroll
            for (int a = 0; a < kMaxK; ++a)
#pragma unroll
                for (int b = 0; b < kMaxK; ++b)
                    if (a < k && b < k && (a == b || mv[a][b])) bits |= 1ull << (a * k + b);
            bits_out[t] = bits;
            float global = 0.0f;
#pragma unroll
            for (int a = 0; a < kMaxK; ++a)
#pragma unroll
                for (int b = 0; b < kMaxK; ++b)
                    if (a < k && b < k && ((bits >> (a * k + b)) & 1))
                        global = fmaf(p[a], p[b], global);  // explicit: one rounding per term
            float* bt = beta_out + t * k * k;
#pragma unroll
            for (int a = 0; a < kMaxK; ++a) {
                if (a >= k) break;
                float src = 0.0f;  // sum of p over the targets of source a
#pragma unroll
                for (int b = 0; b < kMaxK; ++b)
                    if (b < k && ((bits >> (a * k + b)) & 1)) src += p[b];
#pragma unroll
                for (int b = 0; b < kMaxK; ++b) {
                    if (b >= k) break;
                    float v = 0.0f;
                    if ((bits >> (a * k + b)) & 1) {
                        // p_a (p_b / src) rather than a reciprocal: stays exact (beta_aa = p_a
                        // for a source whose only target is itself) when p is subnormal
                        v = beta_mode == 0 ? p[a] * (p[b] / src)
                                           : (beta_mode == 1 ? p[a] * p[b] : p[a] * p[b] / global);
                    }
                    bt[a * k + b] = v;
                }
            }
        }
#pragma unroll
        for (int a = 0; a < kMaxK; ++a)
            if (a < k) atomicOr(&sm.words[wave][e[a]], 1ull << lane);
    }
    __syncthreads();

    // rows of each expert in the earlier waves of this block
    for (int x = tid; x < kMaxN; x += kPathBlock) {
        int run = 0;
        if (x < n) {
#pragma unroll
            for (int v = 0; v < kWaves; ++v) {
                sm.prefix[v][x] = run;
                run += __popcll(sm.words[v][x]);
            }
        }
        sm.scan[x] = run;
    }
    __syncthreads();

    if (PH == kCount) {
        for (int x = tid; x < n; x += kPathBlock) block_counts[(int64_t)blockIdx.x * n + x] = sm.scan[x];
        return;
    }
    for (int x = tid; x < n; x += kPathBlock) sm.scan[x] = block_counts[(int64_t)blockIdx.x * n + x];
    __syncthreads();
    if (valid) {
        const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
        for (int a = 0; a < kMaxK; ++a) {
            if (a >= k) break;
            const int x = e[a];
            const int pos = sm.scan[x] + sm.prefix[wave][x] + __popcll(sm.words[wave][x] & below);
            row_token[pos] = (int32_t)t;
            row_slot[pos] = a;
            row_of[t * k + a] = pos;
        }
    }
}

// T <= 256 in one workgroup: a thread per (token, slot) pair, at most two pairs each. Bound by the
// latency of its dependent loads (ids, then mask bytes) and its barriers: a thread per token, as in
// paths_kernel, left 24 tokens of top-8 on 24 threads with 64 mask loads, sums and divisions in a row
// each: 17.8 us; this way 6.5 us. The operations on each value and their order are paths_kernel's.
constexpr int kSmallThreads = 1024;
__global__ __launch_bounds__(kSmallThreads) void paths_small_kernel(
    const int32_t* __restrict__ ids, const float* __restrict__ w, const uint8_t* __restrict__ mask,
    int T, int n, int k, int beta_mode, uint64_t* __restrict__ bits_out, float* __restrict__ beta_out,
    int32_t* __restrict__ offsets, int32_t* __restrict__ row_token, int32_t* __restrict__ row_slot,
    int32_t* __restrict__ row_of) {
    constexpr int PER = kPathBlock * kMaxK / kSmallThreads;   // pairs per thread
    __shared__ unsigned long long words[kWaves][kMaxN];
    __shared__ int e_s[kPathBlock * kMaxK];
    __shared__ float p_s[kPathBlock * kMaxK];
    __shared__ uint8_t row_s[kPathBlock * kMaxK];   // path bits of each (token, source slot)
    __shared__ int first[kMaxN], wave_tot[kMaxN / 64];
    const int tid = threadIdx.x, R = T * k;
    int e[PER], t[PER], a[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = tid + j * kSmallThreads;
        t[j] = i / k;
        a[j] = i - t[j] * k;
        e[j] = 0;
        if (i < R) {
            const int v = ids[i];
            e[j] = v < 0 ? 0 : (v >= n ? n - 1 : v);
            e_s[i] = e[j];
            p_s[i] = w[i];
        }
    }
    for (int i = tid; i < kWaves * kMaxN; i += kSmallThreads) (&words[0][0])[i] = 0ull;
    __syncthreads();
    float den[PER];   // sum of p over the targets of this pair's source
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = tid + j * kSmallThreads;
        if (i >= R) continue;
        atomicOr(&words[t[j] >> 6][e[j]], 1ull << (t[j] & 63));
        const int t0 = t[j] * k;
        uint8_t mv[kMaxK];   // loaded together
#pragma unroll
        for (int b = 0; b < kMaxK; ++b) mv[b] = b < k ? mask[e[j] * n + e_s[t0 + b]] : 0;
        uint32_t row = 0;
        float src = 0.0f;
#pragma unroll
        for (int b = 0; b < kMaxK; ++b)
            if (b < k && (b == a[j] || mv[b])) {
                row |= 1u << b;
                src += p_s[t0 + b];
            }
        row_s[i] = (uint8_t)row;
        den[j] = src;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = tid + j * kSmallThreads;
        if (i >= R) continue;
        const int t0 = t[j] * k;
        if (a[j] == 0) {
            uint64_t bits = 0;
            for (int q = 0; q < k; ++q) bits |= (uint64_t)row_s[t0 + q] << (q * k);
            bits_out[t[j]] = bits;
        }
        if (beta_mode == 2) {   // over the token's paths, (a, b) ascending, one rounding per term
            den[j] = 0.0f;
            for (int q = 0; q < k; ++q)
                for (int b = 0; b < k; ++b)
                    if ((row_s[t0 + q] >> b) & 1) den[j] = fmaf(p_s[t0 + q], p_s[t0 + b], den[j]);
        }
        const uint32_t row = row_s[i];
        const float pa = p_s[i];
        for (int b = 0; b < k; ++b) {
            const float pb = p_s[t0 + b];
            float v = 0.0f;
            if ((row >> b) & 1) v = beta_mode == 0 ? pa * (pb / den[j]) : (beta_mode == 1 ? pa * pb : pa * pb / den[j]);
            beta_out[(int64_t)i * k + b] = v;
        }
    }
    int own = 0;
    if (tid < n)
#pragma unroll
        for (int q = 0; q < kWaves; ++q) own += __popcll(words[q][tid]);
    int total;
    const int excl = scan_columns(own, wave_tot, &total);
    if (tid < n) first[tid] = offsets[tid] = excl;
    if (tid == 0) offsets[n] = total;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = tid + j * kSmallThreads;
        if (i >= R) continue;
        const int wd = t[j] >> 6;
        int pos = first[e[j]] + __popcll(words[wd][e[j]] & ((1ull << (t[j] & 63)) - 1ull));
#pragma unroll
        for (int q = 0; q < kWaves; ++q)
            if (q < wd) pos += __popcll(words[q][e[j]]);
        row_token[pos] = t[j];
        row_slot[pos] = a[j];
        row_of[i] = pos;
    }
}

// Turn per-block counts [NB][n] into per-block first rows and fill expert_offsets.
__global__ __launch_bounds__(kMaxN) void paths_scan_kernel(int32_t* __restrict__ block_counts,
                                                           int64_t NB, int n,
                                                           int32_t* __restrict__ offsets) {
    __shared__ int scan[kMaxN];
    const int x = threadIdx.x;
    int run = 0;
    if (x < n)
        for (int64_t b0 = 0; b0 < NB; b0 += 16) {  // 16 independent loads, then the running sum
            int c[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) c[j] = b0 + j < NB ? block_counts[(b0 + j) * n + x] : 0;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                if (b0 + j < NB) block_counts[(b0 + j) * n + x] = run;
                run += c[j];
            }
        }
    scan[x] = x < n ? run : 0;
    __syncthreads();
    int own = scan[x];
    for (int d = 1; d < kMaxN; d <<= 1) {
        int v = x >= d ? scan[x - d] : 0;
        __syncthreads();
        scan[x] += v;
        __syncthreads();
    }
    const int excl = scan[x] - own;
    if (x < n) {
        offsets[x] = excl;
        for (int64_t b0 = 0; b0 < NB; b0 += 16) {
            int c[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) c[j] = b0 + j < NB ? block_counts[(b0 + j) * n + x] : 0;
#pragma unroll
            for (int j = 0; j < 16; ++j)
                if (b0 + j < NB) block_counts[(b0 + j) * n + x] = c[j] + excl;
        }
    }
    if (x == kMaxN - 1) offsets[n] = scan[x];
}

// Grouped dispatch with a variable number of entries per token: token t contributes
// counts[t] <= K distinct experts ids[t, 0..counts[t]) (scored routing: the distinct
// sources, or the distinct targets, of its selected paths). Rows are ordered by
// (expert, token) with the same OR-bitset ranks as paths_kernel; row_of[t, a] = -1 for
// a >= counts[t]. blockIdx.y is the side. The scatter phase either reads its first rows from
// block_counts (turned into them by paths_scan_kernel), or, with `reduce`, sums the count table of NB
// blocks itself (one launch fewer; every block reads the whole table).
template <int PH>
__global__ __launch_bounds__(kPathBlock) void dispatch_kernel(DispatchSides sides, int64_t T, int n, int K,
                                                             int64_t NB, int reduce) {
    const DispatchSide d = sides.s[blockIdx.y];
    const int32_t* const ids = d.ids;
    int32_t *const row_of = d.row_of, *const block_counts = d.block_counts;
    __shared__ PathSmem sm;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    for (int i = tid; i < kWaves * kMaxN; i += kPathBlock) (&sm.words[0][0])[i] = 0ull;
    __syncthreads();

    const int64_t t = (int64_t)blockIdx.x * kPathBlock + tid;
    const bool valid = t < T;
    int c = valid ? d.counts[t] : 0;
    c = c < 0 ? 0 : (c > K ? K : c);
    int e[kMaxK];
#pragma unroll
    for (int a = 0; a < kMaxK; ++a) {
        int v = (a < c) ? ids[t * K + a] : 0;
        e[a] = v < 0 ? 0 : (v >= n ? n - 1 : v);
    }
#pragma unroll
    for (int a = 0; a < kMaxK; ++a)
        if (a < c) atomicOr(&sm.words[wave][e[a]], 1ull << lane);
    __syncthreads();

    for (int x = tid; x < kMaxN; x += kPathBlock) {
        int run = 0;
        if (x < n) {
#pragma unroll
            for (int v = 0; v < kWaves; ++v) {
                sm.prefix[v][x] = run;
                run += __popcll(sm.words[v][x]);
            }
        }
        sm.scan[x] = run;
    }
    __syncthreads();

    if (PH == kCount) {
        for (int x = tid; x < n; x += kPathBlock) block_counts[(int64_t)blockIdx.x * n + x] = sm.scan[x];
        return;
    }
    if (PH == kFused) {
        const int total = block_exclusive_scan(sm.scan, n);
        for (int x = tid; x < n; x += kPathBlock) d.offsets[x] = sm.scan[x];
        if (tid == 0) d.offsets[n] = total;
    } else if (reduce) {
        __shared__ int wave_tot[kMaxN / 64];
        int all = 0, before = 0;
        if (tid < n)
            for (int64_t b0 = 0; b0 < NB; b0 += 16) {   // 16 independent loads at a time
                int v[16];
#pragma unroll
                for (int q = 0; q < 16; ++q) v[q] = b0 + q < NB ? block_counts[(b0 + q) * n + tid] : 0;
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    all += v[q];
                    before += b0 + q < blockIdx.x ? v[q] : 0;
                }
            }
        int total;
        const int excl = scan_columns(all, wave_tot, &total);
        if (tid < n) sm.scan[tid] = excl + before;
        if (blockIdx.x == 0) {
            if (tid < n) d.offsets[tid] = excl;
            if (tid == 0) d.offsets[n] = total;
        }
        __syncthreads();
    } else {
        for (int x = tid; x < n; x += kPathBlock) sm.scan[x] = block_counts[(int64_t)blockIdx.x * n + x];
        __syncthreads();
    }
    if (valid) {
        const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
        for (int a = 0; a < kMaxK; ++a) {
            if (a >= K) break;
            if (a >= c) {
                row_of[t * K + a] = -1;
                continue;
            }
            const int x = e[a];
            const int pos = sm.scan[x] + sm.prefix[wave][x] + __popcll(sm.words[wave][x] & below);
            d.row_token[pos] = (int32_t)t;
            d.row_slot[pos] = a;
            row_of[t * K + a] = pos;
        }
    }
}

}  // namespace

size_t build_paths_ws_bytes(int64_t T, int n) {
    const int64_t NB = ceil_div(T, kPathBlock);
    return NB <= 1 ? 0 : align_up((size_t)NB * n * sizeof(int32_t), 256);
}

hipError_t launch_build_paths(const int32_t* ids, const float* w, const uint8_t* mask, int64_t T,
                              int n, int k, int beta_mode, uint64_t* bits, float* beta,
                              int32_t* offsets, int32_t* row_token, int32_t* row_slot,
                              int32_t* row_of, int32_t* block_counts, hipStream_t s) {
    const int64_t NB = ceil_div(T, kPathBlock);
    if (NB <= 1) {
        paths_small_kernel<<<1, kSmallThreads, 0, s>>>(ids, w, mask, (int)T, n, k, beta_mode, bits, beta,
                                                       offsets, row_token, row_slot, row_of);
        return hipGetLastError();
    }
    paths_kernel<kCount><<<(unsigned)NB, kPathBlock, 0, s>>>(ids, w, mask, T, n, k, beta_mode, bits,
                                                             beta, row_token, row_slot, row_of,
                                                             block_counts);
    paths_scan_kernel<<<1, kMaxN, 0, s>>>(block_counts, NB, n, offsets);
    paths_kernel<kScatter><<<(unsigned)NB, kPathBlock, 0, s>>>(ids, w, mask, T, n, k, beta_mode,
                                                               bits, beta, row_token, row_slot, row_of,
                                                               block_counts);
    return hipGetLastError();
}

}  // namespace pcm

namespace pcm {

hipError_t launch_dispatch(const DispatchSides& d, int64_t T, int n, int K, hipStream_t s) {
    const int64_t NB = ceil_div(T, kPathBlock);
    if (NB <= 1) {
        dispatch_kernel<kFused><<<dim3(1, 2), kPathBlock, 0, s>>>(d, T, n, K, NB, 0);
        return hipGetLastError();
    }
    // up to 64 blocks (16384 tokens) a block sums the count table in at most four rounds of loads,
    // less than the scan's launch
    const int reduce = NB <= 64 ? 1 : 0;
    const dim3 grid((unsigned)NB, 2);
    dispatch_kernel<kCount><<<grid, kPathBlock, 0, s>>>(d, T, n, K, NB, 0);
    if (!reduce)
        for (const DispatchSide& side : d.s)
            paths_scan_kernel<<<1, kMaxN, 0, s>>>(side.block_counts, NB, n, side.offsets);
    dispatch_kernel<kScatter><<<grid, kPathBlock, 0, s>>>(d, T, n, K, NB, reduce);
    return hipGetLastError();
}

}  // namespace pcm
