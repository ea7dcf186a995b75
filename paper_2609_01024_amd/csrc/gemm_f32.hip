// Grouped float32 GEMMs for float32 layers (same operations as the bf16 kernels: expansion with
// fused SwiGLU, down projection store or accumulate), on v_mfma_f32_16x16x4_f32: float32 operands,
// products and sums.
#include "gemm_ring.h"

namespace pcm {
namespace {

struct ElemF32 {
    static constexpr int SIZE = 4, NJ = 4;
    using T = floatx4;
    struct Silu {   // float32 layers: the library exponential and an IEEE division
        __device__ static float silu(float g) { return g / (1.0f + expf(-g)); }
    };
    __device__ static T weights(const char* p) { return *(const T*)p; }
    __device__ static T acts(const char* p) { return *(const T*)p; }
    __device__ static floatx4 step(int j, const T& w, const T& a, floatx4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(w[j], a[j], c, 0, 0, 0);
    }
};

// 64 x 64 tiles (three workgroups on a compute unit, so one's epilogue and waits overlap the others'
// MFMAs); 32 x 64 tiles where those would not fill the chip once. Both are bound by the MFMA rate
// (154 TFLOP/s in a large dense product here) where tiles are many: 4000 tokens, 8 experts, top-2,
// H 1024, F 2048: expansion 1051 -> 576 us (117 TFLOP/s), projection with mix and combine 552 ->
// 353 us, against the vector-ALU tiles before. 64 x 128 and 128 x 128 tiles measured 0-5% and 3-40%
// slower (fewer workgroups to overlap, a longer last round), a ring of two slices 2-8%, 32-row tiles for
// the last rows of a group -1% to +8%, a deeper ring for the 32 x 64 tiles 0-30%.
using WideF32 = RCfg<64, 64, 2, 2, 3>;
using NarrowF32 = RCfg<32, 64, 2, 2, 4>;

template <int MODE>
hipError_t launch_mode_f32(const GemmArgs& g, int64_t R, hipStream_t s) {
    // expected tiles: full row blocks, and half a block of remainder for every group with rows.
    // Below 768 (three on each of 256 compute units) the smaller tiles are faster: 32 rows over 32
    // experts 25 against 46 us (projection, F 1024), 300 tokens over 8 experts 19 against 24 us;
    // above, the larger ones: 777 tokens, 16 experts, top-4: 100 against 157 us (expansion, F 960).
    const int64_t groups = g.offsets ? (R < g.n ? R : g.n) : 0;
    const int64_t tiles = (R / 32 + groups + (g.offsets ? 0 : 1)) * ceil_div(g.N, MODE == kExpand ? 32 : 64) / 2;
    return tiles >= 768 ? launch_ring<ElemF32, WideF32, WideF32, MODE>(g, R, s, 1)
                        : launch_ring<ElemF32, NarrowF32, NarrowF32, MODE>(g, R, s, 1);
}

}  // namespace

hipError_t launch_gemm_f32(GemmMode mode, const GemmArgs& g0, int64_t R, hipStream_t s) {
    GemmArgs g = g0;
    g.ksplit = 1;
    switch (mode) {
        case kExpand: return launch_mode_f32<kExpand>(g, R, s);
        case kDownStore: return launch_mode_f32<kDownStore>(g, R, s);
        default: return launch_mode_f32<kDownAccum>(g, R, s);
    }
}

}  // namespace pcm
