// The block-scaled products of the ring kernel (gemm_fp8_ring.hpp): its forms and their launch.
#include "gemm_fp8_ring.hpp"

namespace fp8k {

bool gemm_mxfp8_ring_fits(const GemmOperands& g, int64_t ld_ea, int64_t ld_eb) {
    auto reach = [&](int64_t ld, int64_t rows) { return ld >= 0 ? ld < (1 << 22) : -ld >= rows && -ld * ((g.K + 511) / 512) < (1ll << 26); };
    return gemm_fp8_ring_fits(g) && g.K > 0 && g.K % 128 == 0 && reach(ld_ea, g.M) && reach(ld_eb, g.N);
}

hipError_t launch_gemm_mxfp8_ring(int tile, const GemmOperands& g, int fmt_a, int fmt_b, const uint8_t* ea, int64_t ld_ea,
                                  const uint8_t* eb, int64_t ld_eb, int out_f32, hipStream_t st) {
    if (g.M == 0 || g.N == 0) return hipErrorInvalidValue;
    const MxScales e{ea, eb, ld_ea, ld_eb};
#define FP8K_RING(FA_, FB_) \
    if (fmt_a == FA_ && fmt_b == FB_) return launch_ring_f<FA_, FB_, true>(tile, g, nullptr, &e, 0, 0, out_f32 ? 1 : 0, st)
    FP8K_RING(FMT_E4M3FN, FMT_E4M3FN);
    FP8K_RING(FMT_E5M2, FMT_E4M3FN);
    FP8K_RING(FMT_E4M3FN, FMT_E5M2);
    FP8K_RING(FMT_E5M2, FMT_E5M2);
#undef FP8K_RING
    return hipErrorInvalidValue;
}

}  // namespace fp8k
