// The plain FP8 products of the ring kernel (gemm_fp8_ring.hpp): its forms and their launch.
#include "gemm_fp8_ring.hpp"

namespace fp8k {

bool gemm_fp8_ring_fits(const GemmOperands& g) {
    // 32-bit panel offsets, tile counts within the reach of the kernel's reciprocals
    return g.lda < (1 << 22) && g.ldb < (1 << 22) && ((g.M + 63) / 64) * ((g.N + 63) / 64) < (1 << 15);
}

hipError_t launch_gemm_fp8_ring(int tile, const GemmOperands& g1, const GemmOperands* g2, int fmt_a, int fmt_b, int row_a,
                                int row_b, int mode, hipStream_t st) {
    if (g1.M == 0 || g1.N == 0 || (g2 && (g2->M == 0 || g2->N == 0))) return hipErrorInvalidValue;
#define FP8K_RING(FA_, FB_) \
    if (fmt_a == FA_ && fmt_b == FB_) return launch_ring_f<FA_, FB_, false>(tile, g1, g2, nullptr, row_a, row_b, mode, st)
    FP8K_RING(FMT_E4M3FN, FMT_E4M3FN);
    FP8K_RING(FMT_E5M2, FMT_E4M3FN);
    FP8K_RING(FMT_E4M3FN, FMT_E5M2);
    FP8K_RING(FMT_E5M2, FMT_E5M2);
#undef FP8K_RING
    return hipErrorInvalidValue;
}

}  // namespace fp8k
