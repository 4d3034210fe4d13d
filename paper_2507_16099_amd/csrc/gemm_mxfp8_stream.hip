// The block-scaled products of the persistent kernel (gemm_fp8_stream.hpp): its launch.
#include "gemm_fp8_stream.hpp"

namespace fp8k {

template <int FA, int FB, int AF1>
static hipError_t launch_mx_stream_t(const GemmOperands& g, const uint8_t* ea, int64_t slab_a, const uint8_t* eb, int64_t slab_b, int tiles_m,
                                     int tiles_n, hipStream_t st) {
    using namespace st;
    auto kern = gemm_fp8_stream_kernel<FA, FB, AF1, true>;
    static DynamicLdsOnce attr;
    if (hipError_t e = attr.ensure(reinterpret_cast<const void*>(kern), LDS_BYTES_MX); e != hipSuccess) return e;
    int cus = compute_units();
    if (const int forced = knob(KNOB_GEMM_STREAM); forced >= NUM_XCD) cus = forced;
    if (cus < NUM_XCD) cus = NUM_XCD;
    const int64_t units = (int64_t)tiles_m * tiles_n, need = (units + NUM_XCD - 1) / NUM_XCD * NUM_XCD;
    int64_t grid = cus / NUM_XCD * NUM_XCD;
    if (grid > need) grid = need;
    kern<<<dim3((unsigned)grid), dim3(NT), LDS_BYTES_MX, st>>>(g.a, g.lda, g.b, g.ldb, reinterpret_cast<const float*>(ea), (int)slab_a,
                                                              reinterpret_cast<const float*>(eb), (int)slab_b, (int)g.M, (int)g.N, (int)g.K,
                                                              static_cast<uint16_t*>(g.out), g.ld_out, tiles_m, tiles_n, (int)units);
    return hipGetLastError();
}

// scales in slabs of slab_a / slab_b rows; two groups of four K steps at least
bool gemm_mxfp8_stream_fits(const GemmOperands& g, int64_t slab_a, int64_t slab_b, int out_f32) {
    const int64_t pieces = (g.K + 511) / 512 * 16;
    return g.K % st::BK == 0 && g.K > 512 && gemm_fp8_stream_fits(g.lda, g.ldb, g.ld_out, g.N, g.K, out_f32, 0) && pieces * slab_a < (1ll << 31) &&
           pieces * slab_b < (1ll << 31) && (g.M + 191) / 192 * ((g.N + 255) / 256) < 0x3FFFFFFF;
}

hipError_t launch_gemm_mxfp8_stream(const GemmOperands& g, int fmt_a, const uint8_t* ea, int64_t slab_a, int fmt_b, const uint8_t* eb, int64_t slab_b,
                                    int tile_m, hipStream_t st) {
    using namespace st;
    if (tile_m != 256 && tile_m != 224 && tile_m != 192) return hipErrorInvalidValue;
    const int tiles_m = (int)((g.M + tile_m - 1) / tile_m), tiles_n = (int)((g.N + BN - 1) / BN);
#define FP8K_STREAM(FA_, FB_)                                                                                          \
    if (fmt_a == FA_ && fmt_b == FB_) {                                                                                \
        if (tile_m == 256) return launch_mx_stream_t<FA_, FB_, 4>(g, ea, slab_a, eb, slab_b, tiles_m, tiles_n, st);    \
        if (tile_m == 224) return launch_mx_stream_t<FA_, FB_, 3>(g, ea, slab_a, eb, slab_b, tiles_m, tiles_n, st);    \
        return launch_mx_stream_t<FA_, FB_, 2>(g, ea, slab_a, eb, slab_b, tiles_m, tiles_n, st);                       \
    }
    FP8K_STREAM(FMT_E4M3FN, FMT_E4M3FN)
    FP8K_STREAM(FMT_E5M2, FMT_E4M3FN)
    FP8K_STREAM(FMT_E4M3FN, FMT_E5M2)
    FP8K_STREAM(FMT_E5M2, FMT_E5M2)
#undef FP8K_STREAM
    return hipErrorInvalidValue;
}

}  // namespace fp8k
