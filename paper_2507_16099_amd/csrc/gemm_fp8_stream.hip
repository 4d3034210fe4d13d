// The plain FP8 products of the persistent kernel (gemm_fp8_stream.hpp): its launch.
#include "gemm_fp8_stream.hpp"

namespace fp8k {

template <int FA, int FB, int AF1>
static hipError_t launch_stream_t(const uint8_t* a, int64_t lda, const float* sa, int row_a, const uint8_t* b, int64_t ldb,
                                  const float* sb, int row_b, int M, int N, int K, void* out, int64_t ld_out, int tiles_m,
                                  int tiles_n, int64_t units, hipStream_t st) {
    using namespace st;
    auto kern = gemm_fp8_stream_kernel<FA, FB, AF1>;
    static DynamicLdsOnce attr;
    if (hipError_t e = attr.ensure(reinterpret_cast<const void*>(kern), LDS_BYTES); e != hipSuccess) return e;
    // one workgroup per CU (they do not fit twice), a multiple of the XCD count; the switch GEMM_STREAM >= 8 sets
    // the number of workgroups instead (test aid: few workgroups walk many tiles each, also on small problems)
    int cus = compute_units();
    if (const int forced = knob(KNOB_GEMM_STREAM); forced >= NUM_XCD) cus = forced;
    if (cus < NUM_XCD) cus = NUM_XCD;
    int64_t grid = cus / NUM_XCD * NUM_XCD;
    const int64_t need = (units + NUM_XCD - 1) / NUM_XCD * NUM_XCD;
    if (grid > need) grid = need;
    kern<<<dim3((unsigned)grid), dim3(NT), LDS_BYTES, st>>>(a, lda, b, ldb, sa, row_a, sb, row_b, M, N, K,
                                                           static_cast<uint16_t*>(out), ld_out, tiles_m, tiles_n, (int)units);
    return hipGetLastError();
}

bool gemm_fp8_stream_fits(int64_t lda, int64_t ldb, int64_t ld_out, int64_t N, int64_t K, int out_f32, int act) {
    return !out_f32 && !act && N % 8 == 0 && K > 2 * st::BK && lda < (1 << 23) && ldb < (1 << 23) && ld_out < (1 << 22);
}

// Tile height (256, 224 or 192 rows) for an [M, N] output when the persistent kernel takes every tile: the one
// with the least rounds x height on this device's CUs; 256 when it is no worse (a lower tile moves more operand
// bytes per product).  The switch GEMM_TILE_M forces one.
int gemm_fp8_stream_tile_m(int64_t M, int64_t N) {
    const int forced = knob(KNOB_GEMM_TILE_M);
    if (forced == 256 || forced == 224 || forced == 192) return forced;
    const int64_t cus = compute_units() > 0 ? compute_units() : 256;
    const int64_t tiles_n = (N + st::BN - 1) / st::BN;
    int best = 256;
    int64_t best_cost = 0;
    for (int tm : {256, 224, 192}) {
        const int64_t tiles = (M + tm - 1) / tm * tiles_n;
        const int64_t cost = (tiles + cus - 1) / cus * tm;
        if (tm == 256 || cost < best_cost) { best = tm; best_cost = cost; }
    }
    return best;
}

// tiles [0, units) of the tile order of the non-persistent kernel (tile_m == 256), or every tile of the problem cut
// into tiles of tile_m rows (units == the tile count)
hipError_t launch_gemm_fp8_stream(const uint8_t* a, int64_t lda, int fmt_a, const float* scale_a, int row_a,
                                  const uint8_t* b, int64_t ldb, int fmt_b, const float* scale_b, int row_b,
                                  int64_t M, int64_t N, int64_t K, void* out, int64_t ld_out, int64_t units, int tile_m,
                                  hipStream_t st) {
    using namespace st;
    if (units <= 0) return hipSuccess;
    if (tile_m != 256 && tile_m != 224 && tile_m != 192) return hipErrorInvalidValue;
    const int tiles_m = (int)((M + tile_m - 1) / tile_m), tiles_n = (int)((N + BN - 1) / BN);
    if (units > (int64_t)tiles_m * tiles_n || units > 0x3FFFFFFF) return hipErrorInvalidValue;
    const int m = (int)M, n = (int)N, k = (int)K;
#define FP8K_STREAM(FA_, FB_)                                                                                   \
    if (fmt_a == FA_ && fmt_b == FB_) {                                                                         \
        if (tile_m == 256) return launch_stream_t<FA_, FB_, 4>(a, lda, scale_a, row_a, b, ldb, scale_b, row_b, m, n, k, out, ld_out, tiles_m, tiles_n, units, st); \
        if (tile_m == 224) return launch_stream_t<FA_, FB_, 3>(a, lda, scale_a, row_a, b, ldb, scale_b, row_b, m, n, k, out, ld_out, tiles_m, tiles_n, units, st); \
        return launch_stream_t<FA_, FB_, 2>(a, lda, scale_a, row_a, b, ldb, scale_b, row_b, m, n, k, out, ld_out, tiles_m, tiles_n, units, st); \
    }
    FP8K_STREAM(FMT_E4M3FN, FMT_E4M3FN)
    FP8K_STREAM(FMT_E5M2, FMT_E4M3FN)
    FP8K_STREAM(FMT_E4M3FN, FMT_E5M2)
    FP8K_STREAM(FMT_E5M2, FMT_E5M2)
#undef FP8K_STREAM
    return hipErrorInvalidValue;
}

}  // namespace fp8k
