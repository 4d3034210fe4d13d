// Which kernel the FP8 products are sent to (test infrastructure, no device).
//
// Built by tests/test_gemm_choice.py from this file and gemm_fp8.hip.  The launchers behind the choice are replaced by the stubs
// below, which print what they were asked for; the switches and the number of CUs come from the command line.  Each line of the
// input is a query, each line of the output its answer:
//     one M N K                   a product
//     mx M N K                    the same, block-scaled; mxrows: with plain rows of scales
//     own M N K                   the same, its weight written by the same call; strips: in column strips
//     act M N K                   the same with the sigmoid
//     f32 M N K                   the same with fp32 results
//     large M N K                 of a product sent to the 256 x 256 kernels: its wide tile, or the height of the tiles of one round; large32: fp32 results
//     slabs M N K                 height of the persistent kernel's tiles for a block-scaled product, 0: one 256 x 256 tile per workgroup
//     few M N K                   the split of a few-row product
//     stream M N K                up to 16 rows: persistent workgroups, strided or in runs, or the few-row kernel; streamld M N K ld: rows of
//                                 the weight ld bytes apart
//     cols rows load              columns of a strip of the shared quantization (the third number is not used)
//     two M1 N1 K1 M2 N2 K2       the pair of a backward step
// Arguments: CUs=<n>, <switch number>=<value>.
#include "../paper_2507_16099_amd/csrc/launchers.hpp"
#include "../paper_2507_16099_amd/csrc/tuning.hpp"

#include <cstdio>
#include <cstdlib>
#include <cstring>

namespace fp8k {
static const char* const names[RING_TILES] = {"64x64", "128x64", "64x128", "128x128", "128x256", "256x128", "96x64", "64x192", "160x64", "96x128",
                                                "160x128", "192x128", "128x192", "160x192", "192x192", "160x256", "224x192"};
static int g_cus = 256, g_knobs[KNOB_COUNT];
int knob(Knob k) { return g_knobs[k]; }
int compute_units() { return g_cus; }
bool gemm_fp8_ring_fits(const GemmOperands& g) { return g.lda < (1 << 22) && g.ldb < (1 << 22) && ((g.M + 63) / 64) * ((g.N + 63) / 64) < (1 << 15); }
bool gemm_fp8_snake_fits(int64_t lda, int64_t ldb) { return lda < (1 << 23) && ldb < (1 << 23); }
hipError_t launch_gemm_fp8_ring(int tile, const GemmOperands& g1, const GemmOperands* g2, int, int, int, int, int, hipStream_t) {
    std::printf("ring %s %s%s %d K=%lld\n", names[tile], g2 ? "together" : "alone", ring_hint(tile, g1, g2) ? " hint" : "", ring_waves(tile, g1, g2, false),
                (long long)g1.K);      // (together: K of the one whose workgroups come first)
    return hipSuccess;
}
hipError_t launch_gemm_fp8_skinny(const uint8_t*, int64_t, int, const float*, int, const uint8_t*, int64_t, int, const float*, int, int64_t, int64_t,
                                  int64_t, void*, int64_t, int, hipStream_t) {
    std::printf("few-row\n");
    return hipSuccess;
}
hipError_t launch_gemm_fp8_snake(const uint8_t*, int64_t, int, const float*, int, const uint8_t*, int64_t, int, const float*, int, int64_t, int64_t,
                                 int64_t, void*, int64_t, int, hipStream_t, int) {
    std::printf("256x256\n");
    return hipSuccess;
}
}  // namespace fp8k

int main(int argc, char** argv) {
    using namespace fp8k;
    for (int& k : g_knobs) k = -1;
    for (int i = 1; i < argc; ++i) {
        const char* eq = std::strchr(argv[i], '=');
        if (!eq) return 2;
        if (std::strncmp(argv[i], "CUs=", 4) == 0) g_cus = std::atoi(eq + 1);
        else g_knobs[std::atoi(argv[i])] = std::atoi(eq + 1);
    }
    char kind[16];
    long long M, N, K, M2, N2, K2;
    auto product = [](long long m, long long n, long long k) {
        // (addresses that nothing reads: whole cache lines)
        return GemmOperands{reinterpret_cast<const uint8_t*>(4096), k, nullptr, reinterpret_cast<const uint8_t*>(8192), k, nullptr, m, n, k, nullptr, n};
    };
    while (std::scanf("%15s %lld %lld %lld", kind, &M, &N, &K) == 4) {
        const GemmOperands g = product(M, N, K);
        if (std::strcmp(kind, "two") == 0) {
            if (std::scanf("%lld %lld %lld", &M2, &N2, &K2) != 3) return 2;
            if (launch_gemm_fp8_pair(g, product(M2, N2, K2), 0, 0, 1, 1, nullptr) != hipSuccess) std::printf("apart\n");
        } else if (std::strncmp(kind, "mx", 2) == 0) {
            const bool plain = std::strcmp(kind, "mxrows") == 0;
            const int tile = gemm_mxfp8_ring_choice(g, plain);
            if (tile < 0) std::printf("256x256\n");
            else std::printf("ring %s %d\n", names[tile], ring_waves(tile, g, nullptr, true, plain));
        } else if (std::strcmp(kind, "few") == 0) {
            const FewRowForm f = few_row_form(M, N, K, 0, g_cus);
            std::printf("%d %d %lld %s%s\n", f.nw, f.ks, (long long)f.grid, f.deep ? "deep" : "",
                        few_row_hint((int)(M + 15) / 16, f.nw, f.ks) ? " hint" : "");
        } else if (std::strncmp(kind, "stream", 6) == 0) {
            GemmOperands w = g;
            if (std::strcmp(kind, "streamld") == 0 && std::scanf("%lld", &M2) == 1) w.ldb = M2;
            std::printf("%s\n", !few_row_streams(w, g_cus, g_knobs[KNOB_SKINNY_DMA]) ? "few-row" : few_row_runs(w, g_cus, g_knobs[KNOB_SKINNY_DMA]) ? "runs" : "strided");
        } else if (std::strcmp(kind, "cols") == 0) {
            std::printf("%d\n", strip_columns(M, (double)N, g_cus));
        } else if (std::strcmp(kind, "act") == 0) {
            std::printf("%s\n", gemm_fp8_ring_choice(g) >= 0 ? "ring" : "256x256");
        } else if (std::strcmp(kind, "slabs") == 0) {
            std::printf("%d rows\n", gemm_mxfp8_stream_height(g));
        } else if (std::strncmp(kind, "large", 5) == 0) {
            const bool bf16 = std::strcmp(kind, "large") == 0;
            const int tile = gemm_fp8_wide_choice(g, bf16);
            if (tile >= 0) std::printf("ring %s\n", names[tile]);
            else std::printf("%d rows\n", bf16 ? one_round_height(g, g_cus) : 256);
        } else if (launch_gemm_fp8(g.a, g.lda, 0, nullptr, 1, g.b, g.ldb, 0, nullptr, 1, M, N, K, nullptr, N, std::strcmp(kind, "f32") == 0, nullptr,
                                   std::strcmp(kind, "own") == 0 ? B_WRITTEN : std::strcmp(kind, "strips") == 0 ? B_WRITTEN_IN_STRIPS : B_AT_REST) != hipSuccess) {
            return 3;
        }
    }
    return 0;
}
