// Scaled FP8 GEMM for gfx950 on the CDNA4 matrix cores
// (v_mfma_f32_16x16x128_f8f6f4): out[M,N] = (A[M,K] . B[N,K]^T) / (sa * sb).
//
// The paper (Section 2.1) leaves the FP8 products to the hardware vendor's GEMM
// kernels; this is this library's own fallback for operands that the LDS-DMA kernels' 32-bit offsets do not reach,
// and the dispatch.
//
// Layout of the work
//   - Both operands have the contraction axis contiguous.  A workgroup owns a
//     BM x BN tile of the output and walks K in steps of 128 bytes.
//   - Each K step stages BM + BN rows of 128 bytes in LDS.  A row is eight
//     16-byte chunks; chunk c of a row is stored at chunk position c ^ key(row)
//     so that the 128-bit LDS reads of one MFMA operand (16 rows, same logical
//     chunk) fall into different banks.
//   - One MFMA takes 16 rows x 128 K-bytes of each operand: lane l supplies 32
//     bytes of row l%16, here chunks l/16 and l/16 + 4.  The assignment of K
//     bytes to lanes is the same for both operands, which is all a dot product
//     needs; this one makes every 64-lane 128-bit LDS read touch each of the
//     16 bank groups (16 bytes wide, 256-byte wrap) exactly four times, the
//     conflict-free pattern (chunks 2*(l/16), 2*(l/16)+1 would use only half
//     of the bank groups and run at half the LDS rate).
//   - The B tile is the FIRST MFMA operand and the A tile the second, so a lane
//     ends up with accumulators for one output row m and several n.  The rows
//     of a 64-wide B group are dealt to the four MFMA tiles such that lane l
//     holds 16 CONSECUTIVE n (n = 16*(l/16) + 4*t + r for tile t, register r):
//     the epilogue scales, rounds to bfloat16 and stores 32 contiguous bytes
//     per lane straight from registers.
//   - Workgroup ids are remapped so that each XCD (ids are dealt round-robin to
//     the 8 XCDs) works on one contiguous range of tiles, walked in groups of
//     tile rows, which keeps the operand panels of concurrently running tiles
//     in that XCD's L2.
#include "fp8_device.hpp"
#include "launchers.hpp"
#include "tuning.hpp"

namespace fp8k {

typedef int v8i_t __attribute__((ext_vector_type(8)));
typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef float v4f_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

constexpr int BK = 128;          // bytes of K per step
constexpr int GROUP_M = 4;       // tile rows walked together
constexpr int NUM_XCD = 8;

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    f32x2_t v = {a, b};
    bf16x2_t h = __builtin_convertvector(v, bf16x2_t);
    uint32_t r;
    __builtin_memcpy(&r, &h, 4);
    return r;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int FA, int FB, bool OUT_F32>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64) void gemm_fp8_tn_kernel(
    const uint8_t* __restrict__ A, int64_t lda, const uint8_t* __restrict__ B, int64_t ldb, const float* __restrict__ scale_a,
    int row_a, const float* __restrict__ scale_b, int row_b, int M, int N, int K, void* __restrict__ out, int64_t ld_out,
    int tiles_m, int tiles_n) {
    constexpr int NT = WAVES_M * WAVES_N * 64;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int FM = WM / 16;       // A fragments (16 rows each) per wave
    constexpr int NG = WN / 64;       // 64-wide B groups per wave
    constexpr int FN = NG * 4;        // B fragments per wave
    constexpr int NLA = BM * 8 / NT;  // 16-byte chunks each thread stages per step
    constexpr int NLB = BN * 8 / NT;
    constexpr int STAGE = (BM + BN) * BK;
    static_assert(WM % 16 == 0 && WN % 64 == 0 && (BM * 8) % NT == 0 && (BN * 8) % NT == 0 && (NT / 8) % 32 == 0, "tile");

    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

    // ---- workgroup -> tile
    const int ntiles = tiles_m * tiles_n;
    const int per_xcd = gridDim.x / NUM_XCD;
    const int logical = (blockIdx.x % NUM_XCD) * per_xcd + blockIdx.x / NUM_XCD;
    if (logical >= ntiles) return;
    const int in_group = GROUP_M * tiles_n;
    const int first_m = (logical / in_group) * GROUP_M;
    const int gsize = tiles_m - first_m < GROUP_M ? tiles_m - first_m : GROUP_M;
    const int tm = first_m + (logical % in_group) % gsize;
    const int tn = (logical % in_group) / gsize;
    const int m0 = tm * BM, n0 = tn * BN;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm0 = (wave / WAVES_N) * WM, wn0 = (wave % WAVES_N) * WN;

    // ---- global -> LDS staging: thread t owns LDS chunk slots i*NT + t
    const int srow = tid >> 3, spc = tid & 7;
    const int ca = spc ^ (srow & 7);                                   // logical chunk, A rows
    const int cb = spc ^ ((srow & 3) | ((srow >> 2) & 4));             // logical chunk, B rows
    const uint8_t* a_ptr = A + (int64_t)(m0 + srow) * lda + ca * 16;
    const uint8_t* b_ptr = B + (int64_t)(n0 + srow) * ldb + cb * 16;
    const int64_t a_step = (int64_t)(NT / 8) * lda, b_step = (int64_t)(NT / 8) * ldb;
    uint4 ra[NLA], rb[NLB];
    auto gload = [&](int k0) {
        const bool ka = k0 + ca * 16 < K, kb = k0 + cb * 16 < K;
#pragma unroll
        for (int i = 0; i < NLA; ++i) {
            const bool ok = ka && (m0 + srow + i * (NT / 8) < M);
            ra[i] = ok ? *reinterpret_cast<const uint4*>(a_ptr + i * a_step + k0) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < NLB; ++i) {
            const bool ok = kb && (n0 + srow + i * (NT / 8) < N);
            rb[i] = ok ? *reinterpret_cast<const uint4*>(b_ptr + i * b_step + k0) : make_uint4(0, 0, 0, 0);
        }
    };
    auto lstore = [&](int stage) {
        uint8_t* as = smem + stage * STAGE + tid * 16;
        uint8_t* bs = as + BM * BK;
#pragma unroll
        for (int i = 0; i < NLA; ++i) *reinterpret_cast<uint4*>(as + i * NT * 16) = ra[i];
#pragma unroll
        for (int i = 0; i < NLB; ++i) *reinterpret_cast<uint4*>(bs + i * NT * 16) = rb[i];
    };

    // ---- LDS -> MFMA operands
    const int key = lane & 7;
    const int off_lo = ((lane >> 4) ^ key) << 4, off_hi = (((lane >> 4) + 4) ^ key) << 4;
    const int a_row_off = (wm0 + (lane & 15)) * BK;
    const int b_row_off = (wn0 + 16 * ((lane & 15) >> 2) + (lane & 3)) * BK;

    v4f_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = v4f_t{0.f, 0.f, 0.f, 0.f};

    auto frag = [&](const uint8_t* base) {
        const uint4 lo = *reinterpret_cast<const uint4*>(base + off_lo);
        const uint4 hi = *reinterpret_cast<const uint4*>(base + off_hi);
        return v8i_t{(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
    };
    auto compute = [&](int stage) {
        const uint8_t* as = smem + stage * STAGE + a_row_off;
        const uint8_t* bs = smem + stage * STAGE + BM * BK + b_row_off;
        v8i_t bf[FN];
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int t = 0; t < 4; ++t) bf[g * 4 + t] = frag(bs + (64 * g + 4 * t) * BK);
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const v8i_t af = frag(as + 16 * i * BK);
#pragma unroll
            for (int j = 0; j < FN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(bf[j], af, acc[i][j], FB, FA, 0, 0, 0, 0);
        }
    };

    // ---- main loop, two LDS stages, loads one step ahead
    const int ksteps = (K + BK - 1) / BK;
    // the scales of this tile's rows and columns are requested now, so that their latency lies under the K loop
    // (problems of few tiles are bound by such fixed costs: a trip to memory is about as long as two K steps)
    float sa_raw[FM], sb_raw[NG][16];
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int m = m0 + wm0 + 16 * i + (lane & 15);
        sa_raw[i] = row_a ? (m < M ? scale_a[m] : 1.0f) : scale_a[0];
    }
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int n = n0 + wn0 + 64 * g + 16 * (lane >> 4) + e;
            sb_raw[g][e] = row_b ? (n < N ? scale_b[n] : 1.0f) : scale_b[0];
        }
    if (ksteps > 0) {
        gload(0);
        lstore(0);
        __syncthreads();
        for (int kt = 0; kt < ksteps; ++kt) {
            gload((kt + 1) * BK);
            compute(kt & 1);
            lstore((kt + 1) & 1);
            __syncthreads();
        }
    }

    // ---- epilogue: (acc * 1/sa) * 1/sb, round, store 16 consecutive n per lane
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const int nb = n0 + wn0 + 64 * g + 16 * (lane >> 4);
        float inv_b[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) inv_b[e] = (nb + e < N) ? 1.0f / sb_raw[g][e] : 0.f;
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int m = m0 + wm0 + 16 * i + (lane & 15);
            if (m >= M || nb >= N) continue;
            const float inv_a = 1.0f / sa_raw[i];
            float v[16];
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) v[4 * t + r] = (acc[i][g * 4 + t][r] * inv_a) * inv_b[4 * t + r];
            if constexpr (OUT_F32) {
                float* dst = static_cast<float*>(out) + (int64_t)m * ld_out + nb;
                if (nb + 16 <= N) {
#pragma unroll
                    for (int e = 0; e < 16; e += 4)
                        *reinterpret_cast<float4*>(dst + e) = make_float4(v[e], v[e + 1], v[e + 2], v[e + 3]);
                } else {
                    for (int e = 0; nb + e < N; ++e) dst[e] = v[e];
                }
            } else {
                uint16_t* dst = static_cast<uint16_t*>(out) + (int64_t)m * ld_out + nb;
                uint32_t p[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) p[e] = pack_bf16(v[2 * e], v[2 * e + 1]);
                if (nb + 16 <= N) {
                    *reinterpret_cast<uint4*>(dst) = make_uint4(p[0], p[1], p[2], p[3]);
                    *reinterpret_cast<uint4*>(dst + 8) = make_uint4(p[4], p[5], p[6], p[7]);
                } else {
                    for (int e = 0; nb + e < N; ++e) dst[e] = (uint16_t)(p[e >> 1] >> ((e & 1) * 16));
                }
            }
        }
    }
}

template <int FA, int FB, bool OUT_F32>
static hipError_t launch_tn(const GemmOperands& g, int row_a, int row_b, hipStream_t st) {
    constexpr int BM = 128, BN = 128;
    auto kern = gemm_fp8_tn_kernel<BM, BN, 2, 2, FA, FB, OUT_F32>;
    constexpr int lds = 2 * (BM + BN) * BK;
    static DynamicLdsOnce attr;     // one per instantiation
    if (hipError_t e = attr.ensure(reinterpret_cast<const void*>(kern), lds); e != hipSuccess) return e;
    const int tiles_m = (int)((g.M + BM - 1) / BM), tiles_n = (int)((g.N + BN - 1) / BN);
    const int64_t blocks = ((int64_t)tiles_m * tiles_n + NUM_XCD - 1) / NUM_XCD * NUM_XCD;
    if (blocks > 0x7FFFFFF0) return hipErrorInvalidValue;
    kern<<<dim3((unsigned)blocks), dim3(256), lds, st>>>(g.a, g.lda, g.b, g.ldb, g.scale_a, row_a, g.scale_b, row_b, (int)g.M, (int)g.N,
                                                       (int)g.K, g.out, g.ld_out, tiles_m, tiles_n);
    return hipGetLastError();
}

// ---- kernel choice.  Up to 16 rows: the few-row kernel of gemm_fp8_skinny.hip (it streams B once).  17 to 32 rows: the same where
// there are 64 x 64 ring tiles for less than five eighths of the CUs (us, few-row / ring at 32 rows, weights from HBM: 4096 x 4096
// 7.1 / 11.2, 8192 x 4096 10.2 / 12.0; 11008 x 4096 15.1 / 13.4), else by few_rows_tile below.  Up to 64 rows the few-row kernel
// where there are too few 64 x 64 tiles for the CUs, N <= 8192, and the contraction is long enough for its wavefronts to share (us,
// few-row / best ring tile, N x K at 33, 40, 48, 64 rows, weights from HBM: 4096 x 4096 7.8 / 11.2, 8.0 / 11.5, 8.5 / 12.0, 9.5 /
// 12.8; 8192 x 4096 11.1 / 12.1, 11.5 / 12.4, 11.9 / 12.9, 13.0 / 13.9; 4096 x 14336 18.3 / 30.3 .. 23.6 / 36.9; 4096 x 2048 4.9 /
// 6.1 .. 5.8 / 6.3.  Beyond the lines: 11008 x 4096 18.8 / 13.1 .. 22.3 / 14.8, 14336 x 4096 20.4 / 15.3 .. 23.6 / 16.0, 28672 x
// 8192 60.7 / 50.1 .. 71.8 / 52.1, 8192 x 1024 6.1 / 5.1 .. 6.8 / 5.2.  On them it is close: 8192 x 2048 7.8 / 7.8 .. 9.2 / 8.7,
// 4096 x 1024 4.7 / 4.9 .. 5.3 / 5.1.) More than one round of 256 x 256 tiles (one per CU): the large-product kernels of
// gemm_fp8_snake.hip / gemm_fp8_stream.hip.  In between the cheapest of the ring kernel's tiles (gemm_fp8_ring.hpp) and one round
// of 256 x 256 tiles by this estimate, in us (one launch; rounds of 256 workgroups, K steps of 128 bytes):
//     3 + rounds * (a + steps * b);  256 x 256 tiles: 10 + 1.2 * steps, at most half of the CUs busy (half tiles) 7.2 + 0.91 * steps,
//     one round of 224 x 256 tiles 9.6 + 1.085 * steps, of 192 x 256 ones 9 + 0.97 * steps (one_round_height).
// a: prologue and epilogue of a tile; b: a K step with every CU busy (some 460 / 670 / 970 / 1600 cycles for the tiles below; their
// matrix instructions take 128 / 256 / 512 / 1024, the fragment reads and LDS-DMA writes at 128 bytes a cycle 384 / 576 / 768 /
// 1152). No unit is full: 128 x 128 tiles at 777 x 4096 x 14336 keep the matrix units busy 42 % of the time and the LDS's reads 22
// %. Measured (a HIP graph of twelve, operands alternating; us; K = 1024 / 4096 / 16384; since then 128 x 64 tiles take 0.4 us
// less, 128 x 256 tiles 0.7 up to K = 6144):
//                        64x64              128x64             128x128            128x256            before (other kernels)
//     1024 x 1024     6.0 / 10.5 / 29     7.4 / 13.2 / 36     8.3 / 16.0 / 46    11.3 / 23.9 / 73      7.8 / 14.8 / 45
//     1024 x 2048     9.6 / 18.3 / 66     7.9 / 14.2 / 50     8.6 / 17.2 / 64    11.6 / 24.8 / 99     10.3 / 21.8 / 74
//     2048 x 2048    16.7 / 32.7 / 122   13.0 / 26.7 / 89    11.7 / 20.2 / 73    12.3 / 27.0 / 100    13.8 / 29.1 / 95
//     2048 x 4096    29.9 / 62.1 / 242   22.8 / 49.2 / 176   17.9 / 38.2 / 131   17.6 / 32.7 / 109    14.5 / 36.4 / 157
//     3072 x 4096    43.0 / 100          32.4 / 76           25.6 / 58           23.9 / 56            19.0 / 46.1
//     4096 x 4096    57.8 / 136          43.3 / 113          31.7 / 83           31.7 / 68            20.8 / 53.3
// The tiles between these sizes, one round exactly full of them (16 rows of tiles by 16; us, K = 1024 / 4096 / 8192 / 16384, and what
// the six above and 256 x 256 ones take): 96x64 5.6 / 11.6 / 18.9 / 32.7, before 6.6 / 12.8 / 20.8 / 36.7; 64x192 8.5 / 16.9 /
// 28.1 / 50.2, 8.9 / 17.9 / 29.2 / 51.8; 160x64 7.3 / 15.4 / 24.9 / 44.6, 8.4 / 16.6 / 27.3 / 48.7; 96x128 8.0 / 17.1 / 26.8 /
// 48.0, 8.6 / 17.0 / 28.0 / 50.5; 160x128 10.7 / 22.3 / 37.9 / 69.1, 13.2 / 26.4 / 44.5 / 80.0; 192x128 and 128x192 11.9 / 25.2 /
// 42.9 / 78.9, 13.3 / 27.5 / 47.3 / 85.5; 160x192 16.0 / 29.7 / 50.4 / 99.6, 13.0 / 29.9 / 52.0 / 105.8; 192x192 15.2 / 33.2 / 57.0
// / 111, 17.8 / 41.3 / 69.7 / 150; 160x256 16.6 / 36.3 / 65.4 / 125, 18.3 / 42.1 / 71.8 / 153; 224x192 16.9 / 37.5 / 64.7 / 126,
// 18.5 / 43.3 / 74.4 / 153.
// Switches (tuning and test aid): GEMM_RING = 0 takes the ring kernel out of the choice, 1 + tile forces one of its tiles;
// GEMM_BIG_FROM: number of 128 x 128 tiles from which the 256 x 256 kernels are taken; GEMM_VARIANT forces a kernel:
// 0 = the fallback above, 4 = 256 x 256, 5 = few-row kernel (only where M <= 64), 6 / 7 = ring kernel, 64 x 64 / 128 x 128 tiles.
namespace {
// a of the widest tiles is that of eight wavefronts also beyond K = 6144, where four take 0.7 us more: it decides there only
// between a shared launch of two products on these tiles and other forms, of which the shared launch is the faster (us a backward
// step, 6.3 / 7.0: 2215 x 2048 x 7936 110.8 / 124.3 on 128 x 128 tiles, 4743 x 896 x 16000 272.5 / 300.3; apart 2091 x 2048 x 7168
// 93.3 / 101.9, 3729 x 1152 x 11648 173.0 / 182.6).
struct RingCost { int tm, tn; double a, b; };
constexpr RingCost kRing[RING_TILES] = {{64, 64, 1.0, 0.20},   {128, 64, 1.9, 0.29},  {64, 128, 1.9, 0.29},  {128, 128, 4.0, 0.42}, {128, 256, 6.3, 0.70},
                                        {256, 128, 6.3, 0.70}, {96, 64, 1.3, 0.235},  {64, 192, 2.7, 0.35},  {160, 64, 2.5, 0.31},  {96, 128, 3.2, 0.34},
                                        {160, 128, 4.2, 0.485}, {192, 128, 4.2, 0.56}, {128, 192, 4.2, 0.56}, {160, 192, 5.9, 0.65}, {192, 192, 6.5, 0.75},
                                        {160, 256, 6.1, 0.86}, {224, 192, 7.1, 0.86}};
constexpr int kPathRing = 100;       // + tile: the ring kernel; otherwise a GEMM_VARIANT number

int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
double ring_cost(int tile, const GemmOperands& g, const GemmOperands* g2, int64_t cus) {
    const RingCost& c = kRing[tile];
    auto tiles = [&](const GemmOperands& x) { return cdiv(x.M, c.tm) * cdiv(x.N, c.tn); };
    const double per1 = c.a + (double)cdiv(g.K, BK) * c.b, per2 = g2 ? c.a + (double)cdiv(g2->K, BK) * c.b : 0.0;
    const int64_t n1 = tiles(g), n2 = g2 ? tiles(*g2) : 0;
    const double operands = 1e-5 * (double)(n1 + n2) * (c.tm + c.tn);      // (equal otherwise: fewer operand bytes)
    if (n1 + n2 <= cus) return 3.0 + (per1 > per2 ? per1 : per2) + operands;
    // The low tiles' a is that of one round.  In several 128 x 64 and 64 x 128 tiles take 0.4 us more each (one product, us, 64 x
    // 128 as priced by one round / as now: 319 x 24064 x 10240 160 / 105 on 256 x 256 tiles, 289 x 23680 x 9216 126 / 92, 182 x
    // 34048 x 10368 154 / 115; 35 x 35328 x 5760 51 / 45 on 64 x 64), and beside another product all three 0.8 after the first (a
    // backward step, us: 317 x 6144 x 704 41.1 / 34.0 on 128 x 128 tiles, 2063 x 608 x 14640 117.1 / 109.5; 32 x 14336 x 256 apart
    // 14.3, 64x64 17.7, 64x128 15.1, 128x256 12.1; 84 x 3328 x 2560 128x64 41.8, 64x64 49.2).
    const int64_t r = cdiv(n1 + n2, cus);
    const double later = tile > RING_64x128 ? 0.0 : g2 ? 0.8 * (double)(r - 1) : tile == RING_64x64 ? 0.0 : 0.4 * (double)r;
    const double rounds = (double)r * ((double)n1 * per1 + (double)n2 * per2) / (double)(n1 + n2) + later;
    return 3.0 + (rounds > per1 + per2 ? rounds : per1 + per2) + operands;     // (two unequal products: at least one tile of each in turn)
}
// the cheapest ring tile for one product, or two in one launch
int best_ring(const GemmOperands& g, const GemmOperands* g2, int64_t cus, double* cost) {
    int best = 0;
    for (int t = 0; t < RING_ANY_ROUNDS; ++t) {
        const double c = ring_cost(t, g, g2, cus);
        if (t == 0 || c < *cost) { best = t; *cost = c; }
    }
    return best;
}
// 64 x 192 tiles, which gain least (a twentieth, beyond short contractions), not where a step of them fetches more than one of 96 x 128
// or 128 x 128 tiles does: beyond K = 1024 where rows are no whole lines, beyond 1536 over an odd number of rows of tiles below 16, of
// which the last group in the order of tiles holds one or three.  (us from HBM, with these / with the tiles taken instead; partial lines:
// 172 x 11216 x 5296 42.6 / 35.0, 316 x 8288 x 6944 52.0 / 42.3, 192 x 16024 x 4256 35.6 / 29.5, 105 x 19784 x 2080 19.9 / 18.9, 1222 x 2136
// x 1264 10.2 / 9.2; odd rows: 900 x 3208 x 12800 54.5 / 46.2, 425 x 6864 x 2688 16.1 / 13.4, 415 x 6056 x 4096 21.3 / 17.7, 576 x 4496 x
// 2048 11.7 / 9.8, 185 x 12224 x 3072 20.6 / 18.5.)
bool takes_64x192(const GemmOperands& g) {
    const int64_t rows = cdiv(g.M, 64);
    return g.K <= 1024 || (((g.lda | g.ldb) & 127) == 0 && (g.K <= 1536 || rows % 2 == 0 || rows >= 16));
}
// Tiles that make a round fuller but fetch a weight from HBM more often than those that they replace, one round as well (a served
// model's weight; what the call itself has quantized comes from the cache, where they are 5 to 15 % ahead).  Over rows that are no whole
// lines, in place of 256 x 128 ones, 160 x 192 beyond K = 2560 where those are not much fewer, 128 x 192 beyond 6144 unless in two rows of
// those; in three rows of tiles and more 96 x 128 in place of as many 128 x 128 beyond K = 2048, of nearly as many beyond 4096.  (us a
// forward with the quantization of its activations, the fuller / the others.  160 x 192: 3520 x 1856 x 10416 118 / 102, 448 x 14976 x 7904
// 81 / 71, 953 x 6784 x 5840 65 / 57, 3502 x 1808 x 4384 55.9 / 49.9, but 2618 x 2312 x 2384 28.2 / 29.7, 972 x 6272 x 3488 36.0 / 37.5; 128 x 192:
// 976 x 4720 x 10464 94.8 / 88.1, but 409 x 11864 x 4016 39.8 / 42.6, 387 x 11632 x 10448 81 / 88; 96 x 128: 266 x 10280 x 15488 70.9 / 63.2, 279 x
// 9208 x 7168 36.9 / 34.0, 274 x 8944 x 2688 18.4 / 17.8, 658 x 4096 x 16064 89 / 79, 644 x 3784 x 8576 41.2 / 37.5, but 280 x 9352 x 1648 10 %
// ahead, 525 x 4720 x 3712 1 %, 655 x 4480 x 2864 10 %.)
bool fetches_more(int t, const GemmOperands& g, int64_t cus) {
    auto tiles = [&](int i) { return cdiv(g.M, kRing[i].tm) * cdiv(g.N, kRing[i].tn); };
    const int64_t others = tiles(RING_256x128);
    switch (t) {
        case RING_96x128: return g.M > 256 && ((g.K > 2048 && tiles(t) <= tiles(RING_128x128)) || (g.K > 4096 && 6 * tiles(t) <= 7 * tiles(RING_128x128)));
        case RING_128x192: if (g.K <= 6144 || cdiv(g.M, 256) == 2) return false; break;
        case RING_160x192: if (g.K <= 2560 || 8 * others < 7 * tiles(t)) return false; break;
        default: return false;
    }
    double cost;
    return ((g.lda | g.ldb) & 127) != 0 && others <= cus && best_ring(g, nullptr, cus, &cost) == RING_256x128;
}
// Of the tiles [from, to) between those sizes, which make a round fuller: the cheapest that covers the product in one round, if
// it is cheaper than *cost, else -1.  Over several rounds they are behind (two full ones of 192 x 192 tiles, K = 4096, 65.8 against
// 66.9 us on 256 x 256, three 96.6 / 87.2; of 96 x 64 21.1 / 17.0).  Not against a weight that is streamed for up to 256 rows:
// there the number of times it is fetched counts (ring_hint, one_row).
int best_one_round(const GemmOperands& g, int from, int to, int64_t cus, double* cost, bool at_rest = false) {
    int best = -1;
    if (g.M <= 256 && stream_weight(g.b, g.ldb, g.N, g.K)) return best;
    for (int t = from; t < to; ++t) {
        if (cdiv(g.M, kRing[t].tm) * cdiv(g.N, kRing[t].tn) > cus) continue;
        if ((t == RING_64x192 && !takes_64x192(g)) || (at_rest && fetches_more(t, g, cus))) continue;
        const double c = ring_cost(t, g, nullptr, cus);
        if (c < *cost) { best = t; *cost = c; }
    }
    return best;
}
// Two products in one launch, tile by tile: those of the longer contraction first (long / short: number and us of its tiles), each
// CU taking the next one that is left.  (ring_cost's whole rounds of an average tile are up to a quarter more where a few long tiles
// precede many short ones: 4864 x 1024 x 14336 143 / 123 us, 1286 x 1024 x 5120 33 / 25.)
double tiles_in_turn(int64_t n_long, double t_long, int64_t n_short, double t_short, int64_t cus) {
    const int64_t q = n_long / cus, r = n_long % cus;
    const double level[2] = {(double)q * t_long, (double)(q + (r > 0)) * t_long};      // when the CUs are done with the long ones: cus - r, r of them
    const double ideal = ((double)n_long * t_long + (double)n_short * t_short) / (double)cus;
    auto fit = [&](double end, double from) { return end < from ? (int64_t)0 : (int64_t)((end - from) / t_short + 1e-6); };
    double end = 1e30;
    for (const double from : level) {      // the end lies a whole number of short tiles behind one of the levels
        double k = ideal > from ? (double)(int64_t)((ideal - from) / t_short) : 0.0;
        while ((cus - r) * fit(from + k * t_short, level[0]) + r * fit(from + k * t_short, level[1]) < n_short) k += 1.0;
        if (from + k * t_short < end) end = from + k * t_short;
    }
    return end > level[1] ? end : level[1];
}
// one round of the 256 x 256 kernels (half tiles, the lower tiles of the persistent one)
double large_cost(const GemmOperands& g, bool bf16, int64_t cus) {
    const double steps = (double)cdiv(g.K, BK);
    if (2 * cdiv(g.M, 256) * cdiv(g.N, 256) <= cus) return 7.2 + 0.91 * steps;
    const int h = bf16 ? one_round_height(g, cus) : 256;
    return h == 192 ? 9.0 + 0.97 * steps : h == 224 ? 9.6 + 1.085 * steps : 10.0 + 1.2 * steps;
}
// 17 to 32 rows against a wide weight: the ring kernel's tile, or -1 for the few-row kernel, which has no rounds to fill.  64 x 64
// tiles over one round at most, 64 x 128 ones where those fit one and the contraction pays for them, else 64 x 64 ones where it is
// long enough to make up for a last round that is not full.  (us at 17 rows from HBM, few-row / 64 x 64 / 64 x 128; N x K: 16384 x
// 1024 6.7 / 6.5 / 7.4; 20480 x 512 6.1 / 7.9 / 6.1, x 1024 8.9 / 10.0 / 7.9, x 2048 13.8 / 14.2 / 11.3, x 4096 21.8 / 25.8 / 21.6;
// 28672 x 512 6.5 / 8.3 / 6.9, x 4096 26.3 / 25.1 / 24.3, 32768 x 8192 58.4 / 53.8 / 58.7; 36864 x 2048 20.5 / 21.4 / 22.4, x 8192
// 72.4 / 65.8 / 79.0; 65536 x 2048 25.3 / 31.5 / 25.5, x 3072 36.8 / 39.5 / 37.3, 128256 x 4096 107.2 / 95.6 / 97.8.  On a chip
// just full of 64 x 128 tiles whose rows lie a multiple of 4096 bytes apart the few-row kernel is ahead: 32768 x 4096 27.9 / 30.3 /
// 32.4)
int few_rows_tile(const GemmOperands& g, int64_t cus) {
    const int64_t tiles = cdiv(g.N, 64), K = g.K;
    if (tiles <= cus) return RING_64x64;
    if (tiles <= 2 * cus) {
        if (K < 1024 || (g.ldb % 4096 == 0 && K < 8192 && 8 * tiles > 15 * cus)) return -1;
        return K >= 8192 && 5 * tiles >= 8 * cus ? RING_64x64 : RING_64x128;
    }
    return K >= 6144 || (K >= 4096 && tiles >= 4 * cus) ? RING_64x64 : -1;
}
// kernel for one product; *cost: its estimate (large where there is none); any_rounds: only of the tiles that pairs can take too
int pick_path(const GemmOperands& g, double* cost, bool any_rounds = false) {
    *cost = 1e30;
    const bool fits = gemm_fp8_ring_fits(g), ring = fits && knob(KNOB_GEMM_RING) != 0;
    if (const int r = knob(KNOB_GEMM_RING); r >= 1 && r <= RING_TILES && fits) return kPathRing + r - 1;
    const int v = knob(KNOB_GEMM_VARIANT);
    if (v == 0 || v == 4 || v == 5) return v;
    if (v == 6 || v == 7) return fits ? kPathRing + (v == 6 ? RING_64x64 : RING_128x128) : 0;
    const int64_t cus = compute_units() > 0 ? compute_units() : 256;
    if (g.M <= 16 || (g.M > 32 && g.M <= 64 && g.N <= 8192 && g.K >= 2048 && gemm_fp8_snake_fits(g.lda, g.ldb))) return 5;
    if (g.M <= 32) {
        if (!ring || 8 * cdiv(g.N, 64) < 5 * cus) return 5;
        // Codes that the ring kernel has read take longer to be written anew by the next call's quantization, unless in strips (us
        // a call, few-row / ring: forward by rows 17 x 12288 x 2048 23.9 / 32.3, 32 x 16384 x 1536 25.1 / 29.8, 32 x 14336 x 4096
        // 40.1 / 43.3, per tensor 34.7 / 38.4, 35.7 / 39.8, 66.3 / 66.2, 17 x 28672 x 8192 239.5 / 237.2; dX per tensor 32 x 16384
        // x 1536 40.1 / 43.9, by strips 32 x 20480 x 2048 44.6 / 43.3).
        if (g.b_from == B_WRITTEN && !stream_weight(g.b, g.ldb, g.N, g.K)) return 5;
        const int tile = few_rows_tile(g, cus);
        *cost = ring_cost(tile < 0 ? RING_64x64 : tile, g, nullptr, cus);      // (what the few-row kernel takes too where the contraction is short)
        return tile < 0 ? 5 : kPathRing + tile;
    }
    const int64_t big = cdiv(g.M, 256) * cdiv(g.N, 256);
    if (const int b = knob(KNOB_GEMM_BIG_FROM); b > 0 && cdiv(g.M, 128) * cdiv(g.N, 128) >= b) return 4;
    if (big > cus || !ring) return 4;
    // (fp32 results are priced as bfloat16 ones are, although they have no lower tiles: without those a sum of less than 512 elements
    // would go to 128 x 256 tiles more often, 588 x 13024 x 272 19.5 -> 17.8 us, but 3032 x 2592 x 496 15.0 -> 19.2, 875 x 8264 x 416 16.4 -> 19.5)
    double cost_big = large_cost(g, !any_rounds, cus), operands = 0.0;
    int tile = best_ring(g, nullptr, cus, cost);
    if (tile == RING_128x256 && one_row(g)) tile = RING_256x128;
    if (!any_rounds) {
        // (the lower tiles priced with their operands as ring_cost prices its own: K up to 512 on rather few of them is otherwise left to
        // them where one round of 128 x 256 tiles is faster; us, lower / 128 x 256: 820 x 8576 x 288 11.0 / 9.2, 329 x 19744 x 384 9.8 / 8.6,
        // 560 x 12864 x 512 10.2 / 9.3, 834 x 9056 x 448 10.5 / 9.8, 374 x 20576 x 512 9.9 / 9.9)
        const int h = one_round_height(g, cus);
        const bool at_rest = g.b_from == B_AT_REST;
        if (best_one_round(g, RING_WIDE, RING_TILES, cus, &cost_big, at_rest) < 0 && h != 256) operands = 1e-5 * (double)(cdiv(g.M, h) * cdiv(g.N, 256) * (h + 256));
        if (const int t = best_one_round(g, RING_ANY_ROUNDS, RING_WIDE, cus, cost, at_rest); t >= 0) tile = t;
    }
    if (*cost <= cost_big + operands) return kPathRing + tile;
    *cost = cost_big;
    return 4;
}
}  // namespace

hipError_t launch_gemm_fp8(const uint8_t* a, int64_t lda, int fmt_a, const float* scale_a, int row_a,
                           const uint8_t* b, int64_t ldb, int fmt_b, const float* scale_b, int row_b,
                           int64_t M, int64_t N, int64_t K, void* out, int64_t ld_out, int out_f32,
                           hipStream_t st, BFrom b_from) {
    if (M == 0 || N == 0) return hipSuccess;
    const GemmOperands g{a, lda, scale_a, b, ldb, scale_b, M, N, K, out, ld_out, b_from};
    double cost;
    const int v = pick_path(g, &cost);
    if (v >= kPathRing) return launch_gemm_fp8_ring(v - kPathRing, g, nullptr, fmt_a, fmt_b, row_a, row_b, out_f32 ? 1 : 0, st);
    if (v == 5 && M <= 64 && K > 0)
        return launch_gemm_fp8_skinny(a, lda, fmt_a, scale_a, row_a, b, ldb, fmt_b, scale_b, row_b, M, N, K, out, ld_out,
                                      out_f32, st);
    if (v == 4 && gemm_fp8_snake_fits(lda, ldb))   // else: the 128 x 128 register-staged kernel
        return launch_gemm_fp8_snake(a, lda, fmt_a, scale_a, row_a, b, ldb, fmt_b, scale_b, row_b, M, N, K, out, ld_out,
                                     out_f32, st);
#define FP8K_GEMM(FA_, FB_)                                                                    \
    if (fmt_a == FA_ && fmt_b == FB_)                                                          \
        return out_f32 ? launch_tn<FA_, FB_, true>(g, row_a, row_b, st) : launch_tn<FA_, FB_, false>(g, row_a, row_b, st)
    FP8K_GEMM(FMT_E4M3FN, FMT_E4M3FN);
    FP8K_GEMM(FMT_E5M2, FMT_E4M3FN);
    FP8K_GEMM(FMT_E4M3FN, FMT_E5M2);
    FP8K_GEMM(FMT_E5M2, FMT_E5M2);
#undef FP8K_GEMM
    return hipErrorInvalidValue;
}

// The block-scaled product takes the same tiles; its K steps cost a tenth more with the scales in slabs and a quarter more
// with plain scale rows (a cache line per row and step).  256 x 256 tiles: 9 + 1.05 * steps for at most half of the CUs,
// else 10 + 1.25 * steps (there are no half tiles).  Measured (us, slabs / plain, before: 256 x 256 or register-staged tiles):
//     1024 x 1024 x 4096  64x64 12.6 / 14.3, before 40.7 / 77.2     2048 x 2048 x 4096  128x128 21.7 / 26.5, before 41.1 / 76.9
//     2048 x 4096 x 4096  128x256 34.8 / 39.6, before 42.6 / 43.6   3072 x 4096 x 4096  128x256 59.5 / 67.4, 256x256 48.7 / 46.4
// With the shorter rings and eight wavefronts since, over 300 x 14336 .. 4096 x 4096 and K = 1024 .. 14336 (130 shapes), the tile
// taken is on average 1.2 % (slabs) and 3.0 % (plain rows) behind the best one, at most 40 %, where 256 x 256 tiles are taken for
// K = 1024; plain products 1.8 %.
int gemm_mxfp8_ring_choice(const GemmOperands& g, bool plain_scales) {
    if (const int r = knob(KNOB_GEMM_RING); r >= 0 && r <= RING_MX_TILES) return r - 1;
    const int64_t cus = compute_units() > 0 ? compute_units() : 256;
    const int64_t big = cdiv(g.M, 256) * cdiv(g.N, 256);
    if (big > cus) return -1;
    double cost = 0.0;
    int tile = best_ring(g, nullptr, cus, &cost);
    if (const int t = best_one_round(g, RING_ANY_ROUNDS, RING_MX_TILES, cus, &cost); t >= 0) tile = t;
    const double steps = (double)cdiv(g.K, BK);
    const double cost_big = 2 * big <= cus ? 9.0 + 1.05 * steps : 10.0 + 1.25 * steps;
    return 3.0 + (cost - 3.0) * (plain_scales ? 1.25 : 1.1) <= cost_big ? tile : -1;
}

// Height of the persistent kernel's tiles for a product whose scales lie in slabs, or 0: one 256 x 256 tile per workgroup.  Over
// several rounds the height with the least sum of round lengths, a tile of h rows taking a time like h + 100, a last round of up to
// half of the CUs 0.85 of a full one (us, tile per workgroup / 256 / 224 / 192: 14336 x 4096 x 4096 188 / 184 / 175 / 189; 4096 x
// 14336 x 4096 189 / 183 / 202 / 194; 8192 x 6144 x 4096 152 / 149 / 166 / 181; 6144 x 4096 x 8192 167 / 165 / 156 / 150; 5000 x
// 8192 x 2048 83 / 76 / 73 / 82).  256 rows only up to K = 6144, where the tile boundaries count (us, tile per workgroup / 256:
// 8192 x 16384 x 2048 229 / 211, x 4096 394 / 383, x 8192 760 / 767; 16384 x 16384 x 1024 277 / 243; 16384 x 4096 x 14336 657 / 658).
// In one round only the lower tiles, where they fill it better (3072 x 4096 x 4096 46.5 / 46.2 / 44.1 / 42.9).  Where rows of the output
// start between sectors, only lower tiles and from K = 3072 on (us, tile per workgroup / persistent: 8192 x 8184 x 1024 83 / 109, x 4096 219
// / 232, 6144 x 4080 x 1024 39 / 51, x 2048 58 / 68, x 4096 98 / 99, x 8192 180 / 174; 5000 x 8184 x 2048 90 / 100, x 8192 288 / 276, 6166 x 7856
// x 3584 175 / 159, 4174 x 2312 x 15872 153 / 136; 350 products over several rounds, relative to a tile per workgroup: of 192 rows K = 2048 ..
// 2559 +2 %, 3072 .. 3583 -4 %, 4096 .. 8191 -10 %; of 224 rows 2560 .. 3071 +6 %, 3584 .. 8191 -2 to -5 %; of 256 rows +17 %, +8 %, +5 %).
int gemm_mxfp8_stream_height(const GemmOperands& g) {
    const int64_t M = g.M, N = g.N, K = g.K;
    const int sw = knob(KNOB_GEMM_STREAM), forced = knob(KNOB_GEMM_TILE_M);
    if (forced == 256 || forced == 224 || forced == 192) return forced;
    const int64_t cus = compute_units() > 0 ? compute_units() : 256, cols = cdiv(N, 256);
    if (cdiv(M, 256) * cols <= cus && sw < 2) {
        const int low = one_round_height(g, cus);
        return low == 256 ? 0 : low;
    }
    const bool sectors = rows_on_sectors(g);
    if (!sectors && K < 3072 && sw < 2) return 0;
    int best = 256;
    double least = 0.0;
    for (int tm : {256, 224, 192}) {
        const int64_t tiles = cdiv(M, tm) * cols, rest = tiles % cus;
        const double cost = (tm + 100) * ((double)(tiles / cus) + (rest == 0 ? 0.0 : 2 * rest <= cus ? 0.85 : 1.0));
        if (tm == 256 || cost < least) { best = tm; least = cost; }
    }
    return best == 256 && (K > 6144 || !sectors) && sw < 2 ? 0 : best;
}

int gemm_fp8_ring_choice(const GemmOperands& g) {
    double cost;
    const int v = pick_path(g, &cost);
    if (v >= kPathRing) return v - kPathRing;
    if (v == 4 || knob(KNOB_GEMM_RING) == 0 || !gemm_fp8_ring_fits(g)) return -1;
    return best_ring(g, nullptr, compute_units() > 0 ? compute_units() : 256, &cost);
}

int gemm_fp8_wide_choice(const GemmOperands& g, bool bf16) {
    if (knob(KNOB_GEMM_RING) >= 0 || knob(KNOB_GEMM_VARIANT) >= 0 || knob(KNOB_GEMM_BIG_FROM) > 0 || knob(KNOB_GEMM_STREAM) >= 0 || knob(KNOB_GEMM_TILE_M) >= 0)
        return -1;      // a form is forced
    if (!gemm_fp8_ring_fits(g)) return -1;
    const int64_t cus = compute_units() > 0 ? compute_units() : 256;
    double cost = large_cost(g, bf16, cus);
    return best_one_round(g, RING_WIDE, RING_TILES, cus, &cost);
}

// Two products of the same formats and kinds of scale (bfloat16 results) in ONE launch, for the pair dX, dW of a
// backward step whose products are too small to fill the chip one at a time.  hipErrorNotSupported (nothing launched)
// where one launch each is estimated to be as fast, on the same kinds of tile, or clearly faster on those that only single products
// take: the caller then launches them one after the other.
hipError_t launch_gemm_fp8_pair(const GemmOperands& g1, const GemmOperands& g2, int fmt_a, int fmt_b, int row_a, int row_b,
                                hipStream_t st) {
    if (g1.M == 0 || g1.N == 0 || g2.M == 0 || g2.N == 0 || knob(KNOB_PAIRS) == 0) return hipErrorNotSupported;
    if (!gemm_fp8_ring_fits(g1) || !gemm_fp8_ring_fits(g2)) return hipErrorNotSupported;
    double c1, c2, both = 0.0;
    const int v1 = pick_path(g1, &c1, true), v2 = pick_path(g2, &c2, true);
    if (c1 > 1e29 || c2 > 1e29) {      // no estimate: forced, few rows, or large
        if (v1 < kPathRing || v1 != v2) return hipErrorNotSupported;
        return launch_gemm_fp8_ring(v1 - kPathRing, g1, &g2, fmt_a, fmt_b, row_a, row_b, 0, st);
    }
    const int64_t cus = compute_units() > 0 ? compute_units() : 256;
    const int tile = best_ring(g1, &g2, cus, &both);
    if (both >= c1 + c2) return hipErrorNotSupported;
    // Against the tiles that only single products take (one round of them, or of the persistent kernel's lower ones) estimates do not
    // compare as like with like: a shared launch is up to a fifth faster than its own - no gap between the products, tiles of both to
    // fill the last round.  Beyond that the two go apart, unless a short contraction leaves mostly prologue and epilogue.  (Backward steps,
    // us, shared / apart, by estimated ratio.  From 1.2 on, 91 steps, 4 to 16 % faster apart: 3072 x 3072 x 3072 86 / 78, 4352 x 2048 x
    // 5120 132 / 122, 6144 x 1504 x 5472 163 / 148, 7973 x 1040 x 7984 236 / 203, 1280 x 2048 x 6880 77 / 72.  1.1 .. 1.2: 6144 x 2048 x
    // 6144 183 / 169, 2560 x 2048 x 8192 119 / 114, but 2048 x 5744 x 1904 67 / 75, 3072 x 3728 x 3024 90 / 97, 1170 x 4016 x 2048 40 / 44.
    // Below, 50 of 64 faster shared, by up to 15 %.  Up to 1024 tokens or features: 1012 x 4112 x 2848 58.8 / 63.7, 875 x 2656 x 5120 58.3
    // / 58.4, 768 x 3072 x 4496 53.7 / 51.4.)
    const bool swap = g2.K > g1.K;     // the workgroups of the longer contraction first
    const GemmOperands &first = swap ? g2 : g1, &second = swap ? g1 : g2;
    if (second.K > 1024) {
        const RingCost& c = kRing[tile];
        auto tiles = [&](const GemmOperands& g) { return cdiv(g.M, c.tm) * cdiv(g.N, c.tn); };
        auto each = [&](const GemmOperands& g) { return c.a + (double)cdiv(g.K, BK) * c.b; };
        pick_path(g1, &c1);      // what they take by themselves
        pick_path(g2, &c2);
        if (3.0 + tiles_in_turn(tiles(first), each(first), tiles(second), each(second), cus) > 1.2 * (c1 + c2)) return hipErrorNotSupported;
    }
    return launch_gemm_fp8_ring(tile, first, &second, fmt_a, fmt_b, row_a, row_b, 0, st);
}

}  // namespace fp8k
