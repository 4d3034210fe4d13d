// Product of up to 16 rows against a large weight, on persistent workgroups: out[M, N] = (A[M, K] . B[N, K]^T) / (sa * sb).
//
// The few-row kernel of gemm_fp8_skinny.hip gives every wavefront 32 rows of the weight and fetches A again with each of them; its
// workgroups come and go, each with a ring to fill and K parts to sum while it streams nothing.  Here one workgroup of eight
// wavefronts per CU walks a list of tiles of 16 weight rows.  Wavefront w owns an eighth of K for all of them: its fragments of A sit
// in registers from the start, and only the weight passes through LDS, in a private ring that never drains between tiles.  A comes
// the same way, as the first units of the ring.  At a tile's end the eight parts are summed by one wavefront (each in turn) while the
// others stream on: one barrier a tile.
//
// What bounds it is the weight stream: the same loads without the product take 34.3 us for 28672 x 8192 (6.9 TB/s), at 16 rows the
// product 38.5 (40.0 on the few-row kernel), most of the difference before A has arrived.  Where it is taken: few_row_streams.
#include "fp8_device.hpp"
#include "launchers.hpp"
#include "tuning.hpp"

namespace fp8k {

namespace fs {
typedef int v8i_t __attribute__((ext_vector_type(8)));
typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef float v4f_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
constexpr int WAVES = 8;
constexpr int RING = 8;            // units (16 rows x 128 bytes) in flight per wavefront: what the LDS holds
constexpr int MAX_TILES = 32;      // per workgroup (their scales sit in LDS)

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    f32x2_t v = {a, b};
    bf16x2_t h = __builtin_convertvector(v, bf16x2_t);
    uint32_t r;
    __builtin_memcpy(&r, &h, 4);
    return r;
}
// 16 bytes per lane from a raw buffer into LDS at lds_addr + lane * 16, zeros out of range; the wavefront's own LDS reads of the slot
// are waited for first
template <bool HINT>
__device__ __forceinline__ void lds_dma16(v4i_t rsrc, uint32_t lds_addr, uint32_t voffset) {
    if constexpr (HINT)
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds"
                     :
                     : "s"(lds_addr), "v"(voffset), "s"(rsrc)
                     : "memory", "m0");
    else
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     :
                     : "s"(lds_addr), "v"(voffset), "s"(rsrc)
                     : "memory", "m0");
}
// 4 bytes per lane
__device__ __forceinline__ void lds_dma4(v4i_t rsrc, uint32_t lds_addr, uint32_t voffset) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" : : "s"(lds_addr), "v"(voffset), "s"(rsrc) : "memory", "m0");
}
template <int N_>
__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N_) : "memory"); }
__device__ __forceinline__ void barrier_lds() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
}  // namespace fs

// PER: most K steps of a wavefront.  Workgroup b's tiles: first * b + step * j, either every step-th (first = 1) or a run of `first`.
template <int FA, int FB, int PER, bool HINT>
__global__ __launch_bounds__(64 * fs::WAVES) void gemm_fp8_few_stream_kernel(const uint8_t* __restrict__ A, int64_t lda, const uint8_t* __restrict__ B,
                                                                              int64_t ldb, const float* __restrict__ scale_a, int row_a,
                                                                              const float* __restrict__ scale_b, int row_b, int M, int N, int K,
                                                                              void* __restrict__ out, int64_t ld_out, int out_f32, int first, int step) {
    using namespace fs;
    // LDS: rings; parts [2][WAVES][64 lanes][16 bytes]; reciprocals of the scales of this workgroup's columns; scales of A, a copy
    // per wavefront
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
#ifdef __HIP_DEVICE_COMPILE__      // (the arguments in one trip, see gemm_fp8_ring.hpp)
    asm volatile("" ::"s"(A), "s"(lda), "s"(B), "s"(ldb), "s"(scale_a), "s"(row_a), "s"(scale_b), "s"(row_b), "s"(M), "s"(N), "s"(K), "s"(out), "s"(ld_out),
                 "s"(out_f32), "s"(first), "s"(step));
#endif
    v4f_t* const parts = reinterpret_cast<v4f_t*>(smem + WAVES * RING * 2048);
    float* const inv_sb = reinterpret_cast<float*>(parts + 2 * WAVES * 64);
    float* const sa_tab = inv_sb + MAX_TILES * 16;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4;
    constexpr uint32_t OOB = 0x80000000u;

    const int tiles = (N + 15) >> 4, t0 = first * (int)blockIdx.x;
    const int mine = first == 1 ? (tiles - t0 + step - 1) / step : (tiles - t0 < first ? tiles - t0 : first);      // (first == 1: strided; else runs of `first`)
    if (mine <= 0) return;
    const int ksteps = (K + 127) >> 7, per = (ksteps + WAVES - 1) / WAVES;
    const int s_begin = wave * per;

    // ---- scales: one column per thread, the rows once per wavefront (older than the units, so there with the first of them)
    const uint64_t psa = reinterpret_cast<uint64_t>(scale_a), psb = reinterpret_cast<uint64_t>(scale_b), pa = reinterpret_cast<uint64_t>(A);
    const v4i_t rsrc_sa = {(int)(uint32_t)psa, (int)(uint32_t)(psa >> 32), row_a ? M * 4 : 4, 0x00020000};
    const v4i_t rsrc_sb = {(int)(uint32_t)psb, (int)(uint32_t)(psb >> 32), row_b ? N * 4 : 4, 0x00020000};
    const v4i_t rsrc_a = {(int)(uint32_t)pa, (int)(uint32_t)(pa >> 32), (int)((int64_t)(M - 1) * lda + K), 0x00020000};
    lds_dma4(rsrc_sb, (uint32_t)(size_t)inv_sb + (uint32_t)wave * 256u, row_b ? (uint32_t)((t0 + (tid >> 4) * step) * 16 + (tid & 15)) * 4u : 0u);
    lds_dma4(rsrc_sa, (uint32_t)(size_t)sa_tab + (uint32_t)wave * 256u, row_a ? (uint32_t)(lane & 15) * 4u : 0u);

    // ---- units: first A's, then the weight's.  Load h of a unit fetches rows 8 h + lane / 8; lane's chunk
    //      slot lane % 8 receives chunk slot ^ key(row)
    const int lrow = lane >> 3;
    const int c0 = (lane & 7) ^ ((lrow >> 1) & 7), c1 = (lane & 7) ^ ((4 + (lrow >> 1)) & 7);
    const uint32_t vb0 = (uint32_t)(lrow * (int)ldb + c0 * 16), vb1 = (uint32_t)((8 + lrow) * (int)ldb + c1 * 16);
    const uint32_t va0 = (uint32_t)(lrow * (int)lda + c0 * 16), va1 = (uint32_t)((8 + lrow) * (int)lda + c1 * 16);
    const uint32_t ring = (uint32_t)(size_t)smem + (uint32_t)wave * (RING * 2048u);
    // the unit of the weight that is requested next: step next_k / 128 of the tile that rsrc_b describes, `left` tiles to go
    const int k_begin = s_begin * 128, k_end = k_begin + per * 128;
    int next_k = k_begin, left = mine, rows_left = N - t0 * 16;
    uint64_t pb = reinterpret_cast<uint64_t>(B + (int64_t)t0 * 16 * ldb);
    const uint64_t pb_step = (uint64_t)step * 16 * (uint64_t)ldb;
    v4i_t rsrc_b = {(int)(uint32_t)pb, (int)(uint32_t)(pb >> 32), ((rows_left < 16 ? rows_left : 16) - 1) * (int)ldb + K, 0x00020000};
    auto issue = [&](uint32_t dst) {
        lds_dma16<HINT>(rsrc_b, dst, next_k + c0 * 16 < K ? vb0 + (uint32_t)next_k : OOB);
        lds_dma16<HINT>(rsrc_b, dst + 1024, next_k + c1 * 16 < K ? vb1 + (uint32_t)next_k : OOB);
        next_k += 128;
        if (next_k == k_end) {
            next_k = k_begin;
            pb += pb_step;
            rows_left -= 16 * step;
            left -= 1;
            rsrc_b[0] = (int)(uint32_t)pb;
            rsrc_b[1] = (int)(uint32_t)(pb >> 32);
            rsrc_b[2] = left > 0 ? ((rows_left < 16 ? rows_left : 16) - 1) * (int)ldb + K : 0;
        }
    };
    auto issue_unit = [&](int u, uint32_t dst) {      // number u of the whole sequence, as long as it may be A's
        if (u < per) {
            const int k0 = (s_begin + u) * 128;
            lds_dma16<false>(rsrc_a, dst, k0 + c0 * 16 < K ? va0 + (uint32_t)k0 : OOB);
            lds_dma16<false>(rsrc_a, dst + 1024, k0 + c1 * 16 < K ? va1 + (uint32_t)k0 : OOB);
        } else {
            issue(dst);
        }
    };
#pragma unroll 1
    for (int u = 0; u < RING; ++u) issue_unit(u, ring + u * 2048);

    const int key = (i >> 1) & 7;
    const int f_lo = i * 128 + ((g ^ key) << 4), f_hi = i * 128 + (((g + 4) ^ key) << 4);
    const uint8_t* const ring_p = smem + wave * (RING * 2048);
    int slot = 0;
    auto unit = [&]() {                   // the fragment of the oldest unit: chunks g and g + 4 of row i
        wait_vmem<2 * (RING - 1)>();      // all but the younger units have landed
        const uint8_t* u = ring_p + slot * 2048;
        const uint4 lo = *reinterpret_cast<const uint4*>(u + f_lo), hi = *reinterpret_cast<const uint4*>(u + f_hi);
        return v8i_t{(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
    };
    v8i_t af[PER];
#pragma unroll
    for (int s = 0; s < PER; ++s) {
        af[s] = v8i_t{0, 0, 0, 0, 0, 0, 0, 0};
        if (s < per) {
            af[s] = unit();
            if constexpr (PER > RING) issue_unit(s + RING, ring + (uint32_t)slot * 2048u);
            else issue(ring + (uint32_t)slot * 2048u);
            slot = slot + 1 == RING ? 0 : slot + 1;
        }
    }
    const float inv_a = 1.0f / sa_tab[wave * 64 + i];
    inv_sb[tid] = 1.0f / inv_sb[tid];
    for (int j = 0; j < mine; ++j) {
        v4f_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < PER; ++s) {
            if (s < per) {
                const v8i_t bf = unit();
                acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(bf, af[s], acc, FB, FA, 0, 0, 0, 0);
                issue(ring + (uint32_t)slot * 2048u);
                slot = slot + 1 == RING ? 0 : slot + 1;
            }
        }
        // ---- the parts of K: parked by every wavefront, summed by one (two sets: the next tile's are parked before it is done)
        v4f_t* const set = parts + (j & 1) * (WAVES * 64);
        set[wave * 64 + lane] = acc;
        barrier_lds();
        if (wave != (j & (WAVES - 1))) continue;
        const int nb = (t0 + j * step) * 16 + 4 * g;
        const float4 ib = *reinterpret_cast<const float4*>(inv_sb + j * 16 + 4 * g);
        v4f_t sum = set[lane];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) sum += set[w * 64 + lane];
        if (i >= M || nb >= N) continue;
        const float v[4] = {(sum[0] * inv_a) * ib.x, (sum[1] * inv_a) * ib.y, (sum[2] * inv_a) * ib.z, (sum[3] * inv_a) * ib.w};
        if (out_f32) {
            float* dst = static_cast<float*>(out) + (int64_t)i * ld_out + nb;
            if (nb + 4 <= N) *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
            else for (int r = 0; nb + r < N; ++r) dst[r] = v[r];
        } else {
            uint16_t* dst = static_cast<uint16_t*>(out) + (int64_t)i * ld_out + nb;
            const uint32_t p0 = pack_bf16(v[0], v[1]), p1 = pack_bf16(v[2], v[3]);
            if (nb + 4 <= N) {
                *reinterpret_cast<uint2*>(dst) = make_uint2(p0, p1);
            } else {
                const uint32_t w2[2] = {p0, p1};
                for (int r = 0; nb + r < N; ++r) dst[r] = (uint16_t)(w2[r >> 1] >> ((r & 1) * 16));
            }
        }
    }
    wait_vmem<0>();       // trailing (out-of-range) refills must land before the LDS is handed back
}

template <int FA, int FB, int PER>
static hipError_t launch_fs(const GemmOperands& g, int row_a, int row_b, int out_f32, int first, int step, int grid, hipStream_t st) {
    using namespace fs;
    constexpr int lds = WAVES * RING * 2048 + 2 * WAVES * 1024 + MAX_TILES * 16 * 4 + WAVES * 256;
    static_assert(lds <= 160 * 1024, "LDS");
    auto launch = [&](auto kern, DynamicLdsOnce& attr) {
        if (hipError_t e = attr.ensure(reinterpret_cast<const void*>(kern), lds); e != hipSuccess) return e;
        kern<<<dim3((unsigned)grid), dim3(64 * WAVES), lds, st>>>(g.a, g.lda, g.b, g.ldb, g.scale_a, row_a, g.scale_b, row_b, (int)g.M, (int)g.N, (int)g.K,
                                                                 g.out, g.ld_out, out_f32, first, step);
        return hipGetLastError();
    };
    static DynamicLdsOnce attr[2];
    if (stream_weight(g.b, g.ldb, g.N, g.K)) return launch(gemm_fp8_few_stream_kernel<FA, FB, PER, true>, attr[1]);
    return launch(gemm_fp8_few_stream_kernel<FA, FB, PER, false>, attr[0]);
}

// hipErrorNotSupported (nothing launched) where this form does not apply (few_row_streams); the order of the tiles: few_row_runs.
hipError_t launch_gemm_fp8_few_stream(const GemmOperands& g, int fmt_a, int fmt_b, int row_a, int row_b, int out_f32, hipStream_t st) {
    const int64_t cus = compute_units() > 0 ? compute_units() : 256;
    const int forced = knob(KNOB_SKINNY_DMA);
    if (!few_row_streams(g, cus, forced)) return hipErrorNotSupported;
    const int64_t tiles = (g.N + 15) / 16, grid = tiles < cus ? tiles : cus, run = (tiles + grid - 1) / grid;
    const int per = (int)(((g.K + 127) / 128 + fs::WAVES - 1) / fs::WAVES);
    const bool runs = few_row_runs(g, cus, forced);
    const int first = runs ? (int)run : 1, step = runs ? 1 : (int)grid;
#define FP8K_FS(FA_, FB_, PER_) \
    if (fmt_a == FA_ && fmt_b == FB_ && per <= PER_) return launch_fs<FA_, FB_, PER_>(g, row_a, row_b, out_f32, first, step, (int)grid, st)
#define FP8K_FS3(FA_, FB_) FP8K_FS(FA_, FB_, 4); FP8K_FS(FA_, FB_, 8); FP8K_FS(FA_, FB_, 16)
    FP8K_FS3(FMT_E4M3FN, FMT_E4M3FN);
    FP8K_FS3(FMT_E5M2, FMT_E4M3FN);
    FP8K_FS3(FMT_E4M3FN, FMT_E5M2);
    FP8K_FS3(FMT_E5M2, FMT_E5M2);
#undef FP8K_FS3
#undef FP8K_FS
    return hipErrorNotSupported;
}

}  // namespace fp8k
