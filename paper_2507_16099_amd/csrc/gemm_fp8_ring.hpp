// Scaled FP8 GEMM for gfx950, products of few to middling size:
// out[M,N] = (A[M,K] . B[N,K]^T) / (sa * sb), v_mfma_f32_16x16x128_f8f6f4, and its block-scaled (MX) form
// out[m,n] = sum_blk 2^(ea[m,blk]-127) 2^(eb[n,blk]-127) sum_{k in blk} a[m,k] b[n,k], v_mfma_scale_f32_16x16x128_f8f6f4.
//
// What bounds these products is not the matrix cores but the time from the request of a K step's operands to their
// arrival: a workgroup is alone on its CU (there are fewer tiles than fill the chip many times over), and a K step of
// a 128 x 128 tile is 512 matrix-core cycles next to some 2000 cycles of latency from the Infinity Cache or HBM.  So
// the tiles here are smaller than the 256 x 256 of the large-product kernels, which gives every CU one, and the LDS
// that a smaller tile leaves free holds more K steps in flight: a ring of R stages, filled R steps ahead by
// LDS-DMA (no staging registers), one workgroup barrier per step.  Four wavefronts, one per SIMD; of 128 x 256 tiles eight,
// where the contraction is short: what they save is in the prologue and the epilogue (below).
//
// Most products in between fill part of a round, and a CU without a tile is lost for the whole of it: hence the many heights and
// widths (multiples of 32 rows and 64 columns).  What the choice gains by them, one product, us: 1500 x 2048 x 4096 17.2 -> 15.5 (96 x
// 128), 1400 x 4096 x 4096 25.7 -> 24.2 and 3001 x 2048 x 4096 25.8 -> 24.3 (192 x 128), 2500 x 2048 x 8192 41.9 -> 37.7 (160 x 128),
// 3072 x 3072 x 4096 40.8 -> 32.7 and 702 x 11264 x 10112 95.5 -> 70.9 (192 x 192), 319 x 24064 x 10240 103.9 -> 81.0; block-scaled
// 3072 x 3072 x 4096 42.0 -> 36.0, 1536 x 2048 x 4096 19.7 -> 18.1.
//
//   step s:  wait until stage s + 1 has landed (vmcnt counts the loads of the younger stages) and the wave's own
//            fragment reads of stage s are done; barrier: both now hold for every wave
//            MFMAs of step s from one set of fragment registers; in their shadow the fragments of step s + 1 are
//            read into the other set and stage s is refilled with step s + R
//
// LDS layout, swizzle keys, operand roles (B is the first MFMA operand; a lane ends up with consecutive output
// columns of one row) and the XCD-aware tile order are those of gemm_fp8_snake.hip; B groups can be 32 wide here.
//
// MX: a K step is four blocks of 32, so every stage also holds one dword of E8M0 scales per tile row (one LDS-DMA load per
// 64 rows), and every fragment read is followed by a one-byte read: lane (l % 16, g) passes the scale of block g of row
// l % 16 to the matrix instruction (gemm_mxfp8_snake.hip).  Scale rows in slabs of sixteen blocks cost 8 cache lines per
// 64 rows and step, plain rows 64.
#pragma once
#include "fp8_device.hpp"
#include "launchers.hpp"
#include "tuning.hpp"

#include <type_traits>
#include <utility>

namespace fp8k {

namespace rg {
typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef unsigned v4u_t __attribute__((ext_vector_type(4)));
typedef int v8i_t __attribute__((ext_vector_type(8)));
typedef float v4f_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
constexpr int BK = 128;
constexpr int NUM_XCD = 8;

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    f32x2_t v = {a, b};
    bf16x2_t h = __builtin_convertvector(v, bf16x2_t);
    uint32_t r;
    __builtin_memcpy(&r, &h, 4);
    return r;
}
// 16 bytes per lane from a raw buffer straight into LDS at lds_addr + lane * 16 (lds_addr wave-uniform); lanes out of
// range deliver zeros.  Inline assembly on purpose: a compiler that knew these loads write LDS would drain them before
// every LDS read.
template <bool HINT = false>      // HINT: streaming (non-temporal)
__device__ __forceinline__ void lds_dma16(v4i_t rsrc, uint32_t lds_addr, uint32_t voffset) {
    if constexpr (HINT)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds"
                     :
                     : "s"(lds_addr), "v"(voffset), "s"(rsrc)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     :
                     : "s"(lds_addr), "v"(voffset), "s"(rsrc)
                     : "memory", "m0");
}
// 4 bytes per lane into LDS at lds_addr + lane * 4 (the scales of 64 rows, or the block scales of a step of 64 rows)
__device__ __forceinline__ void lds_dma4(v4i_t rsrc, uint32_t lds_addr, uint32_t voffset) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 :
                 : "s"(lds_addr), "v"(voffset), "s"(rsrc)
                 : "memory", "m0");
}
// at most N_ loads in flight (they complete in issue order), own LDS reads done, workgroup barrier
template <int N_>
__device__ __forceinline__ void wait_vmem_but_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N_) : "memory");
    __builtin_amdgcn_sched_barrier(0);
}
// c += b a on the matrix cores, assembly with the accumulator tied in place: through the builtin the compiler moves
// accumulators and fragments between register files (23 copies per 64 instructions on the 128 x 256 tile).  It inserts
// no wait states for assembly: an operand written by the vector ALU needs two in front of the instruction, a result
// twelve behind it before anything else touches it.  So the vector ALU writes no operand among the steps (fragments and
// scales come from LDS reads), the accumulators are cleared ahead of the prologue's wait and read behind the last barrier.
// tests/test_isa_hazards.py checks the built code.
// ACC_V: the accumulator lives in the ordinary register file (tiles small enough: the epilogue then needs no copies).
// Otherwise the code holds one copy of each step: with a further one for an odd last step, behind the loop, the compiler
// moved the accumulators to other registers and back directly in front of its matrix instructions, which also took 0.5 us
// (odd step counts, 128 x 256 tiles: 2048 x 4096 x 4224 33.2 -> 32.6 us, x 1152 16.0 -> 15.4).  The small tiles keep the
// pair of steps without a branch in it (2048 x 4096 x 4096 on 64 x 64 tiles: 66.8 us, with the branch 70.2).
#define RG_MFMA(CSTR, MOD) asm volatile("v_mfma_f32_16x16x128_f8f6f4 %0, %1, %2, %0" MOD : CSTR(c) : "v"(b), "v"(a))
template <int FA, int FB, bool ACC_V>
__device__ __forceinline__ void mfma(v4f_t& c, const v8i_t& b, const v8i_t& a) {
    if constexpr (ACC_V) {
        if constexpr (FB == 0 && FA == 0) RG_MFMA("+v", "");
        else if constexpr (FB == 1 && FA == 0) RG_MFMA("+v", " cbsz:1");
        else if constexpr (FB == 0 && FA == 1) RG_MFMA("+v", " blgp:1");
        else RG_MFMA("+v", " cbsz:1 blgp:1");
    } else {
        if constexpr (FB == 0 && FA == 0) RG_MFMA("+a", "");
        else if constexpr (FB == 1 && FA == 0) RG_MFMA("+a", " cbsz:1");
        else if constexpr (FB == 0 && FA == 1) RG_MFMA("+a", " blgp:1");
        else RG_MFMA("+a", " cbsz:1 blgp:1");
    }
}
#undef RG_MFMA
// the same with block scales (the low byte of sb / sa)
#define RG_MFMA_MX(CSTR, MOD) \
    asm volatile("v_mfma_scale_f32_16x16x128_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel:[0,0,0] op_sel_hi:[0,0,0]" MOD : CSTR(c) : "v"(b), "v"(a), "v"(sb), "v"(sa))
template <int FA, int FB, bool ACC_V>
__device__ __forceinline__ void mfma_mx(v4f_t& c, const v8i_t& b, const v8i_t& a, uint32_t sb, uint32_t sa) {
    if constexpr (ACC_V) {
        if constexpr (FB == 0 && FA == 0) RG_MFMA_MX("+v", "");
        else if constexpr (FB == 1 && FA == 0) RG_MFMA_MX("+v", " cbsz:1");
        else if constexpr (FB == 0 && FA == 1) RG_MFMA_MX("+v", " blgp:1");
        else RG_MFMA_MX("+v", " cbsz:1 blgp:1");
    } else {
        if constexpr (FB == 0 && FA == 0) RG_MFMA_MX("+a", "");
        else if constexpr (FB == 1 && FA == 0) RG_MFMA_MX("+a", " cbsz:1");
        else if constexpr (FB == 0 && FA == 1) RG_MFMA_MX("+a", " blgp:1");
        else RG_MFMA_MX("+a", " cbsz:1 blgp:1");
    }
}
#undef RG_MFMA_MX
__device__ __forceinline__ float sigmoid(float x) { return __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }
}  // namespace rg

// One product as the kernel sees it.  A launch can carry two of them (same formats, same kinds of scale): blockIdx.y
// picks one (known without a load: a split index among the arguments made every argument fetch wait for it).
struct RingProblem {
    const uint8_t* A; int64_t lda; const uint8_t* B; int64_t ldb;
    const float* scale_a; const float* scale_b; int M, N, K; void* out; int64_t ld_out; int tiles_m, tiles_n;
    // tile order: groups of GROUP_M tile rows; division by the tiles of a group and by the rows of the last group as
    // multiplications by ceil(2^32 / d) (exact below 2^16: a scalar division costs a lone workgroup 0.1 us each)
    int in_group; uint32_t inv_group, inv_tail;
    int per_xcd;             // an eighth of the tiles, rounded up: what each XCD walks
    const uint8_t *EA, *EB; int64_t ld_ea, ld_eb;     // MX: scale rows, ld >= 0: plain, < 0: slabs of -ld rows
};

// mode: 0 = bfloat16 out, 1 = fp32 out, 2 = bfloat16 of the logistic function of the result
template <int FA, int FB, int TM, int TN, int WAVES_M, int WAVES_N, int R, int GROUP_M, bool MX, bool HINT_B>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_fp8_ring_kernel(RingProblem p1, RingProblem p2, int row_a, int row_b, int mode) {
    using namespace rg;
    constexpr int NW = WAVES_M * WAVES_N;            // wavefronts: four, one per SIMD, or eight
    constexpr int WM = TM / WAVES_M, WN = TN / WAVES_N;
    constexpr int FM = WM / 16, FN = WN / 16;        // fragments (16 rows each) per wave
    constexpr int GW = WN % 64 == 0 ? 64 : 32;       // B rows dealt together: a lane holds GW / 4 consecutive columns of a group
    constexpr int GT = GW / 16, NG = WN / GW;        // fragments per group, groups
    constexpr int SH = GW == 64 ? 4 : 3;             // log2(GW / 4)
    constexpr int TILE = (TM + TN) * BK;
    constexpr int UA = (TM + 63) / 64, TMS = 64 * UA, NU = UA + TN / 64;     // scales come 64 rows at a time: units of A, rows of its table, units in all
    constexpr int NLE = MX ? (NU + NW - 1) / NW : 0;              // scale loads (64 rows each) per wave and step
    constexpr int STAGE = TILE + NLE * NW * 256;
    constexpr int NLA = TM / (8 * NW), NLB = TN / (8 * NW), NLD = NLA + NLB;   // data loads per wave and step
    constexpr int NL = NLD + NLE;
    constexpr int NM = FM * FN;
    constexpr bool ACC_V = 4 * NM + (MX ? 18 : 16) * (FM + FN) <= (NW == 8 ? 208 : 192);     // accumulators and both fragment sets fit 256 registers with the rest
    static_assert((NW == 4 || NW == 8) && WM % 16 == 0 && (GW == 64 || GW == 32) && WN % GW == 0 && TM % (8 * NW) == 0 && TN % 64 == 0 && TN % (8 * NW) == 0, "tile");
    static_assert(R >= 3 && (R - 1) * NL <= 63, "vmcnt range");
    constexpr int CPR = WN / 8;                      // 16-byte chunks of an output row of the wave
    constexpr bool POW2 = (CPR & (CPR - 1)) == 0;    // chunk c of a parked row lies at c ^ (row % CPR); else rows are a chunk further apart
    constexpr int PITCH = (CPR + (POW2 ? 0 : 1)) * 16;
    static_assert(NW * WM * PITCH <= R * STAGE, "the epilogue stages through the ring");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

    const RingProblem& p = blockIdx.y ? p2 : p1;
    // All arguments are requested here and waited for once: left to itself the compiler fetches each where it is first used, six
    // trips to memory one behind the other in front of the first load.
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" ::"s"(p.A), "s"(p.lda), "s"(p.B), "s"(p.ldb), "s"(p.scale_a), "s"(p.scale_b), "s"(p.M), "s"(p.N), "s"(p.K), "s"(p.out), "s"(p.ld_out),
                 "s"(p.tiles_m), "s"(p.tiles_n), "s"(p.in_group), "s"(p.inv_group), "s"(p.inv_tail), "s"(p.per_xcd), "s"(row_a), "s"(row_b), "s"(mode));
    if constexpr (MX) asm volatile("" ::"s"(p.EA), "s"(p.EB), "s"(p.ld_ea), "s"(p.ld_eb));
#endif
    const int M = p.M, N = p.N, K = p.K, tiles_m = p.tiles_m, tiles_n = p.tiles_n;

    // ---- workgroup -> tile (ids are dealt round-robin to the XCDs; each XCD walks a contiguous range of tiles)
    const int slot = blockIdx.x / NUM_XCD;
    const int logical = (int)(blockIdx.x % NUM_XCD) * p.per_xcd + slot;
    if (slot >= p.per_xcd || logical >= tiles_m * tiles_n) return;
    const int grp_no = (int)__umulhi((uint32_t)logical, p.inv_group);
    const int first_m = grp_no * GROUP_M, in_grp = logical - grp_no * p.in_group;
    const int gsize = tiles_m - first_m < GROUP_M ? tiles_m - first_m : GROUP_M;
    const int tn = gsize == GROUP_M ? in_grp / GROUP_M : gsize == 1 ? in_grp : (int)__umulhi((uint32_t)in_grp, p.inv_tail);
    const int tm = first_m + in_grp - tn * gsize;
    const int m0 = tm * TM, n0 = tn * TN;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave / WAVES_N) * WM, wn0 = (wave % WAVES_N) * WN;

    // ---- buffer descriptors of this tile's operand panels (the host checks that offsets stay below 2^31)
    const int64_t lda = p.lda, ldb = p.ldb;
    const int rows_a = M - m0 < TM ? M - m0 : TM, rows_b = N - n0 < TN ? N - n0 : TN;
    const uint64_t pa = reinterpret_cast<uint64_t>(p.A + (int64_t)m0 * lda);
    const uint64_t pb = reinterpret_cast<uint64_t>(p.B + (int64_t)n0 * ldb);
    const v4i_t rsrc_a = {(int)(uint32_t)pa, (int)(uint32_t)(pa >> 32), (int)((int64_t)(rows_a - 1) * lda + K), 0x00020000};
    const v4i_t rsrc_b = {(int)(uint32_t)pb, (int)(uint32_t)(pb >> 32), (int)((int64_t)(rows_b - 1) * ldb + K), 0x00020000};

    // ---- scales of the tile's rows and columns, by LDS-DMA into the table behind the ring (64 rows or columns a load: unit u
    //      goes to wave u % NW), ahead of the operands: older than these, they have landed with stage 0.  The table then takes
    //      their reciprocals, rows first.
    float* inv_tab = reinterpret_cast<float*>(smem + R * STAGE);
    if constexpr (!MX) {
        const uint64_t psa = reinterpret_cast<uint64_t>(p.scale_a + (row_a ? m0 : 0)), psb = reinterpret_cast<uint64_t>(p.scale_b + (row_b ? n0 : 0));
        const v4i_t rsrc_sa = {(int)(uint32_t)psa, (int)(uint32_t)(psa >> 32), row_a ? rows_a * 4 : 4, 0x00020000};
        const v4i_t rsrc_sb = {(int)(uint32_t)psb, (int)(uint32_t)(psb >> 32), row_b ? rows_b * 4 : 4, 0x00020000};
#pragma unroll
        for (int h = 0; h < (NU + NW - 1) / NW; ++h) {
            const int u = wave + NW * h, r = 64 * (u < UA ? u : u - UA) + lane;
            const uint32_t at = (uint32_t)(size_t)inv_tab + (uint32_t)u * 256u;
            if (u < UA) lds_dma4(rsrc_sa, at, row_a ? (uint32_t)(r < rows_a ? r : rows_a - 1) * 4u : 0u);
            else if (u < NU) lds_dma4(rsrc_sb, at, row_b ? (uint32_t)(r < rows_b ? r : rows_b - 1) * 4u : 0u);
        }
    }
    auto scale_table = [&]() {
        if constexpr (MX) return;
        if (tid < TM) inv_tab[tid] = 1.0f / inv_tab[tid];
        if (tid < TN) inv_tab[TMS + tid] = 1.0f / inv_tab[TMS + tid];
    };

    // ---- global -> LDS: load i of wave w fills rows 8 NW i + 8 w + lane / 8; lane's chunk slot lane % 8 takes chunk
    //      slot ^ key(row).  A: key = (row >> 1) & 7.  B: ((row >> 1) & 1) | ((row >> SH) & 3) << 1.
    const int lrow = lane >> 3;
    const int ca = (lane & 7) ^ ((4 * (wave & 1) + (lrow >> 1)) & 7);
    const int kb_e = SH == 4 ? (wave >> 1) : wave, kb_o = SH == 4 && NW == 4 ? 2 + (wave >> 1) : kb_e;
    const int cb_e = (lane & 7) ^ (((lrow >> 1) & 1) | ((kb_e & 3) << 1));     // even i
    const int cb_o = (lane & 7) ^ (((lrow >> 1) & 1) | ((kb_o & 3) << 1));     // odd i
    const uint32_t va0 = (uint32_t)((wave * 8 + lrow) * (int)lda + ca * 16);
    const uint32_t vb0_e = (uint32_t)((wave * 8 + lrow) * (int)ldb + cb_e * 16);
    const uint32_t vb0_o = (uint32_t)((wave * 8 + lrow) * (int)ldb + cb_o * 16);
    const uint32_t va_step = (uint32_t)(8 * NW * (int)lda), vb_step = (uint32_t)(8 * NW * (int)ldb);
    const uint32_t lds_base = (uint32_t)(size_t)smem + (uint32_t)wave * 1024u;
    constexpr uint32_t OOB = 0x80000000u;      // puts a lane outside its descriptor: zeros arrive
    auto load_q = [&](int q, uint32_t stage_off, uint32_t ka, uint32_t ke, uint32_t ko) {
        if (q < NLB) lds_dma16<HINT_B>(rsrc_b, lds_base + stage_off + TM * BK + q * (NW * 1024), ((q & 1) ? vb0_o + ko : vb0_e + ke) + (uint32_t)q * vb_step);
        else if (q < NLD) lds_dma16<>(rsrc_a, lds_base + stage_off + (q - NLB) * (NW * 1024), va0 + (uint32_t)(q - NLB) * va_step + ka);
    };
    // MX scales: unit u of a stage is the dwords of 64 rows, A's rows first; wave w loads units w, w + NW (units past the last
    // one deliver zeros into spare room, so that every wave has the same number of loads in flight).  Slabs: rows past the
    // operand's end read the next slab's rows; their products reach only rows and columns that are never stored.
    const bool slab_a = MX && p.ld_ea < 0, slab_b = MX && p.ld_eb < 0;
    v4i_t rsrc_e[NLE ? NLE : 1];
    uint32_t ve[NLE ? NLE : 1], gse[NLE ? NLE : 1];      // lane offset, bytes per four steps
    if constexpr (MX) {
#pragma unroll
        for (int h = 0; h < NLE; ++h) {
            const int u = wave + NW * h;
            const bool is_a = u < UA, none = u >= NU;
            const bool slab = is_a ? slab_a : slab_b;
            const int64_t ld = is_a ? p.ld_ea : p.ld_eb;
            const int r0 = is_a ? m0 : n0, rows = is_a ? rows_a : rows_b;
            const int64_t group = slab ? -ld * 16 : 16;
            const uint64_t pe = reinterpret_cast<uint64_t>((is_a ? p.EA : p.EB) + (int64_t)r0 * (slab ? 16 : ld));
            const int64_t nrec = slab ? (int64_t)((K + 511) / 512) * group - (int64_t)r0 * 16 : (int64_t)(rows - 1) * ld + K / 32;
            rsrc_e[h] = v4i_t{(int)(uint32_t)pe, (int)(uint32_t)(pe >> 32), none ? 0 : (int)nrec, 0x00020000};
            ve[h] = (uint32_t)((64 * (is_a ? u : u - UA) + lane) * (slab ? 16 : (int)ld));
            gse[h] = (uint32_t)group;
        }
    }
    const uint32_t lds_e = (uint32_t)(size_t)smem + (uint32_t)TILE + (uint32_t)wave * 256u;
    auto load_e = [&](uint32_t stage_off, int k0) {
        if constexpr (MX) {
            const uint32_t s4 = (uint32_t)(k0 >> 9), sr = (uint32_t)((k0 >> 7) & 3) * 4;
#pragma unroll
            for (int h = 0; h < NLE; ++h)
                lds_dma4(rsrc_e[h], lds_e + stage_off + h * (NW * 256), k0 < K ? ve[h] + s4 * gse[h] + sr : OOB);
        }
    };
    auto kofs = [&](int k0, int c) { return k0 + c * 16 < K ? (uint32_t)k0 : OOB; };

    // ---- LDS -> fragments
    const int r16 = lane & 15, g = lane >> 4;
    const int key_a = (r16 >> 1) & 7;
    const int key_b = ((r16 >> 1) & 1) | ((r16 >> 2) << 1);
    int offa[2], offb[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        offa[c] = (wm0 + r16) * BK + (((g + 4 * c) ^ key_a) << 4);
        offb[c] = TM * BK + (wn0 + (GW / 4) * (r16 >> 2) + (r16 & 3)) * BK + (((g + 4 * c) ^ key_b) << 4);
    }
    v8i_t af[2][FM], bf[2][FN];
    uint32_t ea[2][FM], eb[2][FN];      // their scales (MX)
    const int offea = TILE + (wm0 + r16) * 4 + g, offeb = TILE + (TMS + wn0 + (GW / 4) * (r16 >> 2) + (r16 & 3)) * 4 + g;
    auto read_q = [&](auto set_t, const uint8_t* s, int q) {      // fragment q: first the B ones, then the A ones
        constexpr int SET = decltype(set_t)::value;
        const bool is_b = q < FN;
        const int ro = is_b ? ((q / GT) * GW + (q % GT) * 4) * BK : (q - FN) * 16 * BK;
        const uint4 x0 = *reinterpret_cast<const uint4*>(s + (is_b ? offb[0] : offa[0]) + ro);
        const uint4 x1 = *reinterpret_cast<const uint4*>(s + (is_b ? offb[1] : offa[1]) + ro);
        const v8i_t v = {(int)x0.x, (int)x0.y, (int)x0.z, (int)x0.w, (int)x1.x, (int)x1.y, (int)x1.z, (int)x1.w};
        if (is_b) bf[SET][q < FN ? q : 0] = v; else af[SET][q < FN ? 0 : q - FN] = v;
        if constexpr (MX) {
            const uint32_t e = s[(is_b ? offeb + ((q / GT) * GW + (q % GT) * 4) * 4 : offea + (q - FN) * 64)];
            if (is_b) eb[SET][q < FN ? q : 0] = e; else ea[SET][q < FN ? 0 : q - FN] = e;
        }
    };

    v4f_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = v4f_t{0.f, 0.f, 0.f, 0.f};

    const int ksteps = (K + BK - 1) / BK;
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int k0 = r * BK;
        const uint32_t ka = kofs(k0, ca), ke = kofs(k0, cb_e), ko = kofs(k0, cb_o);
#pragma unroll
        for (int q = 0; q < NLD; ++q) load_q(q, (uint32_t)(r * STAGE), ka, ke, ko);
        load_e((uint32_t)(r * STAGE), k0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NM; ++i) {              // the accumulators are cleared while the first stage is under way
        if constexpr (ACC_V) asm volatile("" : "+v"(acc[i / FN][i % FN]));
        else asm volatile("" : "+a"(acc[i / FN][i % FN]));
    }
    wait_vmem_but_barrier<(R - 1) * NL>();      // stage 0 has landed for everyone
#pragma unroll
    for (int q = 0; q < FM + FN; ++q) read_q(I0{}, smem, q);
    scale_table();
    __builtin_amdgcn_sched_barrier(0);

    uint32_t cur = 0, nxt = STAGE;              // byte offsets of the stages of steps s and s + 1
    int k_refill = R * BK;
    auto step = [&](auto par_t) {
        constexpr int P = decltype(par_t)::value;
        using NS = std::integral_constant<int, P ^ 1>;
        wait_vmem_but_barrier<(R - 2) * NL>();  // stage s + 1 landed, stage s read out: for everyone
        const uint32_t ka = kofs(k_refill, ca), ke = kofs(k_refill, cb_e), ko = kofs(k_refill, cb_o);
        const uint8_t* rs = smem + nxt;
        // In the shadow of the MFMAs: the reads early (their latency must pass before the next barrier), the refill
        // loads spread evenly - four waves' loads leave the CU's address unit at one per 16 cycles, and a wave that
        // finds its queue full stalls, matrix instructions included.
        constexpr int QR = NM >= 16 ? NM * 5 / 8 : (NM + 1) / 2;
#pragma unroll
        for (int t = 0; t < NM; ++t) {
            const int i = t / FN, j = (i & 1) ? FN - 1 - t % FN : t % FN;   // boustrophedon: one operand stays between neighbours
            if constexpr (MX) mfma_mx<FA, FB, ACC_V>(acc[i][j], bf[P][j], af[P][i], eb[P][j], ea[P][i]);
            else mfma<FA, FB, ACC_V>(acc[i][j], bf[P][j], af[P][i]);
            if (t < QR) {
#pragma unroll
                for (int q = t * (FM + FN) / QR; q < (t + 1) * (FM + FN) / QR; ++q) read_q(NS{}, rs, q);
            }
#pragma unroll
            for (int q = t * NLD / NM; q < (t + 1) * NLD / NM; ++q) load_q(q, cur, ka, ke, ko);
            if (MX && t == NM - 1) load_e(cur, k_refill);
            __builtin_amdgcn_sched_barrier(0);
        }
        cur = nxt;
        nxt = nxt + STAGE == R * STAGE ? 0 : nxt + STAGE;
        k_refill += BK;
    };
    int s = 0;
    if constexpr (ACC_V) {
        for (; s + 2 <= ksteps; s += 2) {
            step(I0{});
            step(I1{});
        }
        if (s < ksteps) step(I0{});
    } else {                    // one copy of each step, see mfma (K = 0: one step of zero codes)
        do {
            step(I0{});
            if (s + 1 < ksteps) step(I1{});
            s += 2;
        } while (s < ksteps);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // trailing (out-of-range) refills must not land in the epilogue's LDS
    __syncthreads();

    // ---- epilogue: (acc * 1/sa) * 1/sb (MX: nothing left to scale)
    constexpr int CE = GW / 4;                          // consecutive columns of a lane in a group
    float inv_b[NG][CE];
#pragma unroll
    for (int grp = 0; grp < NG; ++grp)
#pragma unroll
        for (int e = 0; e < CE; e += 4) {
            if constexpr (MX) break;
            const float4 t4 = *reinterpret_cast<const float4*>(inv_tab + TMS + wn0 + GW * grp + CE * g + e);
            inv_b[grp][e] = t4.x; inv_b[grp][e + 1] = t4.y; inv_b[grp][e + 2] = t4.z; inv_b[grp][e + 3] = t4.w;
        }
    float inv_a[FM];
#pragma unroll
    for (int fi = 0; fi < FM; ++fi) inv_a[fi] = MX ? 1.0f : inv_tab[wm0 + 16 * fi + r16];
    auto result = [&](int fi, int grp, int e) {
        const float v = acc[fi][grp * GT + (e >> 2)][e & 3];
        return MX ? v : (v * inv_a[fi]) * inv_b[grp][e];
    };
    const int64_t ld_out = p.ld_out;
    if (mode == 1) {
#pragma unroll
        for (int fi = 0; fi < FM; ++fi) {
            const int m = m0 + wm0 + 16 * fi + r16;
#pragma unroll
            for (int grp = 0; grp < NG; ++grp)
#pragma unroll
                for (int t = 0; t < GT; ++t) {
                    const int nb = n0 + wn0 + GW * grp + CE * g + 4 * t;
                    float v[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = result(fi, grp, 4 * t + r);
                    if (m < M && nb < N) {
                        float* dst = static_cast<float*>(p.out) + (int64_t)m * ld_out + nb;
                        if (nb + 4 <= N) *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
                        else for (int e = 0; nb + e < N; ++e) dst[e] = v[e];
                    }
                }
        }
        return;
    }
    // bfloat16: the wave's rows are scaled, rounded, parked in its part of the LDS and streamed out as whole rows of the
    // wave's width
    uint8_t* q_lds = smem + wave * (WM * PITCH);
    const bool interior = m0 + TM <= M && n0 + TN <= N;
#pragma unroll
    for (int fi = 0; fi < FM; ++fi) {
        const int r_loc = 16 * fi + r16;
        uint8_t* row = q_lds + r_loc * PITCH;
#pragma unroll
        for (int grp = 0; grp < NG; ++grp) {
            float v[CE];
#pragma unroll
            for (int e = 0; e < CE; ++e) v[e] = result(fi, grp, e);
            if (mode == 2) {
#pragma unroll
                for (int e = 0; e < CE; ++e) v[e] = sigmoid(v[e]);
            }
#pragma unroll
            for (int h = 0; h < CE / 8; ++h) {
                const int c = (GW / 8) * grp + (CE / 8) * g + h;
                *reinterpret_cast<uint4*>(row + ((POW2 ? c ^ (r16 % CPR) : c) << 4)) =
                    make_uint4(pack_bf16(v[8 * h], v[8 * h + 1]), pack_bf16(v[8 * h + 2], v[8 * h + 3]),
                               pack_bf16(v[8 * h + 4], v[8 * h + 5]), pack_bf16(v[8 * h + 6], v[8 * h + 7]));
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int fi = 0; fi < FM; ++fi) {
#pragma unroll
        for (int it = 0; it < CPR / 4; ++it) {
            const int piece = 64 * it + lane, rr = 16 * fi + piece / CPR, c_rd = piece % CPR;
            const uint4 v = *reinterpret_cast<const uint4*>(q_lds + rr * PITCH + ((POW2 ? c_rd ^ ((rr & 15) % CPR) : c_rd) << 4));
            const int m = m0 + wm0 + rr, n_rd = n0 + wn0 + c_rd * 8;
            uint16_t* dst = static_cast<uint16_t*>(p.out) + (int64_t)m * ld_out + n_rd;
            if (interior || (m < M && n_rd + 8 <= N)) {
                *reinterpret_cast<v4u_t*>(dst) = v4u_t{v.x, v.y, v.z, v.w};
            } else if (m < M && n_rd < N) {
                const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
                for (int e = 0; n_rd + e < N; ++e) dst[e] = (uint16_t)(w4[e >> 1] >> ((e & 1) * 16));
            }
        }
    }
}

struct MxScales { const uint8_t *ea, *eb; int64_t ld_ea, ld_eb; };     // of one product

template <int FA, int FB, int TM, int TN, int WAVES_M, int WAVES_N, int R, int GROUP_M, bool MX, bool HINT_B = false>
static hipError_t launch_ring_t(const GemmOperands& g1, const GemmOperands* g2, const MxScales* e, int row_a, int row_b, int mode,
                                hipStream_t st) {
    using namespace rg;
    auto kern = gemm_fp8_ring_kernel<FA, FB, TM, TN, WAVES_M, WAVES_N, R, GROUP_M, MX, HINT_B>;
    constexpr int NW = WAVES_M * WAVES_N;
    constexpr int units = (TM + 63) / 64 + TN / 64;       // of 64 rows of scales
    constexpr int lds = R * ((TM + TN) * BK + (MX ? (units + NW - 1) / NW * (NW * 256) : 0)) + (MX ? 0 : units * 256);
    static_assert(lds <= 160 * 1024, "LDS");
    static DynamicLdsOnce attr;     // one per instantiation
    if (hipError_t err = attr.ensure(reinterpret_cast<const void*>(kern), lds); err != hipSuccess) return err;
    auto problem = [&](const GemmOperands& g) {
        const int tiles_m = (int)((g.M + TM - 1) / TM), tiles_n = (int)((g.N + TN - 1) / TN);
        const int in_group = GROUP_M * tiles_n, tail = tiles_m % GROUP_M ? tiles_m % GROUP_M : GROUP_M;
        auto inv = [](int d) { return (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); };   // (0 for d = 1, which the kernel does not use)
        return RingProblem{g.a, g.lda, g.b, g.ldb, g.scale_a, g.scale_b, (int)g.M, (int)g.N, (int)g.K, g.out, g.ld_out, tiles_m, tiles_n,
                           in_group, inv(in_group), inv(tail), (tiles_m * tiles_n + NUM_XCD - 1) / NUM_XCD,
                           e ? e->ea : nullptr, e ? e->eb : nullptr, e ? e->ld_ea : 0, e ? e->ld_eb : 0};
    };
    const RingProblem p1 = problem(g1), p2 = g2 ? problem(*g2) : p1;
    const int per_xcd = p1.per_xcd > p2.per_xcd ? p1.per_xcd : p2.per_xcd;
    kern<<<dim3((unsigned)(per_xcd * NUM_XCD), g2 ? 2 : 1), dim3(64 * NW), lds, st>>>(p1, p2, row_a, row_b, mode);
    return hipGetLastError();
}

// stages: 128 x 64 and 64 x 128 tiles take four, though six fit: filling them is the longer part of a short product (us, six /
// four: 1024 x 2048 x 1024 6.3 / 6.0, 72 x 14336 x 4096 13.8 / 12.8, 512 x 4096 x 4096 13.4 / 13.0, 256 x 4096 x 14336 32.6 /
// 31.9; block-scaled 1024 x 2048 x 1024 7.4 / 6.9, x 8192 33.7 / 33.1, 72 x 14336 x 4096 17.4 / 17.0).  Otherwise what the LDS holds; rows of tiles walked together: close to square patches.  64 x 64: five stages, which with
// the table of reciprocals is one workgroup per CU; four, for two of them (as in the MX form), cost a long contraction more than
// they give a short one or a second round (us, five / four stages: 1000 x 1000 x 14336 25.2 / 27.1, 512 x 512 x 28672 40.5 / 43.0,
// 1024 x 1024 x 4096 10.5 / 10.5, x 1024 6.0 / 5.8; several rounds, where larger tiles are taken: 2048 x 2048 x 1024 16.3 / 12.9).
template <int FA, int FB, bool MX>
static hipError_t launch_ring_f(int tile, const GemmOperands& g1, const GemmOperands* g2, const MxScales* e, int row_a, int row_b,
                                int mode, hipStream_t st) {
    const bool eight = ring_waves(tile, g1, g2, MX, MX && e->ld_ea >= 0) == 8;
    if constexpr (!MX) {
        if (ring_hint(tile, g1, g2)) {
            if (tile == RING_64x64) return launch_ring_t<FA, FB, 64, 64, 2, 2, 5, 4, false, true>(g1, g2, e, row_a, row_b, mode, st);
            if (tile == RING_64x128) return launch_ring_t<FA, FB, 64, 128, 2, 2, 4, 8, false, true>(g1, g2, e, row_a, row_b, mode, st);
            if (tile == RING_128x128) return launch_ring_t<FA, FB, 128, 128, 2, 2, 4, 4, false, true>(g1, g2, e, row_a, row_b, mode, st);
            if (tile == RING_128x256)
                return eight ? launch_ring_t<FA, FB, 128, 256, 2, 4, 3, 8, false, true>(g1, g2, e, row_a, row_b, mode, st)
                             : launch_ring_t<FA, FB, 128, 256, 2, 2, 3, 8, false, true>(g1, g2, e, row_a, row_b, mode, st);
        }
    }
    switch (tile) {
        case RING_64x64: return launch_ring_t<FA, FB, 64, 64, 2, 2, MX ? 4 : 5, 4, MX>(g1, g2, e, row_a, row_b, mode, st);
        case RING_128x64: return launch_ring_t<FA, FB, 128, 64, 2, 2, 4, 4, MX>(g1, g2, e, row_a, row_b, mode, st);
        case RING_64x128: return launch_ring_t<FA, FB, 64, 128, 2, 2, 4, 8, MX>(g1, g2, e, row_a, row_b, mode, st);
        case RING_128x128: return launch_ring_t<FA, FB, 128, 128, 2, 2, 4, 4, MX>(g1, g2, e, row_a, row_b, mode, st);
        case RING_128x256:
            return eight ? launch_ring_t<FA, FB, 128, 256, 2, 4, 3, 8, MX>(g1, g2, e, row_a, row_b, mode, st)
                         : launch_ring_t<FA, FB, 128, 256, 2, 2, 3, 8, MX>(g1, g2, e, row_a, row_b, mode, st);
        case RING_256x128:
            return eight ? launch_ring_t<FA, FB, 256, 128, 4, 2, 3, 4, MX>(g1, g2, e, row_a, row_b, mode, st)
                         : launch_ring_t<FA, FB, 256, 128, 2, 2, 3, 4, MX>(g1, g2, e, row_a, row_b, mode, st);
        case RING_96x64: return launch_ring_t<FA, FB, 96, 64, 2, 2, 4, 4, MX>(g1, g2, e, row_a, row_b, mode, st);
        case RING_64x192: return launch_ring_t<FA, FB, 64, 192, 2, 2, 4, 8, MX>(g1, g2, e, row_a, row_b, mode, st);
        case RING_160x64: return launch_ring_t<FA, FB, 160, 64, 2, 2, 4, 4, MX>(g1, g2, e, row_a, row_b, mode, st);
        case RING_96x128: return launch_ring_t<FA, FB, 96, 128, 2, 2, 4, 8, MX>(g1, g2, e, row_a, row_b, mode, st);
        case RING_160x128: return launch_ring_t<FA, FB, 160, 128, 2, 2, 4, 4, MX>(g1, g2, e, row_a, row_b, mode, st);
        case RING_192x128:
            return eight ? launch_ring_t<FA, FB, 192, 128, 4, 2, 3, 4, MX>(g1, g2, e, row_a, row_b, mode, st)
                         : launch_ring_t<FA, FB, 192, 128, 2, 2, 3, 4, MX>(g1, g2, e, row_a, row_b, mode, st);
        case RING_128x192: return launch_ring_t<FA, FB, 128, 192, 2, 2, 3, 8, MX>(g1, g2, e, row_a, row_b, mode, st);
        case RING_160x192: return launch_ring_t<FA, FB, 160, 192, 2, 2, 3, 4, MX>(g1, g2, e, row_a, row_b, mode, st);
        case RING_192x192: return launch_ring_t<FA, FB, 192, 192, 2, 2, 3, 4, MX>(g1, g2, e, row_a, row_b, mode, st);
    }
    if constexpr (!MX) {     // (three stages of these with their scales are more than the LDS)
        if (tile == RING_160x256) return launch_ring_t<FA, FB, 160, 256, 2, 2, 3, 8, false>(g1, g2, e, row_a, row_b, mode, st);
        if (tile == RING_224x192) return launch_ring_t<FA, FB, 224, 192, 2, 2, 3, 4, false>(g1, g2, e, row_a, row_b, mode, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace fp8k
