// Quantization of all tensors of a small or middling rowwise step in ONE launch: per-column codes (transposed) from column
// strips that a workgroup keeps in registers, per-row codes from whole rows.
//
// The per-column quantization of a tall matrix takes three launches (column maxima, their second level, transposing cast) and
// reads the matrix twice.  A matrix of a few thousand rows needs neither: a strip of 32 columns x 4096 rows (or 16 x 8192) is
// 256 KB, which the register file of one CU holds.  A workgroup reads its strip once, every load in flight together, reduces the
// maxima across its wavefronts, derives the scales and writes the transposed codes: one launch, no scratch, no order among
// workgroups.  The rowwise codes that the same step needs are made by further workgroups of the same launch.
//
// What bounds it: up to some 64 strips the time of one strip on its CU - a CU takes in a row's piece every five cycles or so, 32 or
// 128 bytes alike (measured; 2 KB pitch and more), so 4096 rows take 10 us to arrive, and conversion and stores follow; that is why
// strips are 16 columns wide where 32 would leave CUs idle, why the loads are plain ones (17 us with the streaming hint) and why
// the conversion carries no clamp.  With more strips HBM: X and W of 4096 x 4096, both orientations, 201 MB in 38 us = 5.3 TB/s.
// Before / now (us, first kernel's start to last one's end): X and W of 1024 x 1024 20.3 / 9.5, of 4096 x 1024 25.0 / 20.1; the
// gradient 1024 x 8192 33.7 / 10.4, 2048 x 4096 39.4 / 14.7, 3072 x 8192 42.3 / 29.9, 4096 x 8192 48.1 / 39.9. Steps: 1024 x 2048 x
// 1024 41.7 / 29.1 (33 before its rows were read plainly), 1024^3 41.1 / 24.5, 3001 x 4096 x 2048 140 / 113, 4096^3 231 / 205 (the
// last three stateless).
#include "fp8_device.hpp"
#include "launchers.hpp"
#include "tuning.hpp"

#include <type_traits>

namespace fp8k {

namespace {
constexpr int XCDS = 8;
constexpr int RPT = 16;        // rows of a thread

struct StripCols {             // one tensor's strips
    const uint16_t* x; int64_t ld; uint8_t* qt; int64_t ld_t; float* scale;
    int rows, cols, fmt;
    int share;                 // strips per workgroup (a power of two): its threads are split evenly among them
    int groups, per_xcd;       // workgroups with work; their eighth, rounded up
};
struct StripRows {             // one tensor's rows
    const uint16_t* x; int64_t ld; uint8_t* q; int64_t ld_q; float* scale;
    int rows, cols, fmt;
    int groups;
};
struct StripArgs { StripCols c[3]; StripRows r[2]; int flags; int hint; };      // hint: rows are read with the streaming hint

// with the lane OFF away within the row of 16, cyclically
template <int OFF>
__device__ __forceinline__ uint32_t pk_absmax_ror(uint32_t v) {
    return pk_absmax(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x120 + OFF, 0xF, 0xF, false));
}

// Strips of workgroup b.  A thread owns RPT consecutive rows of 8 columns: RPT 16-byte loads, LPR lanes a row; its codes leave as
// RPT bytes of eight rows of the transposed output, 64 / LPR * RPT consecutive bytes per wavefront and column.
template <int FMT, int NT, int LPR>
__device__ __forceinline__ void quant_strip(const StripCols& s, int b, int flags, uint32_t* red, float* scales) {
    constexpr int STRIP = 8 * LPR;                            // columns of a strip
    // adjacent strips share cache lines: each XCD (ids are dealt round-robin to them) takes a run of consecutive ones
    const int logical = (b % XCDS) * s.per_xcd + b / XCDS;
    if (b / XCDS >= s.per_xcd || logical >= s.groups) return;
    const int tpw = NT / s.share;                             // threads of a strip
    const int sub = threadIdx.x / tpw, t = threadIdx.x % tpw;
    const int c = (logical * s.share + sub) * STRIP + (t % LPR) * 8;
    const int r0 = t / LPR * RPT;
    const uint16_t* p = s.x + (c < s.cols ? c : 0);
    uint4 v[RPT];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {                           // (a row read twice does not change a maximum)
        const int r = r0 + j < s.rows ? r0 + j : s.rows - 1;
        v[j] = *reinterpret_cast<const uint4*>(p + (int64_t)r * s.ld);
    }
    uint32_t m[4] = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        m[0] = pk_absmax(m[0], v[j].x);
        m[1] = pk_absmax(m[1], v[j].y);
        m[2] = pk_absmax(m[2], v[j].z);
        m[3] = pk_absmax(m[3], v[j].w);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (LPR == 2) m[i] = pk_absmax_ror<2>(m[i]);
        m[i] = pk_absmax_xor<32>(pk_absmax_xor<16>(pk_absmax_xor<8>(pk_absmax_ror<4>(m[i]))));
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane < LPR) *reinterpret_cast<uint4*>(red + (wave * LPR + lane) * 4) = make_uint4(m[0], m[1], m[2], m[3]);
    __syncthreads();
    if (t < STRIP) {
        // one column per thread: its magnitude from every wavefront of the strip
        const int w0 = sub * (tpw / 64), nw = tpw / 64;
        uint32_t mag = 0;
        for (int w = 0; w < nw; ++w) {
            const uint32_t two = red[(w0 + w) * (LPR * 4) + (t >> 1)];
            const uint32_t one = (t & 1) ? two >> 16 : two & 0xFFFFu;
            mag = one > mag ? one : mag;
        }
        const float sc = scale_from_amax(mag_to_float(mag & 0x7FFFu), FMT, flags);
        scales[sub * STRIP + t] = sc;
        const int col = (logical * s.share + sub) * STRIP + t;
        if (col < s.cols) s.scale[col] = sc;
    }
    __syncthreads();
    if (c >= s.cols || r0 >= s.rows) return;
    float sc[8];
    *reinterpret_cast<float4*>(sc) = *reinterpret_cast<const float4*>(scales + sub * STRIP + (t % LPR) * 8);
    *reinterpret_cast<float4*>(sc + 4) = *reinterpret_cast<const float4*>(scales + sub * STRIP + (t % LPR) * 8 + 4);
    auto finish = [&](auto clamp) {
        uint32_t o[8][RPT / 4];
#pragma unroll
        for (int q = 0; q < RPT / 4; ++q) {
            uint2 w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = cast8_own<FMT, decltype(clamp)::value>(v[4 * q + i], sc);
            uint32_t lo[4], hi[4];
            transpose4x4_bytes(w[0].x, w[1].x, w[2].x, w[3].x, lo);
            transpose4x4_bytes(w[0].y, w[1].y, w[2].y, w[3].y, hi);
#pragma unroll
            for (int e = 0; e < 4; ++e) { o[e][q] = lo[e]; o[e + 4][q] = hi[e]; }
        }
        if (r0 + RPT > s.rows) {                              // zero codes in the padding of the output's rows
#pragma unroll
            for (int q = 0; q < RPT / 4; ++q) {
                const int left = s.rows - r0 - 4 * q;
                const uint32_t mask = left >= 4 ? 0xFFFFFFFFu : left <= 0 ? 0u : (1u << (8 * left)) - 1u;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e][q] &= mask;
            }
        }
        uint8_t* dst = s.qt + (int64_t)c * s.ld_t + r0;
#pragma unroll
        for (int e = 0; e < 8; ++e) store_through(dst + e * s.ld_t, make_uint4(o[e][0], o[e][1], o[e][2], o[e][3]));
    };
    const float top = fmaxf(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])), fmaxf(fmaxf(sc[4], sc[5]), fmaxf(sc[6], sc[7])));
    if (__any(top >= CLAMP_FROM)) finish(std::true_type{});
    else finish(std::false_type{});
}

// Rows of workgroup b: groups of 256 threads, each RW consecutive rows, kept in registers between maximum and cast
template <int FMT, int NT, int NV, int RW>
__device__ __forceinline__ void quant_rows(const StripRows& s, int b, int flags, bool hint, uint32_t* red) {
    const int tx = threadIdx.x & 255, g = threadIdx.x >> 8;
    const int nvec = s.cols >> 3;
    const int r0 = (b * (NT / 256) + g) * RW;
    uint4 v[RW][NV];
    auto request = [&](auto load) {
#pragma unroll
        for (int k = 0; k < RW; ++k) {
            const int r = r0 + k < s.rows ? r0 + k : s.rows - 1;
            const uint4* rv = reinterpret_cast<const uint4*>(s.x + (int64_t)r * s.ld);
#pragma unroll
            for (int j = 0; j < NV; ++j) v[k][j] = tx + j * 256 < nvec ? load(rv + tx + j * 256) : make_uint4(0, 0, 0, 0);
        }
    };
    with_loads(hint, request);
#pragma unroll
    for (int k = 0; k < RW; ++k) {
        uint32_t acc = 0;
#pragma unroll
        for (int j = 0; j < NV; ++j) acc = pk_absmax4(acc, v[k][j]);
        const uint32_t m = wave_max_u32<64>(pk_fold(acc));
        if ((threadIdx.x & 63) == 0) red[k * (NT / 64) + (threadIdx.x >> 6)] = m;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < RW; ++k) {
        const int r = r0 + k;
        if (r >= s.rows) break;
        uint32_t m = red[k * (NT / 64) + g * 4];
#pragma unroll
        for (int i = 1; i < 4; ++i) { const uint32_t o = red[k * (NT / 64) + g * 4 + i]; m = o > m ? o : m; }
        const float sc = scale_from_amax(mag_to_float(m), FMT, flags);
        if (tx == 0) s.scale[r] = sc;
        uint2* dst = reinterpret_cast<uint2*>(s.q + (int64_t)r * s.ld_q);
#pragma unroll
        for (int j = 0; j < NV; ++j)
            if (tx + j * 256 < nvec) {
                store_through(dst + tx + j * 256, sc >= CLAMP_FROM ? cast8_own<FMT, true>(v[k][j], sc) : cast8_own<FMT, false>(v[k][j], sc));
            }
    }
}

template <int NV> constexpr int rows_at_once() { return NV == 1 ? 4 : NV == 2 ? 4 : NV == 4 ? 2 : 1; }

template <int NT, int LPR, int NV>
__global__ __launch_bounds__(NT) void quant_strips_kernel(StripArgs a) {
    __shared__ __attribute__((aligned(16))) uint32_t red[NT / 64 * 16];
    __shared__ __attribute__((aligned(16))) float scales[8 * LPR * (NT / 64)];
    constexpr int RW = rows_at_once<NV>();
    int b = blockIdx.x;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int n = a.c[i].per_xcd * XCDS;
        if (b < n) {
            if (a.c[i].fmt == FMT_E4M3FN) quant_strip<FMT_E4M3FN, NT, LPR>(a.c[i], b, a.flags, red, scales);
            else quant_strip<FMT_E5M2, NT, LPR>(a.c[i], b, a.flags, red, scales);
            return;
        }
        b -= n;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if (b < a.r[i].groups) {
            if (a.r[i].fmt == FMT_E4M3FN) quant_rows<FMT_E4M3FN, NT, NV, RW>(a.r[i], b, a.flags, a.hint != 0, red);
            else quant_rows<FMT_E5M2, NT, NV, RW>(a.r[i], b, a.flags, a.hint != 0, red);
            return;
        }
        b -= a.r[i].groups;
    }
}
}  // namespace

hipError_t launch_quant_strips(const StripOperand* ops, int n, int flags, hipStream_t st) {
    if (knob(KNOB_STRIPS) == 0 || knob(KNOB_PAIRS) == 0) return hipErrorNotSupported;
    StripArgs a{};
    a.flags = flags & FLAG_POW2;
    int64_t tall = 0, wide = 0;          // rows of the tallest tensor in strips, columns of the widest in rows
    for (int i = 0; i < n; ++i) {
        const StripOperand& o = ops[i];
        if (o.rows <= 0 || o.cols <= 0 || o.cols % 8 != 0 || o.rows > 0x7FFFFF || o.cols > 0x7FFFFF) return hipErrorNotSupported;
        if (o.q_col_t && o.rows > tall) tall = o.rows;
        if (o.q_row && o.cols > wide) wide = o.cols;
    }
    const int v = knob(KNOB_STRIPS);     // 2, 4: wherever they fit, 16 / 32 columns wide
    if (tall == 0 || tall > (v == 4 ? 4096 : 8192) || wide > 16384) return hipErrorNotSupported;
    // Up to 4096 rows always ahead of the separate launches; beyond, strips are 16 columns wide (32-byte requests), which pays
    // where three tensors share the launch, the stateless backward (us, step before / with: 5000x4096x4096 292 / 272,
    // 8192x4096x4096 397 / 383, 8192^3 1284 / 1287), but not for one or two (8192x2048 gradient 31 / 33, W and X of the
    // 8192x4096x4096 LayerNorm step 458 / 466).
    if (v < 0 && tall > 4096 && n < 3) return hipErrorNotSupported;
    // A tensor wanted in both orientations is read twice, the second time from the 256 MB last-level cache if all of them fit it
    // (X and W of 4096 x 14336, 235 MB: 654 -> 643 us a step; of 4096 x 16384, 268 MB: 756 -> 778).
    int64_t twice = 0, by_rows = 0;
    double load = 0.0;
    for (int i = 0; i < n; ++i) {
        if (ops[i].q_row && ops[i].q_col_t) twice += ops[i].rows * ops[i].cols;
        if (ops[i].q_row) by_rows += ops[i].rows * ops[i].cols;
        load += (ops[i].q_col_t ? 1.0 : 0.5) * (double)((ops[i].cols + 31) / 32) * (double)ops[i].rows / (double)tall;
    }
    if (twice > (int64_t)120 << 20) return hipErrorNotSupported;
    // Rows with the streaming hint beyond 24 Mi elements: the loads are slower by themselves, but what they read does not displace
    // the codes (us a step, hint / plain: 1024x2048x1024 34.4 / 30.3, 2048^3 58.0 / 52.7, 2048x4096x4096 with dW in bfloat16, 24
    // Mi, 153.1 / 150.8, 4096^3 215.9 / 217.1, 600x14336x4096 238 / 246, 4096x14336x2048 416 / 428; all tensors from HBM, 12 Mi
    // 65.5 / 65.5, 16 84.0 / 84.0, 20 95.8 / 92.5, 24 Mi 134.1 / 132.8 and 149.8 / 150.2, 28 177.8 / 179.1 and 191.4 / 193.7, 32
    // 206.2 / 207.5, 40 262.1 / 263.1: even from 24 to 28 Mi).
    a.hint = hint_inputs(by_rows, HINT_PAIR);
    // load: strips of 32 columns, in units of the tallest tensor's, a tensor without strips half
    const int lpr = tall <= 4096 && (v == 2 || v == 4) ? v : strip_columns(tall, load, compute_units() > 0 ? compute_units() : 256) / 8;
    const int threads = tall * lpr <= 4096 ? 256 : tall * lpr <= 8192 ? 512 : 1024;
    // workgroups hold the tallest tensor's strip; of a shorter one each takes several
    const int nv = wide <= 2048 ? 1 : wide <= 4096 ? 2 : wide <= 8192 ? 4 : 8;
    const int rw = nv <= 2 ? 4 : nv == 4 ? 2 : 1;
    int nc = 0, nr = 0;
    int64_t blocks = 0;
    for (int i = 0; i < n; ++i) {
        const StripOperand& o = ops[i];
        if (o.q_col_t) {
            if (nc == 3) return hipErrorNotSupported;
            int share = 1;
            while (share * 2 * 64 <= threads && o.rows * share * 2 * lpr <= (int64_t)threads * RPT) share *= 2;
            const int strips = (int)((o.cols + 8 * lpr - 1) / (8 * lpr)), groups = (strips + share - 1) / share;
            a.c[nc++] = StripCols{static_cast<const uint16_t*>(o.x), o.ld, o.q_col_t, o.ld_col_t, o.scale_col, (int)o.rows, (int)o.cols,
                                  o.fmt, share, groups, (groups + XCDS - 1) / XCDS};
            blocks += (groups + XCDS - 1) / XCDS * XCDS;
        }
        if (o.q_row) {
            if (nr == 2) return hipErrorNotSupported;
            const int per = threads / 256 * rw;
            a.r[nr++] = StripRows{static_cast<const uint16_t*>(o.x), o.ld, o.q_row, o.ld_row, o.scale_row, (int)o.rows, (int)o.cols,
                                  o.fmt, (int)((o.rows + per - 1) / per)};
            blocks += (o.rows + per - 1) / per;
        }
    }
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
#define FP8K_STRIPS(NT, LPR, NV) quant_strips_kernel<NT, LPR, NV><<<dim3((unsigned)blocks), dim3(NT), 0, st>>>(a)
#define FP8K_STRIPS_NV(NT, LPR)                  \
    do {                                         \
        if (nv == 1) FP8K_STRIPS(NT, LPR, 1);    \
        else if (nv == 2) FP8K_STRIPS(NT, LPR, 2); \
        else if (nv == 4) FP8K_STRIPS(NT, LPR, 4); \
        else FP8K_STRIPS(NT, LPR, 8);            \
    } while (0)
    if (lpr == 2) {
        if (threads == 256) FP8K_STRIPS_NV(256, 2);
        else if (threads == 512) FP8K_STRIPS_NV(512, 2);
        else FP8K_STRIPS_NV(1024, 2);
    } else if (threads == 256) FP8K_STRIPS_NV(256, 4);
    else if (threads == 512) FP8K_STRIPS_NV(512, 4);
    else FP8K_STRIPS_NV(1024, 4);
#undef FP8K_STRIPS_NV
#undef FP8K_STRIPS
    return hipGetLastError();
}

}  // namespace fp8k
