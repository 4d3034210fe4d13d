// Internal launch functions behind the C ABI.  Arguments are assumed valid
// (the ABI layer checks them); every function only enqueues work on `st`.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fp8k {

// Whether a quantization of this many elements, all tensors of the launch together, reads its bfloat16 input with the streaming
// hint.  The hint makes a load slower by itself (a strip of 4096 rows arrives in 17 instead of 10 us), but its data does not
// displace what the product reads next (us, hint / plain: see each launcher's lines).
inline bool hint_inputs(int64_t elements, int64_t line) { return elements > line; }
// One tensor before its product: what plain loads gain is small (1 to 3 %), what they cost is large where the weights in turn just
// fit the last-level cache and the input no longer does beside them (us, hint / plain, three weights in turn: 712 x 7840 x 8080
// 65.0 / 81.4, 512 x 14336 x 4096 42.3 / 53.2; six: 1900 x 4096 x 4096 36.3 / 40.0).  So only inputs that are a small part of that
// cache, 4 MB.
constexpr int64_t HINT_ALONE = (int64_t)2 << 20;
constexpr int64_t HINT_BLOCKS = (int64_t)8 << 20;    // the tensors of an MX or blockwise step
constexpr int64_t HINT_PAIR = (int64_t)24 << 20;     // X and W of a step, whose codes are all that the product reads

hipError_t launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t st);

hipError_t launch_amax(const void* x, int64_t rows, int64_t cols, int64_t ld, int gran, float* out,
                       hipStream_t st);

// per-column scales of a tall matrix via a [G, cols] scratch matrix of partial
// maxima (hipErrorNotSupported: shape does not suit it, use launch_amax + launch_scale)
hipError_t launch_col_scales_two_level(const void* x, int64_t rows, int64_t cols, int64_t ld, int fmt, int flags,
                                       float* scale_out, void* scratch, size_t scratch_bytes, hipStream_t st);

// tensorwise quantization of a dense tensor in two launches (per-block maxima, then a cast that derives the
// scale itself); part: scratch for TENSOR_PARTIALS floats
constexpr int TENSOR_PARTIALS = 512;
// flags: FP8_POW2_SCALE, and from bit 8 on the room in part where it is less than TENSOR_PARTIALS (0: it is not)
hipError_t launch_quant_tensor(const void* x, int64_t rows, int64_t cols, int fmt, int flags, int transpose, uint8_t* q,
                               int64_t ld_out, uint8_t* q_plain, int64_t ld_plain, float* scale_out, float* part,
                               hipStream_t st);
// blockwise FP8 (tiles of 1 x 128 or blocks of 128 x 128, power-of-two scales as E8M0 bytes in the MX layout)
hipError_t launch_block_quant(const void* x, int64_t rows, int64_t cols, int64_t ld, int block_rows, int fmt, uint8_t* q,
                              int64_t ld_q, uint8_t* e8m0, int64_t ld_e, hipStream_t st);
// the same of the transposed matrix, written transposed (rows % 128 == 0, cols % 8 == 0)
// q_row / e_row (optional, block_rows == 1, cols % 128 == 0): the tiles along the rows of x from the same read
// FMT_ALONE, or'ed into fmt with q_row given: the codes are the call's result, no product of the same call reads them
constexpr int FMT_ALONE = 256;
hipError_t launch_block_quant_t(const void* x, int64_t rows, int64_t cols, int64_t ld, int block_rows, int fmt, uint8_t* qt,
                                int64_t ld_t, uint8_t* et, int64_t ld_e, hipStream_t st, uint8_t* q_row = nullptr,
                                int64_t ld_row = 0, uint8_t* e_row = nullptr, int64_t ld_er = 0);
hipError_t launch_scale(const float* amax, int64_t n, int fmt, int flags, float* out, hipStream_t st);

// transpose != 0: q is [cols, rows]; q_plain (optional, transpose only) also
// receives the untransposed codes.
hipError_t launch_cast(const void* x, int64_t rows, int64_t cols, int64_t ld, const float* scale, int gran,
                       int fmt, int transpose, uint8_t* q, int64_t ld_out, uint8_t* q_plain, int64_t ld_plain,
                       hipStream_t st);

// single-pass rowwise amax+scale+cast; hipErrorNotSupported if a row is too
// long to keep in registers.
hipError_t launch_quant_row(const void* x, int64_t rows, int64_t cols, int64_t ld, int fmt, int flags, uint8_t* q,
                            int64_t ld_out, float* scale_out, hipStream_t st);

// out[M,N] = (a[M,K] . b[N,K]^T) / (sa * sb); scale_a/scale_b have one entry
// (row_a / row_b == 0) or one per row.
// b_from: who wrote the codes of b, an earlier call or the same one, and then whether as column strips (see ring_hint).
enum BFrom { B_AT_REST = 0, B_WRITTEN, B_WRITTEN_IN_STRIPS };
hipError_t launch_gemm_fp8(const uint8_t* a, int64_t lda, int fmt_a, const float* scale_a, int row_a,
                           const uint8_t* b, int64_t ldb, int fmt_b, const float* scale_b, int row_b,
                           int64_t M, int64_t N, int64_t K, void* out, int64_t ld_out, int out_f32,
                           hipStream_t st, BFrom b_from = B_AT_REST);
// one scaled product out[M, N] = A[M, K] . B[N, K]^T / (scale_a * scale_b), operands as for launch_gemm_fp8
struct GemmOperands {
    const uint8_t* a; int64_t lda; const float* scale_a;
    const uint8_t* b; int64_t ldb; const float* scale_b;
    int64_t M, N, K; void* out; int64_t ld_out;
    BFrom b_from = B_AT_REST;
};
// two small products (bfloat16 results) in one launch; hipErrorNotSupported, with nothing launched, where that does not pay
hipError_t launch_gemm_fp8_pair(const GemmOperands& g1, const GemmOperands& g2, int fmt_a, int fmt_b, int row_a, int row_b,
                                hipStream_t st);

// Whether the rows of a product's weight [N, K] are requested with the streaming hint: from 96 MiB on, for a served model, whose
// layers between two calls push such a weight out of the 256 MB last-level cache.  From HBM it then passes at 5.9 instead of 5.2
// TB/s (us without / with, three weights in turn: 16 x 28672 x 4096 25.3 / 22.0, x 8192 45.8 / 40.2; 64 x 16384 x 8192 32.6 /
// 28.2).  What that costs: a weight called again and again with nothing in between, or just written, is in the cache and comes
// slower with the hint (the same with one weight: 19.9 / 21.1, 36.7 / 39.4, 23.2 / 27.2; 128 x 28672 x 4096 22.8 / 27.4, x 8192
// 39.3 / 53.4, 72 x 16512 x 6528 22.9 / 33.1, 113 x 20992 x 6656 27.5 / 43.1).  Smaller weights gain as much from HBM (16 x 14336 x
// 4096 13.6 / 12.6), but more of them fit the cache between the calls, and lose there (the same, three weights in turn: 11.1 /
// 12.2). Rows have to be whole lines of 128 bytes: a line that two rows or two stages share is fetched twice with the hint (1 x
// 28672 x 4112 24.8 / 36.5, x 8224 52.0 / 62.9, x 8256 53.6 / 60.1; 128 x 28672 x 8224 72.8 / 86.7; x 8320, whole lines, 49.3 /
// 45.0).
inline bool stream_weight(const uint8_t* b, int64_t ldb, int64_t N, int64_t K) {
    return N * K >= (int64_t)96 << 20 && (((uintptr_t)b | (uint64_t)ldb) & 127) == 0;
}

// products of few to middling size on smaller tiles with a deep LDS ring (gemm_fp8_ring.hpp); g2: a second product in
// the same launch, or nullptr; mode 0 = bfloat16, 1 = fp32, 2 = bfloat16 of the sigmoid.  _fits: 32-bit offsets reach
// The tiles up to RING_256x128 are taken over any number of rounds and by pairs of products, those behind only by one product that
// they cover in one round; the last two have no block-scaled form.
enum RingTile { RING_64x64 = 0, RING_128x64, RING_64x128, RING_128x128, RING_128x256, RING_256x128, RING_96x64, RING_64x192, RING_160x64, RING_96x128,
                RING_160x128, RING_192x128, RING_128x192, RING_160x192, RING_192x192, RING_160x256, RING_224x192, RING_TILES };
constexpr int RING_ANY_ROUNDS = RING_256x128 + 1, RING_WIDE = RING_160x192, RING_MX_TILES = RING_160x256;
// Its form for a tile: whether B is read with the streaming hint.  One row of tiles against a weight that stream_weight accepts
// reads it once (us, weights from HBM, without / with: 64 x 28672 x 8192 51.5 / 47.0, 128 rows 56.1 / 53.2, x 4096 32.8 / 30.5).
// Not two rows of 128 x 256 tiles: they read it side by side, but fall out of step where the second is not full, and lines are
// fetched twice (129 rows, x 8192 61.2 / 66.2, x 6144 47.8 / 53.5, x 3584 28.9 / 32.5; 160 rows 63.7 / 64.6, 50.1 / 52.3, 30.5 /
// 31.7; 256 rows 68.4 / 65.7, 56.7 / 54.3, 34.5 / 33.8); one_row below is for them.  Where the same call has quantized B, its codes
// are in the last-level cache: the taller tiles then read them plainly (forward of 128 rows, N x K 28672 x 4096 73.9 / 75.6, x 8192
// 140.3 / 141.7; dX against W^T 28672 x 4096 112.3 / 114.5), low ones with the hint (forward 64 rows 72.0 / 72.4, 136.8 / 137.7,
// 16384 x 8192 82.0 / 82.3; dX 64 rows 106.8 / 105.0, 271.4 / 268.8, 163.8 / 162.1, 16 rows 104.3 / 100.2, 268.8 / 263.7, 156.3 /
// 154.8).
inline bool ring_hint(int tile, const GemmOperands& g, const GemmOperands* g2) {
    if (g2 || !stream_weight(g.b, g.ldb, g.N, g.K)) return false;
    switch (tile) {
        case RING_64x64: case RING_64x128: return g.M <= 64;
        case RING_128x128: case RING_128x256: return g.M <= 128 && g.b_from == B_AT_REST;
    }
    return false;
}
// 129 to 256 rows against such a weight: one row of 256 x 128 tiles in place of two of 128 x 256, which fetches it once (us from
// HBM, 129 / 193 / 256 rows, 128 x 256 plain, with the hint, 256 x 128: 28672 x 8192 61.5 66.2 69.9, 65.3 63.1 65.4, 58.0 62.6
// 67.1; x 6144 47.6 52.6 57.2, 53.6 51.4 54.3, 46.3 50.0 52.7; x 3584 29.2 32.1 34.5, 33.0 32.1 34.0, 28.7 31.6 34.8; 24576 x 4608
// 34.7 38.3 42.0, 39.8 38.2 40.3, 33.5 37.3 38.2).  From the cache the two are close (28672 x 6144 36.1 39.7 40.2 / 35.2 38.8
// 43.2): where the same call has quantized the weight nothing changes.
inline bool one_row(const GemmOperands& g) { return g.M > 128 && g.M <= 256 && g.b_from == B_AT_REST && stream_weight(g.b, g.ldb, g.N, g.K); }
// Wavefronts of a workgroup: four, one per SIMD, or eight on 128 x 256 and 256 x 128 tiles of short contractions, K <= 6144 (us,
// four / eight: 2048 x 4096 x 1024 14.5 / 13.4, 3001 x 2048 x 4096 26.0 / 25.1, 2048 x 4096 x 4096 29.6 / 28.7, 1000 x 4096 x 6144
// 34.2 / 32.7, 4096 x 4096 x 6144 79.5 / 77.1, with the hint 72 x 28672 x 4096 35.8 / 34.7; x 8192 99.6 / 99.2, 2048 x 4096 x 8192
// 50.3 / 51.0, x 14336 +2 %).  Not where a row of full 256 x 128 tiles fetches a large weight (160 / 193 / 224 / 256 rows, 24576 x
// 4608 36.7 37.3 37.8 38.2 / 35.8 37.2 39.0 41.7, 28672 x 6144 50.0 50.0 51.1 52.7 / 48.4 49.0 51.9 55.7, 20480 x 5120 42.1 42.6
// 42.4 44.1 / 41.5 43.9 43.8 47.9). Block-scaled: the same with slabs of scales (1000 x 4096 x 4096 -7 %, 2048 x 4096 x 6144 -1 %).
// Up to K = 1536 with plain rows of scales (from the cache 1000 x 4096 x 1024 / 2048 / 3072 / 4096 -11 / -8 / -3 / +2 %, from HBM
// -13 / +4 / +3 / +11 %), and of 256 x 128 tiles whose B rows are no whole lines (690 x 5968 x 1040 / 2256 / 3088 / 6128 from the
// cache -8 / -4 / -1 / +2 %, from HBM -3 / +4 / +5 / +8 %).
// 192 x 128 tiles: eight up to K = 4096 (3072 x 2048 x 1024 11.9 / 11.5, x 4096 25.2 / 25.1, 1400 x 4096 x 4096 24.8 / 24.2; x 8192 42.9 /
// 43.5, x 16384 78.9 / 80.6).
inline int ring_waves(int tile, const GemmOperands& g, const GemmOperands* g2, bool mx, bool plain_scales = false) {
    const int64_t line = plain_scales || (tile == RING_256x128 && ((g.ldb | (g2 ? g2->ldb : 0)) & 127)) ? 1536 : 6144;
    if (tile == RING_192x128) return g.K <= (plain_scales ? 1536 : 4096) && (!g2 || g2->K <= 4096) ? 8 : 4;
    if (tile != RING_128x256 && tile != RING_256x128) return 4;
    if (tile == RING_256x128 && !mx && !g2 && g.M > 192 && one_row(g)) return 4;
    return g.K <= line && (!g2 || g2->K <= line) ? 8 : 4;
}
bool gemm_fp8_ring_fits(const GemmOperands& g);
int gemm_fp8_ring_choice(const GemmOperands& g);      // its tile where a 256 x 256 tile per workgroup is not the better form, else -1
int gemm_fp8_wide_choice(const GemmOperands& g, bool bf16);      // of a product sent to the 256 x 256 kernels: its wide tile that is the better form, or -1
// Whether every row of a bfloat16 output starts on 64 bytes.  The persistent kernel writes 64 bytes of a row at a time past the caches;
// where those straddle two sectors its stores are slower by as much as its tile boundaries gain, and more.
inline bool rows_on_sectors(const GemmOperands& g) { return (((uintptr_t)g.out | 2 * (uint64_t)g.ld_out) & 63) == 0; }
// Height of the 256 x 256 kernel's tiles where lower ones cover the product in one round on more than half of the CUs: 192 or 224
// rows on the persistent kernel, else 256 (us, 256 rows / 224 / 192: 3001 x 4096 x 2048 26.9 / 24.6 / 23.8; 3072 x 4096 x 1024
// 17.9 / 16.4 / 16.2, x 4096 42.0 / 40.1 / 39.3, x 8192 75.3 / 73.7 / 70.3; 3584 x 4096 x 4096 45.8 / 44.7, x 8192 84.3 / 79.2, of
// a short contraction equal: x 1024 18.2 / 18.7).  One round hides nothing of the epilogue, which takes 3 to 10 us longer where rows do not
// start on sectors (us, 256 rows / the lower ones, N = 4096, 4064, 4048, 4040: 3072 x N x 1024 18.1 18.9 19.1 18.6 / 15.5 15.5 22.7 24.9, x
// 4096 44.6 44.0 44.7 42.3 / 38.3 37.6 44.0 47.0; 3584 x N x 2048 26.8 28.8 28.9 29.2 / 26.8 26.4 34.5 38.8).  There 192 rows only from K =
// 3584 on, 224 from 7168 (200 products, lower ones relative to 256 rows, plain and block-scaled: 192 rows K = 1536 .. 2047 +9 % +15 %, 2560 ..
// 3071 +1 % +4 %, 3584 .. 4095 -1 % 0, 7168 .. 8191 -2 % -4 %, from 12288 -6 % -7 %; 224 rows 3072 .. 3583 +10 % +16 %, 6144 .. 7167 +2 %
// +2 %, 8192 .. 12287 -3 % -2 %, from 12288 -4 % -4 %).
inline int one_round_height(const GemmOperands& g, int64_t cus) {
    const int64_t cols = (g.N + 255) / 256;
    const bool sectors = rows_on_sectors(g);
    if (2 * ((g.M + 255) / 256) * cols <= cus || g.N % 8 || g.K <= 256) return 256;
    if ((g.M + 191) / 192 * cols <= cus) return sectors || g.K >= 3584 ? 192 : 256;
    return (g.M + 223) / 224 * cols <= cus && g.K > (sectors ? 1024 : 7167) ? 224 : 256;
}
hipError_t launch_gemm_fp8_ring(int tile, const GemmOperands& g1, const GemmOperands* g2, int fmt_a, int fmt_b, int row_a,
                                int row_b, int mode, hipStream_t st);

// the block-scaled form (K a multiple of 128; scales as for launch_gemm_mxfp8, g.scale_a / g.scale_b unused)
bool gemm_mxfp8_ring_fits(const GemmOperands& g, int64_t ld_ea, int64_t ld_eb);
int gemm_mxfp8_ring_choice(const GemmOperands& g, bool plain_scales);      // a tile, or -1
int gemm_mxfp8_stream_height(const GemmOperands& g);      // of the persistent kernel's tiles (scales in slabs), or 0: one 256 x 256 tile per workgroup
hipError_t launch_gemm_mxfp8_ring(int tile, const GemmOperands& g, int fmt_a, int fmt_b, const uint8_t* ea, int64_t ld_ea,
                                  const uint8_t* eb, int64_t ld_eb, int out_f32, hipStream_t st);

// Rowwise quantization (codes q, scales scale_out) and the per-column scales
// scale_cols[c] = scale(max_r |x[r, c]|) from a single read of x; scratch holds
// the first-level column maxima.  hipErrorNotSupported if the shape does not suit.
hipError_t launch_quant_row_colmax(const void* x, int64_t rows, int64_t cols, int64_t ld, int fmt, int flags,
                                   uint8_t* q, int64_t ld_out, float* scale_out, float* scale_cols, void* scratch,
                                   size_t scratch_bytes, hipStream_t st);

// a dense tensor [rows, cols] for tensorwise quantization: codes q (transposed [cols, rows] if asked for, then
// optionally also untransposed in q_plain), its scale, and room for TENSOR_PARTIALS floats of per-block maxima
struct TensorOperand {
    const void* x; int64_t rows;
    uint8_t* q; int64_t ld_out; uint8_t* q_plain; int64_t ld_plain; float* scale_out; float* part;
};
// two dense tensors of the same width and format, tensorwise: two launches (instead of four)
hipError_t launch_quant_tensor_pair(const TensorOperand& a, const TensorOperand& b, int64_t cols, int fmt, int flags,
                                    int transpose, hipStream_t st);

// Paired launches: the quantizations of a linear layer come in twos and threes of the same kind; these issue them as
// twin launches (one grid, two problems) with one second-level launch for all column scales.  Results are those of the
// single-tensor functions.  hipErrorNotSupported (nothing launched): a tensor does not suit - quantize one by one.
// fold (optional): quant_fold_bytes(rows, cols) bytes of side storage, 256-byte aligned, for the first-level column
// maxima.  With it the transposing cast derives the column scales itself (one launch less); without it, or where
// quant_fold_bytes is 0, the maxima are parked in the transposed output and a second-level launch reduces them.
constexpr int64_t FOLD_ROWS = 256;
int64_t quant_fold_bytes(int64_t rows, int64_t cols);
struct RowColOperand {      // a tensor [rows, cols] quantized per row (q_row, scale_row) and per column, transposed (q_col_t [cols, rows], scale_col)
    const void* x; int64_t rows, ld;
    uint8_t* q_row; int64_t ld_row; float* scale_row;
    uint8_t* q_col_t; int64_t ld_col_t; float* scale_col;
    void* fold = nullptr;
};
struct ColOperand {         // a tensor [rows, cols] quantized per column, transposed
    const void* x; int64_t rows, ld;
    uint8_t* q_col_t; int64_t ld_col_t; float* scale_col;
    void* fold = nullptr;
};
// two tensors of the same width and format, rowwise: one launch
hipError_t launch_quant_row_pair(const void* x1, int64_t rows1, int64_t ld1, uint8_t* q1, int64_t ld_q1, float* s1, const void* x2,
                                 int64_t rows2, int64_t ld2, uint8_t* q2, int64_t ld_q2, float* s2, int64_t cols, int fmt,
                                 int flags, hipStream_t st);
// one tensor (b == nullptr) or two of the same width and format along both axes: one launch (strips), else three, two with folding.
// q_col_t nullptr: that tensor per row only (strips or hipErrorNotSupported)
hipError_t launch_quant_row_col_pair(const RowColOperand& a, const RowColOperand* b, int64_t cols, int fmt, int flags, hipStream_t st);
// two tensors of the same width and format per column, transposed: one launch, or three (instead of six)
hipError_t launch_quant_col_t_pair(const ColOperand& a, const ColOperand& b, int64_t cols, int fmt, int flags, hipStream_t st);
// the backward of the rowwise recipe: the gradient g along both axes, W and X per column: one launch (strips), else five (instead
// of nine), four with folding.  Without g.q_row, g.q_col_t, w.x or x.x (nullptr) what is left: strips or hipErrorNotSupported
hipError_t launch_quant_bwd_rowwise(const RowColOperand& g, int64_t cols_g, int fmt_g, const ColOperand& w, const ColOperand& x,
                                    int64_t cols_wx, int fmt_wx, int flags, hipStream_t st);

// several tensors in one launch, each per row, per column (transposed), or both; q_row / q_col_t nullptr: not wanted.
// Output rows of q_col_t are padded to 16 bytes at least, the padding belongs to the call (zero codes up to the next 16).
// hipErrorNotSupported (nothing launched) where a tensor does not suit.
struct StripOperand {
    const void* x; int64_t rows, cols, ld; int fmt;
    uint8_t* q_row; int64_t ld_row; float* scale_row;
    uint8_t* q_col_t; int64_t ld_col_t; float* scale_col;
};
hipError_t launch_quant_strips(const StripOperand* ops, int n, int flags, hipStream_t st);

// 256 x 256 kernel on 16x16x128 MFMAs with LDS-DMA loads and the four-phase "snake" schedule; same contract.
// _fits: its 32-bit buffer offsets reach (leading dimensions below 2^23)
bool gemm_fp8_snake_fits(int64_t lda, int64_t ldb);
// act != 0 (bfloat16 output only): the logistic function applied to the fp32 result before rounding
hipError_t launch_gemm_fp8_snake(const uint8_t* a, int64_t lda, int fmt_a, const float* scale_a, int row_a,
                                 const uint8_t* b, int64_t ldb, int fmt_b, const float* scale_b, int row_b,
                                 int64_t M, int64_t N, int64_t K, void* out, int64_t ld_out, int out_f32,
                                 hipStream_t st, int act = 0);

// its block-scaled form, scales in slabs of slab_a / slab_b rows, in tiles of 256, 224 or 192 rows
bool gemm_mxfp8_stream_fits(const GemmOperands& g, int64_t slab_a, int64_t slab_b, int out_f32);
hipError_t launch_gemm_mxfp8_stream(const GemmOperands& g, int fmt_a, const uint8_t* ea, int64_t slab_a, int fmt_b, const uint8_t* eb, int64_t slab_b,
                                    int tile_m, hipStream_t st);
// persistent form of the same kernel (gemm_fp8_stream.hpp): one workgroup per CU walks many tiles, the epilogue of a
// tile is drained inside the K steps of the next.  bfloat16 output, whole tiles [0, units) of the snake kernel's tile
// order; _fits: shapes it takes (N % 8 == 0, more than two K steps, 32-bit offsets reach)
bool gemm_fp8_stream_fits(int64_t lda, int64_t ldb, int64_t ld_out, int64_t N, int64_t K, int out_f32, int act);
// tile_m: 256 (tiles [0, units) of the snake kernel's tile order) or 224 / 192 (then units must be the whole tile count
// of the problem cut into tiles of that height); gemm_fp8_stream_tile_m picks the height for an [M, N] output
int gemm_fp8_stream_tile_m(int64_t M, int64_t N);
hipError_t launch_gemm_fp8_stream(const uint8_t* a, int64_t lda, int fmt_a, const float* scale_a, int row_a,
                                  const uint8_t* b, int64_t ldb, int fmt_b, const float* scale_b, int row_b,
                                  int64_t M, int64_t N, int64_t K, void* out, int64_t ld_out, int64_t units, int tile_m,
                                  hipStream_t st);

// Split of a few-row product (gemm_fp8_skinny.hip).  nw: groups of 16 columns per wavefront; ks: wavefronts of a workgroup that
// share K; deep: five K steps in flight in place of three.  nw_forced: 0, or the switch's value.
struct FewRowForm { int nw, ks; int64_t grid; bool deep; };
// Forms of mt tiles of 16 rows that a weight which stream_weight accepts can come to, and which so exist with the streaming hint:
// against one group of columns N < 6144 and so K > 16384; with 33 rows and more the choice of kernel leaves N <= 8192 and so K >=
// 12288, always four parts of K.
constexpr bool few_row_hint(int mt, int nw, int ks) { return nw == 2 ? mt <= 2 || ks == 4 : nw == 1 && ks == 4; }
inline FewRowForm few_row_form(int64_t M, int64_t N, int64_t K, int nw_forced, int64_t cus) {
    // columns per wavefront: 16 or 32 (64 through the override).  Wider groups reuse every fragment of A
    // for two or four MFMAs but shorten the ring of K steps in flight, narrower ones give more wavefronts;
    // measured: 32 wins or ties from N = 6144 on, 64 never beats 32 (28672 x 8192: 5 % slower)
    const int nw = nw_forced ? nw_forced : N >= 6144 ? 2 : 1;
    const int64_t groups = (N + 16 * nw - 1) / (16 * nw);
    // split K over the wavefronts of a workgroup until about 2048 wavefronts stream B
    int ks = 1;
    while (ks < 4 && groups * ks < 2048 && K / (ks * 2) >= 512) ks *= 2;
    const int64_t grid = (groups + (4 / ks) - 1) / (4 / ks);
    // a long contraction keeps five up to 8 rows on at most half of the CUs, up to 4 rows on three quarters (us from HBM, three /
    // five at 1, 4, 8, 12 rows: 1024 x 11008 8.0 8.0 8.3 8.8 / 7.5 7.7 8.4 9.0, x 28672 16.1 16.4 17.0 18.2 / 14.5 15.3 16.6 18.4;
    // 2560 x 14336 10.5 10.6 10.9 11.6 / 9.9 10.2 10.9 11.8, 3072 x 28672 19.3 19.7 20.4 / 18.5 19.0 20.2; 4096 x 14336 12.7 12.7
    // 12.8 / 12.8 12.9 13.1).  Three weights in turn, from the cache: 1024 x 14336 7.2 7.2 7.2 / 7.0 7.0 7.1, 2560 x 14336 8.1 8.2
    // 8.3 / 8.3 8.4 8.5; shorter ones lose there what they gain from HBM (1024 x 8192 HBM 6.6 6.7 7.0 / 6.4 6.5 6.9, cache 5.0 5.1
    // 5.2 / 5.3 5.3 5.4)
    return {nw, ks, grid, ks == 4 && nw == 1 && K > 10240 && ((M <= 8 && 2 * grid <= cus) || (M <= 4 && 4 * grid <= 3 * cus))};
}

// Whether a product of up to 16 rows goes to persistent workgroups (gemm_fp8_few_stream.hip): weights of 96 MiB and more, where the
// few-row kernel has one of three weaknesses that they have not.  (us from HBM, few-row / persistent, 1 and 16 rows.)
//  * Rows that are no whole cache lines, of which its short-lived workgroups fetch the shared ones twice: 20000 x 5136 24.6 30.6 / 21.6
//    23.2, 9728 x 10416 29.6 37.2 / 23.8 25.3, 16384 x 7184 23.7 29.5 / 23.4 24.8, 8192 x 12304 21.3 25.9 / 21.4 23.0.  (From the cache,
//    called again with nothing in between, the few-row kernel is ahead where one round holds the weight: 16384 x 8240 22.1 / 23.5 at 4
//    rows.)  Not for up to four tokens over two tiles a workgroup, which pass before the ring pays (1, 2, 4 rows from HBM, few-row / persistent:
//    8192 x 12384 22.9 - 23.5 / 23.5 - 23.5, x 12352 21.1 21.0 - / 22.4 22.4 -, x 16336 - 27.4 - / - 28.9 -; from the cache 16.3 / 18.9).
//  * Streams that all start a multiple of 4096 bytes apart, rows and parts of K both: they crowd the same channels.  65536 x 4096 57.7
//    56.3 / 41.9 41.8, 32768 x 8192 57.9 55.1 / 42.9 44.5, 8192 x 16384 30.3 30.7 / 24.8 25.3, 16384 x 16384 57.4 53.7 / 44.8 45.1, 28672 x
//    16384 92.0 93.6 / 74.5 77.0; with parts of 2048 32768 x 4096 22.3 22.6 / 25.6 26.7, 49152 x 4096 31.6 32.2 / 36.0 37.8.
//  * A busiest CU with more rows of the weight than the persistent kernel's has, by a fifth (a tenth where K is long enough for the
//    difference to count): 10240 x 14336 29.0 33.1 / 26.5 27.3, 20480 x 10240 36.0 41.3 / 33.8 34.4, 18432 x 8192 28.0 29.5 / 25.7 25.9,
//    36864 x 4096 28.3 29.6 / 26.8 26.8; by a seventh 28672 x 6144 29.9 32.2 / 28.8 29.1, x 8192 37.5 40.0 / 37.8 38.9, but x 4096 20.5 21.7
//    / 22.3 22.4; as many 24576 x 8192 31.4 32.1 / 33.1 34.2, 8192 x 13312 18.5 19.1 / 20.3 20.7, 16384 x 12288 32.7 34.5 / 33.3 34.7.
// Smaller weights: equal or slower (80 .. 87 MiB 0.92 .. 1.11 times as fast, 42 .. 64 MiB 0.76 .. 1.06, below 40 MiB 0.76 .. 1.05).
// forced: the switch SKINNY_DMA, 2 or 3 = wherever it fits, strided or in runs; 0 or 1 = never.
inline bool few_row_streams(const GemmOperands& g, int64_t cus, int forced = -1) {
    const int64_t tiles = (g.N + 15) / 16;
    if (g.M < 1 || g.M > 16 || g.K < 1 || g.K > 16384 || tiles > 32 * cus || g.lda >= (1 << 23) || g.ldb >= (1 << 23)) return false;
    if (forced >= 0) return forced >= 2;
    if (g.N * g.K < (int64_t)96 << 20) return false;
    if (g.ldb % 128 != 0 && (g.M > 4 || tiles > 2 * cus)) return true;
    const FewRowForm f = few_row_form(g.M, g.N, g.K, 0, cus);
    const int64_t part = ((g.K + 127) / 128 + f.ks - 1) / f.ks * 128;
    if (g.ldb % 4096 == 0 && part % 4096 == 0) return true;
    const int64_t few = (f.grid + cus - 1) / cus * (4 / f.ks) * f.nw * 16, persistent = (tiles + cus - 1) / cus * 16;      // rows of the busiest CU
    return g.K < 6144 ? 5 * few >= 6 * persistent : 10 * few >= 11 * persistent;
}
// Which tiles of 16 weight rows a persistent workgroup takes: a run of neighbouring ones, whose loads come from one stretch of the
// weight, or every grid-th.  Runs where rows are whole cache lines of at most 8 KB and runs do not start multiples of 256 KB apart, with rows of
// up to 4 KB there too (us, runs / strided at 16 rows: 28672 x 8192 38.9 / 39.3, 28672 x 6144 29.1 / 29.6, 36864 x 4096 26.8 / 29.7, 65536 x
// 4096 41.8 / 49.2, 128256 x 4096 82.1 / 93.3, 16400 x 8192 23.7 / 25.2; 16384 x 8192 25.0 / 23.9, 8192 x 16384 28.4 / 25.3, 20480 x 10240
// 35.0 / 34.4, 12288 x 11008 29.4 / 26.6, 28672 x 14336 65.9 / 65.2, 20312 x 6320 28.3 / 26.6, 24344 x 8112 41.9 / 40.2).
inline bool few_row_runs(const GemmOperands& g, int64_t cus, int forced = -1) {
    const int64_t tiles = (g.N + 15) / 16, run = (tiles + cus - 1) / cus;
    if (run < 2) return false;
    if (forced == 2 || forced == 3) return forced == 3;
    return g.ldb % 128 == 0 && g.K <= 8192 && (g.K <= 4096 || run * 16 * g.ldb % (256 << 10) != 0);
}
hipError_t launch_gemm_fp8_few_stream(const GemmOperands& g, int fmt_a, int fmt_b, int row_a, int row_b, int out_f32, hipStream_t st);

// columns of a strip (quant_strips.hip) for tensors of at most tall rows, load strips of 32 columns.  16 where 32 would keep half
// of the CUs busy, unless the strips are short (us, 32 / 16 columns: gradient 4096 x 1024 20.9 / 14.9, x 4096 27.3 / 26.4, x 6144
// 31.8 / 36.0; 2048 x 1024 12.8 / 10.2, x 4096 15.3 / 14.7, x 6144 16.5 / 20.7; 1024 x 1024 8.7 / 9.3, x 4096 10.8 / 12.5); beyond
// 4096 rows 32 do not fit.
inline int strip_columns(int64_t tall, double load, int64_t cus) { return tall > 4096 || (tall > 1024 && 2.0 * load <= (double)cus) ? 16 : 32; }

// few rows of A (M <= 64, the decode shape of inference): B is streamed once
// from HBM by wavefronts that load their MFMA operands straight from global
// memory; same contract otherwise.
hipError_t launch_gemm_fp8_skinny(const uint8_t* a, int64_t lda, int fmt_a, const float* scale_a, int row_a,
                                  const uint8_t* b, int64_t ldb, int fmt_b, const float* scale_b, int row_b,
                                  int64_t M, int64_t N, int64_t K, void* out, int64_t ld_out, int out_f32,
                                  hipStream_t st);

// y[M, N] = fp8(x * s_x)[M, K] . b[N, K]^T / (s_x * scale_b) for up to 16 rows of bfloat16 x, in one launch: the amax of
// x (per row if row_x, else of the whole tensor), its scale (flags: FLAG_POW2) and the cast happen inside the
// few-row product.  hipErrorNotSupported (nothing launched) where that form does not apply.
hipError_t launch_linear_skinny_fused(const void* x, int64_t ldx, int fmt_x, int row_x, int flags, const uint8_t* b,
                                      int64_t ldb, int fmt_b, const float* scale_b, int row_b, int64_t M, int64_t N,
                                      int64_t K, void* out, int64_t ld_out, hipStream_t st);

// bfloat16 GEMM with the contraction on the rows of both operands:
// out[I, J] = a[C, I]^T b[C, J], fp32 accumulate, bfloat16 out (the weight gradient
// dW = dY^T X kept in high precision).  I, J and the leading dimensions are
// multiples of 8 elements, pointers 16-byte aligned.
hipError_t launch_gemm_bf16_at_b(const void* a, int64_t lda, const void* b, int64_t ldb, int64_t I, int64_t J, int64_t C,
                                 void* out, int64_t ld_out, hipStream_t st);

// the same product on the LDS-DMA "snake" schedule with transposing LDS reads (large problems;
// _fits tells whether the 32-bit buffer offsets reach)
bool gemm_bf16_at_b_snake_fits(int64_t lda, int64_t ldb, int64_t I, int64_t J, int64_t C);
hipError_t launch_gemm_bf16_at_b_snake(const void* a, int64_t lda, const void* b, int64_t ldb, int64_t I, int64_t J,
                                       int64_t C, void* out, int64_t ld_out, hipStream_t st);

// gradient through a stored sigmoid output, dz = dy * y * (1 - y): quantized along both axes without being
// materialised (hipErrorNotSupported for shapes the fused kernels do not take), or materialised (dense bf16)
hipError_t launch_quant_row_col_sigmoid_bwd(const void* dy, const void* y, int64_t rows, int64_t cols, int64_t ld,
                                            int fmt, int flags, uint8_t* q_row, int64_t ld_row, float* scale_row,
                                            uint8_t* q_col_t, int64_t ld_col_t, float* scale_col, hipStream_t st);
hipError_t launch_sigmoid_bwd(const void* dy, const void* y, int64_t n, void* dz, hipStream_t st);

// layer normalisation over the rows with the rowwise fp8 quantization of its bfloat16 result fused in
// (cols % 8 == 0, cols <= 16384, else hipErrorNotSupported; h, mean_out, rstd_out optional)
hipError_t launch_layernorm_quant_row(const void* x, int64_t rows, int64_t cols, int64_t ld, const void* gamma,
                                      const void* beta, double eps, int fmt, int flags, void* h, int64_t ld_h, uint8_t* q,
                                      int64_t ld_q, float* scale_out, float* mean_out, float* rstd_out, hipStream_t st);

// MX (microscaling) FP8: blocks of 32 along the contiguous axis, one E8M0 byte per block
// (cols % 32 == 0), and the GEMM whose matrix-core instruction applies the block scales
// (K % 128 == 0, ld_ea and ld_eb multiples of 4, 4-byte aligned scale pointers)
hipError_t launch_mx_quant(const void* x, int64_t rows, int64_t cols, int64_t ld, int fmt, uint8_t* q, int64_t ld_q,
                           uint8_t* e8m0, int64_t ld_e, hipStream_t st);
// blocks of 32 down the columns of x (rows % 32 == 0), output transposed: qt [cols, rows], et [cols, rows / 32];
// with q_row != nullptr also the blocks along the rows (cols % 32 == 0) from the same read: q_row [rows, cols],
// e_row [rows, cols / 32] (ld_er % 4 == 0)
// (FMT_ALONE as above)
hipError_t launch_mx_quant_t(const void* x, int64_t rows, int64_t cols, int64_t ld, int fmt, uint8_t* qt, int64_t ld_t,
                             uint8_t* et, int64_t ld_e, uint8_t* q_row, int64_t ld_row, uint8_t* e_row, int64_t ld_er,
                             hipStream_t st);
// The tensors of a block-scaled linear layer in one launch, all in one format (else, and where a tensor does not suit,
// hipErrorNotSupported and nothing launched).  Two: X and W of a forward, dense rows, MX blocks along them or tiles of 1 x 128 (X)
// and blocks of 128 x 128 (W). Three: dY, W and X of a backward, transposed as by launch_mx_quant_t / launch_block_quant_t (W in
// blocks of 128 x 128), dY with q_row.
struct BlockOperand {
    const void* x; int64_t rows, cols; int fmt;
    uint8_t* q; int64_t ld_q; uint8_t* e; int64_t ld_e;
    uint8_t* q_row; int64_t ld_row; uint8_t* e_row; int64_t ld_er;
};
hipError_t launch_quant_blocks(const BlockOperand* ops, int n, bool mx, hipStream_t st);
bool gemm_mxfp8_takes_slab_scales(int64_t lda, int64_t ldb, int64_t M, int64_t N, int64_t K);
hipError_t launch_gemm_mxfp8(const uint8_t* a, int64_t lda, int fmt_a, const uint8_t* ea, int64_t ld_ea,
                             const uint8_t* b, int64_t ldb, int fmt_b, const uint8_t* eb, int64_t ld_eb, int64_t M,
                             int64_t N, int64_t K, void* out, int64_t ld_out, int out_f32, hipStream_t st);
// the same product on the LDS-DMA "snake" schedule (large problems; leading dimensions below 2^23)
hipError_t launch_gemm_mxfp8_snake(const uint8_t* a, int64_t lda, int fmt_a, const uint8_t* ea, int64_t ld_ea,
                                   const uint8_t* b, int64_t ldb, int fmt_b, const uint8_t* eb, int64_t ld_eb, int64_t M,
                                   int64_t N, int64_t K, void* out, int64_t ld_out, int out_f32, hipStream_t st);

}  // namespace fp8k
