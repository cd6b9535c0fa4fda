// kernels.hpp -- the three passes of the packed four-step convolution.
//
//   col_fwd : N1-point column DFTs of every document column (the left DFT of
//             Algorithm 1) and the per-document twiddle w_P^(u j);
//   row     : m-point row DFTs inside each document only (the block-diagonal
//             right DFT) of the document rows and of the same rows of the
//             filter class grid, the conjugate-symmetry separation of the
//             filter pair, the spectral product and the inverse row DFT;
//   col_inv : the conjugate twiddle and the inverse N1-point column DFT, the
//             store of positions t < L_i.
//
// Grid buffer layout (complex fp32, or complex fp16 for bf16 inputs):
// [pair block][segment grid point][16 pairs],
// grid point of (u, j) in a segment = grid_off + u * m + j.
// The filter "spectrum" is the filter pairs' class grids after the column stage,
// same layout, class grid point of (u, j) = spec_off + u * m + j.  The stored
// grids are the DFTs scaled by 1 / sqrt(N1) (folded into the w_P^r table), the documents'
// times a power of two (Seg::in_scale); a row pass leaves W / m times sqrt(N1), so that with the
// inverse column pass's 1 / sqrt(N1) the result is 1 / P overall and fp16 values stay O(|x|): the
// VALU kernels scale the filter spectra by sqrt(N1) / (2 m), the matrix-core ones split it
// between their operands and their inverse (row_dense.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "plan.hpp"

namespace rubiconv {

// Element type tags.
struct F32 {};
struct BF16 {};

// Power-of-two scales of the complex fp16 grids (device pointers, never null):
// pair[q] = {s, 1 / s} per channel pair q (pair block * 16 + lane pair), glob = {s, m}.
// A column pass into a grid multiplies its fp32 results by pair[q].x * glob->x before
// they are rounded to the grid type; an inverse column pass multiplies its fp32
// outputs by pair[q].y * glob->y.  The filter's per-pair normalisation and a
// call's data prescale travel this way, so every fp16 value stays in range.
struct GridScale {
    const float2* pair;
    const float2* glob;
};

// Where a VALU column pass finds its call's range scale itself: n partial magnitudes (and a
// bf16 element before or after the whole words) of launch_amax; the scale is
// 2^(kDataAmaxExp - e) extra, and workgroup 0 writes {s, (prev ? prev->y : 1) / s} to *out.
struct AmaxSource {
    const uint32_t* parts = nullptr;
    int n = 0;
    const uint16_t* head = nullptr;
    const uint16_t* tail = nullptr;
    float extra = 1.0f;
    const float2* prev = nullptr;
    float2* out = nullptr;
};

struct LaunchTables {
    const Seg* segs;
    const int32_t* col_seg;
    const int32_t* task_seg;
    const float2* tw;      // per-class twiddles
    const float2* tw_n1;   // w_N1^s
    const int32_t* list;   // documents grouped by class / class identity list
};

// `half` selects complex fp16 grid and spectrum elements (complex fp32 otherwise).
hipError_t launch_col_fwd(int r, bool half, int x_dtype, const void* src, int64_t src_row_stride,
                          int D, void* grid, int64_t grid_pb_stride, const LaunchTables& t,
                          GridScale sc, int n_cols, int npb, hipStream_t stream,
                          const AmaxSource& am = AmaxSource());  // with am.parts: in place of sc.glob

hipError_t launch_col_inv(int r, bool half, int y_dtype, const void* grid, int64_t grid_pb_stride,
                          void* dst, int64_t dst_row_stride, int D, const LaunchTables& t,
                          GridScale sc, int n_cols, int npb, hipStream_t stream);

// Row pass: row DFTs of the filter class rows and the document rows, the
// separation and product, the inverse row DFT (generic kernel: long rows).
// Every row launcher takes `corr`: 0 multiplies by the filter spectrum F(f)
// (convolution), 1 by F(-f) = conj F(f) (correlation, the adjoint in x).
hipError_t launch_row_conv(int n1, bool half, void* grid, int64_t grid_pb_stride,
                           const void* fgrid, int64_t fgrid_pb_stride, const LaunchTables& t,
                           int n_tasks, int npb, int lds_bytes, int corr, hipStream_t stream);

// VALU row pass for a listed row size m (row_sizes.hpp) over the nlist documents
// list[0..nlist) of that size: m > kMaxRegM on complex fp32 grids, m > 16 * kMaxDenseBlocks on
// complex fp16 ones (hipErrorInvalidValue otherwise).
hipError_t launch_row_fast(int m, bool half, void* grid, int64_t grid_pb_stride, const void* fgrid,
                           int64_t fgrid_pb_stride, const Seg* segs, const int32_t* list,
                           int nlist, const float2* tw, int n1, int npb, int corr,
                           hipStream_t stream);

// Rows of at most kMaxRegM points on complex fp32 grids, every size class in one launch:
// groups (RowGroup, nb = m) and blocks ((group, rows kRegRows y ..) pairs) as for
// launch_row_groups, the sum as there.
hipError_t launch_row_reg(void* grid, int64_t grid_pb_stride, const void* fgrid, int64_t fgrid_pb_stride,
                          const Seg* segs, const int32_t* docs, const RowGroup* groups, const int32_t* blocks,
                          int nblocks, int npb, int corr, hipStream_t stream, bool sum);

// 16-byte entries of one class's tables of the matrix-core row pass for rows of nb 16-point
// blocks (w = exp(-2 pi i / m)): nb * nb real operands of 64 lanes (the forward transform; the
// inverse takes their conjugates); the partner row's input twiddles w^j, for rows of up to
// kTwinBlocks blocks folded into a second set of operands, for longer ones as 16 nb complex
// fp16 factors w^(-j); 16 nb complex fp32 twiddles kappa w^j, then kappa (the inverse's scale
// over the operands'), fp32; padded to whole 1 KB chunks.
constexpr int partner_pre_u4(int nb) { return nb <= kTwinBlocks ? nb * nb * 64 : 4 * nb; }
constexpr int partner_tab_u4(int nb) { return (nb * nb * 64 + partner_pre_u4(nb) + 8 * nb + 1 + 63) / 64 * 64; }

// Matrix-core row pass (complex fp16 grids) over groups of documents (RowGroup), each
// `count` consecutive entries of `docs` (indices into segs) that share one size class and
// whose second-grid rows are those of the group's first document; blocks: (group, rows
// 4 y ..) pairs, one per workgroup and pair block; no group has more than max_nb 16-point
// blocks per row; tabs = the plan's dense operand tables, addressed through Seg::dense_off.
// The grid of a pair block must span less than 2^31 bytes where a group is batched (nb 0).
// sum: every document of a group brings its own second-grid rows, the products of
// the group's documents are added, and the one inverse transform of the sum is written
// over the first document's rows (the others are left as they were); with sum, dscale
// (a power of two) multiplies the data rows' spectra before they are rounded to fp16,
// and out2 writes the inverse over the first document's second-grid rows instead, which
// leaves the grid itself as it was (both: 1 and false without sum); sum takes corr = 1 only.
hipError_t launch_row_groups(int max_nb, void* grid, int64_t grid_pb_stride, const void* fgrid,
                             int64_t fgrid_pb_stride, const Seg* segs, const int32_t* docs, const RowGroup* groups,
                             const int32_t* blocks, int nblocks, const void* tabs, int npb, int corr,
                             hipStream_t stream, bool sum = false, float dscale = 1.0f, bool out2 = false);

// Long rows (fp16 grids): the first level of the row DFT of one document or class grid
// (LrItem) for its n1 grid rows and npb pair blocks, into its sub-row region, or the
// inverse from the region back (long_rows.hip).  grid_pb_stride in complex elements.
hipError_t launch_lr_step(bool inverse, void* grid, int64_t grid_pb_stride, const LrItem& it,
                          const float2* tw, int n1, int npb, hipStream_t stream);

// Matrix-core column passes (N1 = 256, complex fp16 grids, D a multiple of 32).
// `mtab` holds the MFMA operand tables in lane order (16-byte entries, offsets
// below; see build_mfma_tables).
constexpr int kMtFwd1 = 0;         // forward stage 1: fp32 entries w16^(k1 n1), slots 0 and 1, then 2 and 3
constexpr int kMtInv1 = 128;       // inverse stage 1: fp32 entries w16^(-n2 k2), likewise
constexpr int kMtFwd2 = 256;       // forward stage 2 per k1: re, im
constexpr int kMtInv2 = 2304;      // inverse stage 2 per n2: re, im
constexpr int kMtEntries = 4352;

// first_scale of a pass with amax_out: a power of two from 1 / kMaxScaleGuess to kMaxScaleGuess
constexpr float kMaxScaleGuess = 0x1p60f;

// src_dtype 1: bf16 channels [rows][N][D] (x); 0: fp16 channel pairs [taps][D / 2] from
// launch_transpose_pairs (filter taps).
// amax_out (bf16 sources only; null for none): per column task, the largest bf16 magnitude
// bits of the x it loaded, the pass running at scale first_scale in place of sc.glob.
// amax_in (null for none; 16-byte aligned, from a launch with amax_out over the same tasks):
// this launch takes x's power-of-two range scale s = 2^(3 - e) extra (2^e at or above
// max |x|, extra a power of two), writes {s, p / s} to *used (p = prev->y, or 1 for a null
// prev) and s to *hint (host-mapped, may be null), and redoes the pass at s in place of
// sc.glob unless s equals first_scale (the scale the first launch used).
hipError_t launch_col_fwd_mfma(int src_dtype, const void* src, int64_t src_row_stride, int D,
                               void* grid, int64_t grid_pb_stride, const LaunchTables& t,
                               GridScale sc, const void* mtab, int n_cols, int npb,
                               hipStream_t stream, uint16_t* amax_out = nullptr,
                               const uint16_t* amax_in = nullptr, float2* used = nullptr,
                               float first_scale = 1.0f, float* hint = nullptr, float extra = 1.0f,
                               const float2* prev = nullptr);

hipError_t launch_col_inv_mfma(int y_dtype, const void* grid, int64_t grid_pb_stride, void* dst,
                               int64_t dst_row_stride, int D, const LaunchTables& t,
                               GridScale sc, const void* mtab, int n_cols, int npb,
                               hipStream_t stream);

// Direct-path modes (launch_direct, launch_direct_mfma)
constexpr int kDirectConv = 0;
constexpr int kDirectCorr = 1;
constexpr int kDirectXcorr = 2;

// The direct path on the matrix cores (direct_mfma.hip): the same three modes for bf16 a
// (x, or dy) and b (x, mode 2) of documents of at most kMaxDirectMfma tokens, D a multiple
// of 32, a, b and out 16-byte aligned.  taps: [D][T] bf16 pairs (launch_split_taps), T >=
// min(L, longest document); unused in mode 2.  Outputs: y or dx in bf16, the correlation
// in fp32 (as launch_direct).
hipError_t launch_direct_mfma(int mode, const void* a, const void* b, const uint32_t* taps, int T,
                              const Seg* docs, int n_docs, int N, int D, int L, void* out, hipStream_t stream);
// taps[d][t] = bf16(k[d][t]) | bf16(k[d][t] - bf16(k[d][t])) << 16, t < T (row stride ld of k)
hipError_t launch_split_taps(const float* filters, int D, int T, int ld, uint32_t* taps, hipStream_t stream);

// Documents computed by their defining sums (the direct path; kernels.hip):
// mode 0 out = y from a = x, mode 1 out = dx from a = dy, mode 2 out = the
// per-document correlation of a = dy with b = x at lags tau < min(len, L), written at
// the document's tokens (fp32).  Dtype codes: 0 fp32, 1 bf16.  taps: [T][D] fp32.
// max_len: no document in docs is longer (at most kMaxDirect).
hipError_t launch_direct(int mode, int max_len, int a_dtype, const void* a, int b_dtype,
                         const void* b, const float* taps, const Seg* docs, int n_docs, int N, int D,
                         int L, int out_dtype, void* out, hipStream_t stream);

// The documents of the filter gradient's last sum, by non-increasing length: all n of them, and
// for the lags below lead_lags (a multiple of 32; 0: none) the n_lead that hold the others'
// correlations too (launch_lag_chunks); n_past of the n have lags from lead_lags on.
struct LagDocs {
    const Seg* segs = nullptr;
    int n = 0;
    const Seg* lead = nullptr;
    int n_lead = 0, lead_lags = 0, n_past = 0;
};

// dk[d][tau] = sum over the documents k with tau < min(len_k, L) of
// r[row_k][start_k + tau][d] (r fp32 [B][N][D]); dk [D][L] fp32, fully written.
hipError_t launch_lag_sum(const float* r, const LagDocs& docs, int N, int D, int L, float* dk, hipStream_t stream);

// The same sum's first step at the lags that many documents have: blocks, (chunk, tile)
// pairs, add each chunk's kLagChunk documents at 4 lags onto the chunk's first document (in
// place in r).
hipError_t launch_lag_chunks(float* r, const Seg* segs, const int32_t* blocks, int nblocks, int n_docs, int N, int D,
                             int L, hipStream_t stream);

// Filter taps [D][in_ld] fp32 -> [taps][D / 2] complex fp16 channel pairs (D even).
// partials (may be null): float [*ntiles][D], the sum of |k| of each channel over each
// tile of 32 or 64 taps (the input of launch_filter_scale); *ntiles <= tap_tile_rows(taps).
constexpr int tap_tile_rows(int taps) { return 2 * ((taps + 63) / 64); }
hipError_t launch_transpose_pairs(const float* in, int D, int taps, int in_ld, void* out,
                                  float* partials, int* ntiles, hipStream_t stream);

// out[c][r] = in[r][c] (r < rows, c < cols); partials as above with rows = channels and
// cols = taps (may be null), ceil(cols / 32) tiles.
hipError_t launch_transpose(const float* in, int rows, int cols, int in_ld, float* out,
                            int out_ld, float* partials, hipStream_t stream);

// Per channel pair q < npairs: g = max over its channels of the summed partials (the
// filter's absolute gain, sum over taps of |k|) and s = 2^(kFilterGainExp - e) with
// g < 2^e (1 when g is zero or not finite); pair_scale[q] = {s, 1 / s}.
constexpr int kFilterGainExp = 8;
hipError_t launch_filter_scale(const float* partials, int ntiles, int D, int npairs,
                               float2* pair_scale, hipStream_t stream);

// Exact power-of-two prescale of a [n] bf16 (dtype 1) or fp32 (dtype 0) tensor:
// a = max |v| (partials, then their maximum; no atomics: a fixed result); s = 2^(kDataAmaxExp - e)
// with a < 2^e (1 when a is zero or not finite), times `extra` (a power of two);
// out = {s * extra, (prev ? prev->y : 1) / (s * extra)}.  work: kAmaxParts uint32.
// launch_amax writes the partials and fills parts, n, head and tail of *src (the rest is the
// caller's); a VALU column pass reads them itself, launch_amax_finish writes *src->out for
// the others.
constexpr int kDataAmaxExp = 3;
constexpr int kAmaxParts = 2048;
// A VALU column pass reduces the partials itself while its workgroups together read at most
// this many of them.  Above, a launch of one workgroup costs less than the repeated reads
// (measured, bf16 at D = 767, us, separate launch / always in the pass: steps N = 4096
// 62.0 / 61.1, 8192 86.6 / 87.5, 32768 224.9 / 236.4, 8 x 16384 866 / 923; backward
// 113.3 / 110.9, 168.2 / 170.6, 484.6 / 513.3, 1829 / 2007).
constexpr int64_t kAmaxFoldWords = 5ll << 19;

// 2^(target - e) for a = f 2^e (0.5 <= f < 1): the power of two that brings a into
// [2^(target-1), 2^target); 1 for a zero, negative, infinite or NaN a.
__device__ __forceinline__ float pow2_scale(float a, int target) {
    if (!(a > 0.0f) || !(a <= 3.0e38f)) return 1.0f;
    int e;
    (void)frexpf(a, &e);
    return ldexpf(1.0f, max(-126, min(127, target - e)));
}


hipError_t launch_amax(int dtype, const void* in, int64_t n, uint32_t* work, AmaxSource* src, hipStream_t stream);
hipError_t launch_amax_finish(const AmaxSource& src, hipStream_t stream);

}  // namespace rubiconv
