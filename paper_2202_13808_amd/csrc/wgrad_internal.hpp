// Internal interfaces between the weight-gradient host entry point and its kernels.
#pragma once

#include <algorithm>

#include "common.hpp"

namespace dropit {

struct FcProblem {
    int64_t ntok, cin, cout, k;
};

// the product's tile of dW: 256 x 256 or 128 x 128; 128 x 256 in the in-LDS recover form only
enum class GemmTile { WIDE, SMALL, HALF };
struct FcDensePlan {
    int nkb, nb_count, mb_count, splits, pitch, rows_per_wg;
    GemmTile tile;
    int64_t ntok_pad;                          // rows of the dense operand: the tokens rounded up to whole token blocks
    size_t dense_bytes, partial_bytes;
    // the in-LDS form keeps no dense operand: the pairs regrouped by tile (a word each), the table of tile starts
    // and the table of token-block starts take its place at the front of the workspace
    bool fused;
    size_t packed_bytes, table_bytes, kbptr_bytes;
    size_t operand_bytes() const { return fused ? packed_bytes + table_bytes + kbptr_bytes : dense_bytes; }
    size_t total() const { return operand_bytes() + partial_bytes; }
};

// bf16 fully-connected weight gradient: recover R(a^) densely, then a direct-to-LDS GEMM (wgrad_fc_dense.hip)
bool fc_dense_supported(const FcProblem &p);
// summed: the slice sum runs for one slice too; taps: of the window that the product reads through
FcDensePlan fc_dense_plan(const FcProblem &p, bool fused = false, bool summed = false, int taps = 1);
dropit_status fc_dense_run(const FcProblem &p, const FcDensePlan &plan, const void *vals, const int32_t *idx,
                           const void *dY, float *dW, char *ws, hipStream_t stream);

// the same product with the recover step inside it: the zero-filled tensor exists only as LDS tiles (plan.fused)
bool fc_fused_supported(const FcProblem &p);
dropit_status fc_fused_run(const FcProblem &p, const FcDensePlan &plan, const void *vals, const int32_t *idx,
                           const void *dY, float *dW, char *ws, hipStream_t stream);

// the same from the row form of the cache (col = position in the row, rowptr = pairs before each row)
dropit_status fc_dense_run_rows(const FcProblem &p, const FcDensePlan &plan, const void *vals, const uint16_t *col,
                                const int32_t *rowptr, const void *dY, float *dW, char *ws, hipStream_t stream);

// ... and from the bit-mask form (mask bit per element, blockptr = pairs before each block of DROPIT_MASK_BLOCK);
// only when fc_dense_mask_native(p): c_in % 8 == 0
bool fc_dense_mask_native(const FcProblem &p);
dropit_status fc_dense_run_mask(const FcProblem &p, const FcDensePlan &plan, const void *vals, const uint32_t *mask,
                                const int32_t *blockptr, const void *dY, float *dW, char *ws, hipStream_t stream);

// the GEMM and the K-slice sum alone, on operands that are already dense: dY [ntok][cout], dense [plan.ntok_pad][plan.pitch]
// (rows past ntok zero); `partial` holds plan.partial_bytes
dropit_status fc_dense_gemm(const FcProblem &p, const FcDensePlan &plan, const void *dY, const uint16_t *dense,
                            float *partial, float *dW, hipStream_t stream);

// Quotient of a dividend below 2^31 by a constant of the launch: the multiply-high by ceil(2^32 / d) is the quotient or
// one more, and corrected.  (d = 1 saturates the factor, which is then one less; the correction covers that too.)
struct Divisor {
    uint32_t d, magic;
};
inline Divisor divisor(uint32_t d)
{
    const uint64_t m = ((uint64_t(1) << 32) + d - 1) / d;
    return Divisor{d, uint32_t(std::min<uint64_t>(m, 0xffffffffu))};
}
__device__ inline uint32_t quotient(uint32_t f, Divisor v)
{
    uint32_t q = __umulhi(f, v.magic);
    const int32_t r = int32_t(f - q * v.d);
    if (r < 0) --q;
    else if (uint32_t(r) >= v.d) ++q;
    return q;
}

// A convolution's product with its operand rows read through the window: token t (output position) of the FC form has
// the input elements under its window as columns (u, v, c), which are kh * kw runs of C consecutive elements of the
// recovered input kept token-major, xd [N * H * W][C] followed by one row of zeros (what hangs over the padding reads
// those).  C % 8 == 0.  channel_major: dW is [J][C][taps], else [J][taps][C].
struct ConvWindow {
    int C, H, W, OH, OW, kw, sh, sw, ph, pw, dh, dw, taps;
    bool channel_major;
    uint32_t zero_row;                         // byte offset of the row of zeros
    int adv_y, adv_x;                          // input rows and columns a token block moves on by (beyond whole images)
    int image_step, row_step;                  // input rows and columns that OH output rows, OW output columns move on by
    uint32_t adv, carry_x, carry_y;            // bytes: a token block; the end of an output row; the end of an image
};
ConvWindow conv_window(int64_t N, int64_t C, int64_t H, int64_t W, int64_t OH, int64_t OW, const dropit_conv2d &g,
                       bool channel_major);
bool conv_window_supported(int64_t N, int64_t C, int64_t H, int64_t W);
inline size_t conv_window_bytes(int64_t N, int64_t C, int64_t H, int64_t W) { return round_up(size_t(N * H * W + 1) * C * 2, 256); }
// bytes of `partial` for the product (a channel-major dW always goes through the slice sum, which reorders it)
size_t conv_window_partial_bytes(const FcProblem &p, const FcDensePlan &plan, bool channel_major);
// xd from the pairs of an NHWC tensor; the product (dY token-major)
dropit_status conv_window_recover(const ConvWindow &w, int64_t N, const void *vals, const int32_t *idx, int64_t k,
                                  uint16_t *xd, hipStream_t stream);
dropit_status conv_window_gemm(const FcProblem &p, const FcDensePlan &plan, const ConvWindow &w, const void *dY,
                               const uint16_t *xd, float *partial, float *dW, hipStream_t stream);

// dropit_compress with a cheaper index form as its output (compress.hip); DROPIT_EUNSUPPORTED: convert flat indices instead
enum { FORM_FLAT = 0, FORM_ROWS = 1, FORM_MASK = 2 };
dropit_status compress_form(const void *x, int64_t numel, dropit_dtype dt, int64_t k, void *vals, int32_t *idx, int kind,
                            uint16_t *col, uint32_t *mask, int32_t *starts, uint32_t len, int64_t nstarts, char *ws,
                            hipStream_t stream);

// Row starts of the index-sorted pairs: row_ptr[r] = number of pairs whose flat index lies before row r, r = 0..R
// (row_ptr[R] = k).  The tensor is a run of planes, a plane is cut into `nseg` rows of `seg` consecutive elements (the
// last one may be shorter); one row per plane is the plain case of rows of equal length.  One pass over idx: every
// pair is compared with its predecessor and fills the row starts that fall between them; the entry j == k closes the
// table.  A thread takes PER consecutive pairs: eight (two 16-byte loads when idx is 16-byte aligned), or one where the rows
// are so short or sparse that filling their starts, one store after the other, is the longer part.  Bound by reading
// idx where it is not: 10.3 M pairs take 13.6 us, 4.3 TB/s beside the launch.
template <bool VEC, int PER>
static __global__ void __launch_bounds__(256)
row_starts_kernel(const int32_t *__restrict__ idx, int64_t k, Divisor plane, Divisor seg, uint32_t nseg, int64_t R,
                  uint32_t *__restrict__ row_ptr)
{
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    static_assert(!VEC || PER % 4 == 0, "whole vectors");
    auto row_of = [&](int32_t flat) -> int64_t {
        if (flat < 0) return R;                                           // (a malformed index; valid ones are below 2^31)
        uint32_t r = quotient(uint32_t(flat), plane);
        if (nseg > 1) r = r * nseg + quotient(uint32_t(flat) - r * plane.d, seg);
        return min<int64_t>(r, R);
    };
    const int64_t stride = int64_t(gridDim.x) * blockDim.x * PER;
    for (int64_t j0 = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) * PER; j0 <= k; j0 += stride) {
        int32_t v[PER];
        const int32_t prev = j0 == 0 ? 0 : idx[j0 - 1];
        if (VEC && j0 + PER <= k) {
#pragma unroll
            for (int h = 0; h < PER / 4; ++h) {
                const i32x4 q = *reinterpret_cast<const i32x4 *>(idx + j0 + h * 4);
                v[h * 4] = q[0]; v[h * 4 + 1] = q[1]; v[h * 4 + 2] = q[2]; v[h * 4 + 3] = q[3];
            }
        } else {
#pragma unroll
            for (int e = 0; e < PER; ++e) v[e] = j0 + e < k ? idx[j0 + e] : 0;
        }
        int64_t before = (j0 == 0) ? -1 : row_of(prev);
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int64_t j = j0 + e;
            if (j > k) break;
            const int64_t here = (j == k) ? R : row_of(v[e]);
            for (int64_t r = before + 1; r <= here; ++r) row_ptr[r] = uint32_t(j);
            before = here;
        }
    }
}

// rows of `seg` elements inside planes of `plane` elements
inline void launch_row_starts(const int32_t *idx, int64_t k, uint32_t plane, uint32_t seg, int64_t R, uint32_t *row_ptr,
                              hipStream_t stream)
{
    const uint32_t nseg = (plane + seg - 1) / seg;
    // Fewer than eight pairs per row, or too few pairs for eight to a thread to fill the chip.  (2.5 thousand pairs in 82 thousand rows: 45.4 us with eight to a thread; 500 calls
    // of random shapes and gammas did best with the line at eight, against one and three.)
    const bool one = k < 8 * R || k < (1 << 16);
    const int blocks = int(std::min<int64_t>((k / (one ? 1 : 8) + 1 + 255) / 256, 4096));
    auto launch = [&](auto kernel) {
        kernel<<<blocks, 256, 0, stream>>>(idx, k, divisor(plane), divisor(seg), nseg, R, row_ptr);
    };
    if (one) launch(row_starts_kernel<false, 1>);
    else if (aligned(idx, 16)) launch(row_starts_kernel<true, 8>);
    else launch(row_starts_kernel<false, 8>);
}

inline void launch_row_starts(const int32_t *idx, int64_t k, uint32_t row_len, int64_t R, uint32_t *row_ptr,
                              hipStream_t stream)
{
    launch_row_starts(idx, k, row_len, row_len, R, row_ptr, stream);
}

struct ConvProblem {
    int64_t N, C, H, W, J, k;
};

struct ConvPlan {
    int cb_count, jb_count, bands, rb, pitch_c;
    int wp;                                    // row width the kernel works with: W rounded up to whole groups of 8
    int imgs_per_wg, img_groups;               // a workgroup accumulates over this many images; ceil(N / imgs_per_wg) groups
    size_t lds_bytes, rowptr_bytes, partial_bytes;
    size_t dypad_bytes;                        // zero-padded copy of dY when wp != W, else 0
    size_t total() const { return rowptr_bytes + partial_bytes + dypad_bytes; }
};

// bf16 3x3/s1/p1 convolution weight gradient on the matrix cores (wgrad_conv_mfma.hip)
bool conv_mfma_supported(const ConvProblem &p);
ConvPlan conv_mfma_plan(const ConvProblem &p);
dropit_status conv_mfma_run(const ConvProblem &p, const ConvPlan &plan, const void *vals, const int32_t *idx,
                            const void *dY, float *dW, char *ws, hipStream_t stream);

// The same gradient as one GEMM over token-major operands, for small planes with many channels
// (wgrad_conv_gemm.hip)
struct ConvGemmPlan {
    FcProblem fp;                              // tokens = N*H*W output positions, c_in = 9*C taps, c_out = J
    FcDensePlan gemm;
    int cb, cblocks;                           // input channels per preparing workgroup
    size_t lds_bytes, dyt_bytes, xd_bytes, partial_bytes;
    size_t total() const { return xd_bytes + partial_bytes + dyt_bytes; }
};
bool conv_gemm_supported(const ConvProblem &p);
bool conv_gemm_preferred(const ConvProblem &p);
ConvGemmPlan conv_gemm_plan(const ConvProblem &p);
dropit_status conv_gemm_run(const ConvProblem &p, const ConvGemmPlan &plan, const void *vals, const int32_t *idx,
                            const void *dY, float *dW, char *ws, hipStream_t stream);

// Any geometry, NCHW or NHWC, bf16: zero-filled im2col rows written from the pairs + the FC GEMM
// (wgrad_conv_im2col.hip)
struct ConvGeneral {
    int64_t N, C, H, W, OH, OW, J, k;
    dropit_conv2d g;
    bool nhwc;
};
// 1x1 / stride 1 / unpadded NCHW: the operands multiplied as they lie, no im2col rows (wgrad_conv_pointwise.hip)
struct PointwisePlan {
    int wj;                                    // wavefront groups of 64 output channels per workgroup
    int sp, segs, nseg, tshift;                // positions of a segment in LDS; segments (images) per unit; segments per plane; log2 lanes per run
    int cb_count, jb_count, units, groups;     // workgroup = (channel block, output-channel block, group of units)
    size_t lds_bytes, rowptr_bytes, partial_bytes;
    size_t total() const { return rowptr_bytes + partial_bytes; }
};
struct ConvIm2colPlan {
    FcProblem fp;                              // tokens = N*OH*OW, c_in = C*kh*kw, c_out = J
    FcDensePlan gemm;
    size_t dyt_bytes;                          // token-major copy of dY (NCHW only)
    bool tiled;                                // im2col rows assembled in LDS tiles (else zero fill + scatter)
    int nblocks, blk, bands, rb, rowlen;       // tiled form: column blocks, their width, row bands, rows per band, tile row length
    size_t lds_bytes, rowptr_bytes;
    bool pointwise, window;                    // the forms without im2col rows that take this problem
    PointwisePlan pw;
    size_t xd_bytes;                           // window: the recovered input
    size_t total() const
    {
        return pointwise ? pw.total() : window ? xd_bytes + gemm.partial_bytes : gemm.dense_bytes + gemm.partial_bytes + dyt_bytes + rowptr_bytes;
    }
};
bool conv_pointwise_preferred(const ConvGeneral &p);
PointwisePlan conv_pointwise_plan(const ConvGeneral &p);
dropit_status conv_pointwise_run(const ConvGeneral &p, const PointwisePlan &plan, const void *vals, const int32_t *idx,
                                 const void *dY, float *dW, char *ws, hipStream_t stream);
bool conv_im2col_supported(const ConvGeneral &p);
ConvIm2colPlan conv_im2col_plan(const ConvGeneral &p);
dropit_status conv_im2col_run(const ConvGeneral &p, const ConvIm2colPlan &plan, const void *vals, const int32_t *idx,
                              const void *dY, float *dW, char *ws, hipStream_t stream);

// Exact fp32 products of any shape, geometry and layout, fp32 or bf16 (wgrad_exact.hip)
struct ExactProblem {
    bool conv, nhwc;
    int64_t numel, ntok, cin, cout, k;         // cin: columns of dW (C * kh * kw for a convolution), ntok: output positions
    int64_t C, H, W, OH, OW;                   // convolution only
    dropit_conv2d g;
};
struct ExactPlan {
    int bm, bn, nb_count, mb_count, nkb, splits;
    int tile;                                  // elements of R(a^) per recover workgroup
    size_t dense_bytes, partial_bytes;
    size_t total() const { return dense_bytes + partial_bytes; }
};
ExactPlan exact_plan(const ExactProblem &p, bool f32);
dropit_status exact_run(const ExactProblem &p, const ExactPlan &plan, bool f32, const void *vals, const int32_t *idx,
                        const void *dY, float *dW, char *ws, hipStream_t stream);

}  // namespace dropit
