// Weight gradient from the sparsified cache (Sec. 3.2): recover R(a^) (zeros at
// dropped positions) and take the ordinary dense weight gradient,
//   FC   : dW[j][c]       = sum_n dY[n][j] * R(a^)[n][c]            (Eq. fc_backward_elem_save)
//   conv : dW[j][c][u][v] = sum_{n,oy,ox} dY[n][j][oy][ox] * R(a^)[n][c][oy+u-1][ox+v-1]
//                                                                   (Eq. conv_backward_elem, 3x3/s1/p1)
//
// This file holds the host entry points, the choice of the path, and the one-launch
// kernel of small fully-connected layers.
#include "common.hpp"
#include "wgrad_internal.hpp"
#include "dev_hooks.hpp"
#include <cstdlib>

namespace dropit {
namespace {

__device__ inline float to_f32(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }
__device__ inline float to_f32(uint32_t b) { return __uint_as_float(b); }

__global__ void __launch_bounds__(256) zero_f32_kernel(float *p, int64_t n)
{
    for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
        p[i] = 0.f;
}

// ---- FC, small layers: recover and multiply in ONE launch --------------------------------------------
// A layer whose whole input fits the LDS of a compute unit (numel <= SMALL_NUMEL fp32 values) is bound by
// launches, not by work: the zero fill, the scatter and the product as three kernels cost three dispatch
// slots for a few microseconds of arithmetic.  Here every workgroup rebuilds the whole R(a^) in its own LDS
// (zero fill, then one store per pair: the k pairs are a few thousand), fetches its JB columns of dY,
// and multiplies with true fp32 multiply-adds (bf16 inputs are widened exactly): a thread sums four neighbouring columns
// of a row of dW over its share of the tokens, a contiguous one, in ascending order, and the shares are added in ascending
// order through LDS.  Four rows of dW to a workgroup and up to sixteen shares: the chain of dependent LDS reads, one per
// token, is what a few workgroups of 256 threads with all tokens each spent their time on (calls in a queue
// of calls: 256 tokens of 64 -> 128 10.9 us, 4.8 now; 1024 of 16 -> 64 29.7 and 5.5; 128 of 128 -> 4096 10.2 and 7.1).
// Sixteen rows where four would make more workgroups than the chip holds, or more than one to a compute unit for little work
// (75 tokens of 64 -> 1928 5.0 with four, 4.5 with sixteen; 128 of 128 -> 1928 5.7 and 6.5).
constexpr int SMALL_NUMEL = 16384;         // elements of x: 64 KB of fp32 in LDS
constexpr int SMALL_TOKENS = 1024;         // tokens: the dY slice is SMALL_TOKENS x JB fp32, 64 KB at most
constexpr int SMALL_THREADS = 1024, SMALL_SHARES = 16, SMALL_MAX_JB = 16;

inline int small_rows(int64_t numel, int64_t cout) { return cout <= 1024 || (cout <= 2048 && numel > 8192) ? 4 : SMALL_MAX_JB; }

template <typename RAW, int JB>
__global__ void __launch_bounds__(SMALL_THREADS)
fc_small_kernel(const RAW *__restrict__ vals, const int32_t *__restrict__ idx, int k, const RAW *__restrict__ dY,
                int ntok, int cin, int cout, int shares, float *__restrict__ dW)
{
    extern __shared__ __attribute__((aligned(16))) float small_lds[];
    float *xs = small_lds;                                 // R(a^)  [ntok][cin]; afterwards the shares' sums
    float *gs = small_lds + ntok * cin;                    // dY     [ntok][JB], columns j0 ..
    const int tid = threadIdx.x;
    const int j0 = blockIdx.x * JB;
    const int numel = ntok * cin;                          // a multiple of 4 (cin is)
    // the first pairs and dY are on their way while the zeros are written
    constexpr int PRE = 2;
    int pi[PRE];
    RAW pv[PRE];
#pragma unroll
    for (int u = 0; u < PRE; ++u) {
        const int q = tid + u * SMALL_THREADS;
        pi[u] = q < k ? idx[q] : -1;
        pv[u] = q < k ? vals[q] : RAW(0);
    }
    for (int e = tid; e < ntok * JB; e += SMALL_THREADS) {
        const int n = e / JB, j = j0 + e % JB;
        gs[e] = j < cout ? to_f32(dY[int64_t(n) * cout + j]) : 0.f;
    }
    float4 *xs4 = reinterpret_cast<float4 *>(xs);
    for (int i = tid; i < numel / 4; i += SMALL_THREADS) xs4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    auto place = [&](int i, RAW v) {
        if (i >= 0 && i < numel) xs[i] = to_f32(v);        // an out-of-range index is ignored, never written
    };
#pragma unroll
    for (int u = 0; u < PRE; ++u) place(pi[u], pv[u]);
    for (int q = tid + PRE * SMALL_THREADS; q < k; q += SMALL_THREADS) place(idx[q], vals[q]);
    __syncthreads();
    const int cq = cin / 4, items = JB * cq;               // (row, four columns): the columns run fastest over the lanes
    if (shares > 1) {                                      // items * shares <= SMALL_THREADS
        const int share = tid / items, item = tid % items, j = item / cq, c0 = item % cq * 4;
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
        if (share < shares) {
            const int n1 = ntok * (share + 1) / shares;
#pragma unroll 4
            for (int n = ntok * share / shares; n < n1; ++n) {
                const float g = gs[n * JB + j];
                const float4 b = *reinterpret_cast<const float4 *>(xs + n * cin + c0);
                s.x = __builtin_fmaf(g, b.x, s.x);
                s.y = __builtin_fmaf(g, b.y, s.y);
                s.z = __builtin_fmaf(g, b.z, s.z);
                s.w = __builtin_fmaf(g, b.w, s.w);
            }
        }
        __syncthreads();                                   // R(a^) has been read
        if (share < shares) xs4[tid] = s;
        __syncthreads();
        if (tid < items && j0 + j < cout) {
            for (int h = 1; h < shares; ++h) {
                const float4 o = xs4[h * items + tid];
                s.x += o.x;
                s.y += o.y;
                s.z += o.z;
                s.w += o.w;
            }
            *reinterpret_cast<float4 *>(dW + int64_t(j0 + j) * cin + c0) = s;
        }
    } else {
        for (int item = tid; item < items; item += SMALL_THREADS) {
            const int j = item / cq, c0 = item % cq * 4;
            float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
            for (int n = 0; n < ntok; ++n) {
                const float g = gs[n * JB + j];
                const float4 b = *reinterpret_cast<const float4 *>(xs + n * cin + c0);
                s.x = __builtin_fmaf(g, b.x, s.x);
                s.y = __builtin_fmaf(g, b.y, s.y);
                s.z = __builtin_fmaf(g, b.z, s.z);
                s.w = __builtin_fmaf(g, b.w, s.w);
            }
            if (j0 + j < cout) *reinterpret_cast<float4 *>(dW + int64_t(j0 + j) * cin + c0) = s;
        }
    }
}

template <typename RAW, int JB>
dropit_status launch_fc_small(const void *vals, const int32_t *idx, int64_t k, const void *dY, int64_t ntok, int64_t cin,
                              int64_t cout, float *dW, hipStream_t stream)
{
    static std::atomic<uint64_t> set_up{0};
    if (!once_per_device(set_up, [] {
            return hipFuncSetAttribute(reinterpret_cast<const void *>(fc_small_kernel<RAW, JB>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       int((SMALL_NUMEL + SMALL_TOKENS * JB) * sizeof(float))) == hipSuccess;
        }))
        return DROPIT_EHIP;
    // as many shares of the tokens as threads are left for, four tokens each at least
    const int64_t items = JB * (cin / 4);
    int shares = 1;
    while (shares < SMALL_SHARES && 2 * shares * items <= SMALL_THREADS && 8 * shares <= ntok) shares *= 2;
    const size_t sums = shares > 1 ? size_t(shares) * items * 16 : 0;
    const size_t lds = std::max(size_t(ntok * cin + ntok * JB) * sizeof(float), sums);
    fc_small_kernel<RAW, JB><<<unsigned((cout + JB - 1) / JB), SMALL_THREADS, lds, stream>>>(
        static_cast<const RAW *>(vals), idx, int(k), static_cast<const RAW *>(dY), int(ntok), int(cin), int(cout), shares, dW);
    return launch_status();
}

struct Problem {
    bool conv;
    int64_t numel, ntok, cin, cout;
    int64_t N, C, H, W, OH, OW;
    dropit_conv2d g;
    bool is_3x3_s1_p1;
    bool nhwc;                                   // x [N][H][W][C], dY [N][OH][OW][J], dW [J][kh][kw][C]
};

// Validates shape arguments; returns DROPIT_OK and fills `p`.
dropit_status describe(const int64_t *x_shape, int ndim, dropit_dtype dt, int64_t c_out,
                       const dropit_conv2d *conv, Problem &p, bool nhwc = false)
{
    p.nhwc = nhwc;
    if (dt != DROPIT_F32 && dt != DROPIT_BF16) return DROPIT_EINVAL;
    p.numel = checked_numel(x_shape, ndim);
    if (p.numel < 1 || c_out < 1 || c_out > INT32_MAX) return DROPIT_EINVAL;
    p.cout = c_out;
    p.conv = conv != nullptr;
    p.is_3x3_s1_p1 = false;
    p.g = dropit_conv2d{};
    p.N = p.C = p.H = p.W = p.OH = p.OW = 0;
    if (!p.conv) {
        p.cin = x_shape[ndim - 1];
        p.ntok = p.numel / p.cin;
        if (p.ntok * c_out > int64_t(1) << 40) return DROPIT_EINVAL;
        return DROPIT_OK;
    }
    if (ndim != 4) return DROPIT_EINVAL;
    if (conv->kh < 1 || conv->kw < 1 || conv->stride_h < 1 || conv->stride_w < 1 || conv->pad_h < 0 ||
        conv->pad_w < 0 || conv->dil_h < 1 || conv->dil_w < 1)
        return DROPIT_EINVAL;
    p.g = *conv;
    p.is_3x3_s1_p1 = conv->kh == 3 && conv->kw == 3 && conv->stride_h == 1 && conv->stride_w == 1 && conv->pad_h == 1 &&
                     conv->pad_w == 1 && conv->dil_h == 1 && conv->dil_w == 1;
    p.N = x_shape[0];
    if (nhwc) {
        p.H = x_shape[1]; p.W = x_shape[2]; p.C = x_shape[3];
    } else {
        p.C = x_shape[1]; p.H = x_shape[2]; p.W = x_shape[3];
    }
    constexpr int64_t GEOM_MAX = 65535;              // keeps every index expression far inside 64 bits
    if (conv->kh > 1024 || conv->kw > 1024 || conv->pad_h > GEOM_MAX || conv->pad_w > GEOM_MAX ||
        conv->stride_h > GEOM_MAX || conv->stride_w > GEOM_MAX || conv->dil_h > GEOM_MAX || conv->dil_w > GEOM_MAX)
        return DROPIT_EINVAL;
    const int64_t eh = p.H + 2 * conv->pad_h - conv->dil_h * (conv->kh - 1) - 1;   // output extent: floor(e / stride) + 1
    const int64_t ew = p.W + 2 * conv->pad_w - conv->dil_w * (conv->kw - 1) - 1;
    if (eh < 0 || ew < 0) return DROPIT_EINVAL;                                    // the window does not fit the padded input
    p.OH = eh / conv->stride_h + 1;
    p.OW = ew / conv->stride_w + 1;
    if (p.N * c_out * p.OH * p.OW > INT32_MAX * int64_t(16)) return DROPIT_EINVAL;
    if (c_out * p.C * conv->kh * conv->kw > INT32_MAX) return DROPIT_EINVAL;
    // A channels-last 1x1 / stride 1 / unpadded convolution IS a fully-connected layer over the N*H*W
    // positions: x [N*H*W][C], dY [N*H*W][J], dW [J][1][1][C] = [J][C].  It takes the FC kernels.
    if (nhwc && conv->kh == 1 && conv->kw == 1 && conv->stride_h == 1 && conv->stride_w == 1 && conv->pad_h == 0 &&
        conv->pad_w == 0) {
        p.conv = false;
        p.cin = p.C;
        p.ntok = p.numel / p.C;
    }
    return DROPIT_OK;
}

ExactProblem exact_of(const Problem &p, int64_t k)
{
    if (!p.conv) return ExactProblem{false, false, p.numel, p.ntok, p.cin, p.cout, k, 0, 0, 0, 0, 0, p.g};
    return ExactProblem{true, p.nhwc, p.numel, p.N * p.OH * p.OW, p.C * p.g.kh * p.g.kw, p.cout, k, p.C, p.H, p.W, p.OH, p.OW, p.g};
}

}  // namespace
}  // namespace dropit

using namespace dropit;

static bool use_fc_dense(const FcProblem &fp) { return fc_dense_supported(fp); }

static ConvGeneral general_of(const Problem &p, int64_t k)
{
    return ConvGeneral{p.N, p.C, p.H, p.W, p.OH, p.OW, p.cout, k, p.g, p.nhwc};
}

// Which kernels serve this problem.
static bool fc_small(const Problem &p)
{
    return !p.conv && p.numel <= SMALL_NUMEL && p.ntok <= SMALL_TOKENS && p.cin % 4 == 0 && p.cout <= 4096;
}

// 0: recover into a dense operand in the workspace, then the product; 1: recover inside the product where that
// form exists (see dropit_set_fc_recover).  Per host thread.
static int &fc_recover_form()
{
    static thread_local int form = 0;
    return form;
}

static dropit_wgrad_path choose_path(const Problem &p, dropit_dtype dt, int64_t k)
{
    if (fc_small(p)) return DROPIT_PATH_FC_SMALL;
    if (dt != DROPIT_BF16) return DROPIT_PATH_FMA;
    if (!p.conv) {
        const FcProblem fp = {p.ntok, p.cin, p.cout, k};
        if (!use_fc_dense(fp)) return DROPIT_PATH_FMA;
        return fc_recover_form() == 1 && k >= 1 && fc_fused_supported(fp) ? DROPIT_PATH_FC_FUSED : DROPIT_PATH_FC_MFMA;
    }
    if (p.is_3x3_s1_p1 && !p.nhwc) {
        const ConvProblem cp = {p.N, p.C, p.H, p.W, p.cout, k};
        bool gemm = conv_gemm_preferred(cp);
        if (const long forced = dev_env("DROPIT_CONV_GEMM", -1); forced >= 0) gemm = forced == 1 && conv_gemm_supported(cp);
        if (gemm) return DROPIT_PATH_CONV_GEMM;
        if (conv_mfma_supported(cp)) return DROPIT_PATH_CONV_BANDS;
    }
    return conv_im2col_supported(general_of(p, k)) ? DROPIT_PATH_CONV_IM2COL : DROPIT_PATH_FMA;
}

// Workspace need of the path dropit_weight_grad will take for this problem.
static size_t workspace_need(const Problem &p, dropit_dtype dt, int64_t k)
{
    const ConvProblem cp = {p.N, p.C, p.H, p.W, p.cout, k};
    switch (choose_path(p, dt, k)) {
    case DROPIT_PATH_FC_MFMA: return fc_dense_plan(FcProblem{p.ntok, p.cin, p.cout, k}).total();
    case DROPIT_PATH_FC_FUSED: return fc_dense_plan(FcProblem{p.ntok, p.cin, p.cout, k}, true).total();
    case DROPIT_PATH_CONV_GEMM: return conv_gemm_plan(cp).total();
    case DROPIT_PATH_CONV_BANDS: return conv_mfma_plan(cp).total();
    case DROPIT_PATH_CONV_IM2COL: return conv_im2col_plan(general_of(p, k)).total();
    case DROPIT_PATH_FC_SMALL: return 256;           // nothing is kept outside LDS; a token size so that callers' buffers exist
    default: return exact_plan(exact_of(p, k), dt == DROPIT_F32).total();
    }
}

static dropit_status run(const Problem &p, const void *vals, const int32_t *idx, int64_t k, dropit_dtype dt,
                         const void *dY, float *dW, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (k < 0 || k > p.numel) return DROPIT_EINVAL;
    if (k > 0 && (vals == nullptr || idx == nullptr)) return DROPIT_EINVAL;
    if (k > 0 && (!aligned(vals, dt == DROPIT_F32 ? 4 : 2) || !aligned(idx, 4))) return DROPIT_EINVAL;
    if (dY == nullptr || dW == nullptr || !aligned(dY, 16) || !aligned(dW, 16)) return DROPIT_EINVAL;
    if (workspace == nullptr || !aligned(workspace, 256)) return DROPIT_EINVAL;
    const size_t need = workspace_need(p, dt, k);
    if (workspace_bytes < need) return DROPIT_EWORKSPACE;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    char *ws = static_cast<char *>(workspace);
    if (k == 0) {                                  // everything was dropped: R(a^) = 0, so dW = 0
        const int64_t n = p.conv ? p.cout * p.C * p.g.kh * p.g.kw : p.cout * p.cin;
        zero_f32_kernel<<<int(std::min<int64_t>((n + 255) / 256, 2048)), 256, 0, stream>>>(dW, n);
        return launch_status();
    }
    const ConvProblem cp = {p.N, p.C, p.H, p.W, p.cout, k};
    switch (choose_path(p, dt, k)) {
    case DROPIT_PATH_FC_MFMA: {
        const FcProblem fp = {p.ntok, p.cin, p.cout, k};
        return fc_dense_run(fp, fc_dense_plan(fp), vals, idx, dY, dW, ws, stream);
    }
    case DROPIT_PATH_FC_FUSED: {
        const FcProblem fp = {p.ntok, p.cin, p.cout, k};
        return fc_fused_run(fp, fc_dense_plan(fp, true), vals, idx, dY, dW, ws, stream);
    }
    case DROPIT_PATH_CONV_GEMM: return conv_gemm_run(cp, conv_gemm_plan(cp), vals, idx, dY, dW, ws, stream);
    case DROPIT_PATH_CONV_BANDS: return conv_mfma_run(cp, conv_mfma_plan(cp), vals, idx, dY, dW, ws, stream);
    case DROPIT_PATH_CONV_IM2COL: {
        const ConvGeneral cg = general_of(p, k);
        return conv_im2col_run(cg, conv_im2col_plan(cg), vals, idx, dY, dW, ws, stream);
    }
    case DROPIT_PATH_FC_SMALL: {
        trace_mark(stream);
        auto go = [&](auto raw_) {
            using RAW = decltype(raw_);
            return small_rows(p.numel, p.cout) == 4 ? launch_fc_small<RAW, 4>(vals, idx, k, dY, p.ntok, p.cin, p.cout, dW, stream)
                                           : launch_fc_small<RAW, SMALL_MAX_JB>(vals, idx, k, dY, p.ntok, p.cin, p.cout, dW, stream);
        };
        if (const dropit_status st = dt == DROPIT_BF16 ? go(uint16_t(0)) : go(uint32_t(0)); st != DROPIT_OK) return st;
        trace_mark(stream);
        return launch_status();
    }
    default: break;
    }
    const ExactProblem ep = exact_of(p, k);
    return exact_run(ep, exact_plan(ep, dt == DROPIT_F32), dt == DROPIT_F32, vals, idx, dY, dW, ws, stream);
}

extern "C" dropit_status dropit_set_fc_recover(int form)
{
    if (form != 0 && form != 1) return DROPIT_EINVAL;
    fc_recover_form() = form;
    return DROPIT_OK;
}

extern "C" dropit_wgrad_path dropit_weight_grad_path(const int64_t *x_shape, int ndim, dropit_dtype dt, int64_t k,
                                                     int64_t c_out, const dropit_conv2d *conv)
{
    Problem p;
    if (describe(x_shape, ndim, dt, c_out, conv, p) != DROPIT_OK) return DROPIT_PATH_NONE;
    if (k < 0 || k > p.numel) return DROPIT_PATH_NONE;
    return choose_path(p, dt, k);
}

extern "C" size_t dropit_weight_grad_workspace_bytes(const int64_t *x_shape, int ndim, dropit_dtype dt,
                                                     int64_t k, int64_t c_out, const dropit_conv2d *conv)
{
    Problem p;
    if (describe(x_shape, ndim, dt, c_out, conv, p) != DROPIT_OK) return 0;
    if (k < 0 || k > p.numel) return 0;
    return workspace_need(p, dt, k);
}

extern "C" dropit_status dropit_weight_grad(const void *vals, const int32_t *idx, int64_t k,
                                            const int64_t *x_shape, int ndim, dropit_dtype dt, const void *dY,
                                            int64_t c_out, const dropit_conv2d *conv, float *dW, void *workspace,
                                            size_t workspace_bytes, void *hip_stream)
{
    Problem p;
    const dropit_status st = describe(x_shape, ndim, dt, c_out, conv, p);
    if (st != DROPIT_OK) return st;
    return run(p, vals, idx, k, dt, dY, dW, workspace, workspace_bytes, hip_stream);
}

// ---- channels-last convolutions ------------------------------------------------
extern "C" dropit_wgrad_path dropit_weight_grad_nhwc_path(const int64_t *x_shape, dropit_dtype dt, int64_t k,
                                                          int64_t c_out, const dropit_conv2d *conv)
{
    Problem p;
    if (conv == nullptr || describe(x_shape, 4, dt, c_out, conv, p, true) != DROPIT_OK) return DROPIT_PATH_NONE;
    if (k < 0 || k > p.numel) return DROPIT_PATH_NONE;
    return choose_path(p, dt, k);
}

extern "C" size_t dropit_weight_grad_nhwc_workspace_bytes(const int64_t *x_shape, dropit_dtype dt, int64_t k,
                                                          int64_t c_out, const dropit_conv2d *conv)
{
    Problem p;
    if (conv == nullptr || describe(x_shape, 4, dt, c_out, conv, p, true) != DROPIT_OK) return 0;
    if (k < 0 || k > p.numel) return 0;
    return workspace_need(p, dt, k);
}

extern "C" dropit_status dropit_weight_grad_nhwc(const void *vals, const int32_t *idx, int64_t k,
                                                 const int64_t *x_shape, dropit_dtype dt, const void *dY,
                                                 int64_t c_out, const dropit_conv2d *conv, float *dW,
                                                 void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (conv == nullptr) return DROPIT_EINVAL;
    Problem p;
    const dropit_status st = describe(x_shape, 4, dt, c_out, conv, p, true);
    if (st != DROPIT_OK) return st;
    return run(p, vals, idx, k, dt, dY, dW, workspace, workspace_bytes, hip_stream);
}
