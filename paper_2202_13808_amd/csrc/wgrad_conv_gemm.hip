// 3x3 / stride 1 / pad 1 convolution weight gradient as ONE dense GEMM over token-major operands.
//
// Sec. 3.2 (convolution weight gradient): dW[j][c][u][v] = sum over images and output positions of
// dY[n][j][oy][ox] * R(a^)[n][c][oy + u - 1][ox + v - 1].  Read as a matrix product this is
// dW[j][(u, v, c)] = sum_t dYt[t][j] * B[t][(u, v, c)] with one "token" t per output position
// (n, oy, ox): exactly the fully-connected form dY^T * x^ of the same section, with 9 * C input features.
// The rows of B are never written: they are runs of C elements of the token-major recovered input, which
// the product reads through the window (ConvWindow).
//
// For small planes with many channels (the last stages of a ResNet: 14x14x256, 7x7x512) the product has
// hundreds of (output tile, token block) units, so it runs on the fully-connected GEMM kernel, where the
// row-band kernel of wgrad_conv_mfma.hip spends most of its time staging a few hundred positions per
// workgroup.  Large planes with few channels are the opposite case and stay there.
//
// One small kernel prepares both operands: the recovered input, token-major, is assembled from the
// (value, index) pairs in LDS tiles (one image x a block of channels: its pairs are one contiguous run of
// the sorted arrays); other workgroups of the same launch transpose dY from [N][J][H][W] to [N*H*W][J].
// Bound by the product and the K-slices' partial tiles.  64 images of 256 -> 256 channels at 14 x 14,
// gamma 0.8: this preparation 11 us, where rows of B nine times the input (55 MB) took 29; call 67 -> 48 us;
// 256 images 189 -> 105, 512 channels at 7 x 7 52 -> 46, 16 images of 512 channels at 8 x 8 36 -> 36.6.
#include "wgrad_internal.hpp"

namespace dropit {
namespace {

constexpr int PREP_THREADS = 256;
constexpr int PREP_WINDOW = 32;             // window entries per thread (see for_pairs_in_range)

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int DYT_JB = 64;                    // output channels per transposing workgroup

// dY [N][J][HW] -> dYt [N * HW][J]: workgroup (n, block of 64 output channels) moves a contiguous
// 64 x HW slab through LDS.  J % 8 == 0, so the slab starts on a 16-byte boundary and is whole
// 16-byte vectors: each thread's loads are independent vector loads, all issued before the first
// LDS store; the stores leave as pairs of neighbouring channels.
__device__ inline void dy_to_tokens(const uint16_t *__restrict__ dY, int J, int HW, int unit, int jblocks,
                                    uint16_t *__restrict__ dYt, uint16_t *slab /* [64][HW | 1] */)
{
    const int n = unit / jblocks, j0 = (unit % jblocks) * DYT_JB;
    const int jw = min(DYT_JB, J - j0);                                   // a multiple of 8
    const int ld = HW | 1;                                                // odd pitch: the transposed reads spread over the banks
    const u32x4 *src = reinterpret_cast<const u32x4 *>(dY + (int64_t(n) * J + j0) * HW);
    const int vecs = jw * HW / 8;
    constexpr int BATCH = 4;
    for (int i0 = threadIdx.x; i0 < vecs; i0 += BATCH * PREP_THREADS) {
        u32x4 v[BATCH];
#pragma unroll
        for (int q = 0; q < BATCH; ++q)
            if (i0 + q * PREP_THREADS < vecs) v[q] = src[i0 + q * PREP_THREADS];
#pragma unroll
        for (int q = 0; q < BATCH; ++q) {
            const int i = i0 + q * PREP_THREADS;
            if (i >= vecs) continue;
            int jj = (i * 8) / HW, t = i * 8 - jj * HW;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                slab[jj * ld + t] = uint16_t(v[q][e >> 1] >> ((e & 1) * 16));
                if (++t == HW) {
                    t = 0;
                    ++jj;
                }
            }
        }
    }
    __syncthreads();
    uint32_t *dst = reinterpret_cast<uint32_t *>(dYt + int64_t(n) * HW * J + j0);     // j0 and J are even
    for (int i = threadIdx.x; i < HW * (DYT_JB / 2); i += PREP_THREADS) {
        const int t = i / (DYT_JB / 2), jj = (i % (DYT_JB / 2)) * 2;
        if (jj < jw) dst[(int64_t(t) * J + jj) / 2] = uint32_t(slab[jj * ld + t]) | (uint32_t(slab[(jj + 1) * ld + t]) << 16);
    }
}

// Both operands of the GEMM in one launch.  Workgroup (n, channel block), the first N * cblocks: channels
// [c0, c0 + cw) of the H * W token rows of image n, whose pairs are one contiguous run of the sorted arrays.  The last
// N * jblocks transpose dY; the first of those also clears the row of zeros behind the tokens.
__global__ void __launch_bounds__(PREP_THREADS)
conv_tokens_kernel(const uint16_t *__restrict__ vals, const int32_t *__restrict__ idx, int64_t k, int N, int C, int HW,
                   int cb, int cblocks, int64_t margin, uint16_t *__restrict__ xd, const uint16_t *__restrict__ dY, int J,
                   int jblocks, uint16_t *__restrict__ dYt)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t tile[];      // [HW][cb + 2], or the dY slab
    const int tid = threadIdx.x;
    const int units = N * cblocks;
    if (int(blockIdx.x) >= units) {
        if (int(blockIdx.x) == units)
            for (int i = tid; i < C / 8; i += PREP_THREADS)
                reinterpret_cast<u32x4 *>(xd + int64_t(N) * HW * C)[i] = u32x4{0u, 0u, 0u, 0u};
        dy_to_tokens(dY, J, HW, int(blockIdx.x) - units, jblocks, dYt, tile);
        return;
    }
    const int n = blockIdx.x / cblocks, c0 = (blockIdx.x % cblocks) * cb;
    const int cw = min(cb, C - c0);                                       // a multiple of 8
    const int row = cb + 2;                                               // an odd number of words: the stores of a channel's run spread over the banks
    const int64_t lo = (int64_t(n) * C + c0) * HW, hi = lo + int64_t(cw) * HW;
    auto place = [&](int32_t flat, uint32_t v16) {
        const uint32_t rel = uint32_t(int64_t(flat) - lo);
        if (rel >= uint32_t(cw * HW)) return;                             // another workgroup's pair
        const uint32_t c = rel / uint32_t(HW), t = rel - c * uint32_t(HW);
        tile[t * row + c] = uint16_t(v16);
    };
    // the pairs of [lo, hi): one round of loads around their interpolated position, else a search
    uint32_t *tile4 = reinterpret_cast<uint32_t *>(tile);
    for_pairs_in_range<PREP_THREADS, PREP_WINDOW>(vals, idx, k, int64_t(N) * C * HW, lo, hi, margin, place, [&] {
        for (int i = tid; i < HW * row / 2; i += PREP_THREADS) tile4[i] = 0u;
    });
    __syncthreads();
    const int per_row = cw / 8;
    for (int i = tid; i < HW * per_row; i += PREP_THREADS) {
        const int t = i / per_row, w = i - t * per_row;
        const uint32_t *src = tile4 + t * (row / 2) + w * 4;
        *reinterpret_cast<u32x4 *>(xd + (int64_t(n) * HW + t) * C + c0 + w * 8) = u32x4{src[0], src[1], src[2], src[3]};
    }
}

}  // namespace

ConvGemmPlan conv_gemm_plan(const ConvProblem &p)
{
    ConvGemmPlan plan;
    plan.fp = FcProblem{p.N * p.H * p.W, 9 * p.C, p.J, p.k};
    plan.gemm = fc_dense_plan(plan.fp, false, true, 9);
    const int64_t HW = p.H * p.W;
    // 64 channels: a token's segment is then a whole 128-byte line; fewer where that leaves compute units without a block
    plan.cb = 64;
    while (plan.cb > 16 && p.N * ((p.C + plan.cb - 1) / plan.cb) < 256) plan.cb /= 2;
    plan.cb = int(std::min<int64_t>(plan.cb, p.C));
    plan.cblocks = int((p.C + plan.cb - 1) / plan.cb);
    plan.lds_bytes = size_t(HW) * (plan.cb + 2) * 2;
    plan.xd_bytes = conv_window_bytes(p.N, p.C, p.H, p.W);
    plan.partial_bytes = round_up(conv_window_partial_bytes(plan.fp, plan.gemm, true), 256);
    plan.dyt_bytes = round_up(size_t(plan.fp.ntok) * p.J * 2, 256);
    return plan;
}

bool conv_gemm_supported(const ConvProblem &p)
{
    if (p.C % 8 != 0 || p.J % 8 != 0 || p.H < 1 || p.W < 1) return false;
    const int64_t HW = p.H * p.W;
    if (HW > 256 || p.N * HW >= (int64_t(1) << 31) / (9 * p.C)) return false;
    if (p.N * p.C > INT32_MAX / 2) return false;
    return fc_dense_supported(FcProblem{p.N * HW, 9 * p.C, p.J, p.k});
}

// Taken for small planes with many channels, where a plane fits a preparing workgroup and the product is large enough
// to be worth three dispatches: 56x56x64 and 28x28x128 stay on the row bands (the plane is too large here), planes up
// to the 256 positions the preparation holds come here.  Calls at gamma 0.8, row bands against this form: 64 images of
// 256 channels at 16 x 16 83 -> 56 us, 512 channels 238 -> 105, 128 channels 42.1 -> 39.7; 12 images of 128 channels at
// 16 x 15 38 -> 29.
bool conv_gemm_preferred(const ConvProblem &p)
{
    if (!conv_gemm_supported(p)) return false;
    const int64_t units = (9 * p.C + 255) / 256 * ((p.J + 255) / 256) * ((p.N * p.H * p.W + 31) / 32);   // 256 x 256 tiles times token blocks
    return p.H * p.W <= 256 && p.C >= 128 && units >= 256;
}

dropit_status conv_gemm_run(const ConvProblem &p, const ConvGemmPlan &plan, const void *vals, const int32_t *idx,
                            const void *dY, float *dW, char *ws, hipStream_t stream)
{
    uint16_t *xd = reinterpret_cast<uint16_t *>(ws);
    float *partial = reinterpret_cast<float *>(ws + plan.xd_bytes);
    uint16_t *dYt = reinterpret_cast<uint16_t *>(ws + plan.xd_bytes + plan.partial_bytes);
    const int HW = int(p.H * p.W);

    static std::atomic<uint64_t> attr_set{0};
    if (!once_per_device(attr_set, [] {
            return hipFuncSetAttribute(reinterpret_cast<const void *>(conv_tokens_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024) == hipSuccess;
        }))
        return DROPIT_EHIP;

    trace_mark(stream);
    const int units = int(p.N) * plan.cblocks;
    const int jblocks = int((p.J + DYT_JB - 1) / DYT_JB);
    // half-width of the pair window: 4 standard deviations of an evenly spread selection plus a little
    const int64_t margin = 2 * static_cast<int64_t>(__builtin_sqrt(static_cast<double>(p.k))) + 256;
    const size_t lds = std::max(plan.lds_bytes, size_t(DYT_JB) * (HW | 1) * 2);
    conv_tokens_kernel<<<units + int(p.N) * jblocks, PREP_THREADS, lds, stream>>>(
        static_cast<const uint16_t *>(vals), idx, p.k, int(p.N), int(p.C), HW, plan.cb, plan.cblocks, margin, xd,
        static_cast<const uint16_t *>(dY), int(p.J), jblocks, dYt);
    trace_mark(stream);
    if (launch_status() != DROPIT_OK) return DROPIT_EHIP;
    const dropit_conv2d g = {3, 3, 1, 1, 1, 1, 1, 1};
    return conv_window_gemm(plan.fp, plan.gemm, conv_window(p.N, p.C, p.H, p.W, p.H, p.W, g, true), dYt, xd, partial, dW, stream);
}

}  // namespace dropit
