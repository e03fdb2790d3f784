// Split-K sums of the weight-gradient products (internal header): the K-slices' partial tiles, written in the
// accumulators' own order by wgrad_fc_dense.hip and wgrad_exact.hip, are added in a fixed order and moved to
// row-major dW.  A configuration C names the tile: BM, BN, NTHREADS, WAVES_N, WM, WN, FN (32 x 32 accumulators).
#pragma once

#include <algorithm>

#include "common.hpp"

namespace dropit {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

// Sums the split-K partials in ascending split order, dW = ((p0 + p1) + p2) + ..., and moves
// them from the accumulator order the GEMM wrote (see its epilogue) to row-major dW.
// One thread per 4 accumulator floats: rows m .. m+3 of one column.
template <typename C>
__global__ void __launch_bounds__(256)
splitk_sum_kernel(const f32x4 *__restrict__ partial, int splits, int M, int N, int nb_count, int mb_count,
                  float *__restrict__ dW)
{
    constexpr int TILE4 = C::BM * C::BN / 4;            // float4 groups per tile
    const int64_t tiles = int64_t(nb_count) * mb_count;
    const int64_t total = tiles * TILE4;
    for (int64_t g = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; g < total; g += int64_t(gridDim.x) * blockDim.x) {
        // eight slices at a time: all their loads are issued before the first add
        f32x4 s = partial[g];
        for (int p0 = 1; p0 < splits; p0 += 8) {
            f32x4 part[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (p0 + u < splits) part[u] = partial[(p0 + u) * total + g];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (p0 + u < splits) s += part[u];
        }
        const int tile = int(g / TILE4), r = int(g % TILE4);
        const int tid = r % C::NTHREADS, slot = r / C::NTHREADS;   // slot = (i * FN + j) * 4 + q
        const int q = slot & 3, j = (slot >> 2) % C::FN, i = (slot >> 2) / C::FN;
        const int lane = tid & 63, wave = tid >> 6;
        const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;
        const int mb = tile / nb_count, nb = tile % nb_count;
        const int m = mb * C::BM + wm * C::WM + i * 32 + q * 8 + (lane >> 5) * 4;
        const int n = nb * C::BN + wn * C::WN + j * 32 + (lane & 31);
        if (n < N) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (m + e < M) dW[int64_t(m + e) * N + n] = s[e];
        }
    }
}

// The same sum for many slices of few tiles (a result of one or two tiles is cut into up to 256 slices, one
// per compute unit): 16 threads share an output group, thread p of them adds the slices p, p + 16, ... in
// ascending order, and the 16 sums are added in ascending p through LDS -- a fixed order again, with 16
// times the loads in flight (one thread per group took 20 us for 256 slices of a single tile).
template <typename C>
__global__ void __launch_bounds__(256)
splitk_sum_wide_kernel(const f32x4 *__restrict__ partial, int splits, int M, int N, int nb_count, int mb_count,
                       float *__restrict__ dW)
{
    constexpr int PARTS = 16, GPB = 16;                // slice lanes per group, groups per workgroup
    constexpr int TILE4 = C::BM * C::BN / 4;
    __shared__ f32x4 red[PARTS][GPB];
    const int64_t total = int64_t(nb_count) * mb_count * TILE4;
    const int part = threadIdx.x / GPB, gi = threadIdx.x % GPB;
    const int64_t g = int64_t(blockIdx.x) * GPB + gi;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (g < total) {
        for (int p0 = part; p0 < splits; p0 += 4 * PARTS) {
            f32x4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (p0 + u * PARTS < splits) v[u] = partial[(p0 + u * PARTS) * total + g];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (p0 + u * PARTS < splits) s += v[u];
        }
    }
    red[part][gi] = s;
    __syncthreads();
    if (part != 0 || g >= total) return;
#pragma unroll
    for (int q = 1; q < PARTS; ++q) s += red[q][gi];
    const int tile = int(g / TILE4), r = int(g % TILE4);
    const int tid = r % C::NTHREADS, slot = r / C::NTHREADS;   // slot = (i * FN + j) * 4 + q
    const int q = slot & 3, j = (slot >> 2) % C::FN, i = (slot >> 2) / C::FN;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;
    const int mb = tile / nb_count, nb = tile % nb_count;
    const int m = mb * C::BM + wm * C::WM + i * 32 + q * 8 + (lane >> 5) * 4;
    const int n = nb * C::BN + wn * C::WN + j * 32 + (lane & 31);
    if (n < N) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (m + e < M) dW[int64_t(m + e) * N + n] = s[e];
    }
}

// The same sum where the product's columns are (tap, channel) of a 3 x 3 convolution and dW's are (channel, tap).  A
// workgroup takes eight rows and 32 channels of all nine taps, a wavefront a tap of them; the sums, in ascending split
// order, change places in LDS and leave as whole runs of 288 floats per row.  (Four-byte stores 36 bytes apart straight
// from the sums cost 8 us of a 45 us call: 16 images of 512 -> 512 channels at 8 x 8.)  DEPTH slices are in flight
// per thread: sixteen where a result of few tiles is cut into up to fifty of them, few where there are few, for the
// wavefronts that the registers then leave room for.
constexpr int SUM_TAPS = 9, SUM_CHANNELS = 32;
template <typename C, int DEPTH>
__global__ void __launch_bounds__(64 * SUM_TAPS)
splitk_sum_taps_kernel(const f32x4 *__restrict__ partial, int splits, int M, int channels, int nb_count, int mb_count,
                       float *__restrict__ dW)
{
    constexpr int TILE4 = C::BM * C::BN / 4, ROW = SUM_TAPS * SUM_CHANNELS;
    __shared__ __attribute__((aligned(16))) float turn[8][ROW];
    const int cblocks = (channels + SUM_CHANNELS - 1) / SUM_CHANNELS;
    const int c0 = int(blockIdx.x % unsigned(cblocks)) * SUM_CHANNELS, m0 = int(blockIdx.x / unsigned(cblocks)) * 8;
    const int tap = threadIdx.x >> 6, half = (threadIdx.x >> 5) & 1, l32 = threadIdx.x & 31;
    const int cw = min(SUM_CHANNELS, channels - c0);                // a multiple of 8
    if (l32 < cw) {
        const int n = tap * channels + c0 + l32;
        const int nb = n / C::BN, nr = n % C::BN, wn = nr / C::WN, j = (nr % C::WN) / 32;
        const int mb = m0 / C::BM, mr = m0 % C::BM, wm = mr / C::WM, i = (mr % C::WM) / 32, q = (mr % 32) / 8;
        const int64_t total = int64_t(nb_count) * mb_count * TILE4;
        const f32x4 *src = partial + int64_t(mb * nb_count + nb) * TILE4 + ((i * C::FN + j) * 4 + q) * C::NTHREADS +
                           (wm * C::WAVES_N + wn) * 64 + half * 32 + (nr & 31);
        f32x4 s = src[0];
        for (int p0 = 1; p0 < splits; p0 += DEPTH) {
            f32x4 part[DEPTH];
#pragma unroll
            for (int u = 0; u < DEPTH; ++u)
                if (p0 + u < splits) part[u] = src[(p0 + u) * total];
#pragma unroll
            for (int u = 0; u < DEPTH; ++u)
                if (p0 + u < splits) s += part[u];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) turn[half * 4 + e][l32 * SUM_TAPS + tap] = s[e];
    }
    __syncthreads();
    const int row = threadIdx.x / (ROW / 4), at = threadIdx.x % (ROW / 4) * 4;      // 8 x 72 threads of four floats
    if (m0 + row < M && at < cw * SUM_TAPS)
        *reinterpret_cast<f32x4 *>(dW + (int64_t(m0 + row) * channels + c0) * SUM_TAPS + at) =
            *reinterpret_cast<const f32x4 *>(&turn[row][at]);
}

template <typename C>
inline void launch_splitk_sum_taps(const float *partial, int splits, int M, int channels, int nb_count, int mb_count,
                                   float *dW, hipStream_t stream)
{
    const int64_t blocks = int64_t((M + 7) / 8) * ((channels + SUM_CHANNELS - 1) / SUM_CHANNELS);
    auto launch = [&](auto kernel) {
        kernel<<<int(blocks), 64 * SUM_TAPS, 0, stream>>>(reinterpret_cast<const f32x4 *>(partial), splits, M, channels,
                                                          nb_count, mb_count, dW);
    };
    if (splits > 6) launch(splitk_sum_taps_kernel<C, 16>);
    else launch(splitk_sum_taps_kernel<C, 5>);
}

// Adds the partials of `splits` > 1 slices into dW.
template <typename C>
inline void launch_splitk_sum(const float *partial, int splits, int M, int N, int nb_count, int mb_count, float *dW,
                              hipStream_t stream)
{
    const int64_t groups = int64_t(nb_count) * mb_count * (C::BM * C::BN / 4);
    const f32x4 *p4 = reinterpret_cast<const f32x4 *>(partial);
    if (splits > 16) {
        splitk_sum_wide_kernel<C><<<int((groups + 15) / 16), 256, 0, stream>>>(p4, splits, M, N, nb_count, mb_count, dW);
    } else {
        const int blocks = int(std::min<int64_t>((groups + 255) / 256, 1 << 20));   // one group per thread
        splitk_sum_kernel<C><<<blocks, 256, 0, stream>>>(p4, splits, M, N, nb_count, mb_count, dW);
    }
}

}  // namespace
}  // namespace dropit
