// Sum of per-workgroup partial weight gradients in a fixed order (internal header).
#pragma once

#include "common.hpp"

namespace dropit {
namespace {

// dW[j][c][tap] = sum over the workgroups' partials partial[p][tap][j][c], in a fixed order:
// a workgroup takes 64 consecutive (tap, j, c) outputs; each of its (up to 16) wavefronts adds its share
// of the parts in ascending order (enough loads in flight to cover the memory latency), then the
// first wavefront adds the wavefronts' sums in ascending order.
// VEC = 4 (taken when J * C is a multiple of 4): a thread sums four consecutive outputs with 16-byte loads.
constexpr int RED_GROUPS = 16;
template <int VEC, int TAPS>
__global__ void __launch_bounds__(64 * RED_GROUPS)
conv_reduce_kernel(const float *__restrict__ partial, int parts, int J, int C, float *__restrict__ dW)
{
    typedef float vec_t __attribute__((ext_vector_type(VEC == 1 ? 2 : VEC)));   // (a 1-vector is not indexable: lane 0 of a pair)
    __shared__ vec_t s_sum[RED_GROUPS][64];
    const int groups = blockDim.x / 64;                 // wavefronts of this launch (a power of two up to 16)
    const int64_t jc = int64_t(J) * C;
    const int64_t total = jc * TAPS;
    const int o = threadIdx.x & 63, grp = threadIdx.x >> 6;
    const int64_t i = (int64_t(blockIdx.x) * 64 + o) * VEC;              // first of this thread's outputs
    vec_t s = 0.f;
    if (i < total) {
        const int per = (parts + groups - 1) / groups;
        const int p0 = grp * per, p1 = min(p0 + per, parts);
#pragma unroll 8
        for (int p = p0; p < p1; ++p) {
            if constexpr (VEC == 1) s[0] += partial[int64_t(p) * total + i];
            else s += *reinterpret_cast<const vec_t *>(partial + int64_t(p) * total + i);
        }
    }
    s_sum[grp][o] = s;
    __syncthreads();
    if (grp == 0 && i < total) {
        vec_t t = s_sum[0][o];
        for (int g = 1; g < groups; ++g) t += s_sum[g][o];
        if constexpr (TAPS == 1 && VEC == 4) {
            *reinterpret_cast<vec_t *>(dW + i) = t;
        } else {
            const int64_t tap = i / jc, rem = i - tap * jc;             // i = (tap, j, c); the VEC outputs share tap and j
#pragma unroll
            for (int e = 0; e < VEC; ++e) dW[(rem + e) * TAPS + tap] = t[e];
        }
    }
}

template <int TAPS>
inline void launch_parts_sum(const float *partial, int parts, int64_t J, int64_t C, float *dW, hipStream_t stream)
{
    const int64_t total = J * C * TAPS;
    // wavefronts per 64 (x4) outputs: enough that a thread has about four loads in flight, at most 16
    int groups = 1;
    while (groups * 8 <= parts && groups < RED_GROUPS) groups *= 2;
    if ((J * C) % 4 == 0)
        conv_reduce_kernel<4, TAPS><<<int((total / 4 + 63) / 64), 64 * groups, 0, stream>>>(partial, parts, int(J), int(C), dW);
    else
        conv_reduce_kernel<1, TAPS><<<int((total + 63) / 64), 64 * groups, 0, stream>>>(partial, parts, int(J), int(C), dW);
}

}  // namespace
}  // namespace dropit
