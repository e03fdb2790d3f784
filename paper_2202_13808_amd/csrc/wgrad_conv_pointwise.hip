// Weight gradient of a 1x1 / stride 1 / unpadded NCHW convolution from the sparsified input, bf16 on the matrix cores:
//   dW[j][c] = sum over images n and positions p of dY[n][j][p] * R(a^)[n][c][p]      (Sec. 3.2, Eq. conv_backward_elem)
//
// Both operands keep the positions contiguous, which is the reduction axis: eight consecutive positions of one channel
// are an operand fragment of v_mfma_f32_32x32x16_bf16 as they lie.  dY fragments come straight from global memory
// (16 bytes per lane), R(a^) exists only as LDS rows of 64 channels, zero-filled and filled from the pairs.  No im2col
// rows, no transposed copy of dY.
//
// Bound by memory: the pairs are read once per block of output channels (up to 512 of them share a workgroup), dY once
// per 64 input channels, from the L2 for all but the first (the workgroups of one group of units run on one XCD).  The
// pairs come through three dependent steps (row starts, pairs, LDS), so eight of the sixteen wavefronts do nothing else,
// a unit ahead of the eight that multiply, with the next unit's loads in flight while they place the present one's.
// Whole gradient call, 64 images, gamma 0.8, against im2col rows + transposed dY + product: 256 -> 64 channels at 56 x 56
// 131 -> 68 us, 64 -> 256 129 -> 72, 512 -> 128 at 28 x 28 82 -> 54, 1024 -> 256 at 14 x 14 58 -> 53.  This kernel takes
// 39.5 of the 68 us (42 with one batch of dY in flight, 60 as eight wavefronts that fill and multiply in turn; 28 is what
// the pairs alone take): the 32-byte pieces of 32 rows that a dY load asks for are what is left.
#include "common.hpp"
#include "wgrad_internal.hpp"
#include "parts_sum.hpp"
#include <type_traits>

namespace dropit {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
struct __attribute__((packed, aligned(4))) u32x4_a4 {    // 16 bytes from a 4-byte boundary
    u32x4 v;
};

constexpr int PT = 1024;           // threads: eight wavefronts that fill the LDS rows, eight that multiply
constexpr int PC = 64;             // input channels of a workgroup
constexpr int POSITIONS = 512;     // LDS positions per channel, at most
constexpr int PBATCH = 32;         // positions (two MFMA depths) multiplied per step of a wavefront

struct PointwiseShape {
    int N, C, J, P;                // images, input and output channels, positions of a plane
    int sp, segs, nseg, tshift;    // LDS positions of a segment; segments per unit; segments per plane; log2 lanes per run
    int units, groups, cb_count, jb_count;
};

// until this wavefront's LDS accesses are performed and every wavefront has arrived; global loads stay in flight
__device__ inline void rows_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// A unit is `segs` whole planes of consecutive images (small planes), or one segment of one plane (segs == 1).  The
// pairs of (segment, channel) are one run of the sorted arrays; 64 / segs lanes share a run, a filling wavefront takes
// eight channels of the 64.  The multiplying wavefronts are WJ x (8 / WJ): WJ groups of 64 output channels, the
// others share out the positions and meet in LDS at the end.  At step i the unit i
// is filled into one of two sets of rows and the unit i - 1 multiplied from the other.
// ALIGN: bytes dY's rows are aligned to (16: whole fragments only; 4: pairs of positions).
template <int WJ, int ALIGN>
__global__ void __launch_bounds__(PT) __attribute__((amdgpu_waves_per_eu(4, 4)))
conv_pointwise_kernel(const uint16_t *__restrict__ dY, const uint16_t *__restrict__ vals, const int32_t *__restrict__ idx,
                      uint32_t k, const uint32_t *__restrict__ row_ptr, PointwiseShape g, float *__restrict__ partial)
{
    constexpr int KS = 8 / WJ;
    extern __shared__ __attribute__((aligned(16))) char lds[];      // [2][PC][segs * sp positions | 8], then the parked sums
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave16 = __builtin_amdgcn_readfirstlane(tid >> 6);
    // consecutive numbers on one XCD: the blocks of one group of units read the same rows of dY
    const int v = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    const int blocks = g.cb_count * g.jb_count;
    if (v >= blocks * g.groups) return;
    const int cb = v % g.cb_count, jb = (v / g.cb_count) % g.jb_count, grp = v / blocks;
    const int u_begin = int(int64_t(g.units) * grp / g.groups);
    const int count = int(int64_t(g.units) * (grp + 1) / g.groups) - u_begin;
    const int pitch = (g.segs * g.sp + 8) * 2;                      // an odd number of 16-byte units: conflict-free row reads
    const int wave = wave16 & 7;
    const int wk = wave / WJ, wj = wave % WJ;
    const int half = lane >> 5, l32 = lane & 31;
    f32x16 acc[2][2];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[f][b][e] = 0.f;

    if (wave16 >= 8) {
        // ---- fill: R(a^) of unit i into rows i & 1 ----
        const int q = lane >> g.tshift;                             // this lane's segment of the unit
        const uint32_t t = uint32_t(lane) & ((1u << g.tshift) - 1), step = 1u << g.tshift;
        const int c0 = cb * PC + wave * 8;
        struct Unit {
            int n, p0, seg, len;
            bool ok;
        };
        auto unit = [&](int i) {
            const int u = u_begin + min(i, count - 1);
            const int image0 = g.nseg > 1 ? u / g.nseg : u * g.segs;
            const int seg = g.nseg > 1 ? u - image0 * g.nseg : 0;
            const int p0 = seg * g.sp;
            return Unit{min(image0 + q, g.N - 1), p0, seg, min(g.sp, g.P - p0), image0 + q < g.N};
        };
        uint32_t lo[8], hi[8], lo_raw[8], hi_raw[8];
        auto fetch_bounds = [&](const Unit &u) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t row = uint32_t(u.n * g.C + min(c0 + i, g.C - 1)) * uint32_t(g.nseg) + uint32_t(u.seg);
                lo_raw[i] = row_ptr[row];
                hi_raw[i] = row_ptr[row + 1];
            }
        };
        // four channels: the bounds (clamped: a malformed index array may leave entries unwritten), then two rounds of pairs
        int flat[2][2][4];
        uint32_t val[2][2][4];                                      // full registers: 16-bit destinations get packed in pairs
        auto fetch_pairs = [&](auto half_, bool ok) {
            constexpr int h = decltype(half_)::value;
#pragma unroll
            for (int i = h * 4; i < h * 4 + 4; ++i) {
                lo[i] = min(lo_raw[i], k);
                hi[i] = ok && c0 + i < g.C ? min(hi_raw[i], k) : 0u;
            }
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t at = min(lo[h * 4 + i] + r * step + t, k - 1);   // unconditional, clamped (k > 0)
                    flat[h][r][i] = idx[at];
                    val[h][r][i] = vals[at];
                }
        };
        auto put = [&](char *rows, const Unit &u, int i, uint32_t off, int f, uint32_t w) {
            const uint32_t rel = uint32_t(f - ((u.n * g.C + c0 + i) * g.P + u.p0));
            if (lo[i] + off < hi[i] && rel < uint32_t(u.len))       // (always in the segment, for a sorted index array)
                *reinterpret_cast<uint16_t *>(rows + i * pitch + rel * 2) = uint16_t(w);
        };
        auto place = [&](auto half_, char *rows, const Unit &u) {
            constexpr int h = decltype(half_)::value;
            uint32_t longest = 0;
#pragma unroll
            for (int i = h * 4; i < h * 4 + 4; ++i) longest = max(longest, hi[i] - min(lo[i], hi[i]));
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) put(rows, u, h * 4 + i, r * step + t, flat[h][r][i], val[h][r][i]);
            for (uint32_t off = 2 * step + t; off < longest; off += step) {     // longer runs than the plan expected
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t at = min(lo[h * 4 + i] + off, k - 1);
                    flat[h][0][i] = idx[at];
                    val[h][0][i] = vals[at];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) put(rows, u, h * 4 + i, off, flat[h][0][i], val[h][0][i]);
            }
        };
        constexpr std::integral_constant<int, 0> first_half{};
        constexpr std::integral_constant<int, 1> second_half{};
        Unit cur = unit(0), next = unit(1);
        fetch_bounds(cur);
        fetch_pairs(first_half, cur.ok);
        fetch_pairs(second_half, cur.ok);
        fetch_bounds(next);
        for (int i = 0; i < count; ++i) {
            // this wavefront's own eight rows: its LDS accesses are performed in order, no barrier in between
            char *rows = lds + (i & 1) * (PC * pitch) + wave * 8 * pitch;
            for (int z = lane; z < 8 * pitch / 16; z += 64) reinterpret_cast<u32x4 *>(rows)[z] = u32x4{0, 0, 0, 0};
            asm volatile("" ::: "memory");
            rows += q * g.sp * 2;
            place(first_half, rows, cur);
            fetch_pairs(first_half, next.ok);                       // (past the last unit: its own pairs again, never placed)
            place(second_half, rows, cur);
            fetch_pairs(second_half, next.ok);
            cur = next;
            next = unit(i + 2);
            fetch_bounds(next);
            rows_barrier();
        }
        rows_barrier();
    } else {
        // ---- multiply: this wavefront's batches of 32 positions of unit i - 1 ----
        // Consecutive batches go to one wavefront: a 128-byte line of dY is two batches.  Two batches of fragments are in
        // flight, across the barriers between the units (that is the whole next unit for up to 64 output channels); a
        // fragment past the segment is zeroed where it is used, since a select behind the load would wait for it.
        const int batches = g.segs * g.sp / PBATCH, per_seg = g.sp / PBATCH;
        const int per = (batches + KS - 1) / KS, b0 = wk * per;
        const int steps = max(0, min(per, batches - b0));
        struct Batch {
            int image, p0, at, valid;                               // plane, first position of the segment, of the batch in it, end
        };
        auto batch = [&](int i, int b) {
            const int u = u_begin + i;
            const int image0 = g.nseg > 1 ? u / g.nseg : u * g.segs;
            const int p0 = g.nseg > 1 ? (u - image0 * g.nseg) * g.sp : 0;
            const int s = g.nseg > 1 ? 0 : b / per_seg;
            return Batch{min(image0 + s, g.N - 1), p0, (b - s * per_seg) * PBATCH, image0 + s < g.N ? min(g.sp, g.P - p0) : 0};
        };
        auto fetch = [&](u32x4 (&a)[2][2], const Batch &t) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const int p = t.at + ks * 16 + half * 8;
#pragma unroll
                for (int f = 0; f < 2; ++f) {
                    const int j = min(jb * (WJ * 64) + wj * 64 + f * 32 + l32, g.J - 1);   // rows past J are not stored
                    const uint16_t *row = dY + (int64_t(t.image) * g.J + j) * g.P + t.p0;
                    if constexpr (ALIGN == 16) {
                        a[ks][f] = *reinterpret_cast<const u32x4 *>(row + (p < t.valid ? p : 0));   // P % 8 == 0: inside or past
                    } else {
                        if (p + 8 <= t.valid) {
                            a[ks][f] = reinterpret_cast<const u32x4_a4 *>(row + p)->v;
                        } else {                                    // P % 2 == 0: whole pairs
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                a[ks][f][e] = *reinterpret_cast<const uint32_t *>(row + (p + e * 2 < t.valid ? p + e * 2 : 0));
                        }
                    }
                }
            }
        };
        auto multiply = [&](u32x4 (&a)[2][2], const Batch &t, const char *brow) {
            if (t.at + PBATCH > t.valid) {
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int f = 0; f < 2; ++f)
                            a[ks][f][e] = t.at + ks * 16 + half * 8 + e * 2 < t.valid ? a[ks][f][e] : 0u;
            }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const bf16x8 x0 = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(brow + ks * 32));
                const bf16x8 x1 = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(brow + ks * 32 + 32 * pitch));
#pragma unroll
                for (int f = 0; f < 2; ++f) {
                    const bf16x8 y = __builtin_bit_cast(bf16x8, a[ks][f]);
                    acc[f][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(y, x0, acc[f][0], 0, 0, 0);
                    acc[f][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(y, x1, acc[f][1], 0, 0, 0);
                }
            }
        };
        if (steps == 0) {
            for (int i = 0; i < count; ++i) rows_barrier();
        } else {
            u32x4 ring[2][2][2];
            int i = 0, st = 0, fi = 0, fst = 0;                     // multiplied next, requested next
            auto request = [&](u32x4 (&a)[2][2]) {
                if (fi >= count) return;
                fetch(a, batch(fi, b0 + fst));
                if (++fst == steps) {
                    fst = 0;
                    ++fi;
                }
            };
            auto consume = [&](u32x4 (&a)[2][2]) {
                if (st == 0) rows_barrier();                        // unit i is filled; its predecessor's rows are free
                const char *rows = lds + (i & 1) * (PC * pitch) + l32 * pitch + half * 16;
                multiply(a, batch(i, b0 + st), rows + (b0 + st) * (PBATCH * 2));
                request(a);
                if (++st == steps) {
                    st = 0;
                    ++i;
                }
            };
            request(ring[0]);
            request(ring[1]);
            while (i < count) {
                consume(ring[0]);
                if (i < count) consume(ring[1]);
            }
        }
        rows_barrier();
    }

    // ---- the position groups meet, halves at a time and in a fixed order ----
    const bool multiplies = wave16 < 8;
#pragma unroll
    for (int h = KS / 2; h >= 1; h /= 2) {
        __syncthreads();                                            // rows, or the sums parked before, have been read
        float *park = reinterpret_cast<float *>(lds) + ((wk % h) * WJ + wj) * (64 * WAVE);
        if (multiplies && wk >= h && wk < 2 * h) {
#pragma unroll
            for (int e = 0; e < 64; ++e) park[e * WAVE + lane] = acc[e >> 5][(e >> 4) & 1][e & 15];
        }
        __syncthreads();
        if (multiplies && wk < h) {
#pragma unroll
            for (int e = 0; e < 64; ++e) acc[e >> 5][(e >> 4) & 1][e & 15] += park[e * WAVE + lane];
        }
    }
    if (multiplies && wk == 0) {
        float *dst = partial + int64_t(grp) * g.J * g.C;
#pragma unroll
        for (int e = 0; e < 64; ++e) {
            const int j = jb * (WJ * 64) + wj * 64 + (e >> 5) * 32 + ((e & 15) >> 2) * 8 + half * 4 + (e & 3);
            const int c = cb * PC + ((e >> 4) & 1) * 32 + l32;
            if (j < g.J && c < g.C) dst[int64_t(j) * g.C + c] = acc[e >> 5][(e >> 4) & 1][e & 15];
        }
    }
}

}  // namespace

// Every such problem of the im2col path with an even plane of at least 16 positions: the form was faster at every size
// measured (16 to 4096 positions, 16 to 2048 channels, 2 to 64 images: by 4 % at 256 -> 1024 channels of 14 x 14, by
// 40 to 48 % at 28 x 28 and above).  Odd planes would start dY's rows between words, and planes below 16 positions would
// fill less than half of a segment's 32: they keep the im2col rows.
bool conv_pointwise_preferred(const ConvGeneral &p)
{
    const int64_t P = p.H * p.W;
    return !p.nhwc && p.g.kh == 1 && p.g.kw == 1 && p.g.stride_h == 1 && p.g.stride_w == 1 && p.g.pad_h == 0 &&
           p.g.pad_w == 0 && P % 2 == 0 && P >= 16;
}

PointwisePlan conv_pointwise_plan(const ConvGeneral &p)
{
    PointwisePlan plan;
    const int64_t P = p.H * p.W;
    // A filling wavefront has two rounds of pairs of every run in flight: segments whose expected run, and a little for
    // its spread, two rounds of 64 lanes hold, and (small planes) as few lanes per run as do so.
    const double density = double(p.k) / (double(p.N) * p.C * P);
    auto rounds = [&](int64_t positions) { return int64_t(1.1 * density * positions) + 12; };
    int64_t longest = POSITIONS;
    while (longest > 128 && rounds(longest) > 128) longest -= PBATCH;
    plan.nseg = int((P + longest - 1) / longest);
    plan.sp = int((P + plan.nseg - 1) / plan.nseg + PBATCH - 1) / PBATCH * PBATCH;
    plan.nseg = int((P + plan.sp - 1) / plan.sp);
    int lanes = 4;                                                   // lanes per run: a power of two, at least sp / 8 ...
    while (lanes < 64 && (lanes * 8 < plan.sp || lanes * 2 < rounds(P))) lanes *= 2;
    plan.segs = plan.nseg > 1 ? 1 : 64 / lanes;                      // ... so segs * sp <= POSITIONS
    if (plan.nseg > 1) lanes = 64;
    plan.tshift = 0;
    while ((1 << plan.tshift) < lanes) ++plan.tshift;
    plan.units = plan.nseg > 1 ? int(p.N * plan.nseg) : int((p.N + plan.segs - 1) / plan.segs);
    plan.wj = 1;
    while (plan.wj < 8 && plan.wj * 64 < p.J) plan.wj *= 2;
    plan.cb_count = int((p.C + PC - 1) / PC);
    plan.jb_count = int((p.J + plan.wj * 64 - 1) / (plan.wj * 64));
    const int64_t blocks = int64_t(plan.cb_count) * plan.jb_count;
    int64_t groups = std::min<int64_t>(std::max<int64_t>(256 / blocks, 1), plan.units);   // a workgroup per compute unit
    const int64_t per = (plan.units + groups - 1) / groups;         // units of the longest group: no more groups than it takes
    plan.groups = int((plan.units + per - 1) / per);
    plan.lds_bytes = size_t(2) * PC * (plan.segs * plan.sp + 8) * 2;
    if (plan.wj < 8) plan.lds_bytes = std::max<size_t>(plan.lds_bytes, 4 * 64 * WAVE * 4);   // four parked 64 x 64 sums
    plan.rowptr_bytes = round_up(size_t(p.N * p.C * plan.nseg + 1) * 4, 256);
    plan.partial_bytes = plan.groups > 1 ? round_up(size_t(plan.groups) * p.J * p.C * 4, 256) : 0;
    return plan;
}

dropit_status conv_pointwise_run(const ConvGeneral &p, const PointwisePlan &plan, const void *vals, const int32_t *idx,
                                 const void *dY, float *dW, char *ws, hipStream_t stream)
{
    uint32_t *row_ptr = reinterpret_cast<uint32_t *>(ws);
    float *partial = reinterpret_cast<float *>(ws + plan.rowptr_bytes);
    const int64_t P = p.H * p.W;
    const PointwiseShape g = {int(p.N), int(p.C), int(p.J), int(P), plan.sp, plan.segs, plan.nseg, plan.tshift,
                              plan.units, plan.groups, plan.cb_count, plan.jb_count};
    static std::atomic<uint64_t> attr_set{0};
    if (!once_per_device(attr_set, [] {
            bool ok = true;
            auto set = [&](auto kernel) {
                ok = ok && hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 2 * PC * (POSITIONS + 8) * 2) == hipSuccess;
            };
            set(conv_pointwise_kernel<1, 16>), set(conv_pointwise_kernel<2, 16>), set(conv_pointwise_kernel<4, 16>), set(conv_pointwise_kernel<8, 16>);
            set(conv_pointwise_kernel<1, 4>), set(conv_pointwise_kernel<2, 4>), set(conv_pointwise_kernel<4, 4>), set(conv_pointwise_kernel<8, 4>);
            return ok;
        }))
        return DROPIT_EHIP;
    const int64_t wgs = int64_t(plan.groups) * plan.cb_count * plan.jb_count;
    if (plan.segs * plan.sp > POSITIONS || wgs > INT32_MAX - 8) return DROPIT_EINVAL;
    trace_mark(stream);
    launch_row_starts(idx, p.k, uint32_t(P), uint32_t(plan.nseg > 1 ? plan.sp : P), p.N * p.C * plan.nseg, row_ptr, stream);
    trace_mark(stream);
    float *out = plan.groups > 1 ? partial : dW;
    auto launch = [&](auto kernel) {
        kernel<<<int((wgs + 7) / 8 * 8), PT, plan.lds_bytes, stream>>>(static_cast<const uint16_t *>(dY),
                                                                       static_cast<const uint16_t *>(vals), idx,
                                                                       uint32_t(p.k), row_ptr, g, out);
    };
    if (P % 8 == 0) {
        switch (plan.wj) {
        case 1: launch(conv_pointwise_kernel<1, 16>); break;
        case 2: launch(conv_pointwise_kernel<2, 16>); break;
        case 4: launch(conv_pointwise_kernel<4, 16>); break;
        default: launch(conv_pointwise_kernel<8, 16>); break;
        }
    } else {
        switch (plan.wj) {
        case 1: launch(conv_pointwise_kernel<1, 4>); break;
        case 2: launch(conv_pointwise_kernel<2, 4>); break;
        case 4: launch(conv_pointwise_kernel<4, 4>); break;
        default: launch(conv_pointwise_kernel<8, 4>); break;
        }
    }
    trace_mark(stream);
    if (plan.groups > 1) launch_parts_sum<1>(partial, plan.groups, p.J, p.C, dW, stream);
    trace_mark(stream);
    return launch_status();
}

}  // namespace dropit
