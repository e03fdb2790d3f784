// Recover R(a^) from the (value, index) pairs into a dense matrix in the workspace (internal header), for
// 16-bit (bf16) and 32-bit (fp32) elements.
#pragma once

#include <algorithm>

#include "common.hpp"
#include "dev_hooks.hpp"

namespace dropit {
namespace {

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

#ifndef DROPIT_RECOVER_CFG
#define DROPIT_RECOVER_CFG 256, 16384
#endif
constexpr int recover_cfg[2] = {DROPIT_RECOVER_CFG};
constexpr int RECOVER_THREADS = recover_cfg[0];
// Dense elements one recover workgroup builds in LDS.  Small tiles keep many workgroups resident
// per compute unit, which hides the latency of each one's search; rows wider than that get the
// large tile (64 KB of LDS), rows wider than the large tile take the generic path.
constexpr int RECOVER_ELEMS = recover_cfg[1];
constexpr int RECOVER_ELEMS_MAX = 32768;
constexpr int RECOVER_ELEMS_MIN = 1024;

// ---------------------------------------------------------------------------
// Recover R(a^): workgroup b owns rows [b * rows_per_wg, ...) of the padded dense
// matrix.  Its pairs are one contiguous run of the index-sorted arrays (found by
// search), so the rows are assembled in LDS (zero fill, one 16-bit store per pair)
// and leave as full 16-byte stores: every byte of the dense matrix is written exactly
// once, no separate zero-fill pass.
// The pairs come through for_pairs_in_range: a window around the interpolated positions of the
// rows' first and last flat index, one round of loads, with the exact search as the fallback.
constexpr int RECOVER_WINDOW = 28;                    // window entries per thread, at most

// (The host uses fc_recover_stream_kernel instead when the window would be several times the pairs a
// workgroup needs.)
template <typename RAW>
__global__ void __launch_bounds__(RECOVER_THREADS)
fc_recover_kernel(const RAW *__restrict__ vals, const int32_t *__restrict__ idx, int64_t k, int64_t ntok,
                  int64_t ntok_pad, int cin, int pitch, int rows_per_wg, int64_t numel, int64_t margin, RAW *__restrict__ dense)
{
    extern __shared__ __attribute__((aligned(16))) u32x4 tile16[];   // [rows_per_wg][pitch]
    const int tid = threadIdx.x;
    const int64_t r0 = int64_t(blockIdx.x) * rows_per_wg;
    const int64_t r1 = min(r0 + rows_per_wg, ntok_pad);
    const int rows = int(r1 - r0);
    RAW *tile = reinterpret_cast<RAW *>(tile16);
    constexpr int PER16 = 16 / int(sizeof(RAW));                      // elements per 16-byte unit
    const int chunks = rows * (pitch / PER16);                        // 16-byte units
    const int64_t first = min(r0, ntok) * cin, last = min(r1, ntok) * cin;   // flat index range of these rows
    const uint32_t span = uint32_t(last - first);
    auto place = [&](int32_t flat, uint32_t v) {
        const uint32_t rel = uint32_t(int64_t(flat) - first);
        if (rel >= span) return;                                      // not one of this workgroup's rows
        uint32_t pos = rel;
        if (pitch != cin) {
            const uint32_t row = rel / uint32_t(cin);
            pos = row * uint32_t(pitch) + (rel - row * uint32_t(cin));
        }
        tile[pos] = static_cast<RAW>(v);
    };

    for_pairs_in_range<RECOVER_THREADS, RECOVER_WINDOW>(vals, idx, k, numel, first, last, margin, place, [&] {
        for (int i = tid; i < chunks; i += RECOVER_THREADS) tile16[i] = u32x4{0, 0, 0, 0};
    });
    __syncthreads();
    u32x4 *out16 = reinterpret_cast<u32x4 *>(dense + r0 * pitch);
    for (int i = tid; i < chunks; i += RECOVER_THREADS) out16[i] = tile16[i];
}

// Recover for large k: the error of the interpolated guess grows with sqrt(k) (and with the ties at
// the threshold, which are all kept at the low-index end of the tensor), the pairs of a tile do not, so
// a window per tile would be mostly overlap -- and an exact search per tile costs ~500 scattered probes
// of the index array (measured: 15 of 33 us on a 38 M-element tensor).  Here a workgroup takes several
// consecutive tiles, searches once for the start of its first one, and then walks the pair arrays
// forward: a tile's pairs follow the previous tile's.  A tile is done when a batch of pairs ends with
// an index beyond it.
template <typename RAW>
__global__ void __launch_bounds__(RECOVER_THREADS)
fc_recover_stream_kernel(const RAW *__restrict__ vals, const int32_t *__restrict__ idx, int64_t k, int64_t ntok,
                         int64_t ntok_pad, int cin, int pitch, int rows_per_tile, int tiles_per_wg,
                         RAW *__restrict__ dense)
{
    extern __shared__ __attribute__((aligned(16))) u32x4 tile16[];   // [rows_per_tile][pitch]
    constexpr int NWAVES = RECOVER_THREADS / WAVE;
    constexpr int BATCH = 8;
    __shared__ uint32_t wave_taken[2][NWAVES];
    const int tid = threadIdx.x;
    RAW *tile = reinterpret_cast<RAW *>(tile16);
    constexpr int PER16 = 16 / int(sizeof(RAW));                      // elements per 16-byte unit
    const int64_t tiles = (ntok_pad + rows_per_tile - 1) / rows_per_tile;
    const int64_t t_begin = int64_t(blockIdx.x) * tiles_per_wg, t_end = min(t_begin + tiles_per_wg, tiles);

    int64_t pos, unused;
    {
        const int64_t start = min(t_begin * rows_per_tile, ntok) * cin;
        block_lower_bound2<RECOVER_THREADS>(idx, start, start, 0, k, 0, k, pos, unused);
    }
    int32_t pi[BATCH];
    uint32_t pv[BATCH];             // a full register each (16-bit destinations get packed and the loads serialised)
    auto load_batch = [&]() {       // the pairs at pos, pos + 1, ... : BATCH per thread, all loads in flight together
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int64_t j = pos + int64_t(u) * RECOVER_THREADS + tid;
            if (j < k) {
                pi[u] = idx[j];
                pv[u] = vals[j];
            }
        }
    };
    load_batch();
    uint32_t parity = 0;
    for (int64_t t = t_begin; t < t_end; ++t) {
        const int64_t r0 = t * rows_per_tile, r1 = min(r0 + rows_per_tile, ntok_pad);
        const int chunks = int(r1 - r0) * (pitch / PER16);                // 16-byte units
        const int64_t first = min(r0, ntok) * cin, last = min(r1, ntok) * cin;
        const uint32_t span = uint32_t(last - first);
        for (int i = tid; i < chunks; i += RECOVER_THREADS) tile16[i] = u32x4{0, 0, 0, 0};
        __syncthreads();
        for (;;) {
            uint32_t mine = 0;
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int64_t j = pos + int64_t(u) * RECOVER_THREADS + tid;
                if (j < k && int64_t(pi[u]) < last) {
                    ++mine;
                    const uint32_t rel = uint32_t(int64_t(pi[u]) - first);
                    if (rel < span) {                                 // always, for a sorted index array
                        uint32_t at = rel;
                        if (pitch != cin) {
                            const uint32_t row = rel / uint32_t(cin);
                            at = row * uint32_t(pitch) + (rel - row * uint32_t(cin));
                        }
                        tile[at] = static_cast<RAW>(pv[u]);
                    }
                }
            }
            mine = wave_sum(mine);
            if ((tid & (WAVE - 1)) == 0) wave_taken[parity][tid / WAVE] = mine;
            __syncthreads();                                           // also: this batch's scatter is complete
            uint32_t taken = 0;
#pragma unroll
            for (int w = 0; w < NWAVES; ++w) taken += wave_taken[parity][w];
            parity ^= 1u;
            const int64_t loaded = min<int64_t>(int64_t(BATCH) * RECOVER_THREADS, k - pos);
            pos += taken;
            // The next pairs are fetched right away: more of this tile if the batch lay wholly inside
            // it, else the start of the next tile, whose loads then overlap this tile's write-out.
            const bool more = int64_t(taken) == loaded && pos < k;
            if (more || t + 1 < t_end) load_batch();
            if (!more) break;
        }
        u32x4 *out16 = reinterpret_cast<u32x4 *>(dense + r0 * pitch);
        for (int i = tid; i < chunks; i += RECOVER_THREADS) out16[i] = tile16[i];
        __syncthreads();                                               // tile read before the next one is zeroed
    }
}


// Dense elements of a recover workgroup's tile for a tensor of `numel`: at most `most`, fewer where that leaves compute
// units without a tile: one workgroup on a large tile of a small tensor is a chain of loads (17 thousand elements, gamma 0,
// two tiles of 8192: 12.6 us, and 10 to 16 where zero fill and scatter as two kernels took 4).  Tiles down to 1024 elements
// and 256 of them: within 1 % of 512 and 2048, and of 512 to 2048 tiles, over 700 calls of random shapes.
inline int64_t recover_tile(int64_t numel, int64_t most)
{
    int64_t tile = most;
    while (tile > RECOVER_ELEMS_MIN && (numel + tile - 1) / tile < 256) tile /= 2;
    return tile;
}

// Dense elements of one recover workgroup's tile, and the launch: rows of `cin` elements, `pitch` elements apart in
// the dense matrix (a multiple of 16 bytes), ntok_pad rows of which those from ntok on are zero; `numel` is the
// tensor's size (ntok * cin, or less when the last row is not full).
template <typename RAW>
inline void launch_recover(const RAW *vals, const int32_t *idx, int64_t k, int64_t numel, int64_t ntok, int64_t ntok_pad,
                           int cin, int pitch, int rows_per_wg, RAW *dense, hipStream_t stream)
{
    const int grid = int((ntok_pad + rows_per_wg - 1) / rows_per_wg);
    const size_t lds = size_t(rows_per_wg) * pitch * sizeof(RAW);
    // half-width of the window of pairs a recover workgroup loads around its interpolated positions:
    // 4 standard deviations of an evenly spread selection (sqrt(k)/2 at worst) plus a little
    const int64_t margin = 2 * static_cast<int64_t>(__builtin_sqrt(static_cast<double>(k))) + 256;
    const double pairs_per_wg = static_cast<double>(k) * rows_per_wg * cin / static_cast<double>(std::max<int64_t>(numel, 1));
    bool windowed = pairs_per_wg + 2.0 * margin <= double(RECOVER_WINDOW) * RECOVER_THREADS;
    if (dev_env("DROPIT_RECOVER_STREAM", 0)) windowed = false;
    if (windowed) {
        fc_recover_kernel<RAW><<<grid, RECOVER_THREADS, lds, stream>>>(vals, idx, k, ntok, ntok_pad, cin, pitch,
                                                                       rows_per_wg, numel, margin, dense);
    } else {
        // several consecutive tiles per workgroup, about two workgroups per compute unit (measured best of 1, 2, 4, 8)
        const int tiles_per_wg = std::max(1, (grid + 511) / 512);
        fc_recover_stream_kernel<RAW><<<(grid + tiles_per_wg - 1) / tiles_per_wg, RECOVER_THREADS, lds, stream>>>(
            vals, idx, k, ntok, ntok_pad, cin, pitch, rows_per_wg, tiles_per_wg, dense);
    }
}

}  // namespace
}  // namespace dropit
