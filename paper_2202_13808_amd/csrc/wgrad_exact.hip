// Weight gradient with exact fp32 products on the gfx950 fp32 matrix instructions
// (Sec. 3.2: recover R(a^), then Eq. fc_backward_elem_save / Eq. conv_backward_elem).
//
// Serves fp32 tensors of every geometry and layout, and the bf16 shapes the bf16 matrix-core paths do not take
// (bf16 widens to fp32 exactly).  One product for all of them:
//   dW[j][col] = sum_t dY(t, j) * X(t, col)
// t = token (FC) or output position (n, oy, ox) (convolution), col = input feature or (channel, tap).
//
//   1. recover : R(a^) is rebuilt as a flat dense tensor in the workspace (recover.hpp).
//   2. product : v_mfma_f32_32x32x2_f32, one workgroup per BM x BN tile of dW and K-slice.  This instruction takes
//      64 cycles for 4096 multiply-adds, a sixteenth of the bf16 rate, so the kernel is bound by the matrix pipe
//      with everything else to spare -- 8 to 16 bytes of operands per clock and compute unit -- and the spare
//      goes into the operand fetch: a convolution's im2col rows are never written anywhere, each element of a
//      tile is fetched from R(a^) by its own address (a handful of integer operations per element and 4096 cycles
//      of multiplying per 32-token step), NCHW tensors are read in place without a transposition, and any
//      alignment and ragged edge is served by the same code.  The fetched step waits in registers while the
//      previous one multiplies; one LDS buffer, two barriers per step, two or more workgroups per compute unit
//      to cover them.
//   3. the K-slices' sums are added in a fixed order (splitk.hpp).
// Products and accumulation are true fp32 multiply-adds in a fixed order: dW is bit-reproducible.  (Large fp32 fully-connected
// layers take a faster product, see "fp32 products from bf16 thirds".)
// A window position over the padding is no term of the sum: an infinity or NaN of dY must not meet the zero that stands
// there in the tile.  A workgroup whose sums are not all finite (padded convolutions only: one look at them at the end)
// does its slice again, with the tokens whose dY is not finite taken out of the matrix product and added by vector
// multiply-adds, position by position.
//
// Measured, whole weight-gradient call, against vector multiply-adds on a zero-filled and scattered R(a^) (one
// 64 x 64 tile over all tokens; one workgroup per (j, c) for convolutions): fp32 6304 x 384 -> 1536 637 -> 81 us
// (7.4 GFLOP; 48 us at the 154 TFLOP/s a large fp32 product reaches), fp32 3x3 convolution 32 x 64 x 32 x 32 -> 64
// 442 -> 56 us (2.4 GFLOP, 16 us).
#include "recover.hpp"
#include "splitk.hpp"
#include "wgrad_internal.hpp"
#include "dev_hooks.hpp"
#include <type_traits>

namespace dropit {
namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ inline float widen(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }
__device__ inline float widen(uint32_t b) { return __uint_as_float(b); }

// Tile of 2 x 2 wavefronts.  LDS rows (one token each) are padded by four floats: 16-byte stores stay aligned, and
// stores that walk down the tokens (the NCHW operands) spread over the banks.
template <int BM_, int BN_>
struct ExactCfg {
    static constexpr int BM = BM_, BN = BN_, BK = 32, WAVES_M = 2, WAVES_N = 2, NTHREADS = 256;
    static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N, FM = WM / 32, FN = WN / 32;
    static constexpr int PA = BM + 4, PB = BN + 4;
};

// How an operand tile is fetched: token-major rows with 16-byte loads, token-major rows element by element,
// or one address per element with the lanes along the tokens (NCHW: consecutive positions are consecutive in
// memory) or along the columns (NHWC: consecutive channels are).
enum Fetch { ROWS16, ROWS1, ALONG_TOKENS, ALONG_COLUMNS };

struct ExactGeometry {
    uint32_t OW, P, W, H, C, taps, kw, sh, sw, ph, pw, dh, dw;   // P = OH * OW
    uint32_t xc, xh, xw;                                         // element strides of R(a^): channel, row, column
    int64_t xn, yn;                                              // ... and of an image, in R(a^) and in dY
    Divisor by_P, by_OW;
    uint32_t x_bytes, y_bytes;                                   // of R(a^) and of dY where 32-bit byte offsets reach all of both, else 0
};

// acc[i][j][e] is row 8*(e/4) + 4*(lane/32) + e%4, column lane%32 of its 32x32 block
template <typename C>
__device__ inline void exact_epilogue(const f32x16 (&acc)[C::FM][C::FN], int splits, int split, int nb_count, int mb_count,
                                      int nb, int mb, int M, int N, float *__restrict__ out)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;
    if (splits == 1) {
#pragma unroll
        for (int i = 0; i < C::FM; ++i)
#pragma unroll
            for (int j = 0; j < C::FN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int m = mb * C::BM + wm * C::WM + i * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
                    const int n = nb * C::BN + wn * C::WN + j * 32 + (lane & 31);
                    if (m < M && n < N) out[int64_t(m) * N + n] = acc[i][j][e];
                }
    } else {                                               // the partial tile in accumulator order, see splitk.hpp
        f32x4 *dst = reinterpret_cast<f32x4 *>(out) +
                     (int64_t(split) * (nb_count * mb_count) + (mb * nb_count + nb)) * (C::BM * C::BN / 4) + threadIdx.x;
#pragma unroll
        for (int i = 0; i < C::FM; ++i)
#pragma unroll
            for (int j = 0; j < C::FN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    dst[((i * C::FN + j) * 4 + q) * C::NTHREADS] =
                        f32x4{acc[i][j][q * 4], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]};
    }
}

// SHORT (ALONG_TOKENS): both operands lie within reach of 32-bit byte offsets, so they are read through buffer descriptors:
// what is outside -- padding, a token past the last -- is an offset past the descriptor's end, which reads as zero, and an
// element takes seven vector instructions instead of some twenty with a branch around the load; where a thread has eight
// columns, what it needs to know of them stays in registers (three LDS reads per element otherwise, on an LDS that the tiles
// keep busy).  Rows and columns past the last of dW fetch whatever is there: those sums are not stored.  Whole calls, the same bits:
// fp32 3x3 32 x 64 x 32 x 32 -> 64 58.5 -> 44.9 us, 64 x 64 x 56 x 56 -> 64 245 -> 182, 36 x 232 x 40 x 22 -> 144 409 -> 298;
// bf16 with 129 output channels, 3x3 / stride 2 over 16 x 64 x 56 x 56 86 -> 52.
template <typename RAW, typename C, Fetch FA, Fetch FB, bool SHORT = false>
__global__ void __launch_bounds__(256)
exact_gemm_kernel(const RAW *__restrict__ dY, const RAW *__restrict__ x, int64_t ntok, int M, int N, int nb_count,
                  int mb_count, int nkb, int splits, ExactGeometry g, float *__restrict__ out)
{
    constexpr int BM = C::BM, BN = C::BN, BK = C::BK, NT = C::NTHREADS;
    constexpr bool CONV = FB == ALONG_TOKENS || FB == ALONG_COLUMNS;
    static_assert(sizeof(RAW) == 4 || (FA != ROWS16 && FB != ROWS16), "16-byte fetches are for fp32");
    __shared__ __attribute__((aligned(16))) float sA[BK * C::PA];
    __shared__ __attribute__((aligned(16))) float sB[BK * C::PB];
    __shared__ uint32_t col_off[CONV ? BN : 1], col_y[CONV ? BN : 1], col_x[CONV ? BN : 1];   // of a column: offset of (c, u, v), u * dh, v * dw
    __shared__ uint32_t tok_off[FB == ALONG_COLUMNS ? 2 : 1][BK];                             // of a token: offset of (n, iy0, ix0)
    __shared__ uint32_t tok_y[FB == ALONG_COLUMNS ? 2 : 1][BK], tok_x[FB == ALONG_COLUMNS ? 2 : 1][BK];
    __shared__ uint32_t not_finite[2];                             // bit r: the tile of dY of an even / odd step holds an infinity or NaN for its token r
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;

    // workgroups of one XCD (dealt round-robin) get consecutive tiles: they share operand rows in its L2
    const int total = nb_count * mb_count * splits;
    const int v = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    if (v >= total) return;
    const int nb = v % nb_count, mb = (v / nb_count) % mb_count, split = v / (nb_count * mb_count);
    const int m0 = mb * BM, n0 = nb * BN;
    const int kb_begin = int(int64_t(nkb) * split / splits), kb_end = int(int64_t(nkb) * (split + 1) / splits);

    if constexpr (CONV) {
        for (int q = tid; q < BN; q += NT) {
            const uint32_t col = uint32_t(n0 + q);
            uint32_t c, tap;
            if (FB == ALONG_TOKENS) {              // (channel, tap)
                c = col / g.taps;
                tap = col - c * g.taps;
            } else {                               // (tap, channel)
                tap = col / g.C;
                c = col - tap * g.C;
            }
            const uint32_t u = tap / g.kw, vv = tap - u * g.kw;
            col_y[q] = u * g.dh;
            col_x[q] = vv * g.dw;
            col_off[q] = c * g.xc + u * g.dh * g.xh + vv * g.dw * g.xw;    // modulo 2^32, like the addresses below
        }
    }
    // image and position of a token
    auto locate = [&](int64_t t, uint32_t &n, uint32_t &p) {
        if (ntok <= INT32_MAX) {                   // uniform
            n = quotient(uint32_t(t), g.by_P);
            p = uint32_t(t) - n * g.P;
        } else {
            n = uint32_t(t / g.P);
            p = uint32_t(t - int64_t(n) * g.P);
        }
    };
    // top-left input position of a token's window, as 32-bit words modulo 2^32 (a row or column is inside the
    // tensor iff the word is below H or W: sizes are below 2^31, padding and taps far below 2^31)
    auto window = [&](uint32_t p, uint32_t &iy0, uint32_t &ix0) {
        const uint32_t oy = quotient(p, g.by_OW), ox = p - oy * g.OW;
        iy0 = oy * g.sh - g.ph;
        ix0 = ox * g.sw - g.pw;
    };
    auto fill_tokens = [&](int kb) __attribute__((always_inline)) {   // ALONG_COLUMNS: the step's token table
        if (FB == ALONG_COLUMNS && tid < BK) {
            const int64_t t = int64_t(kb) * BK + tid;
            uint32_t iy0 = 0x80000000u, ix0 = 0;   // past the last token: below no H
            uint32_t off = 0;
            if (t < ntok) {
                uint32_t n, p;
                locate(t, n, p);
                window(p, iy0, ix0);
                off = n * uint32_t(g.xn) + iy0 * g.xh + ix0 * g.xw;
            }
            tok_off[kb & 1][tid] = off;
            tok_y[kb & 1][tid] = iy0;
            tok_x[kb & 1][tid] = ix0;
        }
    };

    // ---- operand fetch: a step's tiles into registers, and from there into LDS ------------------------------
    constexpr int EA = BM * BK / NT, EB = BN * BK / NT;    // elements per thread
    float ra[EA], rb[EB];
    static_assert(!SHORT || (FA == ALONG_TOKENS && FB == ALONG_TOKENS), "the form of NCHW operands");
    constexpr bool HOIST = SHORT && EB <= 8;
    uint32_t my_off[HOIST ? EB : 1], my_y[HOIST ? EB : 1], my_x[HOIST ? EB : 1];
    (void)my_off; (void)my_y; (void)my_x;
    auto short_load = [](const RAW *base, uint32_t bytes, uint32_t offset) -> float {
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<RAW *>(base), 0, int(bytes), 0x00020000);
        if constexpr (sizeof(RAW) == 4) return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, int(offset), 0, 0));
        else return widen(uint16_t(__builtin_amdgcn_raw_buffer_load_b16(rsrc, int(offset), 0, 0)));
    };
    auto fetch = [&](int kb) __attribute__((always_inline)) {   // (two callers)
        const int64_t t0 = int64_t(kb) * BK;
        if constexpr (SHORT) {
            constexpr uint32_t S = sizeof(RAW);
            constexpr int QSTEP = NT / BK;
            const int r = tid % BK, q0 = tid / BK;
            const uint32_t t = uint32_t(t0) + uint32_t(r);
            const bool tok_ok = t < uint32_t(ntok);
            uint32_t n, p, iy0, ix0;
            locate(int64_t(tok_ok ? t : 0u), n, p);
            window(p, iy0, ix0);
            if (!tok_ok) iy0 = 0x80000000u;                // below no H
            uint32_t ya = (n * uint32_t(g.yn) + p + uint32_t(m0 + q0) * g.P) * S;
#pragma unroll
            for (int u = 0; u < EA; ++u) {
                ra[u] = short_load(dY, g.y_bytes, tok_ok ? ya : 0xFFFFFFFFu);
                ya += uint32_t(QSTEP) * g.P * S;
            }
            const uint32_t base = (n * uint32_t(g.xn) + iy0 * g.xh + ix0 * g.xw) * S;
#pragma unroll
            for (int u = 0; u < EB; ++u) {
                const int q = q0 + u * QSTEP;
                const uint32_t off = HOIST ? my_off[HOIST ? u : 0] : col_off[q] * S;
                const uint32_t iy = iy0 + (HOIST ? my_y[HOIST ? u : 0] : col_y[q]), ix = ix0 + (HOIST ? my_x[HOIST ? u : 0] : col_x[q]);
                rb[u] = short_load(x, g.x_bytes, iy < g.H && ix < g.W ? base + off : 0xFFFFFFFFu);
            }
            return;
        }
        if constexpr (FA == ROWS16) {                      // M % 4 == 0
#pragma unroll
            for (int u = 0; u < EA / 4; ++u) {
                const int i = tid + u * NT, r = i / (BM / 4), q = (i % (BM / 4)) * 4;
                f32x4 w = {0.f, 0.f, 0.f, 0.f};
                if (t0 + r < ntok && m0 + q < M) w = *reinterpret_cast<const f32x4 *>(dY + (t0 + r) * M + m0 + q);
#pragma unroll
                for (int e = 0; e < 4; ++e) ra[u * 4 + e] = w[e];
            }
        } else if constexpr (FA == ROWS1) {
#pragma unroll
            for (int u = 0; u < EA; ++u) {
                const int i = tid + u * NT, r = i / BM, q = i % BM;
                ra[u] = (t0 + r < ntok && m0 + q < M) ? widen(dY[(t0 + r) * M + m0 + q]) : 0.f;
            }
        }
        if constexpr (FB == ROWS16) {                      // N % 4 == 0
#pragma unroll
            for (int u = 0; u < EB / 4; ++u) {
                const int i = tid + u * NT, r = i / (BN / 4), q = (i % (BN / 4)) * 4;
                f32x4 w = {0.f, 0.f, 0.f, 0.f};
                if (t0 + r < ntok && n0 + q < N) w = *reinterpret_cast<const f32x4 *>(x + (t0 + r) * N + n0 + q);
#pragma unroll
                for (int e = 0; e < 4; ++e) rb[u * 4 + e] = w[e];
            }
        } else if constexpr (FB == ROWS1) {
#pragma unroll
            for (int u = 0; u < EB; ++u) {
                const int i = tid + u * NT, r = i / BN, q = i % BN;
                rb[u] = (t0 + r < ntok && n0 + q < N) ? widen(x[(t0 + r) * N + n0 + q]) : 0.f;
            }
        } else if constexpr (FB == ALONG_COLUMNS) {
            constexpr int RSTEP = NT / BN;
            const int q = tid % BN;
            const uint32_t off = col_off[q], cy = col_y[q], cx = col_x[q];
            const bool col_ok = n0 + q < N;
#pragma unroll
            for (int u = 0; u < EB; ++u) {
                const int r = tid / BN + u * RSTEP;
                const uint32_t iy = tok_y[kb & 1][r] + cy, ix = tok_x[kb & 1][r] + cx;
                const bool ok = col_ok && iy < g.H && ix < g.W;
                rb[u] = ok ? widen(x[tok_off[kb & 1][r] + off]) : 0.f;
            }
        }
        if constexpr (FA == ALONG_TOKENS || FB == ALONG_TOKENS) {
            const int r = tid % BK, q0 = tid / BK;
            constexpr int QSTEP = NT / BK;
            const int64_t t = t0 + r;
            const bool tok_ok = t < ntok;
            uint32_t n = 0, p = 0, iy0 = 0x80000000u, ix0 = 0;
            if (tok_ok) locate(t, n, p);
            if constexpr (FA == ALONG_TOKENS) {
                const RAW *yp = dY + int64_t(n) * g.yn + p;
#pragma unroll
                for (int u = 0; u < EA; ++u) {
                    const int q = m0 + q0 + u * QSTEP;
                    ra[u] = (tok_ok && q < M) ? widen(yp[int64_t(q) * g.P]) : 0.f;
                }
            }
            if constexpr (FB == ALONG_TOKENS) {
                if (tok_ok) window(p, iy0, ix0);
                // R(a^) has fewer than 2^31 elements: its offsets are 32-bit, intermediate values may wrap
                const uint32_t base = n * uint32_t(g.xn) + iy0 * g.xh + ix0 * g.xw;
#pragma unroll
                for (int u = 0; u < EB; ++u) {
                    const int q = q0 + u * QSTEP;
                    const uint32_t iy = iy0 + col_y[q], ix = ix0 + col_x[q];
                    const bool ok = tok_ok && n0 + q < N && iy < g.H && ix < g.W;
                    rb[u] = ok ? widen(x[base + col_off[q]]) : 0.f;
                }
            }
        }
    };
    auto row_a = [&](int u) {                              // token of this thread's element u of the dY tile
        return FA == ALONG_TOKENS ? tid % BK : FA == ROWS16 ? (tid + u / 4 * NT) / (BM / 4) : (tid + u * NT) / BM;
    };
    auto note_not_finite = [&](int kb) {
#pragma unroll
        for (int u = 0; u < EA; ++u)
            if ((__float_as_uint(ra[u]) & 0x7fffffffu) >= 0x7f800000u && (!SHORT || m0 + tid / BK + u * (NT / BK) < M))
                atomicOr(&not_finite[kb & 1], 1u << row_a(u));
    };
    auto store = [&]() __attribute__((always_inline)) {
        if constexpr (FA == ROWS16) {
#pragma unroll
            for (int u = 0; u < EA / 4; ++u) {
                const int i = tid + u * NT, r = i / (BM / 4), q = (i % (BM / 4)) * 4;
                *reinterpret_cast<f32x4 *>(sA + r * C::PA + q) = f32x4{ra[u * 4], ra[u * 4 + 1], ra[u * 4 + 2], ra[u * 4 + 3]};
            }
        } else {
#pragma unroll
            for (int u = 0; u < EA; ++u) {
                const int q = FA == ALONG_TOKENS ? tid / BK + u * (NT / BK) : (tid + u * NT) % BM;
                sA[row_a(u) * C::PA + q] = ra[u];
            }
        }
        if constexpr (FB == ROWS16) {
#pragma unroll
            for (int u = 0; u < EB / 4; ++u) {
                const int i = tid + u * NT, r = i / (BN / 4), q = (i % (BN / 4)) * 4;
                *reinterpret_cast<f32x4 *>(sB + r * C::PB + q) = f32x4{rb[u * 4], rb[u * 4 + 1], rb[u * 4 + 2], rb[u * 4 + 3]};
            }
        } else {
#pragma unroll
            for (int u = 0; u < EB; ++u) {
                const int r = FB == ALONG_TOKENS ? tid % BK : (tid + u * NT) / BN;
                const int q = FB == ALONG_TOKENS ? tid / BK + u * (NT / BK) : (tid + u * NT) % BN;
                sB[r * C::PB + q] = rb[u];
            }
        }
    };

    f32x16 acc[C::FM][C::FN];
    // a 32x32x2 operand wants, in lane l, row (or column) l % 32 and k = l / 32
    const float *pa = sA + (lane >> 5) * C::PA + wm * C::WM + (lane & 31);
    const float *pb = sB + (lane >> 5) * C::PB + wn * C::WN + (lane & 31);
    // The tokens of `skip` into the sums, window position by window position, and out of the tiles.
    auto take_out = [&](int kb, uint32_t skip) {
        for (uint32_t left = skip; left != 0; left &= left - 1) {
            const int r = __builtin_ctz(left);
            uint32_t n, p, iy0, ix0;
            locate(int64_t(kb) * BK + r, n, p);            // (a token past the last has dY = 0)
            window(p, iy0, ix0);
#pragma unroll
            for (int j = 0; j < C::FN; ++j) {
                const int q = wn * C::WN + j * 32 + (lane & 31);
                const float xv = sB[r * C::PB + q];
                const bool inside = iy0 + col_y[q] < g.H && ix0 + col_x[q] < g.W;
#pragma unroll
                for (int i = 0; i < C::FM; ++i)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const float yv = sA[r * C::PA + wm * C::WM + i * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3)];
                        if (inside) acc[i][j][e] = __builtin_fmaf(yv, xv, acc[i][j][e]);
                        __builtin_amdgcn_sched_barrier(0);  // (one value at a time: this path must not cost the other its registers)
                    }
            }
        }
        __syncthreads();
        for (uint32_t left = skip; left != 0; left &= left - 1) {
            const int r = __builtin_ctz(left);
            for (int q = tid; q < BM; q += NT) sA[r * C::PA + q] = 0.f;
            for (int q = tid; q < BN; q += NT) sB[r * C::PB + q] = 0.f;
        }
        __syncthreads();
    };
    // The slice's product.  CAREFUL: with the tokens whose dY is not finite taken out of the matrix instructions.
    auto accumulate = [&](auto careful_) {
        constexpr bool CAREFUL = decltype(careful_)::value;
#pragma unroll
        for (int i = 0; i < C::FM; ++i)
#pragma unroll
            for (int j = 0; j < C::FN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
        fill_tokens(kb_begin);
        if (CAREFUL && tid < 2) not_finite[tid] = 0;
        __syncthreads();                                   // column and token tables
        if constexpr (HOIST) {
#pragma unroll
            for (int u = 0; u < EB; ++u) {
                const int q = tid / BK + u * (NT / BK);
                my_off[u] = col_off[q] * uint32_t(sizeof(RAW));
                my_y[u] = col_y[q];
                my_x[u] = col_x[q];
            }
        }
        if (!CAREFUL && kb_begin < kb_end) fetch(kb_begin);
        for (int kb = kb_begin; kb < kb_end; ++kb) {
            if constexpr (CAREFUL) {                       // (not a step ahead: take_out has the registers)
                fetch(kb);
                note_not_finite(kb);
            }
            __syncthreads();                               // the previous step's tiles have been read
            store();
            if (CAREFUL && tid == 0) not_finite[(kb + 1) & 1] = 0;
            if (kb + 1 < kb_end) fill_tokens(kb + 1);
            __syncthreads();
            if (!CAREFUL && kb + 1 < kb_end) fetch(kb + 1);
            if constexpr (CAREFUL)
                if (const uint32_t skip = __builtin_amdgcn_readfirstlane(not_finite[kb & 1]); skip != 0) take_out(kb, skip);
#pragma unroll
            for (int kk = 0; kk < BK / 2; ++kk) {
                float a[C::FM], b[C::FN];
#pragma unroll
                for (int i = 0; i < C::FM; ++i) a[i] = pa[kk * 2 * C::PA + i * 32];
#pragma unroll
                for (int j = 0; j < C::FN; ++j) b[j] = pb[kk * 2 * C::PB + j * 32];
#pragma unroll
                for (int i = 0; i < C::FM; ++i)
#pragma unroll
                    for (int j = 0; j < C::FN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
            }
        }
    };
    accumulate(std::false_type{});
    if constexpr (CONV) {
        if ((g.ph | g.pw) != 0) {                          // uniform
            float z = 0.f;
            auto look = [&](auto inside) {
#pragma unroll
                for (int i = 0; i < C::FM; ++i)
#pragma unroll
                    for (int j = 0; j < C::FN; ++j)
#pragma unroll
                        for (int e = 0; e < 16; ++e) z = __builtin_fmaf(inside(i, j, e) ? acc[i][j][e] : 0.f, 0.f, z);
            };
            if (SHORT && (m0 + BM > M || n0 + BN > N))     // uniform; what lies past dW holds other images' sums
                look([&](int i, int j, int e) {
                    return m0 + wm * C::WM + i * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3) < M &&
                           n0 + wn * C::WN + j * 32 + (lane & 31) < N;
                });
            else look([](int, int, int) { return true; });
            if (__syncthreads_or(!(z == 0.f))) accumulate(std::true_type{});
        }
    }

    exact_epilogue<C>(acc, splits, split, nb_count, mb_count, nb, mb, M, N, out);
}

// ---- fp32 products from bf16 thirds -----------------------------------------------------------------
// A fp32 number is the sum of three bf16 numbers, 8 significand bits each (a = a1 + a2 + a3, every difference exact; a2 is at
// most 2^-8, a3 2^-17 of a), so a product of two is the sum of nine bf16 products, exact in fp32.  All but a3 b3, at most
// 2^-34 of |a b|, are summed: 256 cycles of the bf16 matrix instructions for 16 tokens of a 32 x 32 block, where the fp32
// instruction takes 512.  (Without a2 b3 and a3 b2, 2^-24 of |a b| between them, the call below takes 66 us, and a sum of one
// term is off by up to 1.15e-7 of itself instead of the 6e-8 that rounding it takes.)  a1 b1 has sums of its own, so that they
// are rounded once per 16 tokens and not eight times (against 64 bits, 6304 tokens, gamma 0.9: 0.8e-7 in the 2-norm; the
// fp32 instruction 1.4e-7; six products in one set of sums 2.4e-7).
// The thirds are made on the way from the fetch to LDS (five vector instructions per element, beside the other workgroup's
// matrix instructions) and lie there as [third][column][32 tokens], so that an operand is one 16-byte read; the 16-byte unit o
// of column c is kept at o ^ swizzle(c), which spreads the reads (consecutive columns, one o) and the stores over the banks.
// Two workgroups per compute unit, one converting while the other multiplies.  Whole call, fp32 instruction -> this:
// 6304 x 384 -> 1536 86 -> 72 us, 6304 x 1536 -> 384 94 -> 81, 2048 x 1024 -> 1024 56 -> 50, 700 x 1024 -> 1024 36 -> 34.5;
// 120 random layers 0.73 to 0.98 of the time.  (With six products, two LDS stages and one 256 x 128 workgroup of eight
// wavefronts took 10 % more, loads of four bytes instead of eight 15 %.)
// What the thirds cannot carry shows in the sums and in the smallest elements: an infinity, a NaN, or a value that rounds to
// infinity in bf16 makes a sum not finite; and where the last third of a value is below the normal numbers (2^-126, taken as
// lost here), or a product of parts below the subnormal ones, a sum of n terms is off by n 2^-126 of the other operand's
// largest value, n 2^-146 for the products.  A workgroup with a sum that is not finite, or so small that this would be 2^-25
// of it, does its slice again with the fp32 instruction.  A sum that is exactly zero is most often one of no terms at all; it
// counts as small where an element of the tiles but zero is below 2^-103, whose last third may be lost (below 2^-134 all
// three are), or the product of the smallest two is, whose parts' products may be.
constexpr int SPLIT_BM = 128, SPLIT_BN = 128;

__device__ inline void split_thirds(float a, float b, uint32_t &p1, uint32_t &p2, uint32_t &p3)      // a in the lower halves
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    auto pack = [](float lo, float hi) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2)); };
    p1 = pack(a, b);
    a -= __uint_as_float(p1 << 16);
    b -= __uint_as_float(p1 & 0xFFFF0000u);
    p2 = pack(a, b);
    a -= __uint_as_float(p2 << 16);
    b -= __uint_as_float(p2 & 0xFFFF0000u);
    p3 = pack(a, b);
}

// largest over the 64 lanes, in every lane
__device__ inline uint32_t wave_max(uint32_t v)
{
#define DROPIT_DPP_MAX(ctrl, row_mask) v = max(v, uint32_t(__builtin_amdgcn_update_dpp(int(v), int(v), ctrl, row_mask, 0xf, false)))
    DROPIT_DPP_MAX(0x111, 0xf);   // row_shr:1, 2, 4, 8
    DROPIT_DPP_MAX(0x112, 0xf);
    DROPIT_DPP_MAX(0x114, 0xf);
    DROPIT_DPP_MAX(0x118, 0xf);
    DROPIT_DPP_MAX(0x142, 0xa);   // row_bcast:15, 31
    DROPIT_DPP_MAX(0x143, 0xc);
#undef DROPIT_DPP_MAX
    return uint32_t(__builtin_amdgcn_readlane(int(v), WAVE - 1));
}

__global__ void __launch_bounds__(256, 2)
exact_split_kernel(const float *__restrict__ dY, const float *__restrict__ x, int64_t ntok, int M, int N, int nb_count,
                   int mb_count, int nkb, int splits, float *__restrict__ out)
{
    typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    using C = ExactCfg<SPLIT_BM, SPLIT_BN>;
    constexpr int BM = C::BM, BN = C::BN, BK = C::BK, THIRD = BM * BK * 2;      // bytes of a third of an operand tile
    static_assert(BM == BN && BK == 32 && C::NTHREADS == 256 && C::WM == 64 && C::WN == 64, "a wavefront per 8 tokens, two columns per lane");
    __shared__ __attribute__((aligned(16))) char lds[6 * THIRD];
    static_assert(6 * THIRD >= BK * (C::PA + C::PB) * 4, "the fp32 tiles of the other form");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;
    const int total = nb_count * mb_count * splits;
    const int v = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;          // (workgroups of one XCD share operand rows in its L2)
    if (v >= total) return;
    const int nb = v % nb_count, mb = (v / nb_count) % mb_count, split = v / (nb_count * mb_count);
    const int m0 = mb * BM, n0 = nb * BN;
    const int kb_begin = int(int64_t(nkb) * split / splits), kb_end = int(int64_t(nkb) * (split + 1) / splits);
    f32x16 acc[C::FM][C::FN], small[C::FM][C::FN];         // a1 b1, and the others
    auto clear = [&](f32x16 (&s)[C::FM][C::FN]) {
#pragma unroll
        for (int i = 0; i < C::FM; ++i)
#pragma unroll
            for (int j = 0; j < C::FN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) s[i][j][e] = 0.f;
    };

    // a step's tiles: lane = two columns, wavefront = 8 tokens, of dY and of R(a^)
    f32x2 ra[8], rb[8];
    // (columns past the last re-read the last two, those sums are not stored; tokens past the last are zero)
    const int q = lane * 2;
    int qm = min(m0 + q, M - 2), qn = min(n0 + q, N - 2);                       // M and N are even
    auto fetch = [&](int kb) {
        const int64_t t = int64_t(kb) * BK + wave * 8;
        const float *pa = dY + t * M + qm, *pb = x + t * N + qn;
        if (t + 8 <= ntok) {                                                    // uniform
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                ra[r] = *reinterpret_cast<const f32x2 *>(pa + int64_t(r) * M);
                rb[r] = *reinterpret_cast<const f32x2 *>(pb + int64_t(r) * N);
            }
        } else {
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                ra[r] = rb[r] = f32x2{0.f, 0.f};
                if (t + r < ntok) {
                    ra[r] = *reinterpret_cast<const f32x2 *>(pa + int64_t(r) * M);
                    rb[r] = *reinterpret_cast<const f32x2 *>(pb + int64_t(r) * N);
                }
            }
        }
    };
    auto unit = [](int c, int o) { return c * 64 + ((o ^ c ^ (c >> 2)) & 3) * 16; };      // of column c, tokens 8 o .. 8 o + 7
    float most_a = 0.f, most_b = 0.f;                                           // largest magnitudes of this thread's elements
    auto larger = [](float a, float b, float m) {
        asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(a), "v"(b));
        return m;
    };
    uint32_t least_a = ~0u, least_b = ~0u;                                      // smallest ones but zero: twice the bits less one
    auto smaller = [](float a, float b, uint32_t m) {
        return min(min(m, (__float_as_uint(a) << 1) - 1u), (__float_as_uint(b) << 1) - 1u);
    };
    auto store = [&]() {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            most_a = larger(ra[r][0], ra[r][1], most_a);
            most_b = larger(rb[r][0], rb[r][1], most_b);
            least_a = smaller(ra[r][0], ra[r][1], least_a);
            least_b = smaller(rb[r][0], rb[r][1], least_b);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {                                           // dY, R(a^)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                u32x4 third[3];
#pragma unroll
                for (int r = 0; r < 8; r += 2) {
                    uint32_t p1, p2, p3;
                    if (h == 0) split_thirds(ra[r][c], ra[r + 1][c], p1, p2, p3);
                    else split_thirds(rb[r][c], rb[r + 1][c], p1, p2, p3);
                    third[0][r / 2] = p1;
                    third[1][r / 2] = p2;
                    third[2][r / 2] = p3;
                }
#pragma unroll
                for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x4 *>(lds + (h * 3 + p) * THIRD + unit(q + c, wave)) = third[p];
            }
        }
    };
    clear(acc);
    clear(small);
    if (kb_begin < kb_end) fetch(kb_begin);
    for (int kb = kb_begin; kb < kb_end; ++kb) {
        __syncthreads();                                                        // the previous step's tiles have been read
        store();
        __syncthreads();
        if (kb + 1 < kb_end) fetch(kb + 1);
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            bf16x8 a[3][C::FM], b[3][C::FN];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
#pragma unroll
                for (int i = 0; i < C::FM; ++i)
                    a[p][i] = *reinterpret_cast<const bf16x8 *>(lds + p * THIRD + unit(wm * C::WM + i * 32 + (lane & 31), kk * 2 + (lane >> 5)));
#pragma unroll
                for (int j = 0; j < C::FN; ++j)
                    b[p][j] = *reinterpret_cast<const bf16x8 *>(lds + (3 + p) * THIRD + unit(wn * C::WN + j * 32 + (lane & 31), kk * 2 + (lane >> 5)));
            }
            constexpr int PA[8] = {2, 1, 2, 0, 1, 1, 0, 0}, PB[8] = {1, 2, 0, 2, 1, 0, 1, 0};     // small ones first
#pragma unroll
            for (int p = 0; p < 8; ++p)
#pragma unroll
                for (int i = 0; i < C::FM; ++i)
#pragma unroll
                    for (int j = 0; j < C::FN; ++j) {
                        f32x16 &s = p == 7 ? acc[i][j] : small[i][j];
                        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[PA[p]][i], b[PB[p]][j], s, 0, 0, 0);
                    }
        }
    }
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
        for (int j = 0; j < C::FN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] += small[i][j][e];
    // Does a sum need the fp32 instruction?  The extremes of the elements and of the sums, over the workgroup
    uint32_t most_s = 0u, least_s = ~0u, zeros = ~0u;
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
        for (int j = 0; j < C::FN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const uint32_t twice = __float_as_uint(acc[i][j][e]) << 1;
                most_s = max(most_s, twice);
                least_s = min(least_s, twice - 1u);
                zeros = min(zeros, twice);
            }
    __shared__ __attribute__((aligned(16))) uint32_t extremes[4][8];            // the largest of each, a row per wavefront
    {
        // (a NaN element is not the largest; it is in the sums)
        const uint32_t mine[7] = {__float_as_uint(most_a), __float_as_uint(most_b), ~least_a, ~least_b, most_s, ~least_s, ~zeros};
#pragma unroll
        for (int h = 0; h < 7; ++h) {
            const uint32_t m = wave_max(mine[h]);
            if (lane == 0) extremes[wave][h] = m;
        }
    }
    __syncthreads();
    uint32_t most[7];
#pragma unroll
    for (int h = 0; h < 7; ++h) most[h] = max(max(extremes[0][h], extremes[1][h]), max(extremes[2][h], extremes[3][h]));
    // (of elements and sums but zeros: infinity if there are none)
    auto smallest = [](uint32_t inverted) { return inverted == 0u ? __builtin_inff() : __uint_as_float((~inverted >> 1) + 1u); };
    const float least_y = smallest(most[2]), least_x = smallest(most[3]);
    const bool tiny = least_y < 0x1p-103f || least_x < 0x1p-103f || least_y * least_x < 0x1p-103f;
    // n 2^-126 of the operands, n 2^-146 of the products, times 2^25
    const float lost = float((kb_end - kb_begin) * BK) * (0x1p-101f * (__uint_as_float(most[0]) + __uint_as_float(most[1])) + 0x1p-121f);
    if (most[4] >= 0xFF000000u || smallest(most[5]) < lost || (tiny && most[6] == ~0u)) {      // uniform
        float *sA = reinterpret_cast<float *>(lds), *sB = sA + BK * C::PA;
        clear(acc);
        int again = q;
        asm volatile("" : "+v"(again));                                          // (no addresses kept for this through the other loop)
        qm = min(m0 + again, M - 2);
        qn = min(n0 + again, N - 2);
        for (int kb = kb_begin; kb < kb_end; ++kb) {
            fetch(kb);
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                *reinterpret_cast<f32x2 *>(sA + (wave * 8 + r) * C::PA + q) = ra[r];
                *reinterpret_cast<f32x2 *>(sB + (wave * 8 + r) * C::PB + q) = rb[r];
            }
            __syncthreads();
#pragma unroll 1
            for (int kk = 0; kk < BK / 2; ++kk)
#pragma unroll
                for (int i = 0; i < C::FM; ++i)
#pragma unroll
                    for (int j = 0; j < C::FN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(sA[(kk * 2 + (lane >> 5)) * C::PA + wm * C::WM + i * 32 + (lane & 31)],
                                                                         sB[(kk * 2 + (lane >> 5)) * C::PB + wn * C::WN + j * 32 + (lane & 31)],
                                                                         acc[i][j], 0, 0, 0);
        }
    }
    exact_epilogue<C>(acc, splits, split, nb_count, mb_count, nb, mb, M, N, out);
}

constexpr int EXACT_TILE_BYTES = 32 * 1024;                // of R(a^), per recover workgroup, at most

template <typename RAW, typename C>
dropit_status launch_exact(const ExactProblem &p, const ExactPlan &plan, const RAW *dY, const RAW *x, float *partial,
                           float *dW, hipStream_t stream)
{
    const int total = plan.nb_count * plan.mb_count * plan.splits;
    const int grid = (total + 7) / 8 * 8;
    float *out = plan.splits > 1 ? partial : dW;
    ExactGeometry g = {};
    if (p.conv) {
        const int64_t taps = p.g.kh * p.g.kw;
        g = ExactGeometry{uint32_t(p.OW), uint32_t(p.OH * p.OW), uint32_t(p.W), uint32_t(p.H), uint32_t(p.C), uint32_t(taps),
                          uint32_t(p.g.kw), uint32_t(p.g.stride_h), uint32_t(p.g.stride_w), uint32_t(p.g.pad_h),
                          uint32_t(p.g.pad_w), uint32_t(p.g.dil_h), uint32_t(p.g.dil_w),
                          p.nhwc ? 1u : uint32_t(p.H * p.W), p.nhwc ? uint32_t(p.W * p.C) : uint32_t(p.W),
                          p.nhwc ? uint32_t(p.C) : 1u, p.C * p.H * p.W, p.cout * p.OH * p.OW,
                          divisor(uint32_t(p.OH * p.OW)), divisor(uint32_t(p.OW)), 0u, 0u};
        const int64_t xb = p.numel * int64_t(sizeof(RAW)), yb = p.ntok * p.cout * int64_t(sizeof(RAW));
        // (Rows past the last and columns past the last add planes to an offset: it may pass the end or wrap around, and fetch
        // zeros or anything of the operand.  The descriptor bounds it, and those sums are neither stored nor looked at.)
        constexpr int64_t REACH = int64_t(1) << 31;
        if (xb < REACH && yb < REACH && !dev_env("DROPIT_EXACT_LONG", 0)) {
            g.x_bytes = uint32_t(xb);
            g.y_bytes = uint32_t(yb);
        }
    }
    auto go = [&](auto kernel) {
        kernel<<<grid, C::NTHREADS, 0, stream>>>(dY, x, p.ntok, int(p.cout), int(p.cin), plan.nb_count, plan.mb_count,
                                                 plan.nkb, plan.splits, g, out);
    };
    const bool wide_y = p.cout % 4 == 0, wide_x = p.cin % 4 == 0;      // 16-byte rows
    if constexpr (sizeof(RAW) == 4) {
        if (!p.conv) {
            if (wide_y && wide_x && C::BM == SPLIT_BM && !dev_env("DROPIT_EXACT_FMA", 0))
                exact_split_kernel<<<grid, 256, 0, stream>>>(reinterpret_cast<const float *>(dY), reinterpret_cast<const float *>(x),
                                                             p.ntok, int(p.cout), int(p.cin), plan.nb_count, plan.mb_count,
                                                             plan.nkb, plan.splits, out);
            else if (wide_y && wide_x) go(exact_gemm_kernel<RAW, C, ROWS16, ROWS16>);
            else go(exact_gemm_kernel<RAW, C, ROWS1, ROWS1>);
        } else if (!p.nhwc && g.x_bytes) go(exact_gemm_kernel<RAW, C, ALONG_TOKENS, ALONG_TOKENS, true>);
        else if (!p.nhwc) go(exact_gemm_kernel<RAW, C, ALONG_TOKENS, ALONG_TOKENS>);
        else if (wide_y) go(exact_gemm_kernel<RAW, C, ROWS16, ALONG_COLUMNS>);
        else go(exact_gemm_kernel<RAW, C, ROWS1, ALONG_COLUMNS>);
    } else {
        if (!p.conv) go(exact_gemm_kernel<RAW, C, ROWS1, ROWS1>);
        else if (!p.nhwc && g.x_bytes) go(exact_gemm_kernel<RAW, C, ALONG_TOKENS, ALONG_TOKENS, true>);
        else if (!p.nhwc) go(exact_gemm_kernel<RAW, C, ALONG_TOKENS, ALONG_TOKENS>);
        else go(exact_gemm_kernel<RAW, C, ROWS1, ALONG_COLUMNS>);
    }
    if (plan.splits > 1)
        launch_splitk_sum<C>(partial, plan.splits, int(p.cout), int(p.cin), plan.nb_count, plan.mb_count, dW, stream);
    trace_mark(stream);
    return launch_status();
}

template <typename RAW>
dropit_status run_exact(const ExactProblem &p, const ExactPlan &plan, const void *vals, const int32_t *idx, const void *dY,
                        float *dW, char *ws, hipStream_t stream)
{
    RAW *x = reinterpret_cast<RAW *>(ws);
    float *partial = reinterpret_cast<float *>(ws + plan.dense_bytes);
    trace_mark(stream);
    const int64_t rows = (p.numel + plan.tile - 1) / plan.tile;   // R(a^) as rows of a tile each, the last one not full
    launch_recover<RAW>(static_cast<const RAW *>(vals), idx, p.k, p.numel, rows, rows, plan.tile, plan.tile, 1, x, stream);
    trace_mark(stream);
    const RAW *y = static_cast<const RAW *>(dY);
    if (plan.bm == 128) return launch_exact<RAW, ExactCfg<128, 128>>(p, plan, y, x, partial, dW, stream);
    if (plan.bn == 128) return launch_exact<RAW, ExactCfg<64, 128>>(p, plan, y, x, partial, dW, stream);
    return launch_exact<RAW, ExactCfg<64, 64>>(p, plan, y, x, partial, dW, stream);
}

}  // namespace

ExactPlan exact_plan(const ExactProblem &p, bool f32)
{
    ExactPlan plan;
    plan.tile = int(recover_tile(p.numel, EXACT_TILE_BYTES / (f32 ? 4 : 2)));
    plan.dense_bytes = round_up(size_t((p.numel + plan.tile - 1) / plan.tile * plan.tile) * (f32 ? 4 : 2), 256);
    // the tile that pads the result least, the larger one where two pad the same
    plan.bm = plan.bn = 0;
    int64_t least = INT64_MAX;
    const int shapes[3][2] = {{128, 128}, {64, 128}, {64, 64}};
    for (const auto &s : shapes) {
        const int64_t padded = round_up(p.cout, s[0]) * round_up(p.cin, s[1]);
        if (padded < least) {
            least = padded;
            plan.bm = s[0];
            plan.bn = s[1];
        }
    }
    plan.nkb = int((p.ntok + 31) / 32);
    // ... and the smallest where a workgroup per tile and two steps would leave compute units idle: a quarter of the work
    // each (390 tokens, 72 columns, 96 rows: 17.5 us in six workgroups of 128 x 128)
    const int64_t whole = (p.cout + plan.bm - 1) / plan.bm * ((p.cin + plan.bn - 1) / plan.bn);
    if (whole * std::max(plan.nkb / 2, 1) < 256) plan.bm = plan.bn = 64;
    plan.mb_count = int((p.cout + plan.bm - 1) / plan.bm);
    plan.nb_count = int((p.cin + plan.bn - 1) / plan.bn);
    // K-slices: two (128 x 128) to four workgroups per compute unit.  Measured with one / two / three / four: 84 / 81 /
    // 102 / 89 us for 36 tiles of 128 x 128 over 6304 tokens, 91 / 66 / 59 / 56 us for 9 tiles of 64 x 64 over 32768.
    // A slice writes a whole partial tile however little it summed, yet short problems want every compute unit: two
    // 32-token steps per slice at least (435 tokens, 6 tiles of 128 x 128: 15 us with two, 17 with four, 27 with eight),
    // one as long as that makes no more than 256 workgroups (the 28 of 700 small calls that took over 1.2 times the vector
    // kernels' time with two steps were 5 with one; 315 tiles over 41 tokens lost 12 -> 18 us by cutting them).
    const int64_t tiles = int64_t(plan.mb_count) * plan.nb_count;
    const int64_t resident = dev_env("DROPIT_EXACT_WGS", plan.bm * plan.bn >= 128 * 128 ? 512 : 1024);
    const int64_t most = std::max<int64_t>(plan.nkb / 2, std::min<int64_t>(plan.nkb, 256 / std::max<int64_t>(tiles, 1)));
    const int64_t splits = std::min<int64_t>(resident / std::max<int64_t>(tiles, 1), most);
    plan.splits = int(std::max<int64_t>(1, std::min<int64_t>(splits, 256)));
    plan.partial_bytes = plan.splits > 1 ? size_t(plan.splits) * tiles * plan.bm * plan.bn * 4 : 0;
    return plan;
}

dropit_status exact_run(const ExactProblem &p, const ExactPlan &plan, bool f32, const void *vals, const int32_t *idx,
                        const void *dY, float *dW, char *ws, hipStream_t stream)
{
    return f32 ? run_exact<uint32_t>(p, plan, vals, idx, dY, dW, ws, stream)
               : run_exact<uint16_t>(p, plan, vals, idx, dY, dW, ws, stream);
}

}  // namespace dropit
