// Min-k dropping D(a) = {a_Xr, Xr} (Sec. 3.2; Sec. 3.3, min-k strategy; Sec. 4.1)
// as a bandwidth-bound radix select + ordered stream compaction for gfx950.
//
// The magnitude key of an element is its bit pattern with the sign cleared
// (15 bits for bf16, 31 for fp32); unsigned key order == |x| order.
//
// The steps, whichever way they are launched:
//   hist pass : MSB-first digit histogram of the keys that match the digits
//               resolved so far (LDS histogram per workgroup, merged with
//               global atomics), then the digit holding the k-th key is resolved
//   count pass: resolves the last (4/5-bit) digit; every workgroup owns one
//               contiguous chunk of x and records, per chunk, how many keys
//               are above the resolved prefix and a small histogram of the
//               matching ones.  From these follow the threshold key t, the tie
//               budget m = k - #{key > t}, and the exclusive per-chunk offsets
//               of {key > t} and {key == t}.
//   compact   : each workgroup writes the (value, index) pairs of its chunk in
//               ascending index order; of the keys equal to t only the first m
//               by flat index are kept.
// bf16: 11 + 4 bits (one hist pass); fp32: 13 + 13 + 5 bits (two hist passes).
//
// Default: ONE persistent kernel (select_fused_kernel) does all of it with grid
// barriers between the steps, and a serial redo path should the barriers ever give
// up.  It predicts the range of the threshold from a sample and
// stages every element that can still be kept in LDS during its one pass over the
// tensor (see "sampled first digit" and "one read of x" below); the counts are exact,
// so a wrong prediction is noticed and repaired, and the bytes it writes are the same
// either way.  Small tensors take one workgroup.  Alternative: the steps as separate kernels
// (init, hist, count, compact) with a last-workgroup-to-arrive ticket instead of
// barriers.  Nothing here synchronises with the host; counts are integer, so the
// result does not depend on the order in which workgroups run.
//
// Measured, whole call in a queue of calls on rotating inputs, with the earlier form of the persistent kernel (every
// workgroup's exit report behind its output stores; two-level barrier counters; candidates turned through LDS; the whole
// chunk read again where a segment overflowed) -> now:
//   bf16 0.6 M elements 17.7 -> 12.7 us, 3.2 M 22 -> 16.0, 9.7 M 26.3 -> 20.3, 50 M (gamma 0.9) 53.8 -> 44.4,
//   39 M (gamma 0.8) 78.7 -> 48, 51 M (gamma 0.8) 93.6 -> 65.
// fp32, digit histograms of the whole tensor -> sample, staged candidates and the threshold's bin as a list (gamma 0.9):
//   0.07 M elements 24.2 -> 17.5 us, 0.6 M 28.9 -> 19.7, 2.4 M 35.5 -> 21.8, 8.4 M 50.1 -> 29.4, 50 M 166 -> 103.
#include "common.hpp"
#include "wgrad_internal.hpp"
#include "dev_hooks.hpp"
#include <atomic>
#include <cstdlib>
#include <random>
#include <type_traits>

namespace dropit {
namespace {

constexpr int SEL_THREADS = 1024;
constexpr int SEL_MAX_CHUNKS = 512;
constexpr int SEL_UNROLL = 4;
constexpr int MAX_HIST_BITS = 13;
constexpr int MAX_LAST_BINS = 56;       // keys of the range in the per-chunk table: up to seven 8-key bins of a sampled bracket, else 2^LAST_BITS
constexpr int TABLE_PITCH = 64;         // words per chunk in the persistent kernel's table: the range's keys, the keys above it, padding to whole lines

struct SelState {
    uint32_t prefix;     // key digits resolved so far (key >> remaining bits)
    uint32_t k_rem;      // elements still to take among the keys matching prefix
    uint32_t t;          // threshold key (valid after the count pass)
    uint32_t m;          // how many keys equal to t are kept (lowest flat index first)
    uint32_t ticket[4];  // arrival counters, one per pass
    uint32_t form;       // fused kernel, for the tests, 16-bit types at every size: 0 exact digit histograms, 1 sampled bracket confirmed, 2 sampled bracket missed (exact retry)
    uint32_t error;      // hint: some workgroup ran out of patience at a grid barrier (the others stop waiting)
    uint32_t exited;     // fused kernel: low 16 bits = workgroups past their last grid barrier or gone, high 16 bits = how many gave up
    uint32_t path;       // `form` for 16-bit tensors of SAMPLE_LARGE elements or more, 0 below: what readers of this word were told when smaller ones had no sampled form
    unsigned long long ready;    // == the call's generation number once workgroup 0 has cleared the words above and the histograms;
                                 // the last workgroup to leave puts 0 back (no generation is 0), so a launch replayed with
                                 // the same number (a captured graph) waits for its own workgroup 0 again
    uint32_t redo;       // fused kernel, for callers and tests: 1 if the grid barriers gave up and the last workgroup redid the selection alone
    uint32_t staged;     // fused kernel, for the tests: how many workgroups compacted from candidates staged in LDS (one read of x)
    unsigned long long ready_hist;   // 16-bit types: the same for the digit histogram, which only the exact form needs
    uint32_t pad[45];
    uint32_t form32;     // fp32, for the tests: as `form`, + 4 where the threshold's bin went through a histogram and a second table
};
static_assert(sizeof(SelState) == 256, "state block is 256 bytes");
static_assert(MAX_LAST_BINS + 1 <= TABLE_PITCH && TABLE_PITCH == WAVE, "a lane per word of a chunk's line");

// Workspace carving (in bytes from the 256-byte aligned base).
struct SelWorkspace {
    static constexpr size_t state_off = 0;
    static constexpr size_t hist0_off = state_off + sizeof(SelState);
    static constexpr size_t hist1_off = hist0_off + sizeof(uint32_t) * (1u << MAX_HIST_BITS);
    static constexpr size_t table_off = hist1_off + sizeof(uint32_t) * (1u << MAX_HIST_BITS);
    static constexpr size_t offgt_off = table_off + sizeof(uint32_t) * TABLE_PITCH * SEL_MAX_CHUNKS;
    static constexpr size_t offeq_off = offgt_off + sizeof(uint32_t) * SEL_MAX_CHUNKS;
    static constexpr size_t xbar_off = offeq_off + sizeof(uint32_t) * SEL_MAX_CHUNKS;   // 8 arrival counters, 256 B apart
    static constexpr size_t bytes = xbar_off + 8 * 256;
    static constexpr size_t zero_bytes = table_off;   // state + both histograms are cleared per call
};

template <typename RAW> struct KeyTraits;
template <> struct KeyTraits<uint16_t> {
    static constexpr int VEC = 8;
    static constexpr uint32_t MASK = 0x7FFFu;
};
template <> struct KeyTraits<uint32_t> {
    static constexpr int VEC = 4;
    static constexpr uint32_t MASK = 0x7FFFFFFFu;
};

// Calls f(raw_bits, e) for the VEC elements of one 16-byte vector, e ascending.
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;   // plain register vector (no class wrapper)

template <typename V, typename F> __device__ inline void for_each_raw(uint16_t, const V &q, F f)
{
    f(q.x & 0xFFFFu, 0); f(q.x >> 16, 1); f(q.y & 0xFFFFu, 2); f(q.y >> 16, 3);
    f(q.z & 0xFFFFu, 4); f(q.z >> 16, 5); f(q.w & 0xFFFFu, 6); f(q.w >> 16, 7);
}
template <typename V, typename F> __device__ inline void for_each_raw(uint32_t, const V &q, F f)
{
    f(q.x, 0); f(q.y, 1); f(q.z, 2); f(q.w, 3);
}

__global__ void __launch_bounds__(256) init_kernel(uint32_t *ws, uint32_t nwords, uint32_t k)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < nwords; i += gridDim.x * blockDim.x)
        ws[i] = (i == offsetof(SelState, k_rem) / 4) ? k : 0u;
}

// Ticket: true in every thread of exactly one workgroup, the last to arrive.
// The fences make every earlier workgroup's global writes visible to the
// ordinary loads the last workgroup issues afterwards.
__device__ inline bool last_block_to_arrive(uint32_t *ticket)
{
    __shared__ uint32_t s_last;
    __syncthreads();                       // the whole workgroup's global writes are issued
    if (threadIdx.x == 0) {
        __threadfence();                   // release them (one fence per workgroup: it is device-wide)
        const uint32_t t = atomicAdd(ticket, 1u);
        const bool last = t == gridDim.x - 1;
        if (last) __threadfence();         // acquire every other workgroup's writes
        s_last = last ? 1u : 0u;
    }
    __syncthreads();
    return s_last != 0;
}

// One workgroup: find the digit d with  #{digit > d} < k_rem <= #{digit >= d}
// in hist[0..NB), then fold it into the state.
template <int NB, int BITS>
__device__ inline void resolve_digit(const uint32_t *hist, SelState *st, uint32_t *scan /*[SEL_THREADS]*/)
{
    constexpr int PER = (NB + SEL_THREADS - 1) / SEL_THREADS;
    const int tid = threadIdx.x;
    const int lo = tid * PER;
    uint32_t c[PER];
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        c[i] = (lo + i < NB) ? hist[lo + i] : 0u;
        mine += c[i];
    }
    // inclusive suffix sum over threads: scan[tid] = sum of `mine` for threads >= tid
    scan[tid] = mine;
    __syncthreads();
    for (int o = 1; o < SEL_THREADS; o <<= 1) {
        const uint32_t add = (tid + o < SEL_THREADS) ? scan[tid + o] : 0u;
        __syncthreads();
        scan[tid] += add;
        __syncthreads();
    }
    const uint32_t k_rem = st->k_rem;
    const uint32_t prefix = st->prefix;
    uint32_t above = scan[tid] - mine;     // keys with a digit in a higher thread's range
    __syncthreads();                       // every thread has read the state before it changes
    if (above < k_rem && k_rem <= above + mine) {
#pragma unroll
        for (int i = PER - 1; i >= 0; --i) {
            if (above + c[i] >= k_rem) {
                st->prefix = (prefix << BITS) | static_cast<uint32_t>(lo + i);
                st->k_rem = k_rem - above;
                break;
            }
            above += c[i];
        }
    }
}

// Digit histogram of the keys whose higher digits equal the resolved prefix.
// x is walked as `nvf` full 16-byte vectors split into contiguous chunks of
// `vpc` vectors (one per workgroup); the last workgroup also takes the
// numel % VEC ragged elements.  The inner loop is branch-free: a key that does
// not match, or whose digit is 0 (exact zeros are common after ReLU), is
// counted in a per-lane spill slot instead of a shared bin.
template <typename RAW, int SHIFT, int BITS, bool FIRST>
__global__ void __launch_bounds__(SEL_THREADS)
hist_kernel(const RAW *__restrict__ x, int64_t numel, int64_t nvf, int64_t vpc, SelState *st,
            uint32_t *ghist, int pass)
{
    constexpr int VEC = KeyTraits<RAW>::VEC;
    constexpr uint32_t MASK = KeyTraits<RAW>::MASK;
    constexpr int NB = 1 << BITS;
    __shared__ uint32_t lh[NB + 2 * WAVE];
    __shared__ uint32_t scan[SEL_THREADS];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    for (int i = tid; i < NB + 2 * WAVE; i += SEL_THREADS) lh[i] = 0;
    const uint32_t prefix = FIRST ? 0u : st->prefix;
    __syncthreads();

    const uint32_t zslot = NB + lane, dslot = NB + WAVE + lane;
    auto count = [&](uint32_t raw, int) {
        const uint32_t key = raw & MASK;
        const uint32_t d = (key >> SHIFT) & (NB - 1);
        uint32_t a = d ? d : zslot;
        if (!FIRST) a = ((key >> (SHIFT + BITS)) == prefix) ? a : dslot;
        atomicAdd(&lh[a], 1u);
    };
    const uint4 *xv = reinterpret_cast<const uint4 *>(x);
    const int64_t v0 = static_cast<int64_t>(blockIdx.x) * vpc;
    const int64_t v1 = min(v0 + vpc, nvf);
    int64_t vb = v0;
    for (; vb + SEL_THREADS * SEL_UNROLL <= v1; vb += SEL_THREADS * SEL_UNROLL) {
        uint4 q[SEL_UNROLL];
#pragma unroll
        for (int u = 0; u < SEL_UNROLL; ++u) q[u] = xv[vb + u * SEL_THREADS + tid];
#pragma unroll
        for (int u = 0; u < SEL_UNROLL; ++u) for_each_raw(RAW(0), q[u], count);
    }
    for (int64_t v = vb + tid; v < v1; v += SEL_THREADS) for_each_raw(RAW(0), xv[v], count);
    if (blockIdx.x == gridDim.x - 1 && tid == 0)
        for (int64_t i = nvf * VEC; i < numel; ++i) count(x[i], 0);
    __syncthreads();
    if (tid < WAVE) {                      // fold the digit-0 spill slots into bin 0
        const uint32_t z = wave_sum(lh[NB + tid]);
        if (tid == 0) lh[0] += z;
    }
    __syncthreads();
    for (int i = tid; i < NB; i += SEL_THREADS) {
        const uint32_t c = lh[i];
        if (c) atomicAdd(&ghist[i], c);
    }
    if (!last_block_to_arrive(&st->ticket[pass])) return;
    resolve_digit<NB, BITS>(ghist, st, scan);
}

// Last digit + per-chunk bookkeeping for the ordered compaction.
template <typename RAW, int LAST_BITS>
__global__ void __launch_bounds__(SEL_THREADS)
count_kernel(const RAW *__restrict__ x, int64_t numel, int64_t nvf, int64_t vpc, SelState *st,
             uint32_t *table /*[LB+1][G]*/, uint32_t *off_gt, uint32_t *off_eq, int pass)
{
    constexpr int VEC = KeyTraits<RAW>::VEC;
    constexpr uint32_t MASK = KeyTraits<RAW>::MASK;
    constexpr int LB = 1 << LAST_BITS;
    constexpr int NW = SEL_THREADS / WAVE;
    __shared__ uint32_t lh[LB + 1 + WAVE];
    __shared__ uint32_t s_digit;
    __shared__ uint32_t wave_tot2[2 * NW];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int G = gridDim.x;
    for (int i = tid; i < LB + 1 + WAVE; i += SEL_THREADS) lh[i] = 0;
    const uint32_t prefix = st->prefix;    // == (threshold key) >> LAST_BITS
    __syncthreads();

    const uint32_t dslot = LB + 1 + lane;
    uint32_t above = 0;
    auto count = [&](uint32_t raw, int) {
        const uint32_t key = raw & MASK;
        const uint32_t hi = key >> LAST_BITS;
        above += (hi > prefix) ? 1u : 0u;
        atomicAdd(&lh[(hi == prefix) ? (key & (LB - 1)) : dslot], 1u);
    };
    const uint4 *xv = reinterpret_cast<const uint4 *>(x);
    const int64_t v0 = static_cast<int64_t>(blockIdx.x) * vpc;
    const int64_t v1 = min(v0 + vpc, nvf);
    int64_t vb = v0;
    for (; vb + SEL_THREADS * SEL_UNROLL <= v1; vb += SEL_THREADS * SEL_UNROLL) {
        uint4 q[SEL_UNROLL];
#pragma unroll
        for (int u = 0; u < SEL_UNROLL; ++u) q[u] = xv[vb + u * SEL_THREADS + tid];
#pragma unroll
        for (int u = 0; u < SEL_UNROLL; ++u) for_each_raw(RAW(0), q[u], count);
    }
    for (int64_t v = vb + tid; v < v1; v += SEL_THREADS) for_each_raw(RAW(0), xv[v], count);
    if (blockIdx.x == gridDim.x - 1 && tid == 0)
        for (int64_t i = nvf * VEC; i < numel; ++i) count(x[i], 0);
    above = wave_sum(above);
    if (lane == 0 && above) atomicAdd(&lh[LB], above);
    __syncthreads();
    if (tid <= LB) table[tid * G + blockIdx.x] = lh[tid];
    if (!last_block_to_arrive(&st->ticket[pass])) return;

    // ---- last workgroup: resolve the final digit, then per-chunk offsets ----
    // totals per bin: each wavefront sums whole rows of table[b][0..G)
    for (int b = tid / WAVE; b < LB; b += NW) {
        uint32_t s = 0;
        for (int c = lane; c < G; c += WAVE) s += table[b * G + c];
        s = wave_sum(s);
        if (lane == 0) lh[b] = s;
    }
    __syncthreads();
    if (tid == 0) {
        const uint32_t k_rem = st->k_rem;
        uint32_t acc = 0;
        int d = 0;
        for (int b = LB - 1; b >= 0; --b) {
            if (acc + lh[b] >= k_rem) { d = b; break; }
            acc += lh[b];
        }
        st->t = (prefix << LAST_BITS) | static_cast<uint32_t>(d);
        st->m = k_rem - acc;
        s_digit = static_cast<uint32_t>(d);
    }
    __syncthreads();
    const int d = static_cast<int>(s_digit);
    // exclusive scan over chunks of (#{key > t}, #{key == t}); consecutive chunks per thread
    constexpr int CPT = (SEL_MAX_CHUNKS + SEL_THREADS - 1) / SEL_THREADS;
    uint32_t gt[CPT], eq[CPT];
    uint32_t mine_gt = 0, mine_eq = 0;
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int c = tid * CPT + i;
        gt[i] = eq[i] = 0;
        if (c < G) {
            uint32_t g = table[LB * G + c];
#pragma unroll
            for (int b = 0; b < LB; ++b) {
                const uint32_t n = table[b * G + c];
                g += (b > d) ? n : 0u;
                eq[i] = (b == d) ? n : eq[i];
            }
            gt[i] = g;
        }
        mine_gt += gt[i];
        mine_eq += eq[i];
    }
    uint32_t run_gt, run_eq, total_gt, total_eq;
    block_exclusive_scan2<SEL_THREADS>(mine_gt, mine_eq, wave_tot2, run_gt, run_eq, total_gt, total_eq);
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int c = tid * CPT + i;
        if (c < G) {
            off_gt[c] = run_gt;
            off_eq[c] = run_eq;
        }
        run_gt += gt[i];
        run_eq += eq[i];
    }
}

// Ordered compaction of one chunk per workgroup.
template <typename RAW>
__global__ void __launch_bounds__(SEL_THREADS)
compact_kernel(const RAW *__restrict__ x, int64_t numel, int64_t nvf, int64_t vpc,
               const SelState *__restrict__ st, const uint32_t *__restrict__ off_gt,
               const uint32_t *__restrict__ off_eq, RAW *__restrict__ vals, int32_t *__restrict__ idx)
{
    constexpr int VEC = KeyTraits<RAW>::VEC;
    constexpr uint32_t MASK = KeyTraits<RAW>::MASK;
    __shared__ uint32_t wave_tot[SEL_THREADS / WAVE];
    const int tid = threadIdx.x;
    const uint32_t t = st->t;
    const uint32_t m = st->m;
    uint32_t run_gt = off_gt[blockIdx.x];  // #{key > t} before this tile
    uint32_t run_eq = off_eq[blockIdx.x];  // #{key == t} before this tile
    const uint4 *xv = reinterpret_cast<const uint4 *>(x);
    const int64_t v0 = static_cast<int64_t>(blockIdx.x) * vpc;
    const int64_t v1 = min(v0 + vpc, nvf);
    for (int64_t vb = v0; vb < v1; vb += SEL_THREADS) {
        const int64_t v = vb + tid;
        const bool live = v < v1;
        uint4 q = make_uint4(0, 0, 0, 0);
        if (live) q = xv[v];
        uint32_t cnt = 0;                  // low 16 bits: #gt, high 16 bits: #eq (tile <= 8192 elements)
        for_each_raw(RAW(0), q, [&](uint32_t raw, int) {
            const uint32_t key = raw & MASK;
            cnt += (key > t ? 1u : 0u) + (key == t ? 0x10000u : 0u);
        });
        if (!live) cnt = 0;
        uint32_t total;
        const uint32_t excl = block_exclusive_scan<SEL_THREADS>(cnt, wave_tot, total);
        uint32_t my_gt = run_gt + (excl & 0xFFFFu);
        uint32_t my_eq = run_eq + (excl >> 16);
        const int64_t base = v * VEC;
        if (live && cnt) {
            for_each_raw(RAW(0), q, [&](uint32_t raw, int e) {
                const uint32_t key = raw & MASK;
                if (key > t) {
                    const uint32_t pos = my_gt + min(my_eq, m);
                    vals[pos] = static_cast<RAW>(raw);
                    idx[pos] = static_cast<int32_t>(base + e);
                    ++my_gt;
                } else if (key == t) {
                    if (my_eq < m) {
                        const uint32_t pos = my_gt + my_eq;
                        vals[pos] = static_cast<RAW>(raw);
                        idx[pos] = static_cast<int32_t>(base + e);
                    }
                    ++my_eq;
                }
            });
        }
        run_gt += total & 0xFFFFu;
        run_eq += total >> 16;
    }
    // ragged tail (numel % VEC elements) after the last full vector
    if (blockIdx.x == gridDim.x - 1 && tid == 0) {
        for (int64_t i = nvf * VEC; i < numel; ++i) {
            const RAW raw = x[i];
            const uint32_t key = raw & MASK;
            if (key > t) {
                const uint32_t pos = run_gt + min(run_eq, m);
                vals[pos] = raw;
                idx[pos] = static_cast<int32_t>(i);
                ++run_gt;
            } else if (key == t) {
                if (run_eq < m) {
                    const uint32_t pos = run_gt + run_eq;
                    vals[pos] = raw;
                    idx[pos] = static_cast<int32_t>(i);
                }
                ++run_eq;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Fused path: the whole select + compaction as ONE persistent kernel with one
// workgroup per compute unit; the phases are separated by
// grid barriers instead of kernel boundaries.  Every workgroup resolves the digits itself
// from the merged histogram, so the select state lives in registers.
//
// The kernel is an ordinary launch (a cooperative launch costs ~14 us of queue switching before and
// after the kernel on this runtime): the host only checks that the grid fits the device all at once.
// Should the workgroups nevertheless not all become resident (a device shared with other persistent
// kernels), the bounded grid barriers give up, every workgroup leaves, and the last one to leave
// redoes the whole selection on its own (select_serial): slow, but the result is always complete.
//
// Everything workgroups exchange (histogram, per-chunk table, barrier counter) is
// accessed ONLY with device-scope atomics, which are coherent by themselves, so no
// device-wide fence is needed: on this 8-XCD part such a fence writes back and
// invalidates a whole L2 and was measured at 5-8 us per grid barrier.  The ordering
// rests on what the hardware does, not on the language's memory model: a wave's exchanged
// stores and atomics are complete (s_waitcnt at the __syncthreads() in front of the
// arrival) before thread 0 issues the arrival atomic, and nothing exchanged is ever read
// through a non-coherent cache line.  The form the model itself guarantees -- acq_rel on the
// group counter, release on the top counter, an acquire fence after the wait, all at agent
// scope -- was measured beside it: 3.4-4.8 us more per call on every benchmark tensor (one
// barrier per call), for the L2 write-back and invalidate it implies; the relaxed form stays.
// Patience in polls (~0.25 us each); every wave exits even if it runs out.  A resident grid meets at a barrier within
// microseconds (a millisecond for the largest tensors), so the barriers give up after ~15 ms: a grid that is not
// resident all at once then costs those milliseconds plus the serial redo, not a second.  Waiting for workgroup 0's
// clearing pass is another matter: it is dispatched first and needs a few microseconds, and a workgroup that stops
// waiting for it leaves the exit count short (nobody then puts `ready` back to 0), so that wait is long.
// Tensors of up to 64 K elements, whose redo takes some 50 us, wait 0.1 ms: beside a large select on another stream, each with
// workgroups on compute units that the other still needs, they give way (calls of 60 K elements beside ones of 10 M, worst of
// 400 rounds 28 ms, of 1500 now 1).
constexpr uint32_t SPIN_LIMIT = 1u << 16, SPIN_LIMIT_SMALL = 400;
constexpr uint32_t READY_SPIN_LIMIT = 1u << 26;

__device__ inline uint32_t dev_load(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void dev_store(uint32_t *p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline unsigned long long dev_load64(const unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void dev_store64(unsigned long long *p, unsigned long long v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// All workgroups of the grid meet here (`round` = 1, 2, ... counts the barriers of the call).
// A workgroup bumps the counter of its group (launch order modulo 8, counters 256 bytes apart: 256 atomics on ONE
// word take ~10 ns each, one after the other) and its first wavefront polls all eight with one load (eight lanes, a
// counter each): one atomic and one load of latency, where a top counter bumped by the last of each group costs
// another atomic's round trip.  The first poll waits until the arrivals are through (they would queue behind it).
// 256 workgroups arriving together: 1.1 us, against 2.1 with the top counter and 1.9 with the first poll at once.
// The grid is sized so that every workgroup is resident at once, but nothing enforces that the
// device is not shared, so the wait is bounded: returns false (in every thread of the workgroup)
// if the others did not all arrive within `spin_limit` polls or if some workgroup already gave
// up.  The caller then skips to the kernel's exit protocol.  Without any patience (spin_limit 0, mode 3) a workgroup polls once,
// and may find the others there: the exit protocol then sees to it that the selection is redone all the same.
// Every wavefront first waits for its own outstanding stores and atomics: a workgroup barrier alone orders LDS only, and
// without this wait the arrival could overtake the histogram merges of the other wavefronts.  (With 8192 bins to merge it
// is 1.5 us of each fp32 digit pass.)
__device__ inline bool grid_barrier(SelState *st, uint32_t *xbar, uint32_t round, uint32_t spin_limit, uint32_t *ok_slot)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x < WAVE) {
        const uint32_t G = gridDim.x, lane = threadIdx.x;
        if (lane == 0)
            __hip_atomic_fetch_add(&xbar[(blockIdx.x & 7u) * 64], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_sleep(16);           // ~0.5 us
        const uint32_t goal = lane < 8u && lane < G ? round * ((G - lane + 7u) / 8u) : 0u;    // arrivals of group `lane`
        uint32_t spins = 0, ok = 1;
        for (;;) {
            const bool short_of = goal != 0u && dev_load(&xbar[lane * 64]) < goal;
            if (__ballot(short_of) == 0ull) break;
            if (++spins > spin_limit || ((spins & 31u) == 0 && dev_load(&st->error) != 0)) {
                if (lane == 0) dev_store(&st->error, 1u);
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(8);        // 256 pollers compete with the arrivals
        }
        if (lane == 0) *ok_slot = ok;
    }
    __syncthreads();
    return *ok_slot != 0;
}

// How a workgroup says that no grid barrier is ahead of it any more: an atomic on its group's report counter, sent right
// after the last barrier, behind the loads of the table; the last of a group passes the
// group's count on to the common word when it leaves (while its last output stores are on their way).  (One atomic per workgroup on
// one word, sent on leaving behind the output stores, held every workgroup back by 3 to 6 us; sent after the barrier,
// 256 of them slowed the table reads down by a microsecond.)
// A report is 1, or 0x10001 from a workgroup that gave up: the high half counts those.
constexpr int REPORT_TID = SEL_THREADS - WAVE;      // lane 0 of the last wavefront
struct ExitReport {
    uint32_t mine;          // the report, 0 while none has been sent (uniform over the workgroup)
    uint32_t before;        // thread REPORT_TID: the counter before it.  Not touched until report_group: the wait for the
                            // atomic's answer goes where its value is first used
    uint32_t group;         // thread REPORT_TID: what the workgroup added to the common word, 0 if it is not the last of its group
    uint32_t common;        // thread REPORT_TID: the common word before that
};
__device__ inline uint32_t *opaque(uint32_t *p)
{
    uint32_t zero = 0;      // (an address known to be uniform would be turned into a wavefront reduction, which waits for the answer)
    asm volatile("" : "+v"(zero));
    return p + zero;
}
__device__ inline void report_past_barriers(uint32_t *xbar, ExitReport &rep, bool gave_up)
{
    rep.mine = gave_up ? 0x10001u : 1u;
    rep.group = 0u;
    if (threadIdx.x == REPORT_TID)
        rep.before = __hip_atomic_fetch_add(opaque(xbar + (blockIdx.x & 7u) * 64 + 32), rep.mine, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void report_group(SelState *st, ExitReport &rep)
{
    if (threadIdx.x == REPORT_TID) {
        const uint32_t seen = rep.before + rep.mine, members = (gridDim.x - (blockIdx.x & 7u) + 7u) / 8u;
        if ((seen & 0xFFFFu) == members) {
            rep.group = seen;
            rep.common = __hip_atomic_fetch_add(opaque(&st->exited), seen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// Workgroup 0 clears what the workgroups exchange through (barrier counters and state words, histograms) and then publishes
// this call's generation number; the others look for it before their first global atomic.  No separate clearing kernel, and
// a workspace with arbitrary contents is fine: a stale word equals the generation (a per-process random number plus a
// call count) with probability 2^-64.  Device-scope atomics, like everything else that is exchanged.
// clear_words: the counters and state words, by the last wavefront of workgroup 0 and with an exchange instead of a store: its
// answer says when it is done, without a wait for the loads that have been issued since.  `done` is that answer.
__device__ inline void clear_words(SelState *st, uint32_t *xbar, uint32_t &done)
{
    const int i = static_cast<int>(threadIdx.x) - REPORT_TID;
    if (i >= 0 && i < 20) {
        uint32_t *w = i < 16 ? xbar + i * 32 : i == 16 ? &st->error : i == 17 ? &st->exited : i == 18 ? &st->redo : &st->staged;
        done = __hip_atomic_exchange(w, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}
__device__ inline void publish_words(SelState *st, uint32_t done, unsigned long long gen)
{
    if (threadIdx.x >= REPORT_TID) {
        asm volatile("" ::"v"(done));               // (the compiler waits for the answer here; it is the wavefront's, hence all lanes')
        if (threadIdx.x == REPORT_TID) dev_store64(&st->ready, gen);
    }
}
// the digit histograms: stores by the whole workgroup, published once they are done
__device__ inline void clear_hist(uint32_t *hist, int words)
{
    for (int i = threadIdx.x; i < words; i += SEL_THREADS) dev_store(hist + i, 0u);
}
__device__ inline void publish_hist(unsigned long long *ready, unsigned long long gen)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                                // every wavefront's stores are done
    if (threadIdx.x == 0) dev_store64(ready, gen);
}

// How a wait, or the whole parallel selection, ended (the same in every thread of a workgroup): SEL_GAVE_UP if a grid
// barrier ran out of patience, here or in another workgroup, SEL_NEVER_READY if the exchange area was never published.  In
// the last two cases the outputs are incomplete (whatever was written is correct, nothing is out of bounds).
enum SelOutcome { SEL_DONE = 0, SEL_GAVE_UP = 1, SEL_NEVER_READY = 2 };

// Waits until `ready` holds this call's generation number (`seen`: what thread 0 has already read there).
// `error` is the state's word where that is this call's already (the state words have been seen published), else null: a
// workgroup that gave up may have been the one to publish, or the last to leave, which takes `ready` back, so the wait
// ends with that word as a grid barrier does.
__device__ inline SelOutcome wait_published(const unsigned long long *ready, unsigned long long gen, unsigned long long seen,
                                            const uint32_t *error, uint32_t *slot)
{
    if (threadIdx.x == 0) {
        uint32_t spins = 0, outcome = SEL_DONE;
        while (seen != gen) {
            if (++spins > READY_SPIN_LIMIT) {      // workgroup 0 never ran: not this workgroup's patience setting
                outcome = SEL_NEVER_READY;
                break;
            }
            if (error != nullptr && (spins & 31u) == 0 && dev_load(error) != 0) {
                outcome = SEL_GAVE_UP;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
            seen = dev_load64(ready);
        }
        *slot = outcome;
    }
    __syncthreads();
    return static_cast<SelOutcome>(*slot);
}

// Finds the digit d with #{digit > d} < k_rem <= #{digit >= d} in the merged histogram
// and folds it into the workgroup's copy of the select state.  Thread t owns the bins
// of reversed rank t, so an ordinary exclusive prefix scan counts the keys above it.
template <int NB, int BITS>
__device__ inline void resolve_digit_local(const uint32_t *hist, uint32_t &prefix, uint32_t &k_rem,
                                           uint32_t *wave_tot, uint32_t *bcast /*[2]*/)
{
    constexpr int PER = (NB + SEL_THREADS - 1) / SEL_THREADS;
    const int tid = threadIdx.x;
    const int hi_bin = NB - 1 - tid * PER;           // this thread's highest bin; it owns hi_bin, hi_bin-1, ...
    uint32_t c[PER];
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        c[i] = (hi_bin - i >= 0) ? dev_load(hist + hi_bin - i) : 0u;
        mine += c[i];
    }
    uint32_t total;
    uint32_t above = block_exclusive_scan<SEL_THREADS>(mine, wave_tot, total);
    if (above < k_rem && k_rem <= above + mine) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (above + c[i] >= k_rem) {
                bcast[0] = (prefix << BITS) | static_cast<uint32_t>(hi_bin - i);
                bcast[1] = k_rem - above;
                break;
            }
            above += c[i];
        }
    }
    __syncthreads();
    prefix = bcast[0];
    k_rem = bcast[1];
    __syncthreads();
}

// ---- sampled first digit (16-bit element types) ---------------------------------------------------
// The first digit's histogram needs one LDS atomic per element, which is what bounds that pass (the
// LDS atomic unit of a compute unit takes ~16 cycles per wavefront instruction whatever it adds), then
// a merge with global atomics, a grid barrier, and a read-back of the merged histogram.  The bin that
// holds the k-th largest key can be predicted from a sample instead, and without any exchange: EVERY
// workgroup reads the same 512 pieces of 32 bytes (one per equal stretch of the tensor, at a hashed
// position inside it -- many small pieces, so that values that come in runs, like the tokens of an
// activation, do not fool it; served by the L2 caches after the first reader), histograms them in its own LDS and
// derives the same bracket of up to seven adjacent 8-key bins around the sample's quantile, wide enough for
// 5 standard deviations of the sampling error.  (8192 elements: twice as many narrow the bracket by a third of its
// width and cost another microsecond of LDS atomics.)  The bracket is only a prediction: the pass over all
// elements that follows counts exactly how many keys lie above the bracket and how many on each key
// inside it, so a bracket that does not contain the k-th largest key is detected, and the selection
// then runs with the exact histogram.  The result is the same in every case; only the time differs.
constexpr int SAMPLE_PIECES = 512;
constexpr int SAMPLE_STRETCH = 4;                     // a piece starts at a multiple of this many vectors (64 bytes) ...
constexpr int SAMPLE_PIECE = SEL_THREADS / SAMPLE_PIECES;   // ... and is this many vectors long: one vector per thread
constexpr int SAMPLE_ELEMS = SEL_THREADS * 8;
constexpr int64_t SAMPLE_LARGE = int64_t(1) << 21;    // from here on the state's `path` says how the prediction went
constexpr int64_t SAMPLE_MIN_NUMEL = int64_t(1) << 14;
static_assert(SAMPLE_MIN_NUMEL / 8 / SAMPLE_STRETCH >= SAMPLE_PIECES, "a place per stretch at least");
constexpr int SAMPLE_SHIFT = 3, SAMPLE_BINS = 1 << (15 - SAMPLE_SHIFT);    // 8 keys per bin
constexpr int BRACKET_MAX_BINS = MAX_LAST_BINS >> SAMPLE_SHIFT;

// First vector of sample piece i: stretch i of the tensor's places (512 of them, as even as they divide: the last one ends
// at the tensor's end), hashed offset inside it.
__device__ inline int64_t sample_piece(int i, int64_t nvf)
{
    const int64_t places = nvf / SAMPLE_STRETCH;
    const int64_t first = i * places / SAMPLE_PIECES, end = (i + 1) * places / SAMPLE_PIECES;
    const uint32_t h = (static_cast<uint32_t>(i) + 1u) * 0x9E3779B1u;
    return (first + static_cast<int64_t>((h >> 8) % static_cast<uint32_t>(end - first))) * SAMPLE_STRETCH;
}

// The sample ranks around the k-th largest key's quantile, r - margin and r + margin with r = the sample's share of k.
// No sample (lo = 0) if one of them lies outside of it: there is no bracket then, whatever the sample holds (a sample of
// few magnitudes costs up to 5 us of LDS atomics on the same bins).
struct SampleRanks {
    float lo, hi;
};
inline SampleRanks sample_ranks(uint32_t k, int64_t numel, int sample)
{
    const float frac = static_cast<float>(k) / static_cast<float>(numel);
    const float r = frac * static_cast<float>(sample);
    const float margin = 5.0f * __builtin_sqrtf(std::max(r * (1.0f - frac), 1.0f)) + 8.0f;
    const bool inside = r - margin >= 1.0f && r + margin <= static_cast<float>(sample) - 1.0f;
    return inside ? SampleRanks{r - margin, r + margin} : SampleRanks{0.0f, 0.0f};
}

// From the sample's histogram (in LDS; bin 0, the zeros, is not counted: it holds what the others leave of the sample): the
// bins that hold the two ranks.
// Returns false (in every thread) if there is no usable bracket (more than `most` bins).
template <int NB>
__device__ inline bool sample_bracket(const uint32_t *hist, SampleRanks ranks, uint32_t most, uint32_t *wave_tot,
                                      uint32_t *bcast /*[2]*/, uint32_t &b_lo, uint32_t &b_hi)
{
    constexpr int PER = (NB + SEL_THREADS - 1) / SEL_THREADS;
    const int tid = threadIdx.x;
    const int hi_bin = NB - 1 - tid * PER;           // as in resolve_digit_local: descending bins, ascending ranks
    uint32_t c[PER];
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        c[i] = (hi_bin - i >= 0) ? hist[hi_bin - i] : 0u;
        mine += c[i];
    }
    if (tid < 2) bcast[tid] = 0xFFFFFFFFu;           // (ordered before the finders' stores by the scan's barriers)
    uint32_t total;
    const uint32_t above = block_exclusive_scan<SEL_THREADS>(mine, wave_tot, total);
    const uint32_t rank[2] = {static_cast<uint32_t>(ranks.lo), static_cast<uint32_t>(ranks.hi) + 1u};   // higher bin first
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (tid == 0 && rank[q] > total) bcast[q] = 0u;              // among the zeros
        if (above < rank[q] && rank[q] <= above + mine) {
            uint32_t a = above;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                if (a + c[i] >= rank[q]) {
                    bcast[q] = static_cast<uint32_t>(hi_bin - i);
                    break;
                }
                a += c[i];
            }
        }
    }
    __syncthreads();
    b_hi = bcast[0];
    b_lo = bcast[1];
    const bool ok = b_hi != 0xFFFFFFFFu && b_lo != 0xFFFFFFFFu && b_hi - b_lo < most;
    __syncthreads();
    return ok;
}

typedef unsigned long long lane_mask;
// number of set bits of the mask in the lanes before this one, plus base
__device__ inline uint32_t bits_before(lane_mask a, uint32_t base)
{
    return __builtin_amdgcn_mbcnt_hi(uint32_t(a >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(a), base));
}

// ---- one read of x: candidates staged in LDS (16-bit element types) ---------------------------------
// With the range [key_lo, key_lo + nf) known BEFORE the pass over the chunk, everything that can still
// be kept is known too: the elements with key >= key_lo, a share of (1 - gamma) plus the range's width
// (12-15 % at gamma = 0.9).  The pass therefore stages them in LDS, in flat-index order, as one word each
// (value << 16 | position), and both the exact counts and the compaction then walk the staged words
// instead of reading x again.
// Each wavefront owns a contiguous 1/16 of the chunk and a staging segment of its own, so the pass needs
// no workgroup barrier.  It walks its range in rows of 64 vectors (a lane's vector is 8 consecutive elements, so
// lane order is flat order), ST_ROWS of them in flight in registers: an 8-bit candidate mask per lane, one wavefront
// scan of the counts of two rows packed into a word, then eight predicated LDS stores per row, each lane advancing its
// slot where its bit is set.
// When the segment is full the pass only counts; the rows that were not staged are read again once the threshold is
// known, and go through the same segment after its first filling has been written out.
constexpr int ST_ROWS = 4;                                 // rows in flight per wavefront
constexpr int ST_ROW_ELEMS = WAVE * 8;
// Staged words per wavefront: 16 segments are 134 KB, the histograms in their place before anything is staged.  (With 1916
// words and the histograms beside them: row form of 39 M elements at gamma 0.8 134.6 -> 133.5 us a pass, 1x1 convolution of
// 51 M 113.0 -> 110.3.  2360 would fit and give 130.3 and 108.5; what stands against it is only that the tests have 9 M elements
// at gamma 0.05 overflow the segments, which they do not there.)
constexpr int ST_SEGCAP = 2136;
constexpr int ST_PART_OFF = (SEL_THREADS / WAVE) * ST_SEGCAP * 4;
constexpr size_t ST_SMEM_BYTES = ST_PART_OFF + 4 * 2 * size_t(SEL_THREADS / WAVE) * TABLE_PITCH;    // + the table's partial sums
static_assert(ST_PART_OFF % 16 == 0 && ST_SEGCAP % 4 == 0, "the segments are read 16 bytes at a time");
static_assert(ST_SEGCAP >= 2 * ST_ROW_ELEMS, "two rows of nothing but candidates fit an empty segment");
static_assert(ST_SMEM_BYTES >= 4 * ((size_t(1) << 13) + 2 * WAVE), "the serial redo's histogram");
static_assert(ST_PART_OFF >= 4 * SAMPLE_BINS, "the sample's or the digit's histogram is done with before anything is staged");

// Classification of the 8 consecutive 16-bit elements of q against a lowest key, five instructions per 32-bit word: one AND
// clears both signs (keys[]), one unsigned compare per half (the upper half against lowest << 16: the lower half cannot
// change the outcome), and an add-with-carry takes each outcome in.
__device__ inline uint32_t count_candidates(const u32x4 &q, uint32_t lowest, u32x4 &keys)   // how many have key >= lowest
{
    uint32_t n = 0;
    const uint32_t lo = lowest, hi = lowest << 16;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        uint32_t k;
        const uint32_t word = q[w];
        asm("v_and_b32 %1, 0x7fff7fff, %2\n\t"
            "v_cmp_le_u32 vcc, %4, %1\n\t"
            "v_addc_co_u32 %0, vcc, 0, %0, vcc\n\t"
            "v_cmp_le_u16 vcc, %3, %1\n\t"
            "v_addc_co_u32 %0, vcc, 0, %0, vcc"
            : "+v"(n), "=&v"(k)
            : "v"(word), "s"(lo), "s"(hi)
            : "vcc");
        keys[w] = k;
    }
    return n;
}
__device__ inline uint32_t candidate_mask(const u32x4 &q, uint32_t lowest)                  // bit e: element e has key >= lowest
{
    uint32_t mask = 0, k;
    const uint32_t lo = lowest, hi = lowest << 16;
#pragma unroll
    for (int w = 3; w >= 0; --w) {             // last to first: element 0 ends in bit 0
        const uint32_t word = q[w];
        asm("v_and_b32 %1, 0x7fff7fff, %2\n\t"
            "v_cmp_le_u32 vcc, %4, %1\n\t"
            "v_addc_co_u32 %0, vcc, %0, %0, vcc\n\t"
            "v_cmp_le_u16 vcc, %3, %1\n\t"
            "v_addc_co_u32 %0, vcc, %0, %0, vcc"
            : "+v"(mask), "=&v"(k)
            : "v"(word), "s"(lo), "s"(hi)
            : "vcc");
    }
    return mask;
}
// Stores the candidates of q, in the lanes of `valid`, as words value << 16 | position (pos, pos + 1, ...) from LDS byte
// address `addr` on.  Per element: the comparison goes straight into the execution mask, so that the store and the advance
// of the address happen in the lanes whose element is a candidate.
__device__ inline void stage_candidates(const u32x4 &q, const u32x4 &keys, uint32_t lowest, unsigned long long valid,
                                        uint32_t addr, uint32_t pos)
{
    uint32_t t;
    unsigned long long saved;
    const uint32_t lo = lowest, hi = lowest << 16, upper = 0xFFFF0000u;
#define STAGE_WORD(W, K)                                   \
    "v_cmpx_le_u16 vcc, %[lo], " K "\n\t"                  \
    "v_lshl_or_b32 %[t], " W ", 16, %[pos]\n\t"            \
    "ds_write_b32 %[addr], %[t]\n\t"                       \
    "v_add_u32 %[addr], 4, %[addr]\n\t"                    \
    "s_mov_b64 exec, %[valid]\n\t"                         \
    "v_add_u32 %[pos], 1, %[pos]\n\t"                      \
    "v_cmpx_le_u32 vcc, %[hi], " K "\n\t"                  \
    "v_and_or_b32 %[t], " W ", %[upper], %[pos]\n\t"       \
    "ds_write_b32 %[addr], %[t]\n\t"                       \
    "v_add_u32 %[addr], 4, %[addr]\n\t"                    \
    "s_mov_b64 exec, %[valid]\n\t"                         \
    "v_add_u32 %[pos], 1, %[pos]\n\t"
    asm volatile("s_mov_b64 %[saved], exec\n\t"
                 "s_mov_b64 exec, %[valid]\n\t"
                 STAGE_WORD("%[q0]", "%[k0]") STAGE_WORD("%[q1]", "%[k1]") STAGE_WORD("%[q2]", "%[k2]") STAGE_WORD("%[q3]", "%[k3]")
                 "s_mov_b64 exec, %[saved]\n\t"
                 "s_nop 4"                      // (cross-lane operations must not follow a vector write of the mask closely)
                 : [addr] "+&v"(addr), [pos] "+&v"(pos), [t] "=&v"(t), [saved] "=&s"(saved)
                 : [q0] "v"(q[0]), [q1] "v"(q[1]), [q2] "v"(q[2]), [q3] "v"(q[3]), [k0] "v"(keys[0]), [k1] "v"(keys[1]),
                   [k2] "v"(keys[2]), [k3] "v"(keys[3]), [lo] "s"(lo), [hi] "s"(hi), [upper] "s"(upper), [valid] "s"(valid)
                 : "vcc", "memory");
#undef STAGE_WORD
}

// From the per-chunk table of a range of nf keys (a line of TABLE_PITCH words per chunk; word r < nf: the chunk's count of
// key key_lo + r; word nf: of the keys above the range): the threshold t = the k-th largest key, the tie budget m, and the
// counts of keys above t and equal to t in the chunks before this one.  A wavefront takes 16 chunks of every 256, a lane per
// word, and adds them up for all chunks and for the chunks before this one; the wavefronts meet in LDS (`part`,
// 2 * NW * TABLE_PITCH words).  False if the k-th key is not in the range.
// (With a line per KEY a workgroup's 33 to 57 stores went to as many lines, each shared by 32 workgroups, and were
// acknowledged a microsecond later; the sums over lanes cost a scan per row.)
// The workgroup's report goes out behind the table loads, if no barrier comes after it (`last`).
__device__ inline bool resolve_table(const uint32_t *table, uint32_t nf, uint32_t key_lo, uint32_t k, uint32_t *part, uint32_t *bcast,
                                     uint32_t *offs, uint32_t *verdict, uint32_t *xbar, ExitReport &rep, bool last)
{
    constexpr int NW = SEL_THREADS / WAVE, PER = 16;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int G = gridDim.x, me = blockIdx.x;
    uint32_t s = 0, sp = 0;
    for (int c0 = wave * PER; c0 < G; c0 += NW * PER) {
        uint32_t v[PER];
        const uint32_t *line = table + c0 * TABLE_PITCH + lane;       // (the table has a line for every possible chunk)
#pragma unroll
        for (int j = 0; j < PER; ++j) v[j] = dev_load(line + j * TABLE_PITCH);
        if (last && rep.mine == 0) report_past_barriers(xbar, rep, false);
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            s += c0 + j < G ? v[j] : 0u;
            sp += c0 + j < me ? v[j] : 0u;
        }
    }
    if (last && rep.mine == 0) report_past_barriers(xbar, rep, false); // (a wavefront without chunks)
    part[wave * TABLE_PITCH + lane] = s;
    part[(NW + wave) * TABLE_PITCH + lane] = sp;
    __syncthreads();
    if (tid < WAVE) {
        // Lane 0 takes the keys above the range, lanes 1.. the range's keys in descending order, so a
        // prefix scan over the lanes counts the keys above each key.  The k-th largest key is the one
        // with  #above < k <= #above + #equal;  it is in the range iff that holds for a lane >= 1.
        const int rr = static_cast<int>(nf) - lane;
        uint32_t full = 0, before = 0;
        if (rr >= 0) {
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                full += part[w * TABLE_PITCH + rr];
                before += part[(NW + w) * TABLE_PITCH + rr];
            }
        }
        const uint32_t incl = wave_inclusive_scan(full), incl_p = wave_inclusive_scan(before);
        const bool here = lane >= 1 && rr >= 0 && incl - full < k && k <= incl;
        const unsigned long long hit = __ballot(here);
        if (lane == 0) *verdict = hit ? 1u : 0u;
        if (here) {
            bcast[0] = key_lo + static_cast<uint32_t>(rr);     // t
            bcast[1] = k - (incl - full);                       // m: how many keys equal to t are kept
            bcast[2] = full;                                    // ... of how many
            offs[0] = incl_p - before;                          // #{key > t} in the chunks before this one
            offs[1] = before;                                   // #{key == t} there
        }
    }
    __syncthreads();
    return *verdict != 0;
}

// ---- the cheaper index forms straight from the output phase (16-bit element types) -------------------
// FORM_ROWS: 16-bit positions within rows of `len` elements instead of flat indices; FORM_MASK: a bit per element.  Both with
// starts[r] = number of kept elements before element r * len.  A wavefront owns a contiguous range of the tensor, so it owns
// the starts and the mask words in it (ranges begin at multiples of 64 elements), and it meets its kept elements in flat order.
// Against writing flat indices and converting them in a kernel of its own (two for the mask), queued calls: row form of 25 M
// elements at gamma 0.7 43.7 -> 39.1 us, mask 57.2 -> 45.3; 9.7 M at 0.9 23.3 -> 20.1 and 26.2 -> 20.8; rows of two elements,
// one in a hundred kept, 39.8 -> 35.6.
struct FormArgs {
    uint16_t *col;
    uint32_t *mask;
    int32_t *starts;
    Divisor len;
    uint32_t nstarts;                                      // entries of starts but the closing one, which is k
};

// One wavefront's state while it walks its kept elements.
template <int FORM>
struct FormWriter {
    FormArgs a;
    uint32_t last_row;         // row of the last kept element; rows up to it have their starts (uniform)
    uint32_t word, bits;       // FORM_MASK: the word that is being filled (uniform)
    uint32_t *window;          // ... and 256 words of LDS of the wavefront's own

    __device__ void begin(const FormArgs &args, uint32_t first, uint32_t *lds)
    {
        a = args;
        // the rows that start at `first` or later are this wavefront's
        last_row = first == 0 ? 0xFFFFFFFFu : quotient(first - 1, a.len);       // (-1: compared as last_row + 1)
        word = first >> 5;
        bits = 0;
        window = lds;
    }
    // the lanes of `kept`, in lane order: element `flat` goes to output slot `slot`
    __device__ void elements(bool kept, lane_mask b, uint32_t flat, uint32_t slot, uint32_t k)
    {
        if (b == 0) return;
        const int lane = threadIdx.x & (WAVE - 1);
        const uint32_t row = quotient(flat, a.len);
        const lane_mask lower = b & ((lane_mask(1) << lane) - 1);
        const int src = lower ? 63 - __builtin_clzll(lower) : 0;
        uint32_t prev = uint32_t(__builtin_amdgcn_ds_bpermute(src * 4, int(row)));
        prev = lower ? prev : last_row;
        if (kept && slot < k) {                            // (always, for consistent counts)
            if constexpr (FORM == FORM_ROWS) a.col[slot] = static_cast<uint16_t>(flat - row * a.len.d);
            for (uint32_t r = prev + 1; r <= row && r < a.nstarts; ++r) a.starts[r] = static_cast<int32_t>(slot);
        }
        last_row = uint32_t(__builtin_amdgcn_readlane(int(row), 63 - __builtin_clzll(b)));
    }
    // FORM_MASK: the bits of up to 4 x 64 kept elements, in flat order (flat[u] where kept[u])
    __device__ void mask_batch(const bool (&kept)[4], const uint32_t (&flat)[4])
    {
        const int lane = threadIdx.x & (WAVE - 1);
        uint32_t top = 0;                                  // the last kept element's word
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const lane_mask b = __ballot(kept[u]);
            if (b) top = uint32_t(__builtin_amdgcn_readlane(int(flat[u]), 63 - __builtin_clzll(b))) >> 5;
        }
        top = max(top, word);
        for (;;) {                                         // windows of 256 words; one, unless little is kept
            u32x4 zero = {0u, 0u, 0u, 0u};
            *reinterpret_cast<u32x4 *>(window + lane * 4) = zero;
            asm volatile("" ::: "memory");
            if (lane == 0) window[0] = bits;
            asm volatile("" ::: "memory");
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t at = (flat[u] >> 5) - word;
                if (kept[u] && at < 256u) atomicOr(&window[at], 1u << (flat[u] & 31u));
            }
            asm volatile("" ::: "memory");
            const bool more = top - word >= 256u;
            const uint32_t done = more ? 256u : top - word;                    // whole words
            for (uint32_t i = lane; i < done; i += WAVE) a.mask[word + i] = window[i];
            if (!more) {
                bits = uint32_t(__builtin_amdgcn_readfirstlane(int(window[done])));
                word = top;
                break;
            }
            word += 256u;
            bits = 0;
        }
    }
    // the range ends before element `end`, `slot` elements have been kept before it
    __device__ void finish(uint32_t end, uint32_t slot)
    {
        const uint32_t lane = threadIdx.x & (WAVE - 1);
        const uint32_t stop = min(quotient(end - 1, a.len) + 1, a.nstarts);      // rows that start before `end`
        for (uint32_t r = last_row + 1 + lane; r < stop; r += WAVE) a.starts[r] = static_cast<int32_t>(slot);
        if constexpr (FORM == FORM_MASK)
            for (uint32_t w = word + lane; w < (end + 31) >> 5; w += WAVE) a.mask[w] = w == word ? bits : 0u;
    }
};

// The forms from the pairs the serial redo has written (one workgroup; every word and start written whole).
template <int FORM>
__device__ inline void forms_from_pairs(const int32_t *idx, int64_t numel, uint32_t k, const FormArgs &a)
{
    auto before = [&](uint32_t flat) {                     // pairs before element `flat`
        uint32_t lo = 0, hi = k;
        while (lo < hi) {
            const uint32_t mid = (lo + hi) / 2;
            if (static_cast<uint32_t>(idx[mid]) < flat) lo = mid + 1; else hi = mid;
        }
        return lo;
    };
    for (uint32_t r = threadIdx.x; r <= a.nstarts; r += SEL_THREADS)
        a.starts[r] = static_cast<int32_t>(r < a.nstarts ? before(r * a.len.d) : k);
    if constexpr (FORM == FORM_ROWS) {
        for (uint32_t j = threadIdx.x; j < k; j += SEL_THREADS) {
            const uint32_t flat = static_cast<uint32_t>(idx[j]);
            a.col[j] = static_cast<uint16_t>(flat - quotient(flat, a.len) * a.len.d);
        }
    } else {
        for (uint32_t w = threadIdx.x; w < (numel + 31) / 32; w += SEL_THREADS) {
            uint32_t bits = 0;
            for (uint32_t j = before(w * 32); j < k; ++j) {
                const uint32_t at = static_cast<uint32_t>(idx[j]) - w * 32;
                if (at >= 32u) break;
                bits |= 1u << at;
            }
            a.mask[w] = bits;
        }
    }
}

// 16-bit element types.
template <int FORM>
__device__ inline SelOutcome select16_body(const uint16_t *__restrict__ x, int64_t numel, int64_t nvf, int64_t vpc, uint32_t k,
                                           SelState *st, uint32_t *hist0, uint32_t *table, uint16_t *__restrict__ vals,
                                           int32_t *__restrict__ idx, uint32_t spin_limit, unsigned long long gen, SampleRanks ranks,
                                           ExitReport &rep, const FormArgs &form)
{
    constexpr int VEC = 8;
    constexpr uint32_t MASK = KeyTraits<uint16_t>::MASK;
    constexpr int BITS1 = 11, SHIFT1 = 4, NB = 1 << BITS1;      // first digit; the last one has SHIFT1 bits
    constexpr int NW = SEL_THREADS / WAVE;
    extern __shared__ __attribute__((aligned(16))) u32x4 dyn_smem[];
    char *dyn_bytes = reinterpret_cast<char *>(dyn_smem);
    uint32_t *lh = reinterpret_cast<uint32_t *>(dyn_bytes);     // (before anything is staged)
    uint32_t *part = reinterpret_cast<uint32_t *>(dyn_bytes + ST_PART_OFF);
    __shared__ uint32_t bcast[4], offs[2], verdict, spilled;
    __shared__ uint32_t wave_tot[NW];
    __shared__ uint32_t whist[NW][MAX_LAST_BINS + 1];           // per wavefront: its elements on each key of the range, and above it
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const bool last_chunk = blockIdx.x == gridDim.x - 1;
    const u32x4 *xv = reinterpret_cast<const u32x4 *>(x);
    uint32_t *xbar = reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(st) + SelWorkspace::xbar_off);

    // development builds only: phase time stamps of one workgroup into the state block's spare words
    [[maybe_unused]] unsigned long long *stamps = reinterpret_cast<unsigned long long *>(st->pad + 4);
#define STAMP(i) DROPIT_DEV_STAMP(stamps, i, tid == 0 && blockIdx.x == gridDim.x / 2)
    STAMP(0);

    // wavefront `wave` owns vectors [wv0, wv1) of the chunk, in rows of 64; ranges start on 128-byte lines
    const int64_t v0 = static_cast<int64_t>(blockIdx.x) * vpc, v1 = min(v0 + vpc, nvf);
    const int64_t vpw = ((vpc + NW - 1) / NW + 7) / 8 * 8;
    const int64_t wv0 = min(v0 + int64_t(wave) * vpw, v1), wv1 = min(wv0 + vpw, v1);
    const int wvecs = static_cast<int>(wv1 - wv0);
    const int nrows = (wvecs + WAVE - 1) / WAVE;
    const u32x4 *wx = xv + (wv0 < nvf ? wv0 : nvf > 0 ? nvf - 1 : 0);   // (an empty range still has a valid address to load from)
    const int last_vec = max(wvecs - 1, 0);
    uint32_t *seg = reinterpret_cast<uint32_t *>(dyn_bytes) + wave * ST_SEGCAP;
    u32x4 q[ST_ROWS];
    // (loads are unconditional and clamped, so that the wait in front of a row's use can leave the rows behind it in flight)
    auto issue_row = [&](u32x4 &dst, int row) { dst = wx[min(row * WAVE + lane, last_vec)]; };
    auto issue_rows = [&](int row) {
#pragma unroll
        for (int u = 0; u < ST_ROWS; ++u) issue_row(q[u], row + u);
    };

    const bool sampling = ranks.lo > 0.0f;                      // uniform over the grid
    // The threshold lies in the key range [key_lo, key_lo + nf): predicted from the sample here, else (or if the
    // prediction fails) exactly known after the digit histogram.
    uint32_t key_lo = 0, nf = 1u << SHIFT1;
    bool predicted = false, preloaded = false;
    uint32_t cleared = 0;
    if (blockIdx.x == 0) {
        clear_words(st, xbar, cleared);
        clear_hist(hist0, NB);                                  // (published when the exact form turns out to be needed)
    }
    {
        u32x4 sq;
        if (sampling) sq = xv[sample_piece(tid / SAMPLE_PIECE, nvf) + tid % SAMPLE_PIECE];
        STAMP(8);
        if (sampling) {
            for (int i = tid; i < SAMPLE_BINS; i += SEL_THREADS) lh[i] = 0;
            // the rows are asked for once the sample is here: ahead of it, 64 KB per compute unit, they would hold it up
            // (bracket after 6.2 instead of 5.0 us, the whole call 45.5 instead of 44.6, on a 100 MB tensor)
            asm volatile("" : "+v"(sq));
            issue_rows(0);
            preloaded = true;
            __syncthreads();
            for_each_raw(uint16_t(0), sq, [&](uint32_t raw, int) {
                const uint32_t dgt = (raw & MASK) >> SAMPLE_SHIFT;
                if (dgt) atomicAdd(&lh[dgt], 1u);
            });
            if (blockIdx.x == 0) publish_words(st, cleared, gen);
            __syncthreads();
            STAMP(9);
            uint32_t b_lo, b_hi;
            predicted = sample_bracket<SAMPLE_BINS>(lh, ranks, BRACKET_MAX_BINS, wave_tot, bcast, b_lo, b_hi);
            if (predicted) {
                key_lo = b_lo << SAMPLE_SHIFT;
                nf = (b_hi - b_lo + 1) << SAMPLE_SHIFT;
            }
        } else if (blockIdx.x == 0) {
            publish_words(st, cleared, gen);
        }
    }
    unsigned long long early = 0;                               // usually the generation number: asked for long before it is needed
    if (tid == 0) early = dev_load64(&st->ready);
    STAMP(1);

    // The rows' candidates (key >= lowest) from row `first` on into the segment, in flat order; returns the first row that
    // was not staged (nrows, or fewer when the segment is full or a position would not fit 16 bits), n = words staged.
    // Positions count from row `first`.  Rows are staged in pairs.
    auto stage_rows = [&](uint32_t lowest, int first, uint32_t &n) -> int {
        const uint32_t low_s = __builtin_amdgcn_readfirstlane(lowest);
        n = 0;
        if (nrows == 0) return 0;
        if (!preloaded) issue_rows(first);
        preloaded = false;
        const uint32_t seg_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint32_t *)seg));
        int end = nrows;
        for (int row = first; row < end; row += ST_ROWS) {
#pragma unroll
            for (int u = 0; u < ST_ROWS; u += 2) {
                if (row + u < end) {
                    const int left = wvecs - (row + u) * WAVE - lane;              // > 0: the lane's vector of the first row exists
                    const bool in0 = left > 0, in1 = left > WAVE;
                    u32x4 k0, k1;
                    const uint32_t n0 = count_candidates(q[u], low_s, k0), n1 = count_candidates(q[u + 1], low_s, k1);
                    const uint32_t c = (in0 ? n0 : 0u) | (in1 ? n1 << 16 : 0u);
                    const uint32_t ex = wave_inclusive_scan(c) - c;
                    const uint32_t tot = uint32_t(__builtin_amdgcn_readlane(int(ex + c), WAVE - 1));
                    const uint32_t t0 = tot & 0xFFFFu, t1 = tot >> 16;
                    if (n + t0 + t1 > uint32_t(ST_SEGCAP) || (row + u + 2 - first) * ST_ROW_ELEMS > 65536) {
                        end = row + u;                                             // full (no jump out of the body: see issue_row)
                    } else {
                        const uint32_t pos = uint32_t((row + u - first) * ST_ROW_ELEMS + lane * VEC);
                        stage_candidates(q[u], k0, low_s, __ballot(in0), seg_addr + (n + (ex & 0xFFFFu)) * 4u, pos);
                        stage_candidates(q[u + 1], k1, low_s, __ballot(in1), seg_addr + (n + t0 + (ex >> 16)) * 4u, pos + ST_ROW_ELEMS);
                        n += t0 + t1;
                    }
                }
                issue_row(q[u], row + u + ST_ROWS);
                issue_row(q[u + 1], row + u + 1 + ST_ROWS);
            }
        }
        return end;
    };
    // exact counts of the rows from `first` on, without staging them
    auto count_rows = [&](int first, uint32_t &above) {
        const uint32_t lo_s = __builtin_amdgcn_readfirstlane(key_lo), end_s = __builtin_amdgcn_readfirstlane(key_lo + nf);
        issue_rows(first);
        for (int row = first; row < nrows; row += ST_ROWS) {
#pragma unroll
            for (int u = 0; u < ST_ROWS; ++u) {
                if (row + u < nrows) {
                    const bool there = wvecs - (row + u) * WAVE - lane > 0;
                    const uint32_t hi = candidate_mask(q[u], end_s);
                    uint32_t in = there ? candidate_mask(q[u], lo_s) & ~hi : 0u;
                    above += there ? __builtin_popcount(hi) : 0u;
                    while (in) {
                        const int e = __builtin_ctz(in);
                        in &= in - 1;
                        const uint32_t a = (e & 2) ? q[u][1] : q[u][0], b = (e & 2) ? q[u][3] : q[u][2];
                        const uint32_t w = (e & 4) ? b : a;
                        atomicAdd(&whist[wave][(((e & 1) ? w >> 16 : w) & MASK) - key_lo], 1u);
                    }
                }
                issue_row(q[u], row + u + ST_ROWS);
            }
        }
    };

    uint32_t barriers = 0;
    bool ready_seen = false, missed = false;
    uint32_t n_w = 0;          // staged words of this wavefront
    int staged_rows = 0;       // the rows they come from: [0, staged_rows)
    for (;;) {
        if (!predicted) {
            // exact digit: every element of the chunk through an LDS histogram, merged with global atomics
            if (blockIdx.x == 0) publish_hist(&st->ready_hist, gen);
            __syncthreads();
            for (int i = tid; i < NB + WAVE; i += SEL_THREADS) lh[i] = 0;
            __syncthreads();
            auto add = [&](uint32_t raw, int) {
                const uint32_t d = (raw & MASK) >> SHIFT1;
                atomicAdd(&lh[d ? d : NB + lane], 1u);                     // exact zeros go to per-lane slots
            };
            int64_t vb = v0;
            for (; vb + SEL_THREADS * SEL_UNROLL <= v1; vb += SEL_THREADS * SEL_UNROLL) {
                u32x4 h[SEL_UNROLL];
#pragma unroll
                for (int u = 0; u < SEL_UNROLL; ++u) h[u] = xv[vb + u * SEL_THREADS + tid];
#pragma unroll
                for (int u = 0; u < SEL_UNROLL; ++u) for_each_raw(uint16_t(0), h[u], add);
            }
            for (int64_t v = vb + tid; v < v1; v += SEL_THREADS) for_each_raw(uint16_t(0), xv[v], add);
            if (last_chunk && tid == 0)
                for (int64_t i = nvf * VEC; i < numel; ++i) add(x[i], 0);
            __syncthreads();
            if (tid < WAVE) {
                const uint32_t z = wave_sum(lh[NB + tid]);
                if (tid == 0) lh[0] += z;
            }
            __syncthreads();
            if (!ready_seen)
                if (const SelOutcome o = wait_published(&st->ready, gen, early, nullptr, &bcast[3])) return o;
            ready_seen = true;
            if (const SelOutcome o = wait_published(&st->ready_hist, gen, 0ull, &st->error, &bcast[2])) return o;   // (a word of its own: others may still read the first wait's)
            for (int i = tid; i < NB; i += SEL_THREADS) {
                const uint32_t c = lh[i];
                if (c) atomicAdd(&hist0[i], c);
            }
            if (!grid_barrier(st, xbar, ++barriers, spin_limit, &bcast[3])) return SEL_GAVE_UP;
            uint32_t prefix = 0, k_rem = k;
            resolve_digit_local<NB, BITS1>(hist0, prefix, k_rem, wave_tot, bcast);
            key_lo = prefix << SHIFT1;
            nf = 1u << SHIFT1;
            STAMP(2);
        }

        // ---- the one pass, then exact counts over the range and above it ----------------
        // (the histogram row of a wavefront is its own; words and counts of one wavefront need no workgroup barrier)
        uint32_t *wh = whist[wave];
        if (lane <= static_cast<int>(nf)) wh[lane] = 0;
        if (tid == 0) spilled = 0;
        staged_rows = stage_rows(key_lo, 0, n_w);
        STAMP(3);
        __syncthreads();                                         // `spilled` is cleared
        const uint32_t key_end = key_lo + nf;
        uint32_t above = 0;
        for (uint32_t q0 = 0; q0 < n_w; q0 += 4 * WAVE) {
            const uint32_t at = q0 + lane * 4;
            if (at < n_w) {
                const u32x4 w4 = *reinterpret_cast<const u32x4 *>(seg + at);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t key = (w4[j] >> 16) & MASK;
                    const bool there = at + j < n_w;
                    above += (there && key >= key_end) ? 1u : 0u;
                    const uint32_t rel = key - key_lo;
                    if (there && rel < nf) atomicAdd(&wh[rel], 1u);
                }
            }
        }
        if (staged_rows < nrows) {
            count_rows(staged_rows, above);
            if (lane == 0) spilled = 1u;
        }
        above = wave_sum(above);
        if (lane == 0) wh[nf] = above;
        __syncthreads();
        if (!ready_seen)
            if (const SelOutcome o = wait_published(&st->ready, gen, early, nullptr, &bcast[3])) return o;
        ready_seen = true;
        if (tid <= static_cast<int>(nf)) {        // the chunk's column of the table: the wavefronts' counts added up
            uint32_t sum = 0;
#pragma unroll
            for (int w2 = 0; w2 < NW; ++w2) sum += whist[w2][tid];
            if (last_chunk)                        // the tensor's ragged end belongs to the chunk, but to no wavefront's range
                for (int64_t i = nvf * VEC; i < numel; ++i) {
                    const uint32_t key = x[i] & MASK;
                    sum += (tid == static_cast<int>(nf) ? key >= key_end : key == key_lo + tid) ? 1u : 0u;
                }
            dev_store(&table[blockIdx.x * TABLE_PITCH + tid], sum);
        }
        STAMP(4);
        if (!grid_barrier(st, xbar, ++barriers, spin_limit, &bcast[3])) return SEL_GAVE_UP;
        STAMP(5);
        if (resolve_table(table, nf, key_lo, k, part, bcast, offs, &verdict, xbar, rep, true)) break;
        if (!predicted) return SEL_GAVE_UP;     // cannot happen with an exact digit; the serial path would still answer
        predicted = false;                       // the sample misled: once more with the exact histogram
        missed = true;
    }
    const uint32_t t = bcast[0], m = bcast[1];
    if (tid == REPORT_TID) {
        if (spilled == 0) __hip_atomic_fetch_add(&st->staged, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (blockIdx.x == 0) {
            const uint32_t form = missed ? 2u : predicted ? 1u : 0u;
            dev_store(&st->form, form);
            dev_store(&st->path, numel < SAMPLE_LARGE ? 0u : form);
        }
    }
    STAMP(6);

    // ---- ordered output -------------------------------------------------------------
    // A kept element (key > t, or one of the first m keys == t) goes to output slot #gt-before + min(#eq-before, m).
    // #{key > t}, #{key == t} in the wavefronts' ranges, from their histograms: lane l adds up wavefront l's
    const uint32_t trel = t - key_lo;
    uint32_t g = 0, e = 0;
    if (lane < NW) {
        g = whist[lane][nf];
        for (uint32_t r = trel + 1; r < nf; ++r) g += whist[lane][r];
        e = whist[lane][trel];
    }
    const uint32_t gi = wave_inclusive_scan(g), ei = wave_inclusive_scan(e);
    uint32_t my_gt = offs[0] + uint32_t(__builtin_amdgcn_readlane(int(gi - g), wave));
    uint32_t my_eq = offs[1] + uint32_t(__builtin_amdgcn_readlane(int(ei - e), wave));
    const uint32_t chunk_gt = offs[0] + uint32_t(__builtin_amdgcn_readlane(int(gi), NW - 1));
    const uint32_t chunk_eq = offs[1] + uint32_t(__builtin_amdgcn_readlane(int(ei), NW - 1));
    auto keep = [&](uint32_t pos, uint32_t raw, uint32_t i) {
        if (pos < k) {                     // always true for consistent counts
            vals[pos] = static_cast<uint16_t>(raw);
            if constexpr (FORM == FORM_FLAT) idx[pos] = static_cast<int32_t>(i);
        }
    };
    FormWriter<FORM> writer;               // (its window: the first 256 staged words, which are in registers by the time it is used)
    if constexpr (FORM != FORM_FLAT) writer.begin(form, static_cast<uint32_t>(wv0 * VEC), seg);
    // All or none of this wavefront's keys equal to t are kept, except in the one wavefront where the budget runs out.
    const uint32_t wave_eq = uint32_t(__builtin_amdgcn_readlane(int(e), wave));
    const bool split = my_eq < m && my_eq + wave_eq > m;
    const uint32_t least = my_eq < m ? t : t + 1;      // lowest key kept (if not split)
    uint32_t my_slot = my_gt + min(my_eq, m);
    int first = 0;                         // the row the staged words' positions count from
    for (;;) {
        // the staged words, 64 at a time in lane order: neighbouring lanes write neighbouring slots
        const uint32_t flat0 = static_cast<uint32_t>(wv0 * VEC) + static_cast<uint32_t>(first) * ST_ROW_ELEMS;
        for (uint32_t q0 = 0; q0 < n_w; q0 += 4 * WAVE) {
            uint32_t w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = q0 + j * WAVE + lane < n_w ? seg[q0 + j * WAVE + lane] : 0u;
            [[maybe_unused]] bool in[4];
            [[maybe_unused]] uint32_t at[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t key = (w[j] >> 16) & MASK, flat = flat0 + (w[j] & 0xFFFFu);
                const bool there = q0 + j * WAVE + lane < n_w;
                bool kept;
                uint32_t slot;
                if (!split) {              // uniform over the wavefront
                    kept = there && key >= least;
                    const lane_mask b = __ballot(kept);
                    slot = bits_before(b, my_slot);
                    if (kept) keep(slot, w[j] >> 16, flat);
                    my_slot += __builtin_popcountll(b);
                } else {
                    const bool gt = there && key > t, eq = there && key == t;
                    const lane_mask bg = __ballot(gt), be = __ballot(eq);
                    const uint32_t eb = bits_before(be, my_eq), gb = bits_before(bg, my_gt);
                    kept = gt || (eq && eb < m);
                    slot = gb + min(eb, m);
                    if (kept) keep(slot, w[j] >> 16, flat);
                    my_gt += __builtin_popcountll(bg);
                    my_eq += __builtin_popcountll(be);
                }
                if constexpr (FORM != FORM_FLAT) {
                    writer.elements(kept, __ballot(kept), flat, slot, k);
                    in[j] = kept;
                    at[j] = flat;
                }
            }
            if constexpr (FORM == FORM_MASK) writer.mask_batch(in, at);
        }
        if (staged_rows >= nrows) break;
        first = staged_rows;               // the rows that did not fit: read again, only what is kept is staged now
        staged_rows = stage_rows(t, first, n_w);
    }
    STAMP(7);
    if constexpr (FORM != FORM_FLAT) {     // (numel is a multiple of eight: no ragged end)
        if (wvecs > 0) writer.finish(static_cast<uint32_t>(wv1 * VEC), split ? my_gt + min(my_eq, m) : my_slot);
        if (last_chunk && tid == 0) form.starts[form.nstarts] = static_cast<int32_t>(k);
    }
    if (last_chunk && tid == 0) {
        uint32_t run_gt = chunk_gt, run_eq = chunk_eq;
        for (int64_t i = nvf * VEC; i < numel; ++i) {
            const uint32_t raw = x[i], key = raw & MASK;
            if (key > t) {
                keep(run_gt + min(run_eq, m), raw, static_cast<uint32_t>(i));
                ++run_gt;
            } else if (key == t) {
                if (run_eq < m) keep(run_gt + run_eq, raw, static_cast<uint32_t>(i));
                ++run_eq;
            }
        }
    }
#undef STAMP
    return SEL_DONE;
}

// ---- candidates of 32-bit elements ------------------------------------------------------------------
// As count_candidates / stage_candidates above: the four consecutive elements of q against a lowest key; a staged candidate
// is two words, the element and its position.
__device__ inline uint32_t count_candidates(const u32x4 &q, uint32_t lowest, u32x4 &keys, uint32_t)
{
    uint32_t n = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        keys[e] = q[e] & KeyTraits<uint32_t>::MASK;
        n += keys[e] >= lowest ? 1u : 0u;
    }
    return n;
}
__device__ inline void stage_candidates(const u32x4 &q, const u32x4 &keys, uint32_t lowest, unsigned long long valid,
                                        uint32_t addr, uint32_t pos, uint32_t)
{
    unsigned long long saved;
    const uint32_t lo = lowest;
#define STAGE_ELEMENT(W, K)                                      \
    "v_cmpx_le_u32 vcc, %[lo], " K "\n\t"                        \
    "ds_write2_b32 %[addr], " W ", %[pos] offset1:1\n\t"         \
    "v_add_u32 %[addr], 8, %[addr]\n\t"                          \
    "s_mov_b64 exec, %[valid]\n\t"                               \
    "v_add_u32 %[pos], 1, %[pos]\n\t"
    asm volatile("s_mov_b64 %[saved], exec\n\t"
                 "s_mov_b64 exec, %[valid]\n\t"
                 STAGE_ELEMENT("%[q0]", "%[k0]") STAGE_ELEMENT("%[q1]", "%[k1]") STAGE_ELEMENT("%[q2]", "%[k2]") STAGE_ELEMENT("%[q3]", "%[k3]")
                 "s_mov_b64 exec, %[saved]\n\t"
                 "s_nop 4"                      // (cross-lane operations must not follow a vector write of the mask closely)
                 : [addr] "+&v"(addr), [pos] "+&v"(pos), [saved] "=&s"(saved)
                 : [q0] "v"(q[0]), [q1] "v"(q[1]), [q2] "v"(q[2]), [q3] "v"(q[3]), [k0] "v"(keys[0]), [k1] "v"(keys[1]),
                   [k2] "v"(keys[2]), [k3] "v"(keys[3]), [lo] "s"(lo), [valid] "s"(valid)
                 : "vcc", "memory");
#undef STAGE_ELEMENT
}
__device__ inline uint32_t count_candidates(const u32x4 &q, uint32_t lowest, u32x4 &keys, uint16_t) { return count_candidates(q, lowest, keys); }
__device__ inline void stage_candidates(const u32x4 &q, const u32x4 &keys, uint32_t lowest, unsigned long long valid,
                                        uint32_t addr, uint32_t pos, uint16_t)
{
    stage_candidates(q, keys, lowest, valid, addr, pos);
}

// A staged candidate of either type.
template <typename RAW> struct Staged;
template <> struct Staged<uint16_t> {
    typedef uint32_t word;
    __device__ static uint32_t raw(word w) { return w >> 16; }
    __device__ static uint32_t pos(word w) { return w & 0xFFFFu; }
    __device__ static word make(uint32_t raw, uint32_t pos) { return raw << 16 | pos; }
};
template <> struct Staged<uint32_t> {
    typedef unsigned long long word;
    __device__ static uint32_t raw(word w) { return uint32_t(w); }
    __device__ static uint32_t pos(word w) { return uint32_t(w >> 32); }
    __device__ static word make(uint32_t raw, uint32_t pos) { return static_cast<unsigned long long>(pos) << 32 | raw; }
};

// fp32: the sampled form as for 16-bit elements, with a key range of up to 56 bins of 2^16 keys (7 of the sample's 2^19): a
// sample cannot narrow 31-bit keys down to single ones.  The first exchange, the table, tells which bin holds the k-th key and
// how many elements of every chunk it has; few in all (0.2 % of a normal tensor's per bin), so they are exchanged next, as a
// list in flat order, and every workgroup finds the threshold in the list by itself: two exchanges and one read of x, where
// digit histograms (13 + 13 + 5 bits) take three and read the tensor, or its parked head, four times.  A bin of more elements
// than the list holds (large tensors, ties) is histogrammed by the next 11 bits instead, and a second table settles the rest.
// A bracket of 8 to 28 sample bins, as where the threshold lies far below the largest magnitudes, gets bins of 2^17 or 2^18 keys,
// if the sample finds no more elements in a bin of 2^19 than the list holds.
// No bracket, one that fails, or a threshold among the smallest magnitudes: the exact histogram of the first 13 bits gives
// the range, and the same steps follow; for the smallest magnitudes the range is the zeros at first, where a threshold down
// there most likely lies (ReLU): that table alone settles it.
constexpr int SEG32_CAP = 1152;                            // staged elements (8 bytes) per wavefront: 16 segments are 144 KB
constexpr int PART32_OFF = (SEL_THREADS / WAVE) * SEG32_CAP * 8;           // the table's partial sums, the second digit's histogram
constexpr int PART32_WORDS = 2 * (SEL_THREADS / WAVE) * TABLE_PITCH;
constexpr size_t SMEM32_BYTES = PART32_OFF + 4 * size_t(PART32_WORDS);
constexpr int LIST32_PER = 16, LIST32_CAP = LIST32_PER * SEL_THREADS;      // list entries per thread; the list takes the digit histograms' place
constexpr int BITS32_FIRST = 13, BITS32_SECOND = 11;
static_assert(SEG32_CAP >= 2 * 4 * WAVE, "two rows of nothing but candidates fit an empty segment");
static_assert(PART32_OFF >= 4 * ((1 << BITS32_FIRST) + WAVE) && PART32_OFF >= 4 * SAMPLE_BINS, "histograms are done with before anything is staged");
static_assert(PART32_WORDS == 1 << BITS32_SECOND && BITS32_SECOND <= MAX_HIST_BITS, "the second digit's histogram");
static_assert(LIST32_CAP <= 2 << MAX_HIST_BITS, "the two digit histograms hold the list");

__device__ inline SelOutcome select32_body(const uint32_t *__restrict__ x, int64_t numel, int64_t nvf, int64_t vpc, uint32_t k,
                                           SelState *st, uint32_t *hist0, uint32_t *hist1, uint32_t *table,
                                           uint32_t *__restrict__ vals, int32_t *__restrict__ idx, uint32_t spin_limit,
                                           unsigned long long gen, SampleRanks ranks, ExitReport &rep)
{
    constexpr int VEC = 4, ROW_ELEMS = WAVE * VEC;
    constexpr uint32_t MASK = KeyTraits<uint32_t>::MASK;
    constexpr int SAMPLE_SHIFT32 = 31 - 12, BIN_SHIFT = SAMPLE_SHIFT32 - 3;    // a sample bin is eight bins of the table
    constexpr int NW = SEL_THREADS / WAVE;
    typedef unsigned long long word;
    extern __shared__ __attribute__((aligned(16))) u32x4 dyn_smem[];
    uint32_t *lh = reinterpret_cast<uint32_t *>(dyn_smem);                     // (before anything is staged)
    uint32_t *part = reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(dyn_smem) + PART32_OFF);
    __shared__ uint32_t bcast[4], offs[2], verdict;
    __shared__ uint32_t wave_tot[NW];
    __shared__ uint32_t whist[NW][MAX_LAST_BINS + 1];           // per wavefront: its elements in each bin of the range, and above it
    __shared__ __attribute__((aligned(16))) uint32_t digits[3][256];
    __shared__ uint32_t wave_gt[NW], wave_eq[NW], list_gt[NW], list_eq[NW];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const bool last_chunk = blockIdx.x == gridDim.x - 1;
    const u32x4 *xv = reinterpret_cast<const u32x4 *>(x);
    uint32_t *xbar = reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(st) + SelWorkspace::xbar_off);
    uint32_t *list = hist0;                                     // (hist1 follows hist0)

    // development builds only: phase time stamps of one workgroup into the state block's spare words
    [[maybe_unused]] unsigned long long *stamps = reinterpret_cast<unsigned long long *>(st->pad + 4);
#define STAMP(i) DROPIT_DEV_STAMP(stamps, i, tid == 0 && blockIdx.x == gridDim.x / 2)
    STAMP(0);

    // wavefront `wave` owns vectors [wv0, wv1) of the chunk, in rows of 64; ranges start on 128-byte lines
    const int64_t v0 = static_cast<int64_t>(blockIdx.x) * vpc, v1 = min(v0 + vpc, nvf);
    const int64_t vpw = ((vpc + NW - 1) / NW + 7) / 8 * 8;
    const int64_t wv0 = min(v0 + int64_t(wave) * vpw, v1), wv1 = min(wv0 + vpw, v1);
    const int wvecs = static_cast<int>(wv1 - wv0);
    const int nrows = (wvecs + WAVE - 1) / WAVE;
    const uint32_t flat0 = static_cast<uint32_t>(wv0 * VEC);
    const u32x4 *wx = xv + (wv0 < nvf ? wv0 : nvf > 0 ? nvf - 1 : 0);   // (an empty range still has a valid address to load from)
    const int last_vec = max(wvecs - 1, 0);
    word *seg = reinterpret_cast<word *>(dyn_smem) + wave * SEG32_CAP;
    const uint32_t seg_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) word *)seg));
    u32x4 q[ST_ROWS];
    auto issue_row = [&](u32x4 &dst, int row) { dst = wx[min(row * WAVE + lane, last_vec)]; };
    auto issue_rows = [&](int row) {
#pragma unroll
        for (int u = 0; u < ST_ROWS; ++u) issue_row(q[u], row + u);
    };
    const int64_t tail0 = nvf * VEC;                            // the tensor's ragged end belongs to the last chunk, but to no wavefront's range

    const bool sampling = ranks.lo > 0.0f;                      // uniform over the grid
    uint32_t key_lo = 0, nf = 0;                                // the range: nf bins of 2^shift keys from key_lo on
    int shift = BIN_SHIFT;
    bool predicted = false, preloaded = false;
    uint32_t cleared = 0;
    if (blockIdx.x == 0) {
        clear_words(st, xbar, cleared);
        clear_hist(hist0, 2 << MAX_HIST_BITS);                  // (done when this workgroup arrives at its first barrier)
    }
    if (sampling) {
        u32x4 sq[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int s = tid + u * SEL_THREADS;
            sq[u] = xv[sample_piece(s / SAMPLE_STRETCH, nvf) + s % SAMPLE_STRETCH];
        }
        for (int i = tid; i < SAMPLE_BINS; i += SEL_THREADS) lh[i] = 0;
        asm volatile("" : "+v"(sq[0]), "+v"(sq[1]));            // (the rows are asked for once the sample is here)
        issue_rows(0);
        preloaded = true;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 2; ++u)
            for_each_raw(uint32_t(0), sq[u], [&](uint32_t raw, int) {
                const uint32_t dgt = (raw & MASK) >> SAMPLE_SHIFT32;
                if (dgt) atomicAdd(&lh[dgt], 1u);
            });
        if (blockIdx.x == 0) publish_words(st, cleared, gen);
        __syncthreads();
        uint32_t b_lo, b_hi;
        // (a range that reaches down to the smallest keys would make every element a candidate)
        predicted = sample_bracket<SAMPLE_BINS>(lh, ranks, 4 * BRACKET_MAX_BINS, wave_tot, bcast, b_lo, b_hi) && b_lo > 0;
        const uint32_t bins = b_hi - b_lo + 1;
        // wider than the table holds bins of 2^16 keys: bins of 2^17 or 2^18, if the list will hold any of them
        const int wider = bins <= uint32_t(BRACKET_MAX_BINS) ? 0 : bins <= 2 * uint32_t(BRACKET_MAX_BINS) ? 1 : 2;
        if (predicted && wider != 0) {                          // uniform
            const uint32_t most = static_cast<uint32_t>(float(LIST32_CAP) * float(SAMPLE_ELEMS) / static_cast<float>(numel));
            predicted = __syncthreads_or(uint32_t(tid) < bins && lh[b_lo + tid] > most) == 0;
        }
        if (predicted) {
            shift = BIN_SHIFT + wider;
            key_lo = b_lo << SAMPLE_SHIFT32;
            nf = bins << (SAMPLE_SHIFT32 - shift);
        }
    } else if (blockIdx.x == 0) {
        publish_words(st, cleared, gen);
    }
    unsigned long long early = 0;                               // usually the generation number: asked for long before it is needed
    if (tid == 0) early = dev_load64(&st->ready);
    STAMP(1);

    // The rows' candidates (key >= lowest) from row `first` on into the segment, in flat order, with their flat indices;
    // returns the first row that was not staged (nrows, or fewer when the segment is full), n = elements staged.  Rows are
    // staged in pairs.
    auto stage_rows = [&](uint32_t lowest, int first, uint32_t &n) -> int {
        const uint32_t low_s = __builtin_amdgcn_readfirstlane(lowest);
        n = 0;
        if (nrows == 0) return 0;
        if (!preloaded) issue_rows(first);
        preloaded = false;
        int end = nrows;
        for (int row = first; row < end; row += ST_ROWS) {
#pragma unroll
            for (int u = 0; u < ST_ROWS; u += 2) {
                if (row + u < end) {
                    const int left = wvecs - (row + u) * WAVE - lane;              // > 0: the lane's vector of the first row exists
                    const bool in0 = left > 0, in1 = left > WAVE;
                    u32x4 k0, k1;
                    const uint32_t n0 = count_candidates(q[u], low_s, k0, 0u), n1 = count_candidates(q[u + 1], low_s, k1, 0u);
                    const uint32_t c = (in0 ? n0 : 0u) | (in1 ? n1 << 16 : 0u);
                    const uint32_t ex = wave_inclusive_scan(c) - c;
                    const uint32_t tot = uint32_t(__builtin_amdgcn_readlane(int(ex + c), WAVE - 1));
                    const uint32_t t0 = tot & 0xFFFFu, t1 = tot >> 16;
                    if (n + t0 + t1 > uint32_t(SEG32_CAP)) {
                        end = row + u;                                             // full
                    } else {
                        const uint32_t at = flat0 + uint32_t((row + u) * ROW_ELEMS + lane * VEC);
                        stage_candidates(q[u], k0, low_s, __ballot(in0), seg_addr + (n + (ex & 0xFFFFu)) * 8u, at, 0u);
                        stage_candidates(q[u + 1], k1, low_s, __ballot(in1), seg_addr + (n + t0 + (ex >> 16)) * 8u, at + ROW_ELEMS, 0u);
                        n += t0 + t1;
                    }
                }
                issue_row(q[u], row + u + ST_ROWS);
                issue_row(q[u + 1], row + u + 1 + ST_ROWS);
            }
        }
        return end;
    };
    uint32_t n_w = 0;          // staged elements of this wavefront
    int staged_rows = 0;       // the rows they come from: [0, staged_rows)
    // f(key) for the wavefront's candidates: the staged ones, and those of the rows that were not staged, read again
    auto for_candidates = [&](auto f) {
        for (uint32_t j = lane; j < n_w; j += 4 * WAVE) {
            uint32_t raw[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) raw[u] = uint32_t(seg[min(j + u * WAVE, n_w - 1)]);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (j + u * WAVE < n_w) f(raw[u] & MASK);
        }
        if (staged_rows < nrows) {
            issue_rows(staged_rows);
            for (int row = staged_rows; row < nrows; row += ST_ROWS) {
#pragma unroll
                for (int u = 0; u < ST_ROWS; ++u) {
                    if ((row + u) * WAVE + lane < wvecs)
                        for_each_raw(uint32_t(0), q[u], [&](uint32_t raw, int) {
                            if ((raw & MASK) >= key_lo) f(raw & MASK);
                        });
                    issue_row(q[u], row + u + ST_ROWS);
                }
            }
        }
    };
    // Exact counts over the range and above it, the chunk's line of the table, a barrier, the table: false if somebody gave up.
    uint32_t barriers = 0;
    bool ready_seen = false;
    auto exchange_counts = [&]() -> SelOutcome {
        uint32_t *wh = whist[wave];
        if (lane <= static_cast<int>(nf)) wh[lane] = 0;
        uint32_t above = 0;
        const uint32_t bins = nf;
        for_candidates([&](uint32_t key) {
            const uint32_t rel = (key - key_lo) >> shift;      // (a key below the range wraps to a huge one)
            if (key >= key_lo && rel >= bins) ++above;
            if (rel < bins) atomicAdd(&wh[rel], 1u);
        });
        above = wave_sum(above);
        if (lane == 0) wh[nf] = above;
        __syncthreads();
        if (!ready_seen)
            if (const SelOutcome o = wait_published(&st->ready, gen, early, nullptr, &bcast[3])) return o;
        ready_seen = true;
        if (tid <= static_cast<int>(nf)) {
            uint32_t sum = 0;
#pragma unroll
            for (int w2 = 0; w2 < NW; ++w2) sum += whist[w2][tid];
            if (last_chunk)
                for (int64_t i = tail0; i < numel; ++i) {
                    const uint32_t key = x[i] & MASK, rel = (key - key_lo) >> shift;
                    sum += (tid == static_cast<int>(nf) ? key >= key_lo && rel >= nf : key >= key_lo && rel == uint32_t(tid)) ? 1u : 0u;
                }
            dev_store(&table[blockIdx.x * TABLE_PITCH + tid], sum);
        }
        return grid_barrier(st, xbar, ++barriers, spin_limit, &bcast[3]) ? SEL_DONE : SEL_GAVE_UP;
    };

    bool missed = false, first_digit = false;
    for (;;) {
        if (!predicted && first_digit) {               // not the zeros: the smallest magnitudes in 32 bins
            // the table is about to be written again, and others may still be reading it
            if (!grid_barrier(st, xbar, ++barriers, spin_limit, &bcast[3])) return SEL_GAVE_UP;
            nf = 32;
            shift = 31 - BITS32_FIRST - 5;
        } else if (!predicted) {
            // exact first digit: every element of the chunk through an LDS histogram, merged with global atomics
            constexpr int NB = 1 << BITS32_FIRST, SHIFT1 = 31 - BITS32_FIRST;
            if (!missed && blockIdx.x == 0) publish_hist(&st->ready_hist, gen);
            __syncthreads();
            for (int i = tid; i < NB + WAVE; i += SEL_THREADS) lh[i] = 0;
            __syncthreads();
            auto add = [&](uint32_t raw, int) {
                const uint32_t d = (raw & MASK) >> SHIFT1;
                atomicAdd(&lh[d ? d : NB + lane], 1u);                     // exact zeros go to per-lane slots
            };
            int64_t vb = v0;
            for (; vb + SEL_THREADS * SEL_UNROLL <= v1; vb += SEL_THREADS * SEL_UNROLL) {
                u32x4 h[SEL_UNROLL];
#pragma unroll
                for (int u = 0; u < SEL_UNROLL; ++u) h[u] = xv[vb + u * SEL_THREADS + tid];
#pragma unroll
                for (int u = 0; u < SEL_UNROLL; ++u) for_each_raw(uint32_t(0), h[u], add);
            }
            for (int64_t v = vb + tid; v < v1; v += SEL_THREADS) for_each_raw(uint32_t(0), xv[v], add);
            if (last_chunk && tid == 0)
                for (int64_t i = tail0; i < numel; ++i) add(x[i], 0);
            __syncthreads();
            if (tid < WAVE) {
                const uint32_t z = wave_sum(lh[NB + tid]);
                if (tid == 0) lh[0] += z;
            }
            __syncthreads();
            if (!ready_seen)
                if (const SelOutcome o = wait_published(&st->ready, gen, early, nullptr, &bcast[3])) return o;
            ready_seen = true;
            if (!missed)                               // (past a barrier the histograms are known to be cleared)
                if (const SelOutcome o = wait_published(&st->ready_hist, gen, 0ull, &st->error, &bcast[2])) return o;
            for (int i = tid; i < NB; i += SEL_THREADS) {
                const uint32_t c = lh[i];
                if (c) atomicAdd(&hist0[i], c);
            }
            if (!grid_barrier(st, xbar, ++barriers, spin_limit, &bcast[3])) return SEL_GAVE_UP;
            uint32_t prefix = 0, k_rem = k;
            resolve_digit_local<NB, BITS32_FIRST>(hist0, prefix, k_rem, wave_tot, bcast);
            first_digit = true;
            key_lo = prefix << SHIFT1;
            nf = prefix ? 32 : 1;                      // among the smallest magnitudes it is most likely a zero
            shift = prefix ? SHIFT1 - 5 : 0;
        }
        STAMP(2);
        staged_rows = stage_rows(key_lo, 0, n_w);
        STAMP(3);
        if (const SelOutcome o = exchange_counts()) return o;
        STAMP(5);
        // (a bin wider than 2^16 keys is settled by the list alone)
        if (resolve_table(table, nf, 0u, k, part, bcast, offs, &verdict, xbar, rep, false) &&
            (shift <= BIN_SHIFT || bcast[2] <= uint32_t(LIST32_CAP)))
            break;
        if (!predicted && shift != 0) return SEL_GAVE_UP;      // cannot happen with an exact digit; the serial path would still answer
        missed |= predicted;                     // the sample misled: once more with the exact histogram
        predicted = false;
    }
    // The k-th key is the k_rem-th largest of the `left` keys in bin `bin`; offs: the chunks before this one, above that bin
    // and in it.
    const uint32_t bin = bcast[0], left = bcast[2];
    uint32_t k_rem = bcast[1];
    const uint32_t above_before = offs[0], in_before = offs[1];
    const uint32_t bin_lo = key_lo + (bin << shift), bin_size = 1u << shift;
    uint32_t t, m, my_gt, my_eq, chunk_gt, chunk_eq, wave_eq_mine;
    if (shift != 0 && left <= uint32_t(LIST32_CAP)) {
        // ---- the bin's keys as a list in flat order ----
        uint32_t before = 0, mine = whist[wave][bin], all = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            before += w < wave ? whist[w][bin] : 0u;
            all += whist[w][bin];
        }
        const uint32_t own = in_before + before;                 // this wavefront's first entry
        uint32_t at = own;
        auto put = [&](bool in, uint32_t rel) {                   // in lane order
            const lane_mask b = __ballot(in);
            if (in) {
                const uint32_t pos = bits_before(b, at);
                if (pos < uint32_t(LIST32_CAP)) dev_store(&list[pos], rel);     // (always, for consistent counts)
            }
            at += uint32_t(__builtin_popcountll(b));
        };
        for (uint32_t q0 = 0; q0 < n_w; q0 += WAVE) {
            const uint32_t rel = (uint32_t(seg[min(q0 + lane, n_w - 1)]) & MASK) - bin_lo;
            put(q0 + lane < n_w && rel < bin_size, rel);
        }
        for (int row = staged_rows; row < nrows; ++row) {         // (element by element of 64 vectors: the order within a
            u32x4 v;                                              // wavefront's share of the list does not matter)
            issue_row(v, row);
            const bool there = row * WAVE + lane < wvecs;
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const uint32_t rel = (v[e] & MASK) - bin_lo;
                put(there && rel < bin_size, rel);
            }
        }
        if (last_chunk && tid == 0) {
            uint32_t pos = in_before + all;
            for (int64_t i = tail0; i < numel; ++i) {
                const uint32_t rel = (x[i] & MASK) - bin_lo;
                if (rel < bin_size && pos < uint32_t(LIST32_CAP)) dev_store(&list[pos++], rel);
            }
        }
        if (tid < 3 * 256) digits[tid >> 8][tid & 255] = 0u;
        if (!grid_barrier(st, xbar, ++barriers, spin_limit, &bcast[3])) return SEL_GAVE_UP;
        STAMP(6);
        uint32_t e[LIST32_PER], mine0 = 0;
#pragma unroll
        for (int j = 0; j < LIST32_PER; ++j)
            if (uint32_t(j * SEL_THREADS + tid) < left) e[j] = dev_load(list + j * SEL_THREADS + tid);
        if (uint32_t(lane) < mine) mine0 = dev_load(list + own + lane);
        report_past_barriers(xbar, rep, false);
        // two digits of 8 bits, and what a wider bin leaves; every wavefront resolves each for itself, a lane four bins in
        // descending order
        uint32_t rel_t = 0;
        int rem = shift;
        auto next_digit = [&](int pass) {
            const int take = min(rem, 8), low = rem - take;
#pragma unroll
            for (int j = 0; j < LIST32_PER; ++j) {
                const bool in = uint32_t(j * SEL_THREADS + tid) < left && (pass == 0 || e[j] >> rem == rel_t);
                const lane_mask some = __ballot(in);
                if (some == 0) continue;
                // ties: one addition for a wavefront of the same digit (14 K equal entries took 20 us one by one)
                const uint32_t d = in ? (e[j] >> low) & ((1u << take) - 1u) : 0u;
                const int leader = __builtin_ctzll(some);
                const uint32_t d0 = uint32_t(__builtin_amdgcn_readlane(int(d), leader));
                if (__ballot(in && d != d0) != 0) {
                    if (in) atomicAdd(&digits[pass][d], 1u);
                } else if (lane == leader) {
                    atomicAdd(&digits[pass][d0], uint32_t(__builtin_popcountll(some)));
                }
            }
            __syncthreads();
            const u32x4 d4 = reinterpret_cast<const u32x4 *>(digits[pass])[WAVE - 1 - lane];
            const uint32_t c[4] = {d4[3], d4[2], d4[1], d4[0]}, sum = c[0] + c[1] + c[2] + c[3];
            const uint32_t inc = wave_inclusive_scan(sum);
            uint32_t a = inc - sum, digit = 0, rest = 0;
            const lane_mask hit = __ballot(a < k_rem && k_rem <= inc);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (a < k_rem && k_rem <= a + c[i]) {
                    digit = uint32_t((WAVE - 1 - lane) * 4 + 3 - i);
                    rest = k_rem - a;
                }
                a += c[i];
            }
            const int finder = hit ? __builtin_ctzll(hit) : 0;    // (always found)
            rel_t = rel_t << take | uint32_t(__builtin_amdgcn_readlane(int(digit), finder));
            k_rem = uint32_t(__builtin_amdgcn_readlane(int(rest), finder));
            rem = low;
        };
        next_digit(0);
        next_digit(1);
        if (__builtin_expect(rem > 0, 0)) next_digit(2);         // uniform
        t = bin_lo + rel_t;
        m = k_rem;
        // above and equal to t: in the list before this chunk, in this wavefront's own entries and above the bin
        uint32_t lg = 0, le = 0, g = 0, eq = 0;
#pragma unroll
        for (int j = 0; j < LIST32_PER; ++j) {
            const uint32_t i = uint32_t(j * SEL_THREADS + tid);
            if (i < left && i < in_before) {
                lg += e[j] > rel_t ? 1u : 0u;
                le += e[j] == rel_t ? 1u : 0u;
            }
        }
        for (uint32_t j = lane; j < mine; j += WAVE) {
            const uint32_t v = j == uint32_t(lane) ? mine0 : dev_load(list + own + j);
            g += v > rel_t ? 1u : 0u;
            eq += v == rel_t ? 1u : 0u;
        }
        if (uint32_t(lane) <= nf && uint32_t(lane) > bin) g += whist[wave][lane];           // (bin nf: above the range)
        lg = wave_sum(lg);
        le = wave_sum(le);
        g = wave_sum(g);
        eq = wave_sum(eq);
        if (lane == 0) {
            list_gt[wave] = lg;
            list_eq[wave] = le;
            wave_gt[wave] = g;
            wave_eq[wave] = eq;
        }
        __syncthreads();
        const uint32_t gw = lane < NW ? wave_gt[lane] : 0u, ew = lane < NW ? wave_eq[lane] : 0u;
        const uint32_t gi = wave_inclusive_scan(gw), ei = wave_inclusive_scan(ew);
        const uint32_t gt0 = above_before + wave_sum(lane < NW ? list_gt[lane] : 0u), eq0 = wave_sum(lane < NW ? list_eq[lane] : 0u);
        my_gt = gt0 + uint32_t(__builtin_amdgcn_readlane(int(gi - gw), wave));
        my_eq = eq0 + uint32_t(__builtin_amdgcn_readlane(int(ei - ew), wave));
        wave_eq_mine = uint32_t(__builtin_amdgcn_readlane(int(ew), wave));
        chunk_gt = gt0 + uint32_t(__builtin_amdgcn_readlane(int(gi), NW - 1));
        chunk_eq = eq0 + uint32_t(__builtin_amdgcn_readlane(int(ei), NW - 1));
    } else {
        if (shift != 0) {
            // ---- the bin's next 11 bits from a histogram, then single keys from a second table ----
            const int low = shift - BITS32_SECOND;                    // 5 or 2 bits are left after it
            for (int i = tid; i < PART32_WORDS; i += SEL_THREADS) part[i] = 0;
            __syncthreads();
            for_candidates([&](uint32_t key) {
                const uint32_t rel = key - bin_lo;
                if (rel < bin_size) atomicAdd(&part[rel >> low], 1u);
            });
            if (last_chunk && tid == 0)
                for (int64_t i = tail0; i < numel; ++i) {
                    const uint32_t rel = (x[i] & MASK) - bin_lo;
                    if (rel < bin_size) atomicAdd(&part[rel >> low], 1u);
                }
            __syncthreads();
            for (int i = tid; i < PART32_WORDS; i += SEL_THREADS) {
                const uint32_t c = part[i];
                if (c) atomicAdd(&hist1[i], c);
            }
            if (!grid_barrier(st, xbar, ++barriers, spin_limit, &bcast[3])) return SEL_GAVE_UP;
            uint32_t digit = 0;
            resolve_digit_local<1 << BITS32_SECOND, BITS32_SECOND>(hist1, digit, k_rem, wave_tot, bcast);
            key_lo = bin_lo + (digit << low);
            nf = 1u << low;
            shift = 0;
            if (const SelOutcome o = exchange_counts()) return o;
            if (!resolve_table(table, nf, 0u, k, part, bcast, offs, &verdict, xbar, rep, true)) return SEL_GAVE_UP;   // cannot happen
        } else {
            report_past_barriers(xbar, rep, false);              // (bins of one key)
        }
        t = key_lo + bcast[0];
        m = bcast[1];
        const uint32_t trel = bcast[0];
        uint32_t g = 0, eq = 0;
        if (lane < NW) {
            g = whist[lane][nf];
            for (uint32_t r = trel + 1; r < nf; ++r) g += whist[lane][r];
            eq = whist[lane][trel];
        }
        const uint32_t gi = wave_inclusive_scan(g), ei = wave_inclusive_scan(eq);
        my_gt = offs[0] + uint32_t(__builtin_amdgcn_readlane(int(gi - g), wave));
        my_eq = offs[1] + uint32_t(__builtin_amdgcn_readlane(int(ei - eq), wave));
        wave_eq_mine = uint32_t(__builtin_amdgcn_readlane(int(eq), wave));
        chunk_gt = offs[0] + uint32_t(__builtin_amdgcn_readlane(int(gi), NW - 1));
        chunk_eq = offs[1] + uint32_t(__builtin_amdgcn_readlane(int(ei), NW - 1));
    }
    if (tid == REPORT_TID && blockIdx.x == 0) {
        dev_store(&st->form, 0u);                                 // (what these two words say is for 16-bit tensors)
        dev_store(&st->path, 0u);
        dev_store(&st->form32, (missed ? 2u : predicted ? 1u : 0u) + (left <= uint32_t(LIST32_CAP) ? 0u : 4u));
    }
    STAMP(7);

    // ---- ordered output, as for 16-bit elements -----------------------------------
    auto keep = [&](uint32_t pos, uint32_t raw, uint32_t i) {
        if (pos < k) {                     // always true for consistent counts
            vals[pos] = raw;
            idx[pos] = static_cast<int32_t>(i);
        }
    };
    const bool split = my_eq < m && my_eq + wave_eq_mine > m;
    const uint32_t least = my_eq < m ? t : t + 1;      // lowest key kept (if not split)
    uint32_t my_slot = my_gt + min(my_eq, m);
    for (;;) {
        for (uint32_t q0 = 0; q0 < n_w; q0 += 4 * WAVE) {
            word w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = seg[min(q0 + j * WAVE + lane, n_w - 1)];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t raw = uint32_t(w[j]), key = raw & MASK;
                const bool there = q0 + j * WAVE + lane < n_w;
                if (!split) {              // uniform over the wavefront
                    const bool kept = there && key >= least;
                    const lane_mask b = __ballot(kept);
                    if (kept) keep(bits_before(b, my_slot), raw, uint32_t(w[j] >> 32));
                    my_slot += __builtin_popcountll(b);
                } else {
                    const bool gt = there && key > t, eq = there && key == t;
                    const lane_mask bg = __ballot(gt), be = __ballot(eq);
                    const uint32_t eb = bits_before(be, my_eq), gb = bits_before(bg, my_gt);
                    if (gt || (eq && eb < m)) keep(gb + min(eb, m), raw, uint32_t(w[j] >> 32));
                    my_gt += __builtin_popcountll(bg);
                    my_eq += __builtin_popcountll(be);
                }
            }
        }
        if (staged_rows >= nrows) break;
        staged_rows = stage_rows(t, staged_rows, n_w);            // the rows that did not fit: only what is kept is staged now
    }
    if (last_chunk && tid == 0) {
        uint32_t run_gt = chunk_gt, run_eq = chunk_eq;
        for (int64_t i = tail0; i < numel; ++i) {
            const uint32_t raw = x[i], key = raw & MASK;
            if (key > t) {
                keep(run_gt + min(run_eq, m), raw, static_cast<uint32_t>(i));
                ++run_gt;
            } else if (key == t) {
                if (run_eq < m) keep(run_gt + run_eq, raw, static_cast<uint32_t>(i));
                ++run_eq;
            }
        }
    }
#undef STAMP
    return SEL_DONE;
}

// The whole selection by ONE workgroup, phase after phase over the whole tensor: same digits,
// same slot formula, histograms in LDS, nothing read from the workspace.  Only ever runs after
// the parallel path gave up.  `lh` is LDS scratch of (1 << 13) + 2 * WAVE words.
template <typename RAW>
__device__ inline void select_serial(const RAW *__restrict__ x, int64_t numel, int64_t nvf, uint32_t k,
                                     RAW *__restrict__ vals, int32_t *__restrict__ idx, uint32_t *lh,
                                     uint32_t *wave_tot, uint32_t *bcast)
{
    constexpr int VEC = KeyTraits<RAW>::VEC;
    constexpr uint32_t MASK = KeyTraits<RAW>::MASK;
    constexpr bool F32 = sizeof(RAW) == 4;
    constexpr int LAST_BITS = F32 ? 5 : 4;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const u32x4 *xv = reinterpret_cast<const u32x4 *>(x);
    auto for_all = [&](auto f) {
        for (int64_t v = tid; v < nvf; v += SEL_THREADS)
            for_each_raw(RAW(0), xv[v], [&](uint32_t raw, int) { f(raw); });
        if (tid == 0)
            for (int64_t i = nvf * VEC; i < numel; ++i) f(x[i]);
    };
    uint32_t prefix = 0, k_rem = k;
    auto pass = [&](auto shift_c, auto bits_c, auto first_c) {
        constexpr int SHIFT = decltype(shift_c)::value, BITS = decltype(bits_c)::value;
        constexpr bool FIRST = decltype(first_c)::value;
        constexpr int NB = 1 << BITS;
        __syncthreads();
        for (int i = tid; i < NB + 2 * WAVE; i += SEL_THREADS) lh[i] = 0;
        __syncthreads();
        const uint32_t zslot = NB + lane, dslot = NB + WAVE + lane;
        for_all([&](uint32_t raw) {
            const uint32_t key = raw & MASK;
            const uint32_t d = (key >> SHIFT) & (NB - 1);
            uint32_t a = d ? d : zslot;
            if (!FIRST) a = ((key >> (SHIFT + BITS)) == prefix) ? a : dslot;
            atomicAdd(&lh[a], 1u);
        });
        __syncthreads();
        if (tid < WAVE) {
            const uint32_t z = wave_sum(lh[NB + tid]);
            if (tid == 0) lh[0] += z;
        }
        __syncthreads();
        resolve_digit_local<NB, BITS>(lh, prefix, k_rem, wave_tot, bcast);
    };
    if constexpr (F32) {
        pass(std::integral_constant<int, 18>{}, std::integral_constant<int, 13>{}, std::true_type{});
        pass(std::integral_constant<int, 5>{}, std::integral_constant<int, 13>{}, std::false_type{});
    } else {
        pass(std::integral_constant<int, 4>{}, std::integral_constant<int, 11>{}, std::true_type{});
    }
    pass(std::integral_constant<int, 0>{}, std::integral_constant<int, LAST_BITS>{}, std::false_type{});
    const uint32_t t = prefix, m = k_rem;   // all digits resolved: the threshold key and its tie budget

    uint32_t run_gt = 0, run_eq = 0;
    auto keep = [&](uint32_t pos, uint32_t raw, int64_t i) {
        if (pos < k) {
            vals[pos] = static_cast<RAW>(raw);
            idx[pos] = static_cast<int32_t>(i);
        }
    };
    for (int64_t vb = 0; vb < nvf; vb += SEL_THREADS) {
        const int64_t v = vb + tid;
        const bool live = v < nvf;
        u32x4 q = u32x4{0, 0, 0, 0};
        if (live) q = xv[v];
        uint32_t cnt = 0;                  // low 16 bits: #gt, high 16 bits: #eq (tile <= 8192 elements)
        for_each_raw(RAW(0), q, [&](uint32_t raw, int) {
            const uint32_t key = raw & MASK;
            cnt += (key > t ? 1u : 0u) + (key == t ? 0x10000u : 0u);
        });
        if (!live) cnt = 0;
        uint32_t total;
        const uint32_t excl = block_exclusive_scan<SEL_THREADS>(cnt, wave_tot, total);
        uint32_t my_gt = run_gt + (excl & 0xFFFFu);
        uint32_t my_eq = run_eq + (excl >> 16);
        if (cnt) {
            for_each_raw(RAW(0), q, [&](uint32_t raw, int e) {
                const uint32_t key = raw & MASK;
                const bool gt = key > t, eq = key == t;
                if (gt || (eq && my_eq < m)) keep(my_gt + min(my_eq, m), raw, v * VEC + e);
                my_gt += gt ? 1u : 0u;
                my_eq += eq ? 1u : 0u;
            });
        }
        run_gt += total & 0xFFFFu;
        run_eq += total >> 16;
    }
    if (tid == 0) {
        for (int64_t i = nvf * VEC; i < numel; ++i) {
            const RAW raw = x[i];
            const uint32_t key = raw & MASK;
            const bool gt = key > t, eq = key == t;
            if (gt || (eq && run_eq < m)) keep(run_gt + min(run_eq, m), raw, i);
            run_gt += gt ? 1u : 0u;
            run_eq += eq ? 1u : 0u;
        }
    }
}

// ---- small tensors: one workgroup, everything in registers ------------------------------------------
// Up to SMALL_VECTORS 16-byte vectors per thread (32 K fp32 or 64 K 16-bit elements): the tensor is read
// once into registers and the whole selection -- the same tie rule and slot formula as above --
// runs in ONE workgroup with workgroup barriers only.  No workspace, no grid barrier, no residency
// question.  Bound by the instructions of one compute unit: a vector instruction per element is 0.1 us for 16 K elements, an
// LDS atomic per element 2 us, and digit histograms over all elements (13 + 13 + 5 bits for fp32) were three of those.
// Instead one element of every vector is histogrammed (4096 bins, the key's upper 12 bits), which gives a bracket of the
// k-th key as the sample of the large form does; what is not below it, little more than k elements, is staged in LDS in
// flat order, a segment per wavefront and its contiguous range, and everything after that -- the counts that confirm the
// bracket, the digits of the threshold (10 bits at a time; 64 elements or fewer are ranked by a wavefront), the output --
// walks the staged words.  Rows of 64 vectors that the segment does not hold are read again for each of these, and staged
// when it has been written out.  A bracket that fails, and small tensors, take the bin of the exact histogram.
// fp32 of 16 K elements at gamma 0.9 13.2 -> 9.2 us, 32 K 20.0 -> 11.9; 16-bit 32 K 14.2 -> 10.8; all magnitudes equal, fp32
// of 16 K 25.4 -> 22.3.
constexpr int SMALL_VECTORS = 8;
constexpr int SMALL_BINS = 4096, SMALL_DIGIT = 10;
constexpr int SMALL_SAMPLE_MIN = 2048;                         // vectors: below, all elements are as quickly histogrammed
constexpr int SMALL_SEG_BYTES = 9216;                          // per wavefront, at most: 1152 staged fp32 elements, 2304 16-bit ones
template <typename RAW>
inline uint32_t small_cap(int nvf)                             // staged words per wavefront: as many as its range has elements, if they fit
{
    constexpr int VEC = KeyTraits<RAW>::VEC, NW = SEL_THREADS / WAVE;
    const int most = SMALL_SEG_BYTES / int(sizeof(typename Staged<RAW>::word));
    static_assert(SMALL_SEG_BYTES / int(sizeof(typename Staged<RAW>::word)) >= WAVE * VEC + VEC, "a row and a ragged end");
    const int vectors = std::max((nvf + NW - 1) / NW + 3, WAVE) + 1;
    return uint32_t(std::min(vectors * VEC / 4 * 4, most));
}

template <typename RAW>
__global__ void __launch_bounds__(SEL_THREADS)
select_small_kernel(const RAW *__restrict__ x, int numel, int nvf, uint32_t k, SampleRanks ranks, uint32_t cap,
                    RAW *__restrict__ vals, int32_t *__restrict__ idx)
{
    constexpr int VEC = KeyTraits<RAW>::VEC;
    constexpr uint32_t MASK = KeyTraits<RAW>::MASK;
    constexpr int SHIFT = (sizeof(RAW) == 4 ? 31 : 15) - 12;
    constexpr int NW = SEL_THREADS / WAVE;
    typedef typename Staged<RAW>::word word;
    static_assert(SMALL_BINS == 4 * SEL_THREADS && (1 << SMALL_DIGIT) == SEL_THREADS, "four bins, one digit bin per thread");
    extern __shared__ __attribute__((aligned(16))) u32x4 dyn_smem[];
    uint32_t *lh = reinterpret_cast<uint32_t *>(dyn_smem);
    __shared__ uint32_t digit_bins[1 << SMALL_DIGIT], few[WAVE];
    __shared__ uint32_t wave_tot[2][NW], wave_gt[NW], wave_eq[NW];
    __shared__ uint32_t bcast[4], in_n, above_n, few_n;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const u32x4 *xv = reinterpret_cast<const u32x4 *>(x);
    word *seg = reinterpret_cast<word *>(dyn_smem) + wave * cap;      // `cap` staged words: a row of candidates and a ragged end at least
    const uint32_t seg_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) word *)seg));

    // wavefront `wave` owns vectors [wv0, wv0 + wvecs), in rows of 64; the last one also the ragged end, an element per lane
    const int vpw = ((nvf + NW - 1) / NW + 3) / 4 * 4;
    const int wv0 = min(wave * vpw, nvf), wvecs = min(wv0 + vpw, nvf) - wv0;
    const int nrows = (wvecs + WAVE - 1) / WAVE;                    // <= SMALL_VECTORS (checked by the host)
    const int ntail = wave == NW - 1 ? numel - nvf * VEC : 0;
    u32x4 q[SMALL_VECTORS];
#pragma unroll
    for (int i = 0; i < SMALL_VECTORS; ++i)
        q[i] = i * WAVE + lane < wvecs ? xv[wv0 + i * WAVE + lane] : u32x4{0u, 0u, 0u, 0u};
    const uint32_t tail = lane < ntail ? uint32_t(x[nvf * VEC + lane]) : 0u;
    auto load_row = [&](int i) { return i * WAVE + lane < wvecs ? xv[wv0 + i * WAVE + lane] : u32x4{0u, 0u, 0u, 0u}; };
    // f(key) for the elements of the rows from `first` on and of the ragged end, the rows read again: a loop over the
    // registers would be unrolled eight-fold wherever it is used, and fetching instructions bounds the smallest tensors
    auto for_rows = [&](int first, auto f) {
#pragma nounroll
        for (int i = first; i < nrows; ++i) {
            const u32x4 v = load_row(i);
            if (i * WAVE + lane < wvecs) for_each_raw(RAW(0), v, [&](uint32_t raw, int) { f(raw & MASK); });
        }
        if (lane < ntail) f(tail & MASK);
    };
    // counts of a thread's bins, the workgroup's bins in descending order: what lies above the thread's
    auto above_mine = [&](uint32_t mine, int slot, uint32_t &total) -> uint32_t {
        const uint32_t inc = wave_inclusive_scan(mine);
        if (lane == WAVE - 1) wave_tot[slot][wave] = inc;
        __syncthreads();
        const uint32_t t = lane < NW ? wave_tot[slot][lane] : 0u, tinc = wave_inclusive_scan(t);
        total = uint32_t(__builtin_amdgcn_readlane(int(tinc), WAVE - 1));
        return uint32_t(__builtin_amdgcn_readlane(int(tinc - t), wave)) + inc - mine;
    };
    // The candidates (key >= lowest) of row i, v, behind the n words of the segment; false if it does not hold them.
    uint32_t n = 0;
    auto stage_row = [&](const u32x4 &v, int i, uint32_t lowest) -> bool {
        const bool there = i * WAVE + lane < wvecs;
        u32x4 keys;
        const uint32_t cn = count_candidates(v, lowest, keys, RAW(0)), c = there ? cn : 0u;
        const uint32_t inc = wave_inclusive_scan(c);
        const uint32_t total = uint32_t(__builtin_amdgcn_readlane(int(inc), WAVE - 1));
        if (n + total > cap) return false;
        stage_candidates(v, keys, lowest, __ballot(there), seg_addr + (n + inc - c) * uint32_t(sizeof(word)),
                         uint32_t((i * WAVE + lane) * VEC), RAW(0));
        n += total;
        return true;
    };
    auto stage_tail = [&](uint32_t lowest) -> bool {
        const bool in = lane < ntail && (tail & MASK) >= lowest;
        const lane_mask b = __ballot(in);
        const uint32_t total = uint32_t(__builtin_popcountll(b));
        if (n + total > cap) return false;
        if (in) seg[bits_before(b, n)] = Staged<RAW>::make(tail, uint32_t(wvecs * VEC + lane));
        n += total;
        return true;
    };

    uint32_t lo = 0, width = 0, k_rem = k, left = 0;  // keys [lo, lo + width) hold the k-th largest: the k_rem-th largest of the `left` in it
    bool sampled = ranks.lo > 0.0f;                   // uniform
    int staged_rows = 0;                              // rows from here on are not in the segment; the ragged end counts as row nrows
    // f(key) for the wavefront's elements with key >= lo
    auto for_candidates = [&](auto f) {
        for (uint32_t j = lane; j < n; j += WAVE) f(Staged<RAW>::raw(seg[j]) & MASK);
        if (staged_rows <= nrows) for_rows(staged_rows, [&](uint32_t key) { if (key >= lo) f(key); });
    };
    for (;;) {
        reinterpret_cast<u32x4 *>(lh)[tid] = u32x4{0u, 0u, 0u, 0u};
        digit_bins[tid] = 0u;
        if (tid == 0) in_n = above_n = few_n = 0u;
        __syncthreads();
        auto count = [&](uint32_t key) {
            if (key >> SHIFT) atomicAdd(&lh[key >> SHIFT], 1u);      // bin 0, the zeros, holds what the others leave
        };
        if (sampled) {
#pragma unroll
            for (int i = 0; i < SMALL_VECTORS; ++i)
                if (i * WAVE + lane < wvecs) {                       // one element of each vector, another one from vector to vector
                    const uint32_t e = uint32_t(lane + (lane >> 3) + i) % VEC;
                    if constexpr (VEC == 4) {
                        const uint32_t a = e & 1 ? q[i][1] : q[i][0], b = e & 1 ? q[i][3] : q[i][2];
                        count((e & 2 ? b : a) & MASK);
                    } else {
                        const uint32_t a = e & 2 ? q[i][1] : q[i][0], b = e & 2 ? q[i][3] : q[i][2];
                        count((e & 4 ? b : a) >> (e & 1 ? 16 : 0) & MASK);
                    }
                }
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (i * WAVE + lane < wvecs) for_each_raw(RAW(0), q[i], [&](uint32_t raw, int) { count(raw & MASK); });
            for_rows(2, count);
        }
        __syncthreads();
        uint32_t c[4], total;
        {
            const u32x4 w = reinterpret_cast<const u32x4 *>(lh)[SEL_THREADS - 1 - tid];
#pragma unroll
            for (int i = 0; i < 4; ++i) c[i] = w[3 - i];
        }
        const int hi_bin = SMALL_BINS - 1 - tid * 4;
        const uint32_t mine = c[0] + c[1] + c[2] + c[3];
        const uint32_t above = above_mine(mine, 0, total);
        const uint32_t rank[2] = {sampled ? uint32_t(ranks.lo) : k, sampled ? uint32_t(ranks.hi) + 1u : k};   // higher bin first
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            if (tid == 0 && rank[r] > total) {
                bcast[r] = 0u;
                bcast[2] = k - total;
                bcast[3] = uint32_t(numel) - total;
            }
            if (above < rank[r] && rank[r] <= above + mine) {
                uint32_t a = above;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (a < rank[r] && rank[r] <= a + c[i]) {
                        bcast[r] = uint32_t(hi_bin - i);
                        bcast[2] = k - a;              // (of the exact histogram; a sample's mean nothing)
                        bcast[3] = c[i];
                    }
                    a += c[i];
                }
            }
        }
        __syncthreads();                               // (also: the histogram is read, its place is the segments')
        lo = bcast[1] << SHIFT;
        width = (bcast[0] - bcast[1] + 1u) << SHIFT;
        const uint32_t low_s = __builtin_amdgcn_readfirstlane(lo);
        n = 0;
        bool fits = true;
        staged_rows = 0;
#pragma unroll
        for (int i = 0; i < SMALL_VECTORS; ++i)
            if (fits && i < nrows) {                   // uniform over the wavefront
                fits = stage_row(q[i], i, low_s);
                staged_rows += fits ? 1 : 0;
            }
        if (fits && stage_tail(low_s)) staged_rows = nrows + 1;
        if (!sampled) {
            k_rem = bcast[2];
            left = bcast[3];
            break;
        }
        uint32_t in_range = 0, above_range = 0;
        for_candidates([&](uint32_t key) {
            in_range += key - lo < width ? 1u : 0u;
            above_range += key - lo < width ? 0u : 1u;
        });
        in_range = wave_sum(in_range);
        above_range = wave_sum(above_range);
        if (lane == 0) {
            atomicAdd(&in_n, in_range);
            atomicAdd(&above_n, above_range);
        }
        __syncthreads();
        k_rem = k - above_n;
        left = in_n;
        if (above_n < k && k_rem <= left) break;
        sampled = false;                               // the sample misled
        __syncthreads();                               // everybody has read the counts
    }

    // the digits of the k_rem-th largest key of the range, ten bits at a time
    auto for_range = [&](auto f) {
        for_candidates([&](uint32_t key) { if (key - lo < width) f(key - lo); });
    };
    int rem = 32 - __builtin_clz(width - 1u);          // bits of a key's distance from lo that are not known yet (width is 8 at least)
    uint32_t prefix = 0;
    for (bool again = false; rem > 0; again = true) {
        const int take = min(rem, SMALL_DIGIT), shift = rem - take;
        if (again) {
            digit_bins[tid] = 0u;
            __syncthreads();
        }
        for_range([&](uint32_t rel) {
            const uint32_t digit = (rel >> shift) & ((1u << take) - 1u);
            // (0 is what the others leave of `left`: zeros, and values that fill the upper bits only, would crowd it)
            if ((!again || rel >> rem == prefix) && digit != 0) atomicAdd(&digit_bins[digit], 1u);
        });
        __syncthreads();
        const uint32_t cnt = digit_bins[SEL_THREADS - 1 - tid];
        uint32_t total;
        const uint32_t above = above_mine(cnt, 1, total);
        if (tid == 0 && k_rem > total) {
            bcast[0] = 0u;
            bcast[1] = k_rem - total;
            bcast[2] = left - total;
        }
        if (above < k_rem && k_rem <= above + cnt) {
            bcast[0] = uint32_t(SEL_THREADS - 1 - tid);
            bcast[1] = k_rem - above;
            bcast[2] = cnt;
        }
        __syncthreads();
        prefix = prefix << take | bcast[0];
        k_rem = bcast[1];
        rem = shift;
        left = bcast[2];
        if (rem > 0 && left <= uint32_t(WAVE)) {       // uniform: every wavefront ranks what is left
            for_range([&](uint32_t rel) {
                if (rel >> rem == prefix) few[atomicAdd(&few_n, 1u) & (WAVE - 1)] = rel;
            });
            __syncthreads();
            const uint32_t own = few[lane];
            uint32_t gt = 0, eq = 0;
            for (uint32_t j = 0; j < left; ++j) {
                const uint32_t other = uint32_t(__builtin_amdgcn_readlane(int(own), int(j)));
                gt += other > own ? 1u : 0u;
                eq += other == own ? 1u : 0u;
            }
            const lane_mask hit = __ballot(uint32_t(lane) < left && gt < k_rem && k_rem <= gt + eq);
            const int at = hit ? __builtin_ctzll(hit) : 0;                 // (always found)
            prefix = uint32_t(__builtin_amdgcn_readlane(int(own), at));
            k_rem -= uint32_t(__builtin_amdgcn_readlane(int(gt), at));
            rem = 0;
        }
        if (rem > 0) __syncthreads();                  // bins and broadcast words are read
    }
    const uint32_t t = lo + prefix, m = k_rem;         // the threshold key and its tie budget

    // ordered output: slot = #gt-before + min(#eq-before, m)
    uint32_t g = 0, e = 0;
    for_candidates([&](uint32_t key) {
        g += key > t ? 1u : 0u;
        e += key == t ? 1u : 0u;
    });
    g = wave_sum(g);
    e = wave_sum(e);
    if (lane == 0) {
        wave_gt[wave] = g;
        wave_eq[wave] = e;
    }
    __syncthreads();
    const uint32_t og = lane < wave ? wave_gt[lane] : 0u, oe = lane < wave ? wave_eq[lane] : 0u;      // (wave < NW)
    uint32_t my_gt = wave_sum(og), my_eq = wave_sum(oe);
    auto keep = [&](uint32_t pos, word w) {
        if (pos < k) {                                 // always true for consistent counts
            vals[pos] = static_cast<RAW>(Staged<RAW>::raw(w));
            idx[pos] = static_cast<int32_t>(uint32_t(wv0 * VEC) + Staged<RAW>::pos(w));
        }
    };
    for (;;) {
        for (uint32_t q0 = 0; q0 < n; q0 += WAVE) {    // 64 words in lane order: neighbouring lanes write neighbouring slots
            const bool there = q0 + lane < n;
            const word w = there ? seg[q0 + lane] : word(0);
            const uint32_t key = Staged<RAW>::raw(w) & MASK;
            const bool gt = there && key > t, eq = there && key == t;
            const lane_mask bg = __ballot(gt), be = __ballot(eq);
            const uint32_t eb = bits_before(be, my_eq), gb = bits_before(bg, my_gt);
            if (gt || (eq && eb < m)) keep(gb + min(eb, m), w);
            my_gt += uint32_t(__builtin_popcountll(bg));
            my_eq += uint32_t(__builtin_popcountll(be));
        }
        if (staged_rows > nrows) break;
        const uint32_t t_s = __builtin_amdgcn_readfirstlane(t);
        n = 0;                                         // what did not fit: only what can be kept now
        while (staged_rows < nrows && stage_row(load_row(staged_rows), staged_rows, t_s)) ++staged_rows;
        if (staged_rows == nrows && stage_tail(t_s)) staged_rows = nrows + 1;
    }
}

// The same with digit histograms over all elements (11 + 4 bits, fp32 13 + 13 + 5), PER rows of a vector per thread, written row
// by row: the shorter program, which is all that counts up to 16 K 16-bit elements, and the one whose time depends least on
// the values, which counts where much is kept: the form above stages all of that, and reads again what does not fit.
constexpr int ROW_VECTORS = 3 * SEL_THREADS;               // the most that 16-bit tensors come with
template <typename RAW, int PER>
__global__ void __launch_bounds__(SEL_THREADS)
select_row_kernel(const RAW *__restrict__ x, int numel, int nvf, uint32_t k, RAW *__restrict__ vals, int32_t *__restrict__ idx)
{
    constexpr int VEC = KeyTraits<RAW>::VEC, KEY_BITS = sizeof(RAW) == 4 ? 31 : 15, FIRST_BITS = sizeof(RAW) == 4 ? 13 : 11;
    constexpr uint32_t MASK = KeyTraits<RAW>::MASK;
    __shared__ uint32_t lh[(1 << FIRST_BITS) + 2 * WAVE];
    __shared__ uint32_t wave_tot[SEL_THREADS / WAVE];
    __shared__ uint32_t bcast[2];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int ntail = numel - nvf * VEC;                             // the ragged end, in thread 0
    u32x4 q[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int v = i * SEL_THREADS + tid;
        q[i] = v < nvf ? reinterpret_cast<const u32x4 *>(x)[v] : u32x4{0u, 0u, 0u, 0u};
    }
    auto for_all = [&](auto f) {
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (i * SEL_THREADS + tid < nvf) for_each_raw(RAW(0), q[i], [&](uint32_t raw, int) { f(raw); });
        if (tid == 0)
            for (int e = 0; e < ntail; ++e) f(x[nvf * VEC + e]);
    };
    uint32_t prefix = 0, k_rem = k;
    auto pass = [&](auto shift_c, auto bits_c) {
        constexpr int SHIFT = decltype(shift_c)::value, BITS = decltype(bits_c)::value;
        constexpr bool FIRST = SHIFT + BITS == KEY_BITS;
        __syncthreads();
        for (int i = tid; i < (1 << BITS) + 2 * WAVE; i += SEL_THREADS) lh[i] = 0;
        __syncthreads();
        for_all([&](uint32_t raw) {
            const uint32_t key = raw & MASK;
            const uint32_t d = (key >> SHIFT) & ((1u << BITS) - 1u);
            uint32_t a = d ? d : (1u << BITS) + lane;                // zeros, and keys of another prefix, to a slot per lane
            if (!FIRST) a = key >> (SHIFT + BITS) == prefix ? a : (1u << BITS) + WAVE + lane;
            atomicAdd(&lh[a], 1u);
        });
        __syncthreads();
        if (tid < WAVE) {
            const uint32_t z = wave_sum(lh[(1 << BITS) + tid]);
            if (tid == 0) lh[0] += z;
        }
        __syncthreads();
        resolve_digit_local<(1 << BITS), BITS>(lh, prefix, k_rem, wave_tot, bcast);
    };
    if constexpr (sizeof(RAW) == 4) {
        pass(std::integral_constant<int, 18>{}, std::integral_constant<int, 13>{});
        pass(std::integral_constant<int, 5>{}, std::integral_constant<int, 13>{});
        pass(std::integral_constant<int, 0>{}, std::integral_constant<int, 5>{});
    } else {
        pass(std::integral_constant<int, 4>{}, std::integral_constant<int, 11>{});
        pass(std::integral_constant<int, 0>{}, std::integral_constant<int, 4>{});
    }
    const uint32_t t = prefix, m = k_rem;                            // the threshold key and its tie budget
    uint32_t run_gt = 0, run_eq = 0;                                 // before the row
    uint32_t my_gt = 0, my_eq = 0;
    auto emit = [&](uint32_t raw, int i) {
        const uint32_t key = raw & MASK;
        const bool gt = key > t, eq = key == t;
        if (gt || (eq && my_eq < m)) {
            const uint32_t pos = my_gt + min(my_eq, m);
            if (pos < k) {                                           // always true for consistent counts
                vals[pos] = static_cast<RAW>(raw);
                idx[pos] = i;
            }
        }
        my_gt += gt ? 1u : 0u;
        my_eq += eq ? 1u : 0u;
    };
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (i > 0 && i * SEL_THREADS >= nvf) break;                  // uniform
        const int v = i * SEL_THREADS + tid;
        uint32_t cnt = 0;                                            // low 16 bits: #gt, high 16 bits: #eq (8192 elements at most)
        if (v < nvf)
            for_each_raw(RAW(0), q[i], [&](uint32_t raw, int) {
                const uint32_t key = raw & MASK;
                cnt += (key > t ? 1u : 0u) + (key == t ? 0x10000u : 0u);
            });
        uint32_t total;
        const uint32_t before = block_exclusive_scan<SEL_THREADS>(cnt, wave_tot, total);
        my_gt = run_gt + (before & 0xFFFFu);
        my_eq = run_eq + (before >> 16);
        if (cnt) for_each_raw(RAW(0), q[i], [&](uint32_t raw, int e) { emit(raw, v * VEC + e); });
        run_gt += total & 0xFFFFu;
        run_eq += total >> 16;
    }
    if (tid == 0) {
        my_gt = run_gt;
        my_eq = run_eq;
        for (int e = 0; e < ntail; ++e) emit(x[nvf * VEC + e], nvf * VEC + e);
    }
}

template <typename RAW, int FORM = FORM_FLAT>
__global__ void __launch_bounds__(SEL_THREADS)
select_fused_kernel(const RAW *__restrict__ x, int64_t numel, int64_t nvf, int64_t vpc, uint32_t k, SelState *st,
                    uint32_t *hist0, uint32_t *hist1, uint32_t *table, RAW *__restrict__ vals,
                    int32_t *__restrict__ idx, uint32_t spin_limit, unsigned long long gen, SampleRanks ranks, FormArgs form)
{
    ExitReport rep;
    rep.mine = 0u;
    SelOutcome outcome;
    if constexpr (sizeof(RAW) == 2)
        outcome = select16_body<FORM>(x, numel, nvf, vpc, k, st, hist0, table, vals, idx, spin_limit, gen, ranks, rep, form);
    else
        outcome = select32_body(x, numel, nvf, vpc, k, st, hist0, hist1, table, vals, idx, spin_limit, gen, ranks, rep);
    // Exit protocol: every workgroup reports once, when it is past its last grid barrier or gives up at one (the high
    // half counts those).  Whoever's report completes the count sees whether anybody gave up, and
    // then redoes the selection alone when it leaves.  Everything the others store to the outputs is either final or
    // missing, never wrong, and the serial pass below uses no workspace, so it needs no ordering against their
    // remaining traffic (both write the same bytes).
    // A workgroup that cannot rely on the count redoes the selection itself, several doing so write identical bytes:
    // one that never saw the exchange area published (workgroup 0, although dispatched first, did not get through its
    // first few microseconds within the waiting time: not expected to happen), or one that gave up at a barrier of the
    // retry after a missed prediction, when it had already reported (its group's report may then still be its own to pass on).
    extern __shared__ __attribute__((aligned(16))) u32x4 dyn_smem[];
    __shared__ uint32_t s_redo;
    __shared__ uint32_t s_wave_tot[SEL_THREADS / WAVE];
    __shared__ uint32_t s_bcast[2];
    const bool alone = outcome == SEL_NEVER_READY || (outcome == SEL_GAVE_UP && rep.mine != 0);
    if (outcome == SEL_GAVE_UP && rep.mine == 0)
        report_past_barriers(reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(st) + SelWorkspace::xbar_off), rep, true);
    if (rep.mine != 0) report_group(st, rep);
    __syncthreads();
    if (threadIdx.x == REPORT_TID) {
        const uint32_t seen = rep.mine != 0 && rep.group != 0 ? rep.common + rep.group : 0u;
        const bool last = (seen & 0xFFFFu) == gridDim.x;
        const bool redo = alone || (last && ((seen >> 16) != 0 || spin_limit == 0));
        // The last report: nobody will look at the published word any more.  Take it back, so that the next launch that
        // carries the same generation number (a replay of a captured graph) cannot take this call's leftovers for its own.
        if (last) {
            dev_store64(&st->ready, 0ull);
            dev_store64(&st->ready_hist, 0ull);
        }
        if (redo) dev_store(&st->redo, 1u);
        s_redo = redo ? 1u : 0u;
    }
    __syncthreads();
    if (s_redo) {
        select_serial<RAW>(x, numel, nvf, k, vals, idx, reinterpret_cast<uint32_t *>(dyn_smem), s_wave_tot, s_bcast);
        if constexpr (FORM != FORM_FLAT) {
            __threadfence_block();         // the pairs of the workgroup's own threads
            __syncthreads();
            forms_from_pairs<FORM>(idx, numel, k, form);
        }
    }
}

// ---- random dropping (Sec. 3.3, Random Elements) ------------------------------------------------
// Philox4x32 with 10 rounds (Salmon et al., SC'11): per round, counter words 0 and 2 are multiplied by two
// odd constants and the halves of the products are crossed with the other two words and the key; the key
// advances by two Weyl constants between rounds.
__device__ inline void philox_round(uint32_t (&c)[4], uint32_t k0, uint32_t k1)
{
    const uint32_t hi0 = __umulhi(0xD2511F53u, c[0]), lo0 = 0xD2511F53u * c[0];
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c[2]), lo1 = 0xCD9E8D57u * c[2];
    c[0] = hi1 ^ c[1] ^ k0;
    c[1] = lo1;
    c[2] = hi0 ^ c[3] ^ k1;
    c[3] = lo0;
}

// keys[4b .. 4b+3] = the four words of block b, each shifted right by one (31-bit keys, so that the
// select's sign-cleared order of fp32 bit patterns is their integer order).  `blocks` 16-byte stores.
__global__ void __launch_bounds__(256) random_keys_kernel(uint4 *keys, int64_t blocks, uint32_t seed_lo,
                                                          uint32_t seed_hi)
{
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t b = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; b < blocks; b += stride) {
        uint32_t c[4] = {static_cast<uint32_t>(b), 0u, 0u, 0u};
        uint32_t k0 = seed_lo, k1 = seed_hi;
#pragma unroll
        for (int round = 0; round < 10; ++round) {
            if (round > 0) {
                k0 += 0x9E3779B9u;
                k1 += 0xBB67AE85u;
            }
            philox_round(c, k0, k1);
        }
        keys[b] = make_uint4(c[0] >> 1, c[1] >> 1, c[2] >> 1, c[3] >> 1);
    }
}

template <typename RAW>
__global__ void __launch_bounds__(256) gather_kernel(const RAW *__restrict__ x, const int32_t *__restrict__ idx,
                                                     int64_t k, RAW *__restrict__ vals)
{
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t j = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; j < k; j += stride)
        vals[j] = x[idx[j]];
}

inline size_t round_up_256(size_t v) { return (v + 255) / 256 * 256; }

// Workspace of the random strategy: the select's own area, one key per element (padded to whole Philox
// blocks), and the keys the select writes out beside the indices (unused afterwards).
struct RandomWorkspace {
    size_t keys_off, keyvals_off, bytes;
    explicit RandomWorkspace(int64_t numel)
    {
        const size_t key_bytes = round_up_256((static_cast<size_t>(numel) + 3) / 4 * 16);
        keys_off = round_up_256(SelWorkspace::bytes);
        keyvals_off = keys_off + key_bytes;
        bytes = keyvals_off + key_bytes;
    }
};

struct Geometry {
    int64_t nvf, vpc;      // full 16-byte vectors, vectors per chunk
    int chunks;
};

template <typename RAW>
Geometry geometry(int64_t numel)
{
    constexpr int VEC = KeyTraits<RAW>::VEC;
    Geometry g;
    g.nvf = numel / VEC;
    int64_t chunks = (g.nvf + SEL_THREADS - 1) / SEL_THREADS;
    if (chunks > SEL_MAX_CHUNKS) chunks = SEL_MAX_CHUNKS;
    if (chunks < 1) chunks = 1;
    g.vpc = (g.nvf + chunks - 1) / chunks;
    g.vpc = (g.vpc + 7) / 8 * 8;           // chunk starts on 128-byte lines
    if (g.vpc < 8) g.vpc = 8;
    g.chunks = static_cast<int>((g.nvf + g.vpc - 1) / g.vpc);
    if (g.chunks < 1) g.chunks = 1;        // a tensor shorter than one vector still needs a workgroup
    return g;
}

// A number no earlier call of this process has used (a random start, then a count), never 0.
unsigned long long next_generation()
{
    static std::atomic<unsigned long long> counter{[] {
        std::random_device rd;
        return (static_cast<unsigned long long>(rd()) << 32) ^ rd();
    }()};
    unsigned long long g = counter.fetch_add(1) + 1;
    return g ? g : counter.fetch_add(1) + 1;
}

// FORM other than FORM_FLAT: what `form` names, by the persistent kernel (form_emitted says where that is), idx being scratch.
template <typename RAW, int FORM = FORM_FLAT>
dropit_status run_compress(const void *x, int64_t numel, int64_t k, void *vals, int32_t *idx,
                           char *ws, hipStream_t stream, const FormArgs &form = FormArgs{})
{
    const Geometry g = geometry<RAW>(numel);
    SelState *st = reinterpret_cast<SelState *>(ws + SelWorkspace::state_off);
    uint32_t *hist0 = reinterpret_cast<uint32_t *>(ws + SelWorkspace::hist0_off);
    uint32_t *hist1 = reinterpret_cast<uint32_t *>(ws + SelWorkspace::hist1_off);
    uint32_t *table = reinterpret_cast<uint32_t *>(ws + SelWorkspace::table_off);
    uint32_t *off_gt = reinterpret_cast<uint32_t *>(ws + SelWorkspace::offgt_off);
    uint32_t *off_eq = reinterpret_cast<uint32_t *>(ws + SelWorkspace::offeq_off);
    const RAW *xr = static_cast<const RAW *>(x);

    auto clear_state = [&]() {                 // the separate kernels' clearing pass
        trace_mark(stream);
        init_kernel<<<32, 256, 0, stream>>>(reinterpret_cast<uint32_t *>(ws),
                                            static_cast<uint32_t>(SelWorkspace::zero_bytes / 4),
                                            static_cast<uint32_t>(k));
    };
    const int mode = select_mode();
    const SampleRanks spread = numel >= SAMPLE_MIN_NUMEL ? sample_ranks(static_cast<uint32_t>(k), numel, SAMPLE_ELEMS) : SampleRanks{0.0f, 0.0f};
    // Small tensors (default mode only: the other modes are there to exercise the other forms): one workgroup, in the form of
    // rows or the one of staged candidates.
    // fp32: rows where more than 3/8 is kept, whose time the values hardly change (32 K elements at gamma 0.6, normal / ReLU /
    // GELU: 20 / 20 / 21 us; staged 18 / 18 / 23; at 0.3 22 / 23 / 22 and 26 / 34 / 26; at 0.7 20 / 19 / 20 and 17 / 16 / 16).
    // 16-bit: rows up to 16 K elements, and to 24 K where more than an eighth is kept (20 K at gamma 0.6, 0.7, 0.8, 0.9: 11.2,
    // 10.4, 9.8, 9.8 us; staged 12.5, 11.5, 10.5, 9.2; persistent 11.2, 11.0 where it can predict the threshold, 15 where it
    // cannot, as in ReLU at 0.6 and GELU at 0.7).  Above, staged to 32 K where at most a quarter is kept, else the persistent
    // kernel: 11 to 16 us from there to 128 K, staged 15 or 25 at 64 K.  Staged to 64 K where the threshold's rank lies outside
    // a sample.
    const int64_t nvec = numel / KeyTraits<RAW>::VEC;
    const bool sampled = spread.lo != 0.0f;
    const bool rows = sizeof(RAW) == 4 ? 8 * k > 3 * numel : nvec <= 2 * SEL_THREADS || (nvec <= ROW_VECTORS && sampled && 8 * k > numel);
    const bool persistent = sizeof(RAW) == 2 && sampled && !rows && (nvec > SMALL_VECTORS / 2 * SEL_THREADS || 4 * k > numel);
    if (FORM == FORM_FLAT && mode == 0 && nvec <= int64_t(SMALL_VECTORS) * SEL_THREADS && !persistent) {
        trace_mark(stream);
        const int vectors = int(nvec);
        if (rows) {
            const auto run = [&](auto kernel) {
                kernel<<<1, SEL_THREADS, 0, stream>>>(xr, int(numel), vectors, static_cast<uint32_t>(k), static_cast<RAW *>(vals), idx);
                trace_mark(stream);
                return launch_status();
            };
            if (vectors <= SEL_THREADS) return run(select_row_kernel<RAW, 1>);
            if (vectors <= 2 * SEL_THREADS) return run(select_row_kernel<RAW, 2>);
            if constexpr (sizeof(RAW) == 2) return run(select_row_kernel<RAW, 3>);
            else return vectors <= 4 * SEL_THREADS ? run(select_row_kernel<RAW, 4>) : run(select_row_kernel<RAW, SMALL_VECTORS>);
        }
        const SampleRanks ranks = vectors >= SMALL_SAMPLE_MIN ? sample_ranks(static_cast<uint32_t>(k), numel, vectors)
                                                              : SampleRanks{0.0f, 0.0f};
        static std::atomic<uint64_t> set_up{0};
        if (!once_per_device(set_up, [] {
                return hipFuncSetAttribute(reinterpret_cast<const void *>(select_small_kernel<RAW>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, SEL_THREADS / WAVE * SMALL_SEG_BYTES) == hipSuccess;
            }))
            return DROPIT_EHIP;
        const uint32_t cap = small_cap<RAW>(vectors);
        const size_t smem = std::max(size_t(SEL_THREADS / WAVE) * cap * sizeof(typename Staged<RAW>::word), 4 * size_t(SMALL_BINS));
        select_small_kernel<RAW><<<1, SEL_THREADS, smem, stream>>>(xr, int(numel), vectors, static_cast<uint32_t>(k), ranks, cap,
                                                                   static_cast<RAW *>(vals), idx);
        trace_mark(stream);
        return launch_status();
    }
    // Preferred: one persistent kernel, one workgroup per compute unit.
    if (mode != 1) {
        constexpr int VEC = KeyTraits<RAW>::VEC;
        constexpr size_t smem_bytes = sizeof(RAW) == 2 ? ST_SMEM_BYTES : SMEM32_BYTES;
        static_assert(smem_bytes <= 156 * 1024, "of the 160 KB of a compute unit; the rest is static");
        static_assert(smem_bytes >= 4 * ((size_t(1) << 13) + 2 * WAVE), "the serial redo's histogram");
        // how many workgroups of this kernel each device holds at once (asked once per element type and device)
        static std::atomic<uint64_t> asked{0};
        static int capacity_of[64] = {};
        int dev = 0;
        (void)hipGetDevice(&dev);
        int fresh = -1;
        const bool ok = once_per_device(asked, [&] {
            hipDeviceProp_t prop;
            int per_cu = 0;
            if (hipGetDeviceProperties(&prop, dev) == hipSuccess &&
                hipFuncSetAttribute(reinterpret_cast<const void *>(select_fused_kernel<RAW, FORM>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize,
                                    static_cast<int>(smem_bytes)) == hipSuccess &&
                hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, select_fused_kernel<RAW, FORM>, SEL_THREADS,
                                                             smem_bytes) == hipSuccess &&
                per_cu > 0 && prop.multiProcessorCount > 0)
                fresh = std::min(per_cu * prop.multiProcessorCount, SEL_MAX_CHUNKS);
            (void)hipGetLastError();
            if (dev >= 0 && dev < 64) capacity_of[dev] = fresh;
            return true;                       // a device that cannot hold the kernel is an answer too (-1)
        });
        const int capacity = !ok ? -1 : (dev >= 0 && dev < 64) ? capacity_of[dev] : fresh;
        if (capacity > 0) {
            // chunk geometry: at most one workgroup per resident slot, chunks start on 128-byte lines
            int64_t nvf = numel / VEC;
            int64_t chunks = std::min<int64_t>(std::max<int64_t>((nvf + SEL_THREADS - 1) / SEL_THREADS, 1), capacity);
            int64_t vpc = std::max<int64_t>(((nvf + chunks - 1) / chunks + 7) / 8 * 8, 8);
            chunks = std::max<int64_t>((nvf + vpc - 1) / vpc, 1);
            uint32_t k32 = static_cast<uint32_t>(k);
            uint32_t spin_limit = mode == 3 ? 0u : nvec <= int64_t(SMALL_VECTORS) * SEL_THREADS ? SPIN_LIMIT_SMALL : SPIN_LIMIT;
            RAW *vals_t = static_cast<RAW *>(vals);
            unsigned long long gen = next_generation();
            SampleRanks ranks = spread;
            FormArgs form_t = form;
            trace_mark(stream);
            if (mode == 2) {               // the runtime guarantees co-residency, at the price of slow queue switches
                void *args[] = {(void *)&xr, (void *)&numel, (void *)&nvf, (void *)&vpc, (void *)&k32, (void *)&st,
                                (void *)&hist0, (void *)&hist1, (void *)&table, (void *)&vals_t, (void *)&idx,
                                (void *)&spin_limit, (void *)&gen, (void *)&ranks, (void *)&form_t};
                if (hipLaunchCooperativeKernel(reinterpret_cast<const void *>(select_fused_kernel<RAW, FORM>),
                                               dim3(static_cast<unsigned>(chunks)), dim3(SEL_THREADS), args,
                                               smem_bytes, stream) == hipSuccess) {
                    trace_mark(stream);
                    return launch_status();
                }
                (void)hipGetLastError();   // cooperative launch unavailable (e.g. stream capture): ordinary launch
            }
            select_fused_kernel<RAW, FORM><<<dim3(static_cast<unsigned>(chunks)), dim3(SEL_THREADS), smem_bytes, stream>>>(
                xr, numel, nvf, vpc, k32, st, hist0, hist1, table, vals_t, idx, spin_limit, gen, ranks, form_t);
            trace_mark(stream);
            return launch_status();
        }
    }
    if constexpr (FORM != FORM_FLAT) return DROPIT_EUNSUPPORTED;     // (the caller converts flat indices)
    clear_state();
    const dim3 grid(g.chunks), block(SEL_THREADS);
    trace_mark(stream);
    if constexpr (sizeof(RAW) == 2) {
        hist_kernel<RAW, 4, 11, true><<<grid, block, 0, stream>>>(xr, numel, g.nvf, g.vpc, st, hist0, 0);
        trace_mark(stream);
        count_kernel<RAW, 4><<<grid, block, 0, stream>>>(xr, numel, g.nvf, g.vpc, st, table, off_gt, off_eq, 1);
    } else {
        hist_kernel<RAW, 18, 13, true><<<grid, block, 0, stream>>>(xr, numel, g.nvf, g.vpc, st, hist0, 0);
        trace_mark(stream);
        hist_kernel<RAW, 5, 13, false><<<grid, block, 0, stream>>>(xr, numel, g.nvf, g.vpc, st, hist1, 1);
        trace_mark(stream);
        count_kernel<RAW, 5><<<grid, block, 0, stream>>>(xr, numel, g.nvf, g.vpc, st, table, off_gt, off_eq, 2);
    }
    trace_mark(stream);
    compact_kernel<RAW><<<grid, block, 0, stream>>>(xr, numel, g.nvf, g.vpc, st, off_gt, off_eq,
                                                    static_cast<RAW *>(vals), idx);
    trace_mark(stream);
    return launch_status();
}

}  // namespace
}  // namespace dropit

// The select with one of the cheaper index forms as its output, idx being scratch of k words.  DROPIT_EUNSUPPORTED, and nothing
// done, where it has to write flat indices: fp32, tensors of one workgroup, a ragged end, separate kernels.
dropit_status dropit::compress_form(const void *x, int64_t numel, dropit_dtype dt, int64_t k, void *vals, int32_t *idx, int kind,
                                    uint16_t *col, uint32_t *mask, int32_t *starts, uint32_t len, int64_t nstarts, char *ws,
                                    hipStream_t stream)
{
    if (dt != DROPIT_BF16 || numel % 8 != 0 || k < 1 || select_mode() == 1) return DROPIT_EUNSUPPORTED;
    if (numel <= int64_t(SMALL_VECTORS) * SEL_THREADS * 8 || x == nullptr || !aligned(x, 16) || vals == nullptr || !aligned(vals, 2))
        return DROPIT_EUNSUPPORTED;                        // (dropit_compress says what is wrong)
    const FormArgs form = {col, mask, starts, divisor(len), uint32_t(nstarts)};
    return kind == FORM_ROWS ? run_compress<uint16_t, FORM_ROWS>(x, numel, k, vals, idx, ws, stream, form)
                             : run_compress<uint16_t, FORM_MASK>(x, numel, k, vals, idx, ws, stream, form);
}

dropit::TraceState &dropit::trace_state()
{
    static thread_local TraceState t = {nullptr, 0, 0};
    return t;
}

int &dropit::select_mode()
{
    static thread_local int mode = 0;
    return mode;
}

using namespace dropit;

extern "C" dropit_status dropit_set_select_mode(int mode)
{
    if (mode < 0 || mode > 3) return DROPIT_EINVAL;
    select_mode() = mode;
    return DROPIT_OK;
}

extern "C" void dropit_trace_events(void **events, int count)
{
    TraceState &t = trace_state();
    t.events = reinterpret_cast<hipEvent_t *>(events);
    t.count = (events != nullptr && count > 0) ? count : 0;
    t.next = 0;
}

extern "C" const char *dropit_status_string(dropit_status s)
{
    switch (s) {
    case DROPIT_OK: return "DROPIT_OK";
    case DROPIT_EINVAL: return "DROPIT_EINVAL: invalid argument";
    case DROPIT_EWORKSPACE: return "DROPIT_EWORKSPACE: workspace too small";
    case DROPIT_EUNSUPPORTED: return "DROPIT_EUNSUPPORTED: geometry not implemented";
    case DROPIT_EHIP: return "DROPIT_EHIP: HIP launch failed";
    }
    return "DROPIT: unknown status";
}

extern "C" int64_t dropit_keep_count(int64_t numel, double gamma)
{
    if (numel < 0 || numel > INT32_MAX) return -1;
    if (!(gamma >= 0.0 && gamma <= 1.0)) return -1;   // also rejects NaN
    // floor((1-gamma)*numel) == numel - ceil(gamma*numel); gamma*numel < 2^31 is exact enough in double
    const double dropped = __builtin_ceil(gamma * static_cast<double>(numel));
    int64_t k = numel - static_cast<int64_t>(dropped);
    if (k < 0) k = 0;
    return k;
}

extern "C" size_t dropit_compress_workspace_bytes(int64_t numel, dropit_dtype dt)
{
    if (numel < 1 || numel > INT32_MAX) return 0;
    if (dt != DROPIT_F32 && dt != DROPIT_BF16) return 0;
    return SelWorkspace::bytes;
}

extern "C" dropit_status dropit_compress(const void *x, const int64_t *shape, int ndim, dropit_dtype dt,
                                         double gamma, void *vals, int32_t *idx, void *workspace,
                                         size_t workspace_bytes, void *hip_stream)
{
    if (dt != DROPIT_F32 && dt != DROPIT_BF16) return DROPIT_EINVAL;
    const int64_t numel = checked_numel(shape, ndim);
    if (numel < 1) return DROPIT_EINVAL;
    const int64_t k = dropit_keep_count(numel, gamma);
    if (k < 0) return DROPIT_EINVAL;
    if (x == nullptr || !aligned(x, 16)) return DROPIT_EINVAL;
    if (k == 0) return DROPIT_OK;
    if (vals == nullptr || idx == nullptr) return DROPIT_EINVAL;
    if (!aligned(vals, dt == DROPIT_F32 ? 4 : 2) || !aligned(idx, 4)) return DROPIT_EINVAL;
    if (workspace == nullptr || !aligned(workspace, 256)) return DROPIT_EINVAL;
    if (workspace_bytes < SelWorkspace::bytes) return DROPIT_EWORKSPACE;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    char *ws = static_cast<char *>(workspace);
    if (dt == DROPIT_BF16) return run_compress<uint16_t>(x, numel, k, vals, idx, ws, stream);
    return run_compress<uint32_t>(x, numel, k, vals, idx, ws, stream);
}

// ---- dropit_compress for callers that cannot allocate ----------------------------------------------
// The select's exchange area (state, histograms, per-chunk table: SelWorkspace::bytes, about 200 KB, the
// same for every tensor size) as a device array of this library instead of a caller's workspace.  In
// host code `scratch` is only a handle for the runtime: the array's device address is asked for once
// per device (each device holds its own copy) and that pointer is what the kernels get.
static __device__ __align__(256) unsigned char scratch[SelWorkspace::bytes];

namespace {
// Device address of `scratch` on the current device, nullptr if the runtime will not tell.
char *static_scratch()
{
    static std::atomic<uint64_t> known{0};
    static void *address_on[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return nullptr;
    void *fresh = nullptr;
    const bool ok = once_per_device(known, [&] {
        if (hipGetSymbolAddress(&fresh, HIP_SYMBOL(scratch)) != hipSuccess || fresh == nullptr) {
            (void)hipGetLastError();
            return false;
        }
        if (dev >= 0 && dev < 64) address_on[dev] = fresh;
        return true;
    });
    if (!ok) return nullptr;
    return static_cast<char *>((dev >= 0 && dev < 64) ? address_on[dev] : fresh);
}
}  // namespace

extern "C" dropit_status dropit_compress_static(const void *x, const int64_t *shape, int ndim, dropit_dtype dt,
                                                double gamma, void *vals, int32_t *idx, void *hip_stream)
{
    if (dt != DROPIT_F32 && dt != DROPIT_BF16) return DROPIT_EINVAL;
    const int64_t numel = checked_numel(shape, ndim);       // -1 beyond DROPIT_STATIC_MAX_NUMEL
    if (numel < 1) return DROPIT_EINVAL;
    const int64_t k = dropit_keep_count(numel, gamma);
    if (k < 0) return DROPIT_EINVAL;
    if (x == nullptr || !aligned(x, 16)) return DROPIT_EINVAL;
    if (k == 0) return DROPIT_OK;
    if (vals == nullptr || idx == nullptr) return DROPIT_EINVAL;
    if (!aligned(vals, dt == DROPIT_F32 ? 4 : 2) || !aligned(idx, 4)) return DROPIT_EINVAL;
    char *ws = static_scratch();
    if (ws == nullptr) return DROPIT_EHIP;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (dt == DROPIT_BF16) return run_compress<uint16_t>(x, numel, k, vals, idx, ws, stream);
    return run_compress<uint32_t>(x, numel, k, vals, idx, ws, stream);
}

extern "C" size_t dropit_compress_random_workspace_bytes(int64_t numel, dropit_dtype dt)
{
    if (numel < 1 || numel > INT32_MAX) return 0;
    if (dt != DROPIT_F32 && dt != DROPIT_BF16) return 0;
    return RandomWorkspace(numel).bytes;
}

extern "C" dropit_status dropit_compress_random(const void *x, const int64_t *shape, int ndim, dropit_dtype dt,
                                                double gamma, uint64_t seed, void *vals, int32_t *idx,
                                                void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (dt != DROPIT_F32 && dt != DROPIT_BF16) return DROPIT_EINVAL;
    const int64_t numel = checked_numel(shape, ndim);
    if (numel < 1) return DROPIT_EINVAL;
    const int64_t k = dropit_keep_count(numel, gamma);
    if (k < 0) return DROPIT_EINVAL;
    if (x == nullptr || !aligned(x, 16)) return DROPIT_EINVAL;
    if (k == 0) return DROPIT_OK;
    if (vals == nullptr || idx == nullptr) return DROPIT_EINVAL;
    if (!aligned(vals, dt == DROPIT_F32 ? 4 : 2) || !aligned(idx, 4)) return DROPIT_EINVAL;
    if (workspace == nullptr || !aligned(workspace, 256)) return DROPIT_EINVAL;
    const RandomWorkspace rw(numel);
    if (workspace_bytes < rw.bytes) return DROPIT_EWORKSPACE;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    char *ws = static_cast<char *>(workspace);
    uint4 *keys = reinterpret_cast<uint4 *>(ws + rw.keys_off);
    const int64_t blocks = (numel + 3) / 4;
    const unsigned grid = static_cast<unsigned>(std::min<int64_t>((blocks + 255) / 256, 256 * 16));
    trace_mark(stream);
    random_keys_kernel<<<grid, 256, 0, stream>>>(keys, blocks, static_cast<uint32_t>(seed & 0xFFFFFFFFu),
                                                 static_cast<uint32_t>(seed >> 32));
    // the drawn keys are 31-bit patterns: the fp32 select ranks them as integers
    dropit_status st = run_compress<uint32_t>(keys, numel, k, ws + rw.keyvals_off, idx, ws, stream);
    if (st != DROPIT_OK) return st;
    const unsigned ggrid = static_cast<unsigned>(std::min<int64_t>((k + 255) / 256, 256 * 16));
    if (dt == DROPIT_BF16)
        gather_kernel<uint16_t><<<ggrid, 256, 0, stream>>>(static_cast<const uint16_t *>(x), idx, k,
                                                           static_cast<uint16_t *>(vals));
    else
        gather_kernel<uint32_t><<<ggrid, 256, 0, stream>>>(static_cast<const uint32_t *>(x), idx, k,
                                                           static_cast<uint32_t *>(vals));
    trace_mark(stream);
    return launch_status();
}
