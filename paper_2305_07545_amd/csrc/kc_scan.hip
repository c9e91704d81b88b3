// Multi-workgroup exclusive prefix sums: block sums, then a rescan of each
// block with the sum of the blocks before it (key-list classification, the
// batched form's outputs and bin offsets), and a one-pass scan of the tiles'
// counts (the single-set pipeline's ordered outputs).
#include <hip/hip_runtime.h>

#include "kc_kernels.hpp"

namespace kc {

namespace {

constexpr int kScanThreads = 256;
constexpr int kScanPer = 16;
constexpr int kScanBlock = kScanThreads * kScanPer;  // elements per workgroup

// Exclusive sum of one value per thread over the workgroup: wave scans by
// shuffles, then the wave totals.  s_wave: kScanThreads / 64 entries.
template <typename T>
__device__ __forceinline__ T wg_exclusive_sum(T v, T *s_wave, T &total) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    T incl = v;
#pragma unroll
    for (uint32_t d = 1; d < 64; d <<= 1) {
        T o = __shfl_up(incl, d, 64);
        if (lane >= d)
            incl += o;
    }
    if (lane == 63)
        s_wave[wave] = incl;
    __syncthreads();
    T before = 0;
    total = 0;
#pragma unroll
    for (uint32_t w = 0; w < kScanThreads / 64; w++) {
        const T t = s_wave[w];
        if (w < wave)
            before += t;
        total += t;
    }
    __syncthreads();
    return before + incl - v;
}

// Sum of each workgroup's kScanBlock elements (coalesced: element i*256+tid).
template <typename TIn, typename TOut>
__global__ void __launch_bounds__(kScanThreads) k_scan_reduce(const TIn *__restrict__ in, uint64_t n,
                                                             TOut *__restrict__ partial) {
    __shared__ TOut s_wave[kScanThreads / 64];
    const uint64_t base = (uint64_t)blockIdx.x * kScanBlock + threadIdx.x;
    TOut sum = 0;
#pragma unroll
    for (int i = 0; i < kScanPer; i++) {
        const uint64_t x = base + (uint64_t)i * kScanThreads;
        if (x < n)
            sum += (TOut)in[x];
    }
    TOut total;
    (void)wg_exclusive_sum<TOut>(sum, s_wave, total);
    if (threadIdx.x == 0)
        partial[blockIdx.x] = total;
}

// LDS slot of element e of a block: one pad word after every kScanPer
// elements, so that thread t's run (elements 16t .. 16t+15) and the
// coalesced rows (elements i*256 + t) are both free of bank conflicts.
__device__ __forceinline__ uint32_t pad_at(uint32_t e) { return e + e / kScanPer; }

// Exclusive scan of each workgroup's elements, offset by base and the sums
// of the workgroups before it (each workgroup adds up those block sums
// itself: a few KB from L2, one launch fewer than a separate scan of the
// sums): coalesced loads into LDS, a sequential scan of 16 consecutive
// elements per thread, the workgroup scan of the thread sums, coalesced
// stores.  The last workgroup writes the grand total (without base).
template <typename TIn, typename TOut>
__global__ void __launch_bounds__(kScanThreads) k_scan_down(const TIn *__restrict__ in, uint64_t n,
                                                           const TOut *__restrict__ partial,
                                                           const TOut *__restrict__ base,
                                                           TOut *__restrict__ out,
                                                           TOut *__restrict__ total_out) {
    __shared__ TOut s_buf[kScanBlock + kScanBlock / kScanPer];
    __shared__ TOut s_wave[kScanThreads / 64];
    TOut before = 0;
    for (uint32_t i = threadIdx.x; i < blockIdx.x; i += kScanThreads)
        before += partial[i];
    TOut pre;
    (void)wg_exclusive_sum<TOut>(before, s_wave, pre);
    const TOut offset = (base ? *base : (TOut)0) + pre;
    const uint64_t b0 = (uint64_t)blockIdx.x * kScanBlock;
#pragma unroll
    for (int i = 0; i < kScanPer; i++) {
        const uint32_t e = (uint32_t)i * kScanThreads + threadIdx.x;
        s_buf[pad_at(e)] = b0 + e < n ? (TOut)in[b0 + e] : (TOut)0;
    }
    __syncthreads();
    TOut v[kScanPer];
    TOut sum = 0;
#pragma unroll
    for (int i = 0; i < kScanPer; i++) {
        v[i] = s_buf[pad_at(threadIdx.x * kScanPer + i)];
        sum += v[i];
    }
    TOut total;
    TOut run = offset + wg_exclusive_sum<TOut>(sum, s_wave, total);
#pragma unroll
    for (int i = 0; i < kScanPer; i++) {
        s_buf[pad_at(threadIdx.x * kScanPer + i)] = run;
        run += v[i];
    }
    if (total_out && threadIdx.x == 0 && blockIdx.x + 1 == gridDim.x)
        *total_out = pre + total;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kScanPer; i++) {
        const uint32_t e = (uint32_t)i * kScanThreads + threadIdx.x;
        if (b0 + e < n)
            out[b0 + e] = s_buf[pad_at(e)];
    }
}

template <typename TIn, typename TOut>
hipError_t scan_impl(const TIn *in, TOut *out, uint64_t n, const TOut *base, TOut *total,
                     TOut *partial, hipStream_t s) {
    uint64_t nb = (n + kScanBlock - 1) / kScanBlock;
    if (nb == 0)
        nb = 1;
    hipLaunchKernelGGL((k_scan_reduce<TIn, TOut>), dim3((unsigned)nb), dim3(kScanThreads), 0, s,
                       in, n, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL((k_scan_down<TIn, TOut>), dim3((unsigned)nb), dim3(kScanThreads), 0, s, in,
                       n, (const TOut *)partial, base, out, total);
    return hipGetLastError();
}

// Exclusive sums of the tiles' distinct and trustworthy counts in one pass
// (decoupled look-back): a workgroup sums its kScanTiles tiles, publishes the
// sums, adds up what the workgroups before it published (their own sums, or
// already the sums up to them) and writes its tiles' offsets.  Workgroups
// number themselves by a ticket, so that every workgroup another one waits
// for has started, and each publishes its own sums before it waits.
// Bound by its launch and the chain of workgroups: 13 us for 150 M positions.
// It replaces two scans of two launches each, the copy of the running count
// and the launch that moved the counters (97 us there, 31 of 112 us of a call
// of 30 K bases).
//
// state: [0] the ticket, then per workgroup a distinct and a trustworthy word:
// kind << 62 | value (0 nothing yet, 1 the workgroup's own sum, 2 the sum up
// to and with it).
constexpr uint64_t kOwn = 1ull << 62, kUpTo = 2ull << 62, kValue = kOwn - 1;

__device__ __forceinline__ void publish(uint64_t *p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t published(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum of what workgroups 0 .. id - 1 published at state[stride * block]
// (a wavefront, 64 workgroups at a time, nearest first).
__device__ uint64_t look_back(const uint64_t *state, uint32_t id) {
    const uint32_t lane = threadIdx.x & 63u;
    uint64_t sum = 0;
    for (int64_t top = (int64_t)id - 1; top >= 0; top -= 64) {
        const int64_t at = top - (int64_t)lane;
        uint64_t v = kUpTo;  // before the first workgroup: nothing
        if (at >= 0)
            do {
                v = published(state + 2 * at);
            } while ((v >> 62) == 0);
        // the nearest workgroup that knows the sum up to it ends the search
        const uint64_t ends = __ballot((v >> 62) == 2);
        const uint32_t end = ends ? (uint32_t)__builtin_ctzll(ends) : 63u;
        uint64_t x = lane <= end ? v & kValue : 0ull;
        for (uint32_t d = 32; d >= 1; d >>= 1)
            x += __shfl_xor(x, d, 64);
        sum += x;
        if (ends)
            break;
    }
    return sum;
}

__global__ void __launch_bounds__(kScanThreads)
k_tile_scan(const uint32_t *__restrict__ tile_d, const uint32_t *__restrict__ tile_t,
            uint64_t n_tiles, int split, uint64_t *__restrict__ state,
            uint64_t *__restrict__ off_d, uint64_t *__restrict__ off_t,
            uint64_t *__restrict__ totals, TileScan T) {
    constexpr int kPer = (int)(kScanTiles / kScanThreads);
    __shared__ uint64_t s_wave[kScanThreads / 64];
    __shared__ uint64_t s_base[2];
    __shared__ uint32_t s_id;
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) {
        s_id = (uint32_t)atomicAdd((unsigned long long *)state, 1ull);
        s_base[0] = *T.n_distinct;  // read before this workgroup publishes anything
    }
    __syncthreads();
    const uint32_t id = s_id;
    const uint64_t call_base = s_base[0];
    __syncthreads();
    // a tile has at most 1024 of either: a workgroup's sums fit 32 bits each
    const uint64_t t0 = (uint64_t)id * kScanTiles + threadIdx.x * kPer;
    uint64_t v[kPer], sum = 0;  // trustworthy << 32 | distinct
#pragma unroll
    for (int u = 0; u < kPer; u++) {
        const uint64_t t = t0 + u;
        v[u] = t < n_tiles ? (uint64_t)tile_d[t] | (split ? (uint64_t)tile_t[t] << 32 : 0ull) : 0ull;
        sum += v[u];
    }
    if (T.tile_v && T.n_windows) {
        uint32_t w = 0;
#pragma unroll
        for (int u = 0; u < kPer; u++)
            w += t0 + u < n_tiles ? T.tile_v[t0 + u] : 0u;
        for (uint32_t d = 32; d >= 1; d >>= 1)
            w += __shfl_xor(w, d, 64);
        if (lane == 0 && w)
            atomicAdd((unsigned long long *)T.n_windows, (unsigned long long)w);
    }
    uint64_t total;
    const uint64_t before = wg_exclusive_sum<uint64_t>(sum, s_wave, total);
    const uint64_t own_d = total & 0xFFFFFFFFull, own_t = total >> 32;
    uint64_t *mine = state + 1 + 2 * (uint64_t)id;
    if (wave < 2) {  // wavefront 0: distinct, 1: trustworthy
        const uint64_t own = wave ? own_t : own_d;
        if (lane == 0)
            publish(mine + wave, (id ? kOwn : kUpTo) | own);
        const uint64_t pre = id ? look_back(state + 1 + wave, id) : 0ull;
        if (lane == 0) {
            if (id)
                publish(mine + wave, kUpTo | (pre + own));
            s_base[wave] = pre;
        }
    }
    __syncthreads();
    uint64_t run_d = call_base + s_base[0] + (before & 0xFFFFFFFFull);
    uint64_t run_t = s_base[1] + (before >> 32);
#pragma unroll
    for (int u = 0; u < kPer; u++) {
        const uint64_t t = t0 + u;
        if (t < n_tiles) {
            off_d[t] = run_d;
            if (split)
                off_t[t] = run_t;
        }
        run_d += v[u] & 0xFFFFFFFFull;
        run_t += v[u] >> 32;
    }
    // the last workgroup knows the totals; every other one has read the
    // running count by then (it published its sums afterwards)
    if (threadIdx.x == 0 && id + 1 == gridDim.x) {
        const uint64_t nd = s_base[0] + own_d, nt = s_base[1] + own_t;
        totals[3] = call_base;
        *T.n_distinct = call_base + nd;
        if (T.n_windows && !T.tile_v)
            *T.n_windows += totals[5];
        bool over = call_base + nd > T.cap_d;
        if (T.n_trust) {
            *T.n_trust = nt;
            *T.n_err = nd - nt;
            over = over || nt > T.cap_te || nd - nt > T.cap_te;
        }
        if (over)
            atomicOr(T.status, kStatusRange);
    }
}

}  // namespace

hipError_t launch_tile_scan(const Workspace &W, uint64_t n_tiles, bool split, const TileScan &T,
                            hipStream_t s) {
    const uint64_t blocks = (n_tiles + kScanTiles - 1) / kScanTiles;
    hipLaunchKernelGGL(k_tile_scan, dim3((unsigned)blocks), dim3(kScanThreads), 0, s,
                       (const uint32_t *)W.tile_a, (const uint32_t *)W.tile_b, n_tiles,
                       split ? 1 : 0, W.off_c, W.off_a, W.off_b, W.totals, T);
    return hipGetLastError();
}

uint64_t scan_partials(uint64_t n) { return (n + kScanBlock - 1) / kScanBlock + 1; }

hipError_t scan_u32_u64(const uint32_t *in, uint64_t *out, uint64_t n, const uint64_t *base,
                        uint64_t *total, uint64_t *partial, hipStream_t s) {
    return scan_impl<uint32_t, uint64_t>(in, out, n, base, total, partial, s);
}

hipError_t scan_u32_u32(const uint32_t *in, uint32_t *out, uint64_t n, uint32_t *total,
                        uint32_t *partial, hipStream_t s) {
    return scan_impl<uint32_t, uint32_t>(in, out, n, (const uint32_t *)nullptr, total, partial, s);
}

}  // namespace kc
