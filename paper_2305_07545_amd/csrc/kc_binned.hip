// Binned insertion: the countBF update and the first-seen resolution done in
// LDS, one workgroup per filter region, with no global atomics on counters.
//
// A filter region is 2^shift consecutive cells whose eta*2^shift counters fit
// the LDS arrays.  For one chunk of positions [c0, c1) (t = p - c0) the
// windows' entries are sorted by region (kc_blocks.hip), then each region is
// updated by one workgroup of a persistent grid: in LDS, hits[c] += 1 and
// first[c] = min(first[c], t) over the region's entries; then counter =
// min(2^alpha - 1, old + hits) per counter, and the occurrence first[c] is
// distinct when the counter was zero before the chunk (the sequential Query-I
// result).  Entry order inside a region never matters: sums and minima are
// order-independent, so the outputs are deterministic.
//
// Here: the plan of an insert, and the passes that turn first-seen records
// into flags.
#include <hip/hip_runtime.h>

#include <cstdlib>

#include "kc_blocks.hpp"
#include "kc_device.hpp"
#include "kc_kernels.hpp"
#include "kc_region.hpp"

namespace kc {

// Workgroups of the persistent region pass: as many as the CUs hold at once
// (one per CU with 128 KiB of counters, two with 64 KiB), at most one
// per region.
uint32_t region_grid(uint32_t n_regions, uint32_t counters) {
    static int n_cu = 0;
    if (n_cu == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
            v > 0)
            n_cu = v;
        else
            n_cu = 256;
    }
    const uint32_t g = (uint32_t)n_cu * (counters == (uint32_t)kSmallRegionCounters ? 2u : 1u);
    return n_regions < g ? n_regions : g;
}

// ---------------------------------------------------------------------------
// winner passes (records mode): the region pass's first-seen records, grouped
// by region, become distinct and trustworthy bits.  Records are
// distributed by position in two counting-sort passes (by t >> 24, then by
// the next 5 bits) into blocks of 2^19 positions, whose bits are built in
// LDS.  Runs are appended to each bucket at an atomic cursor (the
// order of records inside a bucket does not matter: a bitmap is built from
// them), in areas of the two entry buffers.  A position is first seen by each
// of its hash functions at most, so an area has k_h records of room for every
// position it covers.
// ---------------------------------------------------------------------------
constexpr uint32_t kWinA = 24;             // level-A digit: t >> 24 (256 buckets)
constexpr uint32_t kWinB = 19;             // level-B digit: (t >> 19) & 31 (2^19 positions)
constexpr int kWinThreads = 1024;
constexpr int kWinBatch = 8192;            // records per LDS batch
constexpr uint32_t kWinRegions = 64;       // regions per level-A workgroup
constexpr uint32_t kWinSlices = 64;        // level-B workgroups per level-A bucket
constexpr uint32_t kWinBuckets = 256;
constexpr uint32_t kWinBlocksPerBucket = 1u << (kWinA - kWinB);

constexpr int kWinPer = kWinBatch / kWinThreads;  // records per thread and batch
static_assert(kWinBuckets <= 256 && kWinBlocksPerBucket <= 256, "digits are staged as bytes");

// A batch of records appended to buckets by digit d = (rec >> shift) & (nd
// - 1): record u of this thread is v[u] (present where bit u of ok is set).
// The records are ranked within their digit by LDS atomics, the digit
// counts scanned and each digit's run reserved at its bucket's cursor; the
// kept records (keep(rec)) are then staged in LDS in digit order and written
// out in that order, consecutive threads to consecutive addresses of a run
// (the order of records inside a run does not matter).  Buckets' areas are
// `room` records apart.  Ends with a barrier.
template <typename Rec, typename Keep>
__device__ void win_append(const Rec (&v)[kWinPer], uint32_t ok, uint32_t n, uint32_t shift,
                           uint32_t nd, uint32_t bucket0, uint64_t room, uint32_t *s_cnt,
                           uint32_t *s_start, uint32_t *s_base, uint32_t *s_wave,
                           uint32_t *s_stage, uint8_t *s_tag, uint32_t *__restrict__ cursor,
                           uint32_t *__restrict__ out, Keep keep) {
    for (uint32_t i = threadIdx.x; i < nd; i += kWinThreads)
        s_cnt[i] = 0;
    __syncthreads();
    uint32_t rk[kWinPer];
#pragma unroll
    for (int u = 0; u < kWinPer; u++)
        if (ok & (1u << u))
            rk[u] = atomicAdd(&s_cnt[(uint32_t)(v[u] >> shift) & (nd - 1u)], 1u);
    __syncthreads();
    // exclusive scan of the nd (<= 256) counts, 64 per wavefront
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t c = threadIdx.x < nd ? s_cnt[threadIdx.x] : 0u;
    uint32_t incl = c;
    if (threadIdx.x < nd) {
        for (uint32_t d = 1; d < 64; d <<= 1) {
            const uint32_t o = __shfl_up(incl, d, 64);
            if (lane >= d)
                incl += o;
        }
        if (lane == 63 || threadIdx.x == nd - 1)
            s_wave[wave] = incl;
    }
    __syncthreads();
    if (threadIdx.x < nd) {
        uint32_t before = 0;
        for (uint32_t w = 0; w < wave; w++)
            before += s_wave[w];
        s_start[threadIdx.x] = before + incl - c;
        s_base[threadIdx.x] = c ? atomicAdd(&cursor[bucket0 + threadIdx.x], c) : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kWinPer; u++)
        if (ok & (1u << u)) {
            const uint32_t d = (uint32_t)(v[u] >> shift) & (nd - 1u);
            const uint32_t j = s_start[d] + rk[u];
            s_stage[j] = keep(v[u]);
            s_tag[j] = (uint8_t)d;
        }
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < n; j += kWinThreads) {
        const uint32_t d = s_tag[j];
        out[(bucket0 + d) * room + s_base[d] + (j - s_start[d])] = s_stage[j];
    }
    __syncthreads();
}

// Level A: the records of regions [kWinRegions * blockIdx.x, ...) (region r's
// n_win[r] records start at its first entry) -> bucket t >> 24, record
// (t & (2^24 - 1)) | mark << 24.  The regions' record counts are scanned in
// LDS first, so that the workgroup's records are one index range whose
// batches are filled by all threads at once (record i is found in its
// region by a binary search of the scan), not region after region.
__global__ void __launch_bounds__(kWinThreads) k_win_a(uint32_t n_regions,
                                                       const uint32_t *__restrict__ offsets,
                                                       uint64_t off_stride,
                                                       const uint32_t *__restrict__ n_win,
                                                       const uint32_t *__restrict__ e_word,
                                                       const uint16_t *__restrict__ e_half,
                                                       uint32_t *__restrict__ cursor,
                                                       uint32_t *__restrict__ out,
                                                       uint32_t k_h) {
    static_assert(kWinRegions == 64, "one wavefront scans the regions' counts");
    __shared__ uint32_t s_stage[kWinBatch];
    __shared__ uint8_t s_tag[kWinBatch];
    __shared__ uint32_t s_cnt[kWinBuckets], s_start[kWinBuckets], s_base[kWinBuckets];
    __shared__ uint32_t s_wave[kWinThreads / 64];
    __shared__ uint32_t s_first[kWinRegions];    // each region's first entry
    __shared__ uint32_t s_pre[kWinRegions + 1];  // records before each region
    const uint32_t r0 = blockIdx.x * kWinRegions;
    const uint32_t nr = r0 + kWinRegions < n_regions ? kWinRegions : n_regions - r0;
    if (threadIdx.x < 64) {
        const uint32_t i = threadIdx.x;
        const uint32_t n = i < nr ? n_win[r0 + i] : 0u;
        s_first[i] = i < nr ? offsets[(uint64_t)(r0 + i) * off_stride] : 0u;
        uint32_t incl = n;
        for (uint32_t d = 1; d < 64; d <<= 1) {
            const uint32_t o = __shfl_up(incl, d, 64);
            if (i >= d)
                incl += o;
        }
        s_pre[i + 1] = incl;
        if (i == 0)
            s_pre[0] = 0;
    }
    __syncthreads();
    const uint32_t total = s_pre[kWinRegions];
    auto keep = [](uint64_t r) -> uint32_t {
        return ((uint32_t)r & ((1u << kWinA) - 1u)) | ((uint32_t)(r >> 32) << kWinA);
    };
    for (uint32_t q = 0; q < total; q += kWinBatch) {
        const uint32_t m = total - q < (uint32_t)kWinBatch ? total - q : (uint32_t)kWinBatch;
        uint64_t v[kWinPer];
        uint32_t ok = 0;
#pragma unroll
        for (int u = 0; u < kWinPer; u++) {
            const uint32_t i = threadIdx.x + (uint32_t)u * kWinThreads;
            v[u] = 0;
            if (i < m) {
                const uint32_t idx = q + i;
                uint32_t j = 0;  // the last region with s_pre[j] <= idx
#pragma unroll
                for (uint32_t step = kWinRegions / 2; step; step >>= 1)
                    if (s_pre[j + step] <= idx)
                        j += step;
                const uint64_t x = (uint64_t)s_first[j] + (idx - s_pre[j]);
                v[u] = ((uint64_t)e_half[x] << 32) | e_word[x];
                ok |= 1u << u;
            }
        }
        win_append(v, ok, m, kWinA, kWinBuckets, 0, (uint64_t)k_h << kWinA, s_cnt, s_start, s_base, s_wave,
                   s_stage, s_tag, cursor, out, keep);
    }
}

// Level B: slice blockIdx.y of level-A bucket a = blockIdx.x -> block
// (a << 5) | ((t24 >> 19) & 31), record (t & (2^19 - 1)) | mark << 19.
__global__ void __launch_bounds__(kWinThreads) k_win_b(const uint32_t *__restrict__ in,
                                                       const uint32_t *__restrict__ cursor_a,
                                                       uint32_t *__restrict__ cursor_b,
                                                       uint32_t *__restrict__ out,
                                                       uint32_t k_h) {
    __shared__ uint32_t s_stage[kWinBatch];
    __shared__ uint8_t s_tag[kWinBatch];
    __shared__ uint32_t s_cnt[kWinBlocksPerBucket], s_start[kWinBlocksPerBucket],
        s_base[kWinBlocksPerBucket];
    __shared__ uint32_t s_wave[kWinThreads / 64];
    const uint32_t a = blockIdx.x;
    const uint32_t n = cursor_a[a];
    // the bucket's records in equal slices of whole batches
    const uint32_t per = ((n + kWinSlices - 1) / kWinSlices + kWinBatch - 1) / kWinBatch * kWinBatch;
    const uint32_t q0 = blockIdx.y * per;
    const uint32_t q1 = q0 + per < n ? q0 + per : n;
    const uint32_t *src = in + a * ((uint64_t)k_h << kWinA);
    auto keep = [](uint32_t v) -> uint32_t {
        return (v & ((1u << kWinB) - 1u)) | ((v >> kWinA) << kWinB);
    };
    for (uint32_t q = q0; q < q1; q += kWinBatch) {
        const uint32_t m = q1 - q < (uint32_t)kWinBatch ? q1 - q : (uint32_t)kWinBatch;
        uint32_t v[kWinPer];
        uint32_t ok = 0;
#pragma unroll
        for (int u = 0; u < kWinPer; u++) {
            const uint32_t i = threadIdx.x + (uint32_t)u * kWinThreads;
            v[u] = i < m ? src[q + i] : 0u;
            if (i < m)
                ok |= 1u << u;
        }
        // digit (t24 >> 19) & 31 of the record (t24 | mark << 24)
        win_append(v, ok, m, kWinB, kWinBlocksPerBucket, a * kWinBlocksPerBucket,
                   (uint64_t)k_h << kWinB, s_cnt, s_start, s_base, s_wave, s_stage, s_tag, cursor_b,
                   out, keep);
    }
}

// Dense records (position | mark << 30) -> their buckets of 2^log positions: a
// tile is sorted in LDS and appended in runs, one atomic per tile and bucket.
// Bound: its traffic, 12 bytes a record.
__global__ void __launch_bounds__(1024)
k_sort_records(const uint32_t *__restrict__ in, const uint32_t *__restrict__ n_in,
               uint32_t *__restrict__ out, uint64_t room, uint32_t log,
               uint32_t *__restrict__ cursor) {
    constexpr int kPer = 8;
    constexpr uint32_t kRecords = kPer * 1024;
    static_assert(kMarkBuckets <= 1024, "a bucket a thread");
    __shared__ uint32_t s_rec[kRecords];
    __shared__ uint32_t s_count[kMarkBuckets], s_place[kMarkBuckets], s_sum[kMarkBuckets / 64];
    const uint32_t n = *n_in, lane = threadIdx.x & 63u, wave = wave_id(), tid = threadIdx.x;
    for (uint32_t q = blockIdx.x * kRecords; q < n; q += gridDim.x * kRecords) {
        if (tid < kMarkBuckets)
            s_count[tid] = 0;
        uint32_t v[kPer], rank[kPer];
#pragma unroll
        for (int u = 0; u < kPer; u++) {
            const uint32_t i = q + tid + (uint32_t)u * 1024u;
            v[u] = i < n ? in[i] : 0u;  // no record is 0: its mark is not
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPer; u++)
            rank[u] = v[u] ? atomicAdd(&s_count[(v[u] & 0x3FFFFFFFu) >> log], 1u) : 0u;
        __syncthreads();
        uint32_t c = 0, incl = 0;
        if (tid < kMarkBuckets) {
            c = s_count[tid];
            incl = wave_inclusive(c);
            if (lane == 63)
                s_sum[wave] = incl;
        }
        __syncthreads();
        if (tid < kMarkBuckets) {
#pragma unroll
            for (uint32_t w = 0; w < kMarkBuckets / 64; w++)
                incl += w < wave ? s_sum[w] : 0u;
            s_count[tid] = incl - c;
            const uint32_t place = c ? atomicAdd(&cursor[tid], c) : 0u;
            s_place[tid] = tid * (uint32_t)room + place - (incl - c);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPer; u++)
            if (v[u])
                s_rec[s_count[(v[u] & 0x3FFFFFFFu) >> log] + rank[u]] = v[u];
        __syncthreads();
        const uint32_t m = n - q < kRecords ? n - q : kRecords;
        for (uint32_t i = tid; i < m; i += 1024u) {
            const uint32_t x = s_rec[i], t = x & 0x3FFFFFFFu;
            out[s_place[t >> log] + i] = (t & ((1u << log) - 1u)) | (x >> 30 << log);
        }
        __syncthreads();  // the next tile rewrites the sums and records
    }
}

hipError_t launch_sort_records(const uint32_t *in, const uint32_t *n, uint32_t *out, uint64_t room,
                               uint32_t log, uint32_t *cursor, hipStream_t s) {
    hipLaunchKernelGGL(k_sort_records, dim3(512), dim3(1024), 0, s, in, n, out, room, log, cursor);
    return hipGetLastError();
}

// The distinct and trustworthy bits of bucket g = blockIdx.x, the 2^log
// positions from g << log of the chunk, and their tiles' counts, from the
// bucket's cursor[g] records (position | mark << log, `room` apart): bitmaps
// in LDS, every word of the bucket's tiles written.  clean: the cursor is left
// zero for the next chunk.  c0 is a multiple of the tile.
// Bound by its clears and LDS atomics at one or two workgroups per CU: 0.09 ms
// over 150 M positions; the byte flags cost 0.20 ms to store at random and
// 0.17 ms to read again in the compaction (0.07 from bits).
// kLog: the bitmaps' room; the smaller ones leave room for several workgroups
// per CU where a chunk's buckets are small.
template <uint32_t kLog>  // log <= kLog
__global__ void __launch_bounds__(kLog >= 17 ? 1024 : 256)
k_marks(const uint32_t *__restrict__ in, uint64_t room, uint32_t log, uint32_t *__restrict__ cursor,
        int clean, uint64_t c0, uint64_t len, uint32_t *__restrict__ dbits,
        uint32_t *__restrict__ tbits, uint32_t *__restrict__ tile_d,
        uint32_t *__restrict__ tile_t) {
    __shared__ uint32_t s_bits[2u << (kLog - 5)];  // the distinct words, then the trustworthy ones
    const uint32_t words = 1u << (log - 5);
    uint32_t *s_d = s_bits, *s_t = s_bits + words;
    const uint32_t g = blockIdx.x;
    for (uint32_t i = threadIdx.x; i < 2 * words; i += blockDim.x)
        s_bits[i] = 0;
    const uint32_t n = cursor[g];
    __syncthreads();
    if (clean && threadIdx.x == 0)
        cursor[g] = 0;
    const uint32_t *src = in + (uint64_t)g * room;
    constexpr int kUnroll = 4;
    for (uint32_t i = threadIdx.x; i < n; i += kUnroll * blockDim.x) {
        uint32_t v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; u++)
            v[u] = i + u * blockDim.x < n ? src[i + u * blockDim.x] : 0u;  // no record has mark 0
#pragma unroll
        for (int u = 0; u < kUnroll; u++) {
            const uint32_t mark = v[u] >> log, p = v[u] & ((1u << log) - 1u);
            if (mark)
                atomicOr(&s_d[p >> 5], 1u << (p & 31u));
            if (mark & 2u)
                atomicOr(&s_t[p >> 5], 1u << (p & 31u));
        }
    }
    __syncthreads();
    const uint64_t p0 = (uint64_t)g << log;
    const uint64_t left = (len - p0 + kTile - 1) / kTile * (kTile / 32);  // words to the chunk's end
    const uint32_t nw = left < words ? (uint32_t)left : words;
    const uint64_t w0 = (c0 + p0) / 32;
    for (uint32_t i = threadIdx.x; i < nw; i += blockDim.x) {
        const uint32_t d = s_d[i], t = s_t[i];
        dbits[w0 + i] = d;
        tbits[w0 + i] = t;
        // a tile is 32 words: half a wavefront's
        uint32_t nd = (uint32_t)__popc(d), nt = (uint32_t)__popc(t);
        for (uint32_t k = 16; k >= 1; k >>= 1) {
            nd += __shfl_xor(nd, k, 32);
            nt += __shfl_xor(nt, k, 32);
        }
        if ((i & 31u) == 0) {
            tile_d[(w0 + i) / 32] = nd;
            tile_t[(w0 + i) / 32] = nt;
        }
    }
}

// The marks of a chunk's n_buckets buckets.
hipError_t launch_marks(const uint32_t *in, uint64_t room, uint32_t log, uint32_t *cursor,
                        bool clean, uint64_t c0, uint64_t len, uint64_t n_bases,
                        const Workspace &W, hipStream_t s) {
    const uint32_t n = (uint32_t)((len + (1ull << log) - 1) >> log);
    const auto kernel = log <= 13 ? k_marks<13> : log <= 15 ? k_marks<15> : log <= 17 ? k_marks<17>
                                                                                     : k_marks<19>;
    hipLaunchKernelGGL(kernel, dim3(n), dim3(log > 15 ? 1024 : 256), 0, s, in, room, log, cursor,
                       clean ? 1 : 0, c0, len, distinct_bits(W), trust_bits(W, n_bases), W.tile_a,
                       W.tile_b);
    return hipGetLastError();
}

// Records mode, in which the winner passes distribute the regions' records:
// for chunks of more than 2^28 positions, whose records the region pass cannot
// sort by bucket itself (512 buckets of 2^19 positions).
// KMERCO_WINNER_RECORDS=1 forces it for every chunk, 0 turns it off: chunks
// are 2^28 positions at most then (max_part_chunk).
int records_from_env() {
    const char *e = std::getenv("KMERCO_WINNER_RECORDS");
    return e && *e ? (std::atoi(e) != 0 ? 1 : 0) : -1;
}

bool records_mode(uint64_t len) { return records_from_env() == 1 || len > kBinChunk; }

uint64_t max_part_chunk() { return records_from_env() == 0 ? kBinChunk : kPartChunk; }

// The winner passes of one chunk [c0, c0 + len): its records, at most k_h a
// position, region r's n_win[r] of them at offsets[r * off_stride] of the word
// and half arrays; area_a, area_b: the entry buffers (k_h entries of 8 bytes a
// position, of which the areas take 4), the records' own not the first.
hipError_t winner_passes(uint32_t k_h, uint32_t n_regions, const uint32_t *offsets, uint64_t off_stride,
                         const uint32_t *n_win, const uint32_t *rec_word,
                         const uint16_t *rec_half, uint64_t c0, uint64_t len, uint64_t n_bases,
                         uint32_t *area_a, uint32_t *area_b, const Workspace &W, hipStream_t s, Profiler *P) {
    uint32_t *cursors = W.win_cursors;  // kWinBuckets level-A, then the blocks' level-B cursors
    const uint32_t n_a = (uint32_t)((len + (1ull << kWinA) - 1) >> kWinA);
    if (P)
        P->begin(kPhWinners, s);
    static_assert(kWinBuckets + kWinBuckets * kWinBlocksPerBucket == kWinCursors, "cursors");
    hipError_t e = fill_u32(cursors, kWinCursors, 0u, s);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_win_a, dim3((n_regions + kWinRegions - 1) / kWinRegions),
                           dim3(kWinThreads), 0, s, n_regions, offsets, off_stride, n_win,
                           rec_word, rec_half, cursors, area_a, k_h);
        e = hipGetLastError();
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_win_b, dim3(n_a, kWinSlices), dim3(kWinThreads), 0, s,
                           (const uint32_t *)area_a, (const uint32_t *)cursors,
                           cursors + kWinBuckets, area_b, k_h);
        e = hipGetLastError();
    }
    if (e == hipSuccess) {
        e = launch_marks(area_b, (uint64_t)k_h << kWinB, kWinB, cursors + kWinBuckets, false, c0, len,
                         n_bases, W, s);
    }
    if (P)
        P->end(s);
    return e;
}

hipError_t launch_record_winners(uint32_t k_h, uint32_t n_regions, const uint32_t *off, const uint32_t *n,
                                 const uint32_t *word, const uint16_t *half, uint64_t c0,
                                 uint64_t len, uint64_t n_bases, const Workspace &W, hipStream_t s,
                                 Profiler *P) {
    return winner_passes(k_h, n_regions, off, 1, n, word, half, c0, len, n_bases, (uint32_t *)W.entries,
                         (uint32_t *)W.bucketed, W, s, P);
}

bool carry_fits(const BinPlan &plan) {
    // the region's cells are staged in the region pass's s_cell array
    // (kSparseCells = counters / 8 entries)
    return (1u << plan.region_shift) <= plan.region_counters / 8u;
}

Carry carry_of(const Workspace &W, const BinPlan &plan, uint64_t chunk_positions,
               uint64_t n_chunks) {
    Carry c{};
    if (n_chunks < 2 || !carry_fits(plan))
        return c;
    const uint64_t prev = n_chunks - 1;
    if (!W.carry || W.carry_cap < prev * chunk_positions ||
        W.carry_idx_cap < prev * plan.n_regions)
        return c;
    c.n_prev = (uint32_t)prev;
    c.stride = plan.n_regions;
    c.cap = chunk_positions;
    c.word = (uint32_t *)W.carry;
    c.half = W.carry + 2 * W.carry_cap;
    c.off = W.carry_off;
    c.n = W.carry_n;
    return c;
}

hipError_t launch_carried_winners(const BinPlan &plan, const Carry &carry, uint32_t j, uint64_t c0,
                                  uint64_t len, uint64_t n_bases, const Workspace &W, hipStream_t s,
                                  Profiler *P) {
    const uint64_t at = (uint64_t)j * carry.stride;
    // carried calls have one hash function
    return winner_passes(1, plan.n_regions, carry.off + at, 1, carry.n + at,
                         carry.word + (uint64_t)j * carry.cap, carry.half + (uint64_t)j * carry.cap,
                         c0, len, n_bases, (uint32_t *)W.bucketed, (uint32_t *)W.entries, W, s, P);
}

// ---------------------------------------------------------------------------
// launcher
// ---------------------------------------------------------------------------
bool bin_plan(const FilterArgs &F, uint64_t chunk_positions, BinPlan &B, uint32_t part_log,
              uint32_t region_counters) {
    if (region_counters != kRegionCounters && region_counters != kSmallRegionCounters)
        return false;
    // largest power-of-two cell count whose eta counters fit the LDS arrays
    uint32_t shift = 0;
    while (((2ull << shift) * F.eta) <= (uint64_t)region_counters)
        shift++;
    if (((1ull << shift) * F.eta) > (uint64_t)region_counters)
        return false;
    if (part_log > kPartLog)
        part_log = kPartLog;
    const uint64_t n_words = F.X * F.Y;
    const uint64_t n_regions = (n_words + (1ull << shift) - 1) >> shift;
    B = BinPlan{};
    B.region_shift = shift;
    B.region_counters = region_counters;
    const uint64_t np = (n_regions + (1ull << part_log) - 1) >> part_log;
    if (np > kMaxParts)
        return false;
    B.n_regions = (uint32_t)n_regions;
    if (np > 1) {  // partitioned
        B.n_parts = (uint32_t)np;
        B.part_log = part_log;
        uint64_t g = (kPartRooms + np - 1) / np;
        g = g > kMaxPartRooms ? kMaxPartRooms : g;
        B.rooms = (uint32_t)(g * n_regions > kMaxMatrix ? kMaxMatrix / n_regions : g);
        return true;
    }
    // small chunks of the countBF have kRoomSpread rooms at most: a reservation
    // covers every smaller insert
    uint64_t tile = (chunk_positions + kRoomSpread - 1) / kRoomSpread;
    tile = (tile + kBinWG - 1) / kBinWG * kBinWG;
    tile = tile < kRoomFloor ? kRoomFloor : (tile > kRoomMin ? kRoomMin : tile);
    while ((chunk_positions + tile - 1) / tile * n_regions > kMaxMatrix)
        tile *= 2;
    const uint64_t g = (chunk_positions + tile - 1) / tile;
    B.rooms = (uint32_t)(g > kRoomSpread ? g : kRoomSpread);
    return true;
}

hipError_t launch_binned_chunk(const FilterArgs &F, const ReadsArgs &R, uint64_t c0, uint64_t c1,
                               const BinPlan &plan, const Workspace &W, bool classify,
                               uint32_t tau, const Carry &carry, hipStream_t s, Profiler *P) {
    if (c0 & 63u)
        return hipErrorInvalidValue;  // chunks start at whole words of the masks
    if (carry.mode != Carry::kNone && (!carry_fits(plan) || carry.stride != plan.n_regions))
        return hipErrorInvalidValue;  // the region pass stages the cells it classifies against
    // entries (positions x hash functions) are counted in 32 bits
    if ((plan.n_parts == 0 && c1 - c0 > kBinChunk) || (c1 - c0) * F.k_h >= (1ull << 32))
        return hipErrorInvalidValue;
    BlockPlan blocks;
    if (!block_plan(plan, F.k_h, c1 - c0, blocks))
        return hipErrorInvalidValue;
    return launch_blocks_chunk(F, R, c0, c1, plan, blocks, W, classify, tau, carry,
                               carry.mode != Carry::kOut && records_mode(c1 - c0), s, P);
}

}  // namespace kc
