// Binned insertion over block-sorted entry lists.
//
// The hashing workgroup of a block (at most 16384 entries) sorts them by
// region in LDS and writes them as one contiguous run, with a table of the
// 16-bit offset of every region's run inside the block.  Nothing has to be
// counted before: a block's place in the list is fixed, so there are no count
// matrices, no scans and no separate distribution passes.  The region pass
// then gathers its region's short runs from every block: one workgroup per
// region counts hits and first occurrences in LDS as before.
//
// Against counted binning (slot ids written, two counted distribution passes
// of 6-byte entries, their count matrices transposed and scanned), the
// bacterial workload's 150 M bases take 1.44 instead of 1.98 ms, 1 M bases
// into 37 regions 67 instead of 112 us.
//
// An entry is 32 bits: the counter within the region (14 bits) and the
// position within the block (14 bits); the block gives the rest of the
// position.
#include <hip/hip_runtime.h>

#include "kc_bin_hash.hpp"
#include "kc_blocks.hpp"
#include "kc_device.hpp"
#include "kc_kernels.hpp"
#include "kc_region.hpp"

namespace kc {

namespace {

static_assert(kBlockLog + kLocalBits <= 32, "an entry holds the counter and the position");

// Inclusive sum over the wavefront (row shifts, then row broadcasts).
__device__ __forceinline__ uint32_t wave_inclusive(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);
    return x;
}

}  // namespace

// Hash every valid window of the block once and write the block's entries
// sorted by region.  kEpt: entries per thread (kKh hash functions x
// positions); kFast, kWide as k_bin_count.
//
// The block's valid windows are first listed in LDS (in the space the sorted
// entries take later), so that every lane hashes one at each step.  A
// thread's entries stay in registers between hashing, where the histogram's
// atomic also gives each entry's rank in its region, and staging.  Bound by
// its vector instructions (82% busy; 144 per 64 windows, 117 of them the
// hash): 0.55 ms for the bacterial workload's 116 M windows, where hashing
// alone and writing slot ids took 0.42.
template <int kWG, int kEpt, int kKh, bool kFast, bool kWide>
__global__ void __launch_bounds__(kWG, 4)
k_hash_sort(FilterArgs F, ReadsArgs R, uint64_t c0, uint64_t c1, BlockPlan B, uint32_t shift,
            uint32_t n_regions, uint32_t *__restrict__ list, uint16_t *__restrict__ table,
            unsigned long long *__restrict__ n_valid) {
    constexpr int kSteps = kEpt / kKh;
    constexpr uint32_t kPos = kSteps * kWG;    // positions per block
    constexpr uint32_t kEntries = kEpt * kWG;  // room for its entries
    static_assert(kEntries <= kBlockEntries, "entries are staged in LDS");
    extern __shared__ uint32_t s_hist[];  // counts, then starts, per region
    __shared__ __align__(16) uint32_t s_stage[kEntries];
    __shared__ uint32_t s_wave[kWG / 64];
    uint16_t *s_list = reinterpret_cast<uint16_t *>(s_stage);
    const uint32_t lane = threadIdx.x & 63u, wave = wave_id();
    constexpr uint32_t kWaves = kWG / 64;
    for (uint32_t i = threadIdx.x; i < n_regions; i += kWG)
        s_hist[i] = 0;
    const uint64_t p0 = c0 + (uint64_t)blockIdx.x * kPos;
    uint32_t nv;
    {
        // each wavefront lists the valid positions of its share of the block:
        // 64 of them per step, stored by consecutive lanes
        constexpr uint32_t kWords = kPos / 32u / kWaves;  // validity words per wavefront
        static_assert(kWords <= 64 && kWords % 2 == 0, "a word per lane, two per step");
        const uint32_t w0 = wave * kWords;
        uint32_t v = 0;
        if (lane < kWords && p0 + 32u * (w0 + lane) < c1)
            v = R.valid[(p0 >> 5) + w0 + lane];
        const uint32_t incl = wave_inclusive((uint32_t)__popc(v));
        if (lane == 63)
            s_wave[wave] = incl;
        __syncthreads();
        uint32_t at = 0;
        nv = 0;
#pragma unroll
        for (uint32_t w = 0; w < kWaves; w++) {
            const uint32_t t = s_wave[w];
            at += w < wave ? t : 0u;
            nv += t;
        }
        at = __builtin_amdgcn_readfirstlane(at);
        for (uint32_t i = 0; i < kWords; i += 2) {
            const uint64_t m = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)v, i + 1) << 32) |
                               (uint32_t)__builtin_amdgcn_readlane((int)v, i);
            if (__builtin_amdgcn_inverse_ballot_w64(m))
                s_list[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                    (uint16_t)(32u * (w0 + i) + lane);
            at += (uint32_t)__popcll(m);
        }
    }
    __syncthreads();
    const uint32_t *__restrict__ codes = R.codes + (p0 >> 4);
    const uint32_t K = R.k, k_h = kFast ? 1u : F.k_h;
    uint32_t ent[kEpt];  // counter | position << kLocalBits
    uint32_t key[kEpt];  // region | rank << 16
    // A step's code words are requested a step before they are hashed, and a
    // rank is taken in a step after its atomic, so that neither is waited for.
    auto position = [&](int j) -> uint32_t {
        const uint32_t i = (uint32_t)j * kWG + threadIdx.x;
        return i < nv ? s_list[i] : 0u;
    };
    uint32_t q = position(0), q_next = kSteps > 1 ? position(1) : 0u;
    WindowWords<kWide> w(codes, q);
    uint32_t rank[kKh];
#pragma unroll
    for (int j = 0; j < kSteps; j++) {
        const uint32_t i = (uint32_t)j * kWG + threadIdx.x;
        const WindowWords<kWide> wn(codes, q_next);
        const uint32_t q_after = j + 2 < kSteps ? position(j + 2) : 0u;
        uint32_t old[kKh];
        if (i < nv)
            window_entries<kFast, kWide, kKh>(
                F, w, q, K, shift, [&](int a, uint32_t r, uint32_t local) {
                    ent[j * kKh + a] = local | (q << kLocalBits);
                    key[j * kKh + a] = r;
                    old[a] = atomicAdd(&s_hist[r], 1u);
                });
        if (j > 0) {
#pragma unroll
            for (int a = 0; a < kKh; a++)
                key[(j - 1) * kKh + a] |= rank[a] << 16;
        }
#pragma unroll
        for (int a = 0; a < kKh; a++)
            rank[a] = old[a];
        q = q_next;
        q_next = q_after;
        w = wn;
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int a = 0; a < kKh; a++)
        key[(kSteps - 1) * kKh + a] |= rank[a] << 16;
    __syncthreads();
    {  // counts -> starts, in place: each wavefront scans a share of the
       // regions, 64 at a time, then adds the shares before its own
        const uint32_t share = (n_regions + kWG - 1) / kWG * 64u;
        const uint32_t r0 = wave * share;
        uint32_t run = 0;
        for (uint32_t u = 0; u < share; u += 64) {
            const uint32_t r = r0 + u + lane;
            const uint32_t c = r < n_regions ? s_hist[r] : 0u;
            const uint32_t incl = wave_inclusive(c);
            if (r < n_regions)
                s_hist[r] = run + incl - c;
            run += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        }
        if (lane == 0)
            s_wave[wave] = run;
        __syncthreads();
        uint32_t before = 0;
#pragma unroll
        for (uint32_t w = 0; w < kWaves; w++)
            before += w < wave ? s_wave[w] : 0u;
        for (uint32_t u = 0; u < share; u += 64) {
            const uint32_t r = r0 + u + lane;
            if (r < n_regions)
                s_hist[r] += before;
        }
    }
    __syncthreads();
    const uint32_t total = nv * k_h;
    uint16_t *__restrict__ trow = table + (uint64_t)blockIdx.x * B.row;
    for (uint32_t i = threadIdx.x; i <= n_regions; i += kWG)
        trow[i] = (uint16_t)(i < n_regions ? s_hist[i] : total);
#pragma unroll
    for (int j = 0; j < kSteps; j++)
        if ((uint32_t)j * kWG + threadIdx.x < nv) {
#pragma unroll
            for (int a = 0; a < kKh; a++)
                if (kKh == 1 || (uint32_t)a < k_h) {
                    const uint32_t k = key[j * kKh + a];
                    s_stage[s_hist[k & 0xFFFFu] + (k >> 16)] = ent[j * kKh + a];
                }
        }
    __syncthreads();
    uint4 *__restrict__ out = reinterpret_cast<uint4 *>(list + (uint64_t)blockIdx.x * B.cap);
    const uint4 *src = reinterpret_cast<const uint4 *>(s_stage);
    for (uint32_t i = threadIdx.x; i < (total + 3u) / 4u; i += kWG)
        out[i] = src[i];
    if (threadIdx.x == 0)
        atomicAdd(n_valid, (unsigned long long)nv);
}

// Table of a chunk, one row of run starts per block -> one row of blocks per
// region (64 x 64 tiles through LDS): the region pass of short runs then
// reads the starts of 64 blocks at once.
__global__ void __launch_bounds__(256)
k_turn_table(const uint16_t *__restrict__ in, uint16_t *__restrict__ out, uint32_t n_blocks,
             uint32_t row, uint32_t out_row) {
    __shared__ uint16_t t[64][66];
    const uint32_t r0 = blockIdx.x * 64, b0 = blockIdx.y * 64;
    const uint32_t x = threadIdx.x & 31u, y = threadIdx.x >> 5;
    for (uint32_t j = y; j < 64; j += 8) {
        uint32_t v = 0;
        if (b0 + j < n_blocks && r0 + 2 * x < row)  // rows are whole 32-bit words
            v = *reinterpret_cast<const uint32_t *>(in + (uint64_t)(b0 + j) * row + r0 + 2 * x);
        *reinterpret_cast<uint32_t *>(&t[j][2 * x]) = v;
    }
    __syncthreads();
    for (uint32_t j = y; j < 64; j += 8)
        if (r0 + j < row && b0 + 2 * x < out_row)
            *reinterpret_cast<uint32_t *>(out + (uint64_t)(r0 + j) * out_row + b0 + 2 * x) =
                (uint32_t)t[2 * x][j] | ((uint32_t)t[2 * x + 1][j] << 16);
}

// The region pass over the blocks' runs.  kCounters: counters per region (as
// k_region).  kCells: the cells each thread updates, held in registers (the
// plan's region has kCells * kRegionWG cells), or 0 for regions of fewer cells than
// threads.  kLanes: lanes that take a run together (by its expected length),
// or 0 for short runs: a wavefront takes the runs of 64 blocks at once (their
// starts are a segment of the turned table's rows) and lays their entries end
// to end over its lanes, so that every lane counts an entry at each step; the
// lane's run is found by counting the run heads at and before it.
//
// Persistent.  The regions that the workgroups of one XCD (every eighth
// workgroup) hold at a time are consecutive, so that the blocks' neighbouring
// runs, which share cache lines, are read through one L2.
// On the bacterial workload's 3914 regions, 0.51 ms: 0.20 of it stores flag
// bytes at random positions, the rest is LDS atomics and laying out the runs
// (6 entries each).  A plain read before the minimum's atomic took off 0.06,
// blocks of 32768 entries instead of 16384 0.2.
//
// The next region's cells and first bounds are requested before the current
// region's stores, since a wavefront's loads and stores complete in order.
template <int kCounters, int kCells, int kLanes>
__global__ void __launch_bounds__(kRegionWG)
k_region_runs(FilterArgs F, uint64_t c0, BinPlan P, BlockPlan B,
              const uint32_t *__restrict__ list, const uint16_t *__restrict__ table,
              uint8_t *__restrict__ flags, int classify, uint32_t tau, RecordSpace rec, Carry C) {
    constexpr uint32_t kSparseCells = kCounters / 8;
    constexpr bool kTile = (uint32_t)kCells * kRegionWG <= kSparseCells;
    constexpr int kHold = kCells ? kCells : 1;
    constexpr int kChunks = 8;  // kLanes = 0: 64-entry steps in flight
    constexpr uint32_t kWindow = 64u * kChunks;
    constexpr int kWaves = kRegionWG / 64;
    __shared__ uint32_t hits[kCounters];
    __shared__ uint32_t first[kCounters];
    // the region's final cells (for carried records); before them, of each
    // run: list index of its entries less their place, position base
    constexpr uint32_t kRunWords = kLanes ? 0 : kWaves * 64;
    __shared__ unsigned long long s_mem[(kTile && kSparseCells > kRunWords) ? kSparseCells
                                                                            : kRunWords + 1];
    unsigned long long *s_cell = s_mem;
    auto s_run = reinterpret_cast<uint2(*)[64]>(s_mem);
    __shared__ uint32_t s_nwin, s_total, s_base;
    __shared__ uint32_t s_head[kLanes ? 1 : kWaves][2 * kChunks];
    const uint32_t shift = P.region_shift, S = 1u << shift;
    const uint64_t n_words = F.X * F.Y;
    const bool carry_out = C.mode == Carry::kOut;
    const bool carry_in = kTile && C.mode == Carry::kIn && C.n_prev > 0;
    const bool records = carry_out || rec.n != nullptr;
    for (uint32_t i = threadIdx.x; i < (uint32_t)kCounters; i += kRegionWG) {
        hits[i] = 0;
        first[i] = kIdle;
    }
    if (threadIdx.x == 0) {
        s_nwin = 0;
        s_total = 0;
    }
    const uint32_t grid = gridDim.x;
    const uint32_t lane = threadIdx.x & 63u, wave = wave_id();
    auto count = [&](uint32_t e, uint32_t tb) {
        const uint32_t local = e & ((1u << kLocalBits) - 1u);
        const uint32_t t = tb + (e >> kLocalBits);
        atomicAdd(&hits[local], 1u);
        // most entries are not the first of their counter: a plain read (any
        // value read is at least the minimum so far) saves their atomic
        if (t < first[local])
            atomicMin(&first[local], t);
    };
    // cells of region r: those of a region past the last are not read
    auto load_cells = [&](uint32_t r, uint64_t(&cell)[kHold]) {
        const uint64_t wbase = (uint64_t)r << shift;
#pragma unroll
        for (int k = 0; k < kHold; k++) {
            const uint32_t w = threadIdx.x + (uint32_t)k * kRegionWG;
            cell[k] = (kCells && r < P.n_regions && wbase + w < n_words) ? F.words[wbase + w] : 0ull;
        }
    };
    // bounds of the run of region r in block b
    auto bounds = [&](uint32_t r, uint32_t b, uint32_t &s, uint32_t &e) {
        s = e = 0;
        if (b < B.n_blocks && r < P.n_regions) {
            const uint16_t *t = kLanes == 0 ? table + (uint64_t)r * B.turned + b
                                            : table + (uint64_t)b * B.row + r;
            s = t[0];
            e = t[kLanes == 0 ? B.turned : 1u];
        }
    };
    constexpr int kTeam = kLanes ? kLanes : 64;
    constexpr uint32_t kTeams = kRegionWG / kTeam;
    const uint32_t team = threadIdx.x / kTeam, sub = threadIdx.x % kTeam;
    constexpr int kUnroll = kLanes ? 2 : 1;  // runs a team of lanes has in flight
    // the first block whose bounds a thread takes, and its step
    const uint32_t b_first = kLanes ? team : threadIdx.x;
    constexpr uint32_t b_step = kLanes ? kTeams : kRegionWG;
    uint32_t r = (grid & 7u) == 0 ? (blockIdx.x & 7u) * (grid >> 3) + (blockIdx.x >> 3) : blockIdx.x;
    uint64_t cell[kHold];
    uint32_t ns[kUnroll], ne[kUnroll];
    load_cells(r, cell);
#pragma unroll
    for (int u = 0; u < kUnroll; u++)
        bounds(r, b_first + u * b_step, ns[u], ne[u]);
    __syncthreads();  // counters clean, sums zero
    for (; r < P.n_regions; r += grid) {
        const uint64_t wbase = (uint64_t)r << shift;
        const uint32_t nw = wbase + S <= n_words ? S : (uint32_t)(n_words - wbase);
        uint32_t mine = 0;  // entries of the runs whose length this lane has
        if constexpr (kLanes == 0) {
            for (uint32_t b0 = wave * 64u; b0 < B.n_blocks; b0 += kRegionWG) {
                const uint32_t b = b0 + lane;
                const uint32_t s = ns[0], len = ne[0] - ns[0];
                const uint32_t incl = wave_inclusive(len);
                const uint32_t pre = incl - len;
                const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                const uint64_t some = __ballot(len != 0);
                mine += len;
                if (len) {
                    const uint32_t i = __builtin_amdgcn_mbcnt_hi(
                        (uint32_t)(some >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)some, 0u));
                    s_run[wave][i] = make_uint2(b * B.cap + s - pre, b << B.pos_log);
                }
                bounds(r, b + kRegionWG, ns[0], ne[0]);
                for (uint32_t w0 = 0; w0 < n; w0 += kWindow) {
                    if (lane < 2u * kChunks)
                        s_head[wave][lane] = 0;
                    __builtin_amdgcn_wave_barrier();
                    if (len && pre >= w0 && pre - w0 < kWindow)
                        atomicOr(&s_head[wave][(pre - w0) >> 5], 1u << (pre & 31u));
                    // runs that start before the window
                    uint32_t runs = (uint32_t)__popcll(__ballot(len && pre < w0));
                    __builtin_amdgcn_wave_barrier();
                    uint32_t x[kChunks], tb[kChunks];
#pragma unroll
                    for (int c = 0; c < kChunks; c++) {
                        const uint32_t at = w0 + 64u * c + lane;
                        if (w0 + 64u * c < n) {
                            const uint32_t m0 = (uint32_t)__builtin_amdgcn_readfirstlane(
                                (int)s_head[wave][2 * c]);
                            const uint32_t m1 = (uint32_t)__builtin_amdgcn_readfirstlane(
                                (int)s_head[wave][2 * c + 1]);
                            const uint64_t m = ((uint64_t)m1 << 32) | m0;
                            // heads at or before the lane, less one: its run
                            const uint64_t h = m >> 1;
                            const uint32_t i = runs + (m0 & 1u) - 1u +
                                               __builtin_amdgcn_mbcnt_hi(
                                                   (uint32_t)(h >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)h, 0u));
                            runs += (uint32_t)__popcll(m);
                            if (at < n) {
                                const uint2 d = s_run[wave][i];
                                x[c] = list[d.x + at];
                                tb[c] = d.y;
                            }
                        }
                    }
#pragma unroll
                    for (int c = 0; c < kChunks; c++)
                        if (w0 + 64u * c + lane < n)
                            count(x[c], tb[c]);
                    __builtin_amdgcn_wave_barrier();
                }
            }
        } else {
            for (uint32_t b0 = team; b0 < B.n_blocks; b0 += kUnroll * kTeams) {
                // a first 16-byte group of entries of every run, and the next
                // runs' bounds, are requested before any entry is counted
                uint32_t s[kUnroll], e[kUnroll], g[kUnroll];
                uint4 x[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; u++) {
                    s[u] = ns[u];
                    e[u] = ne[u];
                    g[u] = (s[u] & ~3u) + 4u * sub;
                    if (g[u] < e[u])
                        x[u] = *reinterpret_cast<const uint4 *>(
                            list + (uint64_t)(b0 + (uint32_t)u * kTeams) * B.cap + g[u]);
                    mine += sub == 0 ? e[u] - s[u] : 0u;
                    bounds(r, b0 + (uint32_t)(u + kUnroll) * kTeams, ns[u], ne[u]);
                }
#pragma unroll
                for (int u = 0; u < kUnroll; u++) {
                    const uint32_t b = b0 + (uint32_t)u * kTeams;
                    const uint32_t tb = b << B.pos_log;
                    const uint32_t *blk = list + (uint64_t)b * B.cap;
                    while (g[u] < e[u]) {
                        const uint32_t gn = g[u] + 4u * kTeam;
                        uint4 y = make_uint4(0u, 0u, 0u, 0u);
                        if (gn < e[u])
                            y = *reinterpret_cast<const uint4 *>(blk + gn);
                        if (g[u] >= s[u])
                            count(x[u].x, tb);
                        if (g[u] + 1u >= s[u] && g[u] + 1u < e[u])
                            count(x[u].y, tb);
                        if (g[u] + 2u >= s[u] && g[u] + 2u < e[u])
                            count(x[u].z, tb);
                        if (g[u] + 3u >= s[u] && g[u] + 3u < e[u])
                            count(x[u].w, tb);
                        x[u] = y;
                        g[u] = gn;
                    }
                }
            }
        }
        if (records && mine)
            atomicAdd(&s_total, mine);
        __syncthreads();
        if (records) {
            // room for a record of every entry of the region
            if (threadIdx.x == 0)
                s_base = s_total ? atomicAdd(rec.cursor, s_total) : 0u;
            __syncthreads();
        }
        uint64_t celln[kHold];
        load_cells(r + grid, celln);
#pragma unroll
        for (int u = 0; u < kUnroll; u++)
            bounds(r + grid, b_first + u * b_step, ns[u], ne[u]);
        const uint64_t base = records ? s_base : 0u;
        const WinnerSink out{flags,
                             c0,
                             carry_out ? C.word + (uint64_t)C.chunk * C.cap
                                       : (rec.n ? rec.word : nullptr),
                             carry_out ? C.half + (uint64_t)C.chunk * C.cap : rec.half,
                             base,
                             &s_nwin,
                             carry_out};
        if (kCells) {
#pragma unroll
            for (int k = 0; k < kHold; k++) {
                const uint32_t w = threadIdx.x + (uint32_t)k * kRegionWG;
                if (w < nw) {
                    const uint64_t next = region_cell(F, shift, wbase, w, cell[k], hits, first, out,
                                                      classify, tau);
                    if (kTile && C.mode == Carry::kIn)
                        s_cell[w] = next;
                }
            }
        } else {
            for (uint32_t w = threadIdx.x; w < nw; w += kRegionWG) {
                const uint64_t next = region_cell(F, shift, wbase, w, F.words[wbase + w], hits,
                                                  first, out, classify, tau);
                if (kTile && C.mode == Carry::kIn)
                    s_cell[w] = next;
            }
        }
        __syncthreads();  // the region's LDS work and its winner count are complete
        if (carry_in)
            mark_carried(F, shift, C, r, s_cell, tau);
        if (records) {
            if (threadIdx.x == 0) {
                if (carry_out) {
                    C.off[(uint64_t)C.chunk * C.stride + r] = (uint32_t)base;
                    C.n[(uint64_t)C.chunk * C.stride + r] = s_nwin;
                } else {
                    rec.off[r] = (uint32_t)base;
                    rec.n[r] = s_nwin;
                }
                s_nwin = 0;
                s_total = 0;
            }
        }
        if (records || carry_in)
            __syncthreads();  // the sums and s_cell are rewritten by the next region
#pragma unroll
        for (int k = 0; k < kHold; k++)
            cell[k] = celln[k];
    }
}

namespace {

using SortKernel = void (*)(FilterArgs, ReadsArgs, uint64_t, uint64_t, BlockPlan, uint32_t,
                            uint32_t, uint32_t *, uint16_t *, unsigned long long *);
using RunsKernel = void (*)(FilterArgs, uint64_t, BinPlan, BlockPlan, const uint32_t *,
                            const uint16_t *, uint8_t *, int, uint32_t, RecordSpace, Carry);

template <int kKh, bool kFast, bool kWide>
SortKernel sort_kernel_of(const BlockPlan &B) {
    if (B.wg == 1024)
        return k_hash_sort<1024, 32, kKh, kFast, kWide>;
    return B.ept == 32 ? k_hash_sort<512, 32, kKh, kFast, kWide>
                       : k_hash_sort<512, 8, kKh, kFast, kWide>;
}

template <int kKh, bool kFast>
SortKernel sort_kernel_for(const BlockPlan &B, uint32_t k) {
    return k > 32 ? sort_kernel_of<kKh, kFast, true>(B) : sort_kernel_of<kKh, kFast, false>(B);
}

SortKernel sort_kernel(const FilterArgs &F, uint32_t k, const BlockPlan &B) {
    switch (B.kh) {
    case 1:
        return fast_layout(F) ? sort_kernel_for<1, true>(B, k) : sort_kernel_for<1, false>(B, k);
    case 2:
        return sort_kernel_for<2, false>(B, k);
    case 4:
        return sort_kernel_for<4, false>(B, k);
    default:
        return sort_kernel_for<8, false>(B, k);
    }
}

template <int kCounters, int kCells>
RunsKernel runs_kernel_of(const BinPlan &P, const BlockPlan &B) {
    if (B.turned)
        return k_region_runs<kCounters, kCells, 0>;
    return B.cap / P.n_regions <= 64 ? k_region_runs<kCounters, kCells, 4>
                                     : k_region_runs<kCounters, kCells, 16>;
}

// The region pass's instance: counters per region, cells per thread, and
// lanes per run by the run's expected length.
template <int kCounters>
RunsKernel runs_kernel(const BinPlan &P, const BlockPlan &B) {
    switch ((1u << P.region_shift) / kRegionWG) {
    case 0:
        return runs_kernel_of<kCounters, 0>(P, B);
    case 1:
        return runs_kernel_of<kCounters, 1>(P, B);
    case 2:
        return runs_kernel_of<kCounters, 2>(P, B);
    case 4:
        return runs_kernel_of<kCounters, 4>(P, B);
    default:  // two counters a cell
        return runs_kernel_of<kCounters, 8>(P, B);
    }
}

}  // namespace

bool block_plan(const BinPlan &plan, uint32_t k_h, uint64_t len, BlockPlan &B) {
    if (plan.n_parts || plan.n_regions > kBlockRegions || len == 0)
        return false;
    B = BlockPlan{};
    B.kh = 1;
    while (B.kh < k_h)
        B.kh *= 2;
    // large blocks make long runs; chunks that would leave the chip idle take
    // small ones
    B.wg = plan.n_regions > kHalfRegions ? 1024u : 512u;
    B.ept = 32;
    if (len * B.kh < 512ull * 32 * 512) {
        B.wg = 512;
        B.ept = 8;
    }
    while ((1u << B.pos_log) < B.ept * B.wg / B.kh)
        B.pos_log++;
    // a multiple of 4 (blocks start at 16-byte boundaries), and no power of
    // two: the same region's runs of consecutive blocks fall on different
    // memory channels
    B.cap = (k_h << B.pos_log) + kBlockPad;
    B.n_blocks = (uint32_t)((len + (1ull << B.pos_log) - 1) >> B.pos_log);
    B.row = (plan.n_regions + 2u) & ~1u;
    B.turned = B.cap / plan.n_regions <= kShortRun ? (B.n_blocks + 1u) & ~1u : 0u;
    return true;
}

hipError_t launch_blocks_chunk(const FilterArgs &F, const ReadsArgs &R, uint64_t c0, uint64_t c1,
                               const BinPlan &plan, const BlockPlan &B, const Workspace &W,
                               bool classify, uint32_t tau, const Carry &carry, bool records,
                               hipStream_t s, Profiler *P) {
    // the table: in the count matrix's room, or in the slot ids' where that is
    // larger (their rooms are sized for more than this path needs)
    const uint64_t n_table = (uint64_t)B.n_blocks * B.row;
    uint16_t *table = (uint16_t *)W.matrix;
    if (n_table > 2 * W.matrix_cap) {
        table = (uint16_t *)W.slots;
        if (n_table > 2 * W.slots_cap)
            return hipErrorInvalidValue;
    }
    // the list: about 4 of the 8 bytes per entry of W.entries; the turned
    // table: in the second count matrix's room, or behind the list
    const uint64_t last = c1 - c0 - ((uint64_t)(B.n_blocks - 1) << B.pos_log);
    const uint64_t n_list = ((uint64_t)(B.n_blocks - 1) * B.cap + last * F.k_h + 3) / 4 * 4;
    if (n_list > (W.entries_cap + 1) / 2 * 4 || n_list >= (1ull << 32))
        return hipErrorInvalidValue;
    uint32_t *list = (uint32_t *)W.entries;
    const uint64_t n_turned = (uint64_t)B.turned * B.row;
    uint16_t *turned = (uint16_t *)W.matrix_t;
    if (n_turned > 2 * W.matrix_cap) {
        turned = (uint16_t *)(list + n_list);
        if (4 * n_list + 2 * n_turned > 8 * W.entries_cap)
            return hipErrorInvalidValue;
    }
    const size_t lds = (size_t)plan.n_regions * sizeof(uint32_t);
    if (P)
        P->begin(kPhBinCount, s);
    hipLaunchKernelGGL(sort_kernel(F, R.k, B), dim3(B.n_blocks), dim3(B.wg), lds, s, F, R, c0,
                       c1, B, plan.region_shift, plan.n_regions, list, table,
                       (unsigned long long *)(W.totals + 5));
    if (P)
        P->end(s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    if (B.turned) {
        if (P)
            P->begin(kPhBinRegion, s);
        hipLaunchKernelGGL(k_turn_table, dim3((B.row + 63) / 64, (B.n_blocks + 63) / 64), dim3(256),
                           0, s, (const uint16_t *)table, turned, B.n_blocks, B.row, B.turned);
        if (P)
            P->end(s);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    }
    RecordSpace rec{};
    if (records || carry.mode == Carry::kOut) {
        rec.cursor = W.n_entries + 3;
        if ((e = fill_u32(rec.cursor, 1, 0u, s)) != hipSuccess)
            return e;
        if (records) {
            if (2ull * plan.n_regions > W.coarse_cap)
                return hipErrorInvalidValue;
            rec.word = (uint32_t *)W.bucketed;
            rec.half = (uint16_t *)(rec.word + W.entries_cap);
            rec.off = W.coarse;
            rec.n = W.coarse + plan.n_regions;
        }
    }
    if (P)
        P->begin(kPhRegion, s);
    hipLaunchKernelGGL(plan.region_counters == (uint32_t)kSmallRegionCounters
                           ? runs_kernel<kSmallRegionCounters>(plan, B)
                           : runs_kernel<kRegionCounters>(plan, B),
                       dim3(region_grid(plan.n_regions, plan.region_counters)), dim3(kRegionWG), 0,
                       s, F, c0, plan, B, (const uint32_t *)list,
                       (const uint16_t *)(B.turned ? turned : table), W.flags8,
                       classify ? 1 : 0, tau, rec, carry);
    if (P)
        P->end(s);
    e = hipGetLastError();
    if (e == hipSuccess && records)
        e = launch_record_winners(plan.n_regions, rec.off, rec.n, rec.word, rec.half, c0, c1 - c0,
                                  W, s, P);
    return e;
}

}  // namespace kc
