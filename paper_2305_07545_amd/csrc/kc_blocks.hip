// Binned insertion over block-sorted entry lists.
//
// The hashing workgroup of a block (at most 32768 entries) sorts them by
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
// position within the block (15 bits); the block gives the rest of the
// position.  The two-level form, for many regions, adds the region within its
// bucket, in 40 bits in all.
#include <hip/hip_runtime.h>

#include <utility>

#include "kc_bin_hash.hpp"
#include "kc_blocks.hpp"
#include "kc_device.hpp"
#include "kc_kernels.hpp"
#include "kc_region.hpp"

namespace kc {

namespace {

static_assert(kBlockLog + kLocalBits <= 32, "an entry holds the counter and the position");
constexpr int kSubShift = kBlockLog + kLocalBits;  // two-level form: the region within the bucket
static_assert(kSubShift + kMaxSubLog <= 40, "a 5-byte entry holds it");
static_assert(kLocalBits + kSuperLog <= 40, "a 5-byte entry holds the counter and a position");

// fn(0) .. fn(n - 1), each with its number as a constant: the hashing steps
// keep their results in registers, so they have to be unrolled whatever the
// size of one.
template <int... kJ, typename Fn>
__device__ __forceinline__ void unrolled(std::integer_sequence<int, kJ...>, Fn fn) {
    (fn(std::integral_constant<int, kJ>{}), ...);
}

}  // namespace

// Hash every valid window of the block once and write the block's entries
// sorted by bin: by region, or, in the two-level form (kTwo), by bucket of
// 2^sub_log regions, the region within the bucket being the 11 high bits of a
// 5-byte entry (the fifth bytes in an array of their own).  kEpt: entries per
// thread (kKh hash functions x positions).  kFast: the fast layout
// (fast_layout); kWide: two-word keys.
//
// The block's valid windows are first listed in LDS (in the space the sorted
// entries take later), so that every lane hashes one at each step.  A
// thread's entries stay in registers between hashing, where the histogram's
// atomic also gives each entry's rank in its region, and staging.  Bound by
// its vector instructions (77 to 82% busy; 153 per 64 windows, 155 in the
// two-level form, 117 of them the hash): 0.585 ms for 116 M windows over 3914
// regions, where hashing alone and writing slot ids took 0.43 and the sorting
// passes after it 0.88.
template <int kWG, int kEpt, int kKh, bool kFast, bool kWide, bool kTwo>
__global__ void __launch_bounds__(kWG, 4)
k_hash_sort(FilterArgs F, ReadsArgs R, uint64_t n_words, uint64_t c0, uint64_t c1, BlockPlan B,
            uint32_t shift,
            uint32_t *__restrict__ list, uint8_t *__restrict__ list_hi,
            uint16_t *__restrict__ table, unsigned long long *__restrict__ n_valid) {
    constexpr int kSteps = kEpt / kKh;
    constexpr uint32_t kPos = kSteps * kWG;    // positions per block
    constexpr uint32_t kEntries = kEpt * kWG;  // room for its entries
    static_assert(kEntries <= kBlockEntries, "entries are staged in LDS");
    extern __shared__ uint32_t s_hist[];  // counts, then starts, per bin
    __shared__ __align__(16) uint32_t s_stage[kEntries];
    __shared__ uint32_t s_wave[kWG / 64];
    uint16_t *s_list = reinterpret_cast<uint16_t *>(s_stage);
    const uint32_t lane = threadIdx.x & 63u, wave = wave_id(), n_bins = B.n_bins;
    constexpr uint32_t kWaves = kWG / 64;
    for (uint32_t i = threadIdx.x; i < n_bins; i += kWG)
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
        // validity of the words' windows, from the masks here (25 us over 150 M
        // positions): a bitmap of its own took a launch and 28 us there, 5 us
        // in calls of 1 M bases
        if (lane < kWords && p0 + 32u * (w0 + lane) < c1)
            v = valid_word(R.inv, R.rs, n_words, (p0 >> 5) + w0 + lane, R.k, R.n_bases);
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
    uint32_t key[kEpt];  // bin | rank << 16
    uint32_t high[kTwo ? (kEpt + 3) / 4 : 1];  // the entries' fifth bytes
    // A step's code words are requested a step before they are hashed, and a
    // rank is taken in a step after its atomic, so that neither is waited for.
    auto position = [&](int j) -> uint32_t {
        const uint32_t i = (uint32_t)j * kWG + threadIdx.x;
        return i < nv ? s_list[i] : 0u;
    };
    uint32_t q = position(0), q_next = kSteps > 1 ? position(1) : 0u;
    WindowWords<kWide> w(codes, q);
    uint32_t rank[kKh];
    unrolled(std::make_integer_sequence<int, kSteps>{}, [&](auto step) {
        constexpr int j = decltype(step)::value;
        const uint32_t i = (uint32_t)j * kWG + threadIdx.x;
        const WindowWords<kWide> wn(codes, q_next);
        const uint32_t q_after = j + 2 < kSteps ? position(j + 2) : 0u;
        uint32_t old[kKh];
        if (i < nv)
            window_entries<kFast, kWide, kKh>(
                F, w, q, K, shift, [&](int a, uint32_t r, uint32_t local) {
                    constexpr int kFifth = 8;
                    const int u = j * kKh + a;
                    ent[u] = local | (q << kLocalBits);
                    uint32_t bin = r;
                    if (kTwo) {
                        const uint32_t rl = r & ((1u << B.sub_log) - 1u);
                        bin = r >> B.sub_log;
                        ent[u] |= rl << kSubShift;
                        const uint32_t hi = rl >> (32 - kSubShift);
                        high[u / 4] = u % 4 ? high[u / 4] | (hi << (kFifth * (u % 4))) : hi;
                    }
                    key[u] = bin;
                    old[a] = atomicAdd(&s_hist[bin], 1u);
                });
        if constexpr (j > 0) {
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
    });
#pragma unroll
    for (int a = 0; a < kKh; a++)
        key[(kSteps - 1) * kKh + a] |= rank[a] << 16;
    __syncthreads();
    {  // counts -> starts, in place: each wavefront scans a share of the
       // regions, 64 at a time, then adds the shares before its own
        const uint32_t share = (n_bins + kWG - 1) / kWG * 64u;
        const uint32_t r0 = wave * share;
        uint32_t run = 0;
        for (uint32_t u = 0; u < share; u += 64) {
            const uint32_t r = r0 + u + lane;
            const uint32_t c = r < n_bins ? s_hist[r] : 0u;
            const uint32_t incl = wave_inclusive(c);
            if (r < n_bins)
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
            if (r < n_bins)
                s_hist[r] += before;
        }
    }
    __syncthreads();
    const uint32_t total = nv * k_h;
    uint16_t *__restrict__ trow = table + (uint64_t)blockIdx.x * B.row;
    for (uint32_t i = threadIdx.x; i <= n_bins; i += kWG)
        trow[i] = (uint16_t)(i < n_bins ? s_hist[i] : total);
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
    if (kTwo) {  // the fifth bytes, sorted the same way in the same room
        __syncthreads();
        uint8_t *s_byte = reinterpret_cast<uint8_t *>(s_stage);
#pragma unroll
        for (int j = 0; j < kSteps; j++)
            if ((uint32_t)j * kWG + threadIdx.x < nv) {
#pragma unroll
                for (int a = 0; a < kKh; a++)
                    if (kKh == 1 || (uint32_t)a < k_h) {
                        const int u = j * kKh + a;
                        s_byte[s_hist[key[u] & 0xFFFFu] + (key[u] >> 16)] =
                            (uint8_t)(high[u / 4] >> (8 * (u % 4)));
                    }
            }
        __syncthreads();
        uint4 *__restrict__ outb = reinterpret_cast<uint4 *>(list_hi + (uint64_t)blockIdx.x * B.cap);
        for (uint32_t i = threadIdx.x; i < (total + 15u) / 16u; i += kWG)
            outb[i] = src[i];
    }
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

// Up to 64 runs of entries, one a lane, whose aligned groups of four entries lie
// end to end over a wavefront's lanes.
struct LaneRuns {
    uint32_t s, e;   // the lane's run
    uint32_t incl;   // groups up to and with it
    uint32_t n;      // groups of all runs (uniform)

    __device__ __forceinline__ void set(uint32_t start, uint32_t end) {
        s = start;
        e = end;
        incl = wave_inclusive(e > s ? (e - 1u) / 4u + 1u - s / 4u : 0u);
        n = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    }
    // Group f0 + lane (f0 < n, uniform): its run i (< 64), first entry g, and
    // which of its entries are the run's (none past the last group).
    __device__ __forceinline__ uint32_t at(uint32_t f0, uint32_t lane, uint32_t &i,
                                           uint32_t &g) const {
        const uint32_t f = f0 + lane, limit = f0 + 64u < n ? f0 + 64u : n;
        // as many runs as end at or before the group
        uint32_t j = (uint32_t)__popcll(__ballot(incl <= f0));
        i = j;
        for (; j < 63u; j++) {
            const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)incl, (int)j);
            if (end >= limit)
                break;
            i += f >= end ? 1u : 0u;
        }
        i = i < 63u ? i : 63u;
        const uint32_t rs = (uint32_t)__shfl((int)s, (int)i), re = (uint32_t)__shfl((int)e, (int)i);
        // groups count back from the run's last
        g = ((re - 1u) / 4u + 1u - ((uint32_t)__shfl((int)incl, (int)i) - f)) * 4u;
        const uint32_t lo = g < rs ? rs - g : 0u, hi = re - g < 4u ? re - g : 4u;
        return f < n ? (1u << hi) - (1u << lo) : 0u;
    }
};

// The share `part` (of 2^split) of run [s, e): at least kPart entries, so that a
// short run stays whole.  With eight superblocks or fewer, most of the region
// pass's 16 wavefronts would have no run, and one a region's whole list: a
// k-mer repeated over 94% of 3 M bases, 17.2 -> 2.4 ms (with the lanes of one
// counter counted together, here and in the second level).
constexpr uint32_t kPart = 128;
__device__ __forceinline__ void share_run(uint32_t s, uint32_t e, uint32_t part, uint32_t split,
                                          LaneRuns &R) {
    const uint32_t len = e - s, piece = (len + (1u << split) - 1u) >> split;
    const uint32_t each = piece > kPart ? piece : kPart;
    const uint32_t lo = part * each, hi = lo + each;
    R.set(s + (lo < len ? lo : len), s + (hi < len ? hi : len));
}

// Second level: the entries of bucket b in superblock sb (`super` blocks) ->
// sorted by region, entries of 5 bytes again (the counter and the position
// within the superblock).  Their place in the list needs no scan: the
// superblock's room is its blocks' room, and the buckets before b hold as many
// of its entries as b's runs start at, summed over the blocks.  starts[sb]
// receives the place of every region's run.
//
// Bound: memory latency behind the runs' short pieces (about 65 entries), so
// every entry is requested at once (a wavefront takes every 16th block's run,
// LaneRuns) and stays in registers with the rank that its region's count gives
// it, two workgroups of 16 wavefronts per CU (1.7 G entries over 122 K regions in
// 478 buckets: 4.3 ms, 4.0 TB/s; runs read twice by teams of 16 lanes, eight
// wavefronts each, and stored entry by entry: 7.5 ms).  The sorted entries lie in LDS as
// the list's 16-byte groups do, and leave in those.  Buckets of more entries
// than fit (favoured by the input) are read again and placed straight in the
// list.  Workgroups of one XCD take neighbouring buckets of a superblock at a
// time, whose runs and table rows share cache lines.
__global__ void __launch_bounds__(kMergeWG, 8)
k_merge(BlockPlan B, uint32_t n_regions, const uint32_t *__restrict__ list,
        const uint8_t *__restrict__ list_hi, const uint16_t *__restrict__ table,
        uint32_t *__restrict__ out, uint8_t *__restrict__ out_hi, uint32_t *__restrict__ starts) {
    // each with room for lanes without an entry behind it
    constexpr uint32_t kNoPlace = kMergeTile + 4, kNoSub = 1u << kMaxSubLog;
    __shared__ __align__(16) uint32_t s_word[kNoPlace + 64];
    __shared__ __align__(16) uint8_t s_high[kNoPlace + 64];
    __shared__ uint32_t s_cursor[kNoSub + 64];
    __shared__ uint32_t s_wave[kMergeWG / 64];
    __shared__ uint32_t s_sum, s_over;
    constexpr uint32_t kWaves = kMergeWG / 64;
    constexpr int kGroups = 4;
    constexpr uint32_t kStep = 64u * kGroups;
    const uint32_t lane = threadIdx.x & 63u, wave = wave_id();
    const uint32_t per = (B.n_bins + 7u) / 8u;  // buckets per XCD
    const uint32_t b = (blockIdx.x & 7u) * per + (blockIdx.x >> 3) % per;
    const uint32_t sb = (blockIdx.x >> 3) / per;
    if (b >= B.n_bins)
        return;
    const uint32_t n_sub = 1u << B.sub_log;
    const uint32_t k0 = sb * B.super;
    const uint32_t n_k = B.n_blocks - k0 < B.super ? B.n_blocks - k0 : B.super;
    // the lane's run (a superblock has at most 64 runs a wavefront)
    uint32_t bs = 0, be = 0;
    const uint32_t kl = lane * kWaves + wave;
    if (kl < n_k) {
        const uint16_t *t = table + (uint64_t)(k0 + kl) * B.row + b;
        bs = t[0];
        be = t[1];
    }
    for (uint32_t i = threadIdx.x; i < n_sub; i += kMergeWG)
        s_cursor[i] = 0;
    if (threadIdx.x == 0) {
        s_sum = 0;
        s_over = 0;
    }
    LaneRuns R;
    R.set(bs, be);
    uint4 x[kGroups];
    uint32_t h[kGroups], which[kGroups];  // entries; block, and (from bit 28) those in the run
    auto load = [&](uint32_t w0) {
#pragma unroll
        for (int c = 0; c < kGroups; c++) {
            which[c] = 0;
            if (w0 + 64u * c < R.n) {
                uint32_t i, g;
                const uint32_t m = R.at(w0 + 64u * c, lane, i, g);
                const uint32_t k = i * kWaves + wave;
                if (m) {
                    const uint32_t at = (k0 + k) * B.cap + g;
                    x[c] = *reinterpret_cast<const uint4 *>(list + at);
                    h[c] = *reinterpret_cast<const uint32_t *>(list_hi + at);
                    which[c] = k | (m << 28);
                }
            }
        }
    };
    // visit(entry's number in the step, word, fifth byte, block - k0, is it
    // the run's); lanes past their run's end visit too, so that a chunk's LDS
    // operations are in flight together
    auto each = [&](uint32_t w0, auto visit) {
#pragma unroll
        for (int c = 0; c < kGroups; c++)
            if (w0 + 64u * c < R.n) {
                const uint32_t m = which[c], k = m & 0xFFFFu;
                visit(4 * c, x[c].x, h[c] & 0xFFu, k, ((m >> 28) & 1u) != 0);
                visit(4 * c + 1, x[c].y, (h[c] >> 8) & 0xFFu, k, ((m >> 29) & 1u) != 0);
                visit(4 * c + 2, x[c].z, (h[c] >> 16) & 0xFFu, k, ((m >> 30) & 1u) != 0);
                visit(4 * c + 3, x[c].w, h[c] >> 24, k, (m >> 31) != 0);
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    auto sub_of = [](uint32_t w, uint32_t h) -> uint32_t {
        return (w >> kSubShift) | (h << (32 - kSubShift));
    };
    // a place of region `sub` for each lane here: the lanes of the first one's
    // region, often all of them in a bucket that holds this many, take theirs
    // together
    auto take = [&](uint32_t sub) -> uint32_t {
        const uint32_t s0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)sub);
        const uint64_t same = __ballot(sub == s0);
        const uint32_t i = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
        uint32_t at = 0;
        if (sub != s0 || i == 0)
            at = atomicAdd(&s_cursor[sub], sub == s0 ? (uint32_t)__popcll(same) : 1u);
        const uint32_t at0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
        return sub == s0 ? at0 + i : at;
    };
    __syncthreads();
    uint32_t rank[kGroups * 2];  // of two entries a word: read for buckets of at most kMergeTile
#pragma unroll
    for (int j = 0; j < kGroups * 2; j++)
        rank[j] = 0;
    for (uint32_t w0 = kStep; w0 < R.n; w0 += kStep) {  // what is not held
        load(w0);
        each(w0, [&](int, uint32_t w, uint32_t h, uint32_t, bool in) {
            if (in)
                take(sub_of(w, h));
        });
    }
    load(0);
    each(0, [&](int j, uint32_t w, uint32_t h, uint32_t, bool in) {
        const uint32_t x = atomicAdd(&s_cursor[in ? sub_of(w, h) : kNoSub + lane], 1u);
        rank[j / 2] = j % 2 ? rank[j / 2] | (x << 16) : x & 0xFFFFu;
    });
    const uint32_t sum = wave_inclusive(bs);
    if (lane == 63) {
        atomicAdd(&s_sum, sum);
        if (R.n > kStep)
            s_over = 1;
    }
    __syncthreads();
    const uint32_t base = k0 * B.cap + s_sum;  // list places are below 2^32
    // counts -> starts: each wavefront a share of the regions
    const uint32_t share = (n_sub + kMergeWG - 1) / kMergeWG * 64u;
    uint32_t run = 0;
    for (uint32_t u = 0; u < share; u += 64) {
        const uint32_t i = wave * share + u + lane;
        const uint32_t c = i < n_sub ? s_cursor[i] : 0u;
        const uint32_t incl = wave_inclusive(c);
        if (i < n_sub)
            s_cursor[i] = run + incl - c;
        run += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    }
    if (lane == 0)
        s_wave[wave] = run;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (uint32_t w = 0; w < kWaves; w++) {
        before += w < wave ? s_wave[w] : 0u;
        total += s_wave[w];
    }
    uint32_t *__restrict__ row = starts + (uint64_t)sb * (n_regions + 1u);
    const uint32_t r0 = b << B.sub_log;
    for (uint32_t u = 0; u < share; u += 64) {
        const uint32_t i = wave * share + u + lane;
        if (i < n_sub) {
            const uint32_t c = s_cursor[i] + before;
            s_cursor[i] = c;
            if (r0 + i < n_regions)
                row[r0 + i] = base + c;
        }
    }
    if (threadIdx.x == 0 && b + 1u == B.n_bins)
        row[n_regions] = base + total;
    const bool held = total <= kMergeTile && !s_over;  // uniform
    __syncthreads();
    // an entry of the superblock: its word and fifth byte
    auto merged = [&](uint32_t w, uint32_t k, uint8_t &high) -> uint32_t {
        const uint32_t t = (k << B.pos_log) | ((w >> kLocalBits) & ((1u << kBlockLog) - 1u));
        high = (uint8_t)(t >> (32 - kLocalBits));
        return (w & ((1u << kLocalBits) - 1u)) | (t << kLocalBits);
    };
    if (__builtin_expect(!held, 0)) {  // (else the registers of both paths spill)
        uint32_t *__restrict__ o = out + base;
        uint8_t *__restrict__ oh = out_hi + base;
        for (uint32_t w0 = 0; w0 < R.n; w0 += kStep) {
            load(w0);
            each(w0, [&](int, uint32_t w, uint32_t h, uint32_t k, bool in) {
                if (in) {
                    const uint32_t at = take(sub_of(w, h));
                    o[at] = merged(w, k, oh[at]);
                }
            });
        }
        return;
    }
    const uint32_t skew = base & 3u;  // the first entry's place in its 16-byte group
    // the entries as new values: else their regions' numbers stay in registers
    // beside them across the scan
#pragma unroll
    for (int c = 0; c < kGroups; c++)
        asm volatile(""
                     : "+v"(x[c].x), "+v"(x[c].y), "+v"(x[c].z), "+v"(x[c].w), "+v"(h[c]),
                       "+v"(which[c]));
    each(0, [&](int j, uint32_t w, uint32_t h, uint32_t k, bool in) {
        const uint32_t r = (rank[j / 2] >> (16 * (j % 2))) & 0xFFFFu;
        const uint32_t at =
            in ? s_cursor[sub_of(w, h) & (kNoSub - 1u)] + r + skew : kNoPlace + lane;
        s_word[at] = merged(w, k, s_high[at]);
    });
    __syncthreads();
    uint32_t *__restrict__ o = out + (base - skew);
    uint8_t *__restrict__ oh = out_hi + (base - skew);
    const uint32_t end = skew + total;
    for (uint32_t i = 4u * threadIdx.x; i < end; i += 4u * kMergeWG) {
        if (i >= skew && i + 4u <= end) {
            *reinterpret_cast<uint4 *>(o + i) = *reinterpret_cast<const uint4 *>(s_word + i);
            *reinterpret_cast<uint32_t *>(oh + i) = *reinterpret_cast<const uint32_t *>(s_high + i);
        } else {
            for (uint32_t j = i < skew ? skew : i; j < i + 4u && j < end; j++) {
                o[j] = s_word[j];
                oh[j] = s_high[j];
            }
        }
    }
}

// The region pass over the blocks' runs.  kCounters: counters per region.
// kCells: the cells each thread updates, held in registers (the
// plan's region has kCells * kRegionWG cells), or 0 for regions of fewer cells than
// threads.  kTwo: runs of superblocks, 5-byte entries.  kLanes (one-level form):
// lanes that take a run together (by its expected length), or 0 for short
// runs: a wavefront takes the runs of 64 blocks at once (their starts are a
// segment of the turned table's rows) and lays their entries end to end over
// its lanes, so that every lane counts an entry at each step; the lane's run is
// found by counting the run heads at and before it.
//
// Persistent.  The regions that the workgroups of one XCD (every eighth
// workgroup) hold at a time are consecutive, so that the blocks' neighbouring
// runs, which share cache lines, are read through one L2.
//
// kSorted: first-seen occurrences leave as records sorted by bucket of positions
// (LDS counting sort, runs appended by one atomic per region and bucket), which
// k_marks turns into bits.  Byte flags stored at random positions (94 G/s)
// took 0.20 of the 0.51 ms this pass had on 120 M windows over 3914 regions;
// it is 0.375 ms now, and the marks 0.09.  Else the records are in room of the
// region's own (RecordSpace, carried chunks).
//
// Bound: latency, with one 128 KiB workgroup per CU (vector units 49% busy,
// LDS 25%, on 1.7 G entries over 122 K regions: 6.1 ms).  So what the next
// region needs is requested before the current region's counters are updated
// (its cells, its first bounds; kTwo: its entries, 7.2 -> 6.1 ms), and taken in
// before the update's first store.
template <int kCounters, int kCells, int kLanes, bool kTwo, bool kSorted>
__global__ void __launch_bounds__(kRegionWG)
k_region_runs(FilterArgs F, uint64_t c0, BinPlan P, BlockPlan B,
              const uint32_t *__restrict__ list, const uint8_t *__restrict__ list_hi,
              const void *__restrict__ table, int classify, uint32_t tau, RecordSpace rec, Carry C) {
    constexpr uint32_t kSparseCells = kCounters / 8;
    constexpr bool kTile = (uint32_t)kCells * kRegionWG <= kSparseCells;
    constexpr int kHold = kCells ? kCells : 1;
    constexpr int kWin = kCounters / kRegionWG;  // counters whose outcome a thread takes
    constexpr int kEta = kWin / kHold;           // counters per held cell, at most
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
    // records sorted by bucket: counts, then starts; list place less start; wavefronts' sums
    __shared__ uint32_t s_bucket[kMarkBuckets], s_place[kMarkBuckets], s_sum[kWaves];
    __shared__ uint32_t s_head[kLanes ? 1 : kWaves][2 * kChunks];
    const uint32_t shift = P.region_shift, S = 1u << shift;
    const uint64_t n_words = F.X * F.Y;
    const bool carry_out = !kSorted && C.mode == Carry::kOut;
    const bool carry_in = kTile && C.mode == Carry::kIn && C.n_prev > 0;
    constexpr bool by_region = !kSorted;  // records in room of the region's own
    for (uint32_t i = threadIdx.x; i < (uint32_t)kCounters; i += kRegionWG) {
        hits[i] = 0;
        first[i] = kIdle;
    }
    for (uint32_t i = threadIdx.x; i < kMarkBuckets; i += kRegionWG)
        s_bucket[i] = 0;
    if (threadIdx.x == 0) {
        s_nwin = 0;
        s_total = 0;
    }
    const uint32_t grid = gridDim.x;
    const uint32_t lane = threadIdx.x & 63u, wave = wave_id();
    // entry of word e and (kTwo) fifth byte h, its position counted from tb
    auto count = [&](uint32_t e, uint32_t h, uint32_t tb) {
        const uint32_t local = e & ((1u << kLocalBits) - 1u);
        const uint32_t t = tb + ((e >> kLocalBits) | (h << (32 - kLocalBits)));
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
    uint32_t r = (grid & 7u) == 0 ? (blockIdx.x & 7u) * (grid >> 3) + (blockIdx.x >> 3) : blockIdx.x;
    uint64_t cell[kHold];
    load_cells(r, cell);
    // The end of region r, whose entries are counted (mine: those of the runs
    // whose length this lane has); the next region's cells are in `cell` then.
    // prefetch: the caller's loads for the next region.  A wavefront's loads
    // and stores complete in order, so that a load waited for after a store
    // waits for that store: every load in flight (settle: the caller's) is
    // taken in before the first store.
    auto finish = [&](uint32_t r, uint32_t mine, auto prefetch, auto settle) {
        const uint64_t wbase = (uint64_t)r << shift;
        const uint32_t nw = wbase + S <= n_words ? S : (uint32_t)(n_words - wbase);
        if (by_region && mine)
            atomicAdd(&s_total, mine);
        __syncthreads();
        uint64_t celln[kHold];
        load_cells(r + grid, celln);
        prefetch();
        // room for a record of every entry of the region, asked for before the
        // counters' update and taken after it
        uint32_t got = 0;
        if (by_region && threadIdx.x == 0 && s_total)
            got = atomicAdd(rec.cursor, s_total);
        // The counters' update, and the thread's first-seen occurrences: bit j
        // of won, its position wt[j], bit j of sure when it is trustworthy.
        // Counters are left clean (hits 0, first kIdle).
        uint32_t wt[kWin], won = 0, sure = 0;
        uint32_t changed = 0;  // cells to be written
        // the thread's number as a value of this region: else the compiler
        // keeps every counter's address in a register across all regions
        uint32_t tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const uint32_t fm = (uint32_t)F.field_max;  // counters are at most 32 bits wide
        if constexpr (kCells != 0) {
#pragma unroll
            for (int k = 0; k < kHold; k++) {
                const uint32_t w = tid + (uint32_t)k * kRegionWG;
                const uint64_t pre = cell[k];
                uint64_t next = pre;
#pragma unroll
                for (int l = 0; l < kEta; l++)
                    if ((uint32_t)l < F.eta) {
                        const int j = k * kEta + l;
                        const uint32_t idx = ((uint32_t)l << shift) | w;
                        const uint32_t h = hits[idx];
                        wt[j] = first[idx];
                        hits[idx] = 0;
                        first[idx] = kIdle;
                        const uint32_t sh = F.alpha * l;
                        const uint32_t pf = (uint32_t)(pre >> sh) & fm;
                        const uint32_t room = fm - pf;
                        const uint32_t inc = h < room ? h : room;
                        next += (uint64_t)inc << sh;  // the field grows without carrying out
                        won |= (h != 0 && pf == 0) ? 1u << j : 0u;
                        sure |= inc > tau ? 1u << j : 0u;
                        if (j % 4 == 3)  // four counters' reads in flight: the registers' limit
                            __builtin_amdgcn_sched_barrier(0);
                    }
                changed |= next != pre ? 1u << k : 0u;
                cell[k] = next;
                if (kTile && C.mode == Carry::kIn)
                    s_cell[w] = next;
            }
        } else {
            // fewer cells than threads: a cell's owner leaves each counter's
            // outcome in place, and every thread then takes its share
            for (uint32_t w = tid; w < nw; w += kRegionWG) {
                const uint64_t pre = F.words[wbase + w];
                uint64_t next = pre;
                for (uint32_t l = 0; l < F.eta; l++) {
                    const uint32_t idx = (l << shift) | w;
                    const uint32_t h = hits[idx];
                    if (h == 0)
                        continue;
                    const uint32_t sh = F.alpha * l;
                    const uint32_t pf = (uint32_t)(pre >> sh) & fm;
                    const uint32_t room = fm - pf;
                    const uint32_t inc = h < room ? h : room;
                    next += (uint64_t)inc << sh;
                    hits[idx] = pf ? 0u : (inc > tau ? 3u : 1u);
                }
                if (next != pre)
                    F.words[wbase + w] = next;
                if (kTile && C.mode == Carry::kIn)
                    s_cell[w] = next;
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < kWin; j++) {
                const uint32_t idx = tid + (uint32_t)j * kRegionWG;
                const uint32_t h = hits[idx];
                wt[j] = first[idx];
                hits[idx] = 0;
                first[idx] = kIdle;
                won |= h ? 1u << j : 0u;
                sure |= h == 3u ? 1u << j : 0u;
            }
        }
        if (!classify)
            sure = 0;
        auto store_cells = [&]() {
#pragma unroll
            for (int k = 0; k < kHold; k++)
                asm volatile("" : "+v"(celln[k]));
            settle();
#pragma unroll
            for (int k = 0; k < kHold; k++) {
                if ((changed >> k) & 1u)
                    F.words[wbase + tid + (uint32_t)k * kRegionWG] = cell[k];
                cell[k] = celln[k];
            }
        };
        if constexpr (!by_region) {
            // sorted by bucket of positions in the hits' room, then appended to
            // the buckets in runs
            uint32_t rank[(kWin + 1) / 2];
#pragma unroll
            for (int j = 0; j < kWin; j++) {
                uint32_t x = 0;
                if ((won >> j) & 1u)
                    x = atomicAdd(&s_bucket[wt[j] >> rec.log], 1u);
                rank[j / 2] = j % 2 ? rank[j / 2] | (x << 16) : x;
            }
            __syncthreads();
            uint32_t incl = 0, c = 0;
            if (tid < kMarkBuckets) {
                c = s_bucket[tid];
                incl = wave_inclusive(c);
                if (lane == 63)
                    s_sum[wave] = incl;
            }
            __syncthreads();
            uint32_t total = 0;
#pragma unroll
            for (uint32_t w = 0; w < kMarkBuckets / 64; w++) {
                incl += w < wave ? s_sum[w] : 0u;
                total += s_sum[w];
            }
            uint32_t place = 0;
            if (tid < kMarkBuckets) {
                s_bucket[tid] = incl - c;
                if (c)
                    place = atomicAdd(&rec.cursor[tid], c);
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < kWin; j++)
                if ((won >> j) & 1u)
                    hits[s_bucket[wt[j] >> rec.log] + ((rank[j / 2] >> (16 * (j % 2))) & 0xFFFFu)] =
                        wt[j] | (((sure >> j) & 1u ? 3u : 1u) << 30);
            if (tid < kMarkBuckets)
                s_place[tid] =
                    tid * (uint32_t)rec.room + place - s_bucket[tid];
            __syncthreads();
            store_cells();
            for (uint32_t i = tid; i < total; i += kRegionWG) {
                const uint32_t x = hits[i], t = x & 0x3FFFFFFFu;
                hits[i] = 0;
                rec.sorted[s_place[t >> rec.log] + i] =
                    (t & ((1u << rec.log) - 1u)) | (x >> 30 << rec.log);
            }
            for (uint32_t i = tid; i < kMarkBuckets; i += kRegionWG)
                s_bucket[i] = 0;
        } else {
            // a wavefront's records together, from one step of the LDS counter
            const uint32_t mine_n = (uint32_t)__popc(won);
            const uint32_t incl = wave_inclusive(mine_n);
            uint32_t at = 0;
            if (lane == 63 && incl)
                at = atomicAdd(&s_nwin, incl);
            at = (uint32_t)__builtin_amdgcn_readlane((int)at, 63) + incl - mine_n;
            if (tid == 0)
                s_base = got;
            __syncthreads();
            store_cells();
            uint32_t *word = (carry_out ? C.word + (uint64_t)C.chunk * C.cap : rec.word) + s_base;
            uint16_t *half = (carry_out ? C.half + (uint64_t)C.chunk * C.cap : rec.half) + s_base;
#pragma unroll
            for (int j = 0; j < kWin; j++)
                if ((won >> j) & 1u) {
                    const uint32_t idx = kCells ? ((uint32_t)(j % kEta) << shift) |
                                                      (tid + (uint32_t)(j / kEta) * kRegionWG)
                                                : tid + (uint32_t)j * kRegionWG;
                    word[at] = wt[j];
                    half[at] = (uint16_t)(carry_out ? idx : ((sure >> j) & 1u ? 3u : 1u));
                    at++;
                }
        }
        __syncthreads();  // the counters are clean, the region's records counted
        if (carry_in)
            mark_carried(F, shift, C, r, s_cell, tau);
        if (by_region && tid == 0) {
            if (carry_out) {
                C.off[(uint64_t)C.chunk * C.stride + r] = s_base;
                C.n[(uint64_t)C.chunk * C.stride + r] = s_nwin;
            } else {
                rec.off[r] = s_base;
                rec.n[r] = s_nwin;
            }
            s_nwin = 0;
            s_total = 0;
        }
        if (by_region || carry_in)
            __syncthreads();  // the sums and s_cell are rewritten by the next region
    };
    __syncthreads();  // counters clean, sums zero
    if constexpr (kLanes == 0) {
        const uint16_t *__restrict__ turned = (const uint16_t *)table;
        auto bounds = [&](uint32_t r, uint32_t b, uint32_t &s, uint32_t &e) {
            s = e = 0;
            if (lane < B.share && b < B.n_blocks && r < P.n_regions) {
                s = turned[(uint64_t)r * B.turned + b];
                e = turned[(uint64_t)(r + 1u) * B.turned + b];
            }
        };
        // a wavefront takes `share` consecutive blocks of a set of 16 * share
        const uint32_t set = B.share * (uint32_t)kWaves, at0 = wave * B.share + lane;
        uint32_t ns, ne;
        bounds(r, at0, ns, ne);
        for (; r < P.n_regions; r += grid) {
            uint32_t mine = 0;
            for (uint32_t b0 = 0; b0 + wave * B.share < B.n_blocks; b0 += set) {
                const uint32_t b = b0 + at0;
                const uint32_t s = ns, len = ne - ns;
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
                bounds(r, b + set, ns, ne);
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
                            count(x[c], 0u, tb[c]);
                    __builtin_amdgcn_wave_barrier();
                }
            }
            finish(
                r, mine, [&]() { bounds(r + grid, at0, ns, ne); },
                [&]() { asm volatile("" : "+v"(ns), "+v"(ne)); });
        }
    } else if constexpr (kTwo) {
        // A wavefront takes every kWaves-th superblock's run, and lays their
        // 16-byte groups of entries end to end over its lanes.  The groups of
        // the next region (of as many as a step takes: nearly always all) are
        // requested before the current region's counters are updated, and the
        // bounds of the one after behind them.
        constexpr int kGroups = kSorted ? 4 : 5;  // beside the records, what the registers hold
        constexpr uint32_t kSet = kWaves * 64;
        const uint32_t *__restrict__ starts = (const uint32_t *)table;
        uint32_t bs, be;  // the lane's run: its entries in the list
        // run x of a set of kSet: superblock x >> split, that share of it
        const uint32_t part = wave & ((1u << B.split) - 1u);
        auto bounds = [&](uint32_t r, uint32_t b0) {
            const uint32_t b = (b0 + lane * kWaves + wave) >> B.split;
            const bool in = b < B.n_super && r < P.n_regions;
            const uint32_t *t = starts + (in ? (uint64_t)b * (P.n_regions + 1u) + r : 0ull);
            bs = t[0];
            be = in ? t[1] : bs;
        };
        LaneRuns R;
        uint4 x[kGroups];
        uint32_t h[kGroups], which[kGroups];  // entries; run, and (from bit 28) those in the run
        auto load = [&](uint32_t w0) {
#pragma unroll
            for (int c = 0; c < kGroups; c++) {
                which[c] = 0;
                if (w0 + 64u * c < R.n) {
                    uint32_t i, g;
                    const uint32_t m = R.at(w0 + 64u * c, lane, i, g);
                    if (m) {
                        x[c] = *reinterpret_cast<const uint4 *>(list + g);
                        h[c] = *reinterpret_cast<const uint32_t *>(list_hi + g);
                        which[c] = i | (m << 28);
                    }
                }
            }
        };
        auto tally = [&](uint32_t b0) {
#pragma unroll
            for (int c = 0; c < kGroups; c++) {
                const uint32_t m = which[c];
                if (m >> 28) {
                    const uint32_t b = (b0 + (m & 63u) * kWaves + wave) >> B.split;
                    const uint32_t tb = (b * B.super) << B.pos_log;
                    if ((m >> 28) & 1u)
                        count(x[c].x, h[c] & 0xFFu, tb);
                    if ((m >> 29) & 1u)
                        count(x[c].y, (h[c] >> 8) & 0xFFu, tb);
                    if ((m >> 30) & 1u)
                        count(x[c].z, (h[c] >> 16) & 0xFFu, tb);
                    if (m >> 31)
                        count(x[c].w, h[c] >> 24, tb);
                }
            }
        };
        bounds(r, 0);
        share_run(bs, be, part, B.split, R);
        load(0);
        bounds(r + grid, 0);
        for (; r < P.n_regions; r += grid) {
            uint32_t mine = R.e - R.s;
            tally(0);
            for (uint32_t w0 = 64u * kGroups; w0 < R.n; w0 += 64u * kGroups) {
                load(w0);
                tally(0);
            }
            for (uint32_t b0 = kSet; b0 < B.n_super; b0 += kSet) {
                bounds(r, b0);
                share_run(bs, be, part, B.split, R);
                mine += R.e - R.s;
                for (uint32_t w0 = 0; w0 < R.n; w0 += 64u * kGroups) {
                    load(w0);
                    tally(b0);
                }
                if (b0 + kSet >= B.n_super)
                    bounds(r + grid, 0);
            }
            share_run(bs, be, part, B.split, R);
            load(0);
            bounds(r + 2u * grid, 0);
            finish(
                r, mine, [&]() {},
                [&]() {
#pragma unroll
                    for (int c = 0; c < kGroups; c++)
                        asm volatile(""
                                     : "+v"(x[c].x), "+v"(x[c].y), "+v"(x[c].z), "+v"(x[c].w),
                                       "+v"(h[c]));
                    asm volatile("" : "+v"(bs), "+v"(be));
                });
        }
    } else {
        // a team of lanes takes a run, kUnroll runs in flight
        constexpr uint32_t kTeams = kRegionWG / kLanes;
        constexpr int kUnroll = 2;
        const uint32_t team = threadIdx.x / kLanes, sub = threadIdx.x % kLanes;
        uint32_t ns[kUnroll], ne[kUnroll];
        auto bounds = [&](uint32_t r, uint32_t b, uint32_t &s, uint32_t &e) {
            s = e = 0;
            if (b < B.n_blocks && r < P.n_regions) {
                const uint16_t *t = (const uint16_t *)table + (uint64_t)b * B.row + r;
                s = t[0];
                e = t[1];
            }
        };
#pragma unroll
        for (int u = 0; u < kUnroll; u++)
            bounds(r, team + u * kTeams, ns[u], ne[u]);
        for (; r < P.n_regions; r += grid) {
            uint32_t mine = 0;
            for (uint32_t b0 = team; b0 < B.n_blocks; b0 += kUnroll * kTeams) {
                // a first 16-byte group of entries of every run, and the next
                // runs' bounds, are requested before any entry is counted
                uint32_t s[kUnroll], e[kUnroll], g[kUnroll];
                uint4 x[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; u++) {
                    const uint32_t b = b0 + (uint32_t)u * kTeams;
                    s[u] = ns[u];
                    e[u] = ne[u];
                    g[u] = (s[u] & ~3u) + 4u * sub;
                    if (g[u] < e[u])
                        x[u] = *reinterpret_cast<const uint4 *>(list + (uint64_t)b * B.cap + g[u]);
                    mine += sub == 0 ? e[u] - s[u] : 0u;
                    bounds(r, b0 + (uint32_t)(u + kUnroll) * kTeams, ns[u], ne[u]);
                }
#pragma unroll
                for (int u = 0; u < kUnroll; u++) {
                    const uint32_t b = b0 + (uint32_t)u * kTeams, tb = b << B.pos_log;
                    while (g[u] < e[u]) {
                        const uint32_t gn = g[u] + 4u * kLanes;
                        uint4 y = make_uint4(0u, 0u, 0u, 0u);
                        if (gn < e[u])
                            y = *reinterpret_cast<const uint4 *>(list + (uint64_t)b * B.cap + gn);
                        if (g[u] >= s[u])
                            count(x[u].x, 0u, tb);
                        if (g[u] + 1u >= s[u] && g[u] + 1u < e[u])
                            count(x[u].y, 0u, tb);
                        if (g[u] + 2u >= s[u] && g[u] + 2u < e[u])
                            count(x[u].z, 0u, tb);
                        if (g[u] + 3u >= s[u] && g[u] + 3u < e[u])
                            count(x[u].w, 0u, tb);
                        x[u] = y;
                        g[u] = gn;
                    }
                }
            }
            finish(
                r, mine,
                [&]() {
#pragma unroll
                    for (int u = 0; u < kUnroll; u++)
                        bounds(r + grid, team + u * kTeams, ns[u], ne[u]);
                },
                [&]() {
#pragma unroll
                    for (int u = 0; u < kUnroll; u++)
                        asm volatile("" : "+v"(ns[u]), "+v"(ne[u]));
                });
        }
    }
}

// The region pass of sparse regions (a few thousand entries over 16384
// counters), two-level form: by entry instead of by counter.  Entries are
// counted as above; then the one that holds its counter's first position
// updates the cell, cleans the counter, and leaves a record (position | mark
// << 30) if it found the counter zero.
//
// kCells: cells a thread holds; the workgroup has them in LDS (1: regions of up
// to 1024 cells, 2: 2048).  0: regions of 4096 or 8192 cells, which do not fit
// beside the counters; each first entry reads its cell and adds to it in memory.
//
// The sweep over all counters cost 5.8 us a region and workgroup however few
// entries it had; this takes 3.1 with 50 and 4.0 with 1.9 K entries (62 K
// regions: 1.67 -> 0.98 ms), bound by memory latency behind 32 KB of cells and
// 20 KB of entries and records a region.  Two barriers a region here, and what
// the next region needs (cells, entries; bounds of the one after) is requested
// before its entries are counted.
//
// kRecords: where the records go.
// kFlat: dense in `flat`, their room asked for when a region's records are
// counted, and taken after the next region's update, the records held in
// registers until then.
// kFew (regions of kFewEntries entries on average): dense in `flat`, where
// the records of many regions leave together from LDS.  The room comes from
// one address, at 4.5 ns an atomic: one a region cost 74 of 204 us over 16 K
// regions of 15 new k-mers, now 173; the call over 10 K regions of 180 206 us
// in kFlat, 189 in this form, over 100 K of 220 1.650 and 1.641 ms, of 250 1.688
// and 1.693.
// kOwn (chunks above 2^28 positions, carried chunks): the records go to room of
// the region's own for each of its entries, as k_region_runs' do.
enum RecordForm { kOwn, kFlat, kFew };
constexpr uint64_t kFewEntries = 256;

template <int kCells, RecordForm kRecords>
__global__ void __launch_bounds__(kRegionWG)
k_region_sparse(FilterArgs F, BinPlan P, BlockPlan B, const uint32_t *__restrict__ list,
                const uint8_t *__restrict__ list_hi, const uint32_t *__restrict__ starts,
                int classify, uint32_t tau, uint32_t *__restrict__ cursor,
                uint32_t *__restrict__ flat, RecordSpace own, Carry C) {
    constexpr uint32_t kWaves = kRegionWG / 64;
    constexpr bool kOwn = kRecords == RecordForm::kOwn;
    // larger chunks' runs are shorter: more groups of fewer entries
    constexpr int kGroups = kOwn ? 3 : 2, kHeld = 4 * kGroups;
    constexpr uint32_t kStep = 64u * kGroups;
    __shared__ uint32_t hits[kRegionCounters];
    __shared__ uint32_t first[kRegionCounters];
    constexpr int kHold = kCells ? kCells : 1;
    __shared__ unsigned long long s_cell[kCells ? kCells * kRegionWG : 1];
    // records that wait in LDS: all of a region of up to kBatch (kFew), and those
    // of entries that are not held
    constexpr uint32_t kRecRoom = kOwn ? 1 : 2048, kBatch = 320;
    __shared__ uint32_t s_rec[kRecRoom];
    // by the region's parity: records of held entries, of others (!kOwn), and
    // the room for this region's (!kOwn: the region before's), read at once
    struct Tally {
        uint32_t n, more, base, pad;
    };
    __shared__ __align__(16) Tally s_tally[2];
    __shared__ uint32_t s_flush;
    __shared__ uint32_t s_total[2], s_over[2];  // kOwn, by the region's parity
    const uint32_t lane = threadIdx.x & 63u, wave = wave_id(), grid = gridDim.x;
    const uint32_t shift = P.region_shift, S = 1u << shift;
    const uint64_t n_words = F.X * F.Y;
    const uint32_t fm = (uint32_t)F.field_max;  // counters are at most 32 bits wide
    for (uint32_t i = threadIdx.x; i < (uint32_t)kRegionCounters; i += kRegionWG) {
        hits[i] = 0;
        first[i] = kIdle;
    }
    if (threadIdx.x == 0)
        s_tally[0].n = s_tally[1].n = s_tally[0].more = s_tally[1].more = s_total[0] =
            s_total[1] = s_over[0] = s_over[1] = 0;
    const bool carry_out = kOwn && C.mode == Carry::kOut;
    const bool carry_in = kOwn && kCells && C.mode == Carry::kIn && C.n_prev > 0;
    auto load_cells = [&](uint32_t r, uint64_t(&cell)[kHold]) {
        const uint64_t wbase = (uint64_t)r << shift;
#pragma unroll
        for (int k = 0; k < kCells; k++) {
            const uint32_t w = threadIdx.x + (uint32_t)k * kRegionWG;
            const bool in = (kCells > 1 || w < S) && r < P.n_regions && wbase + w < n_words;
            cell[k] = in ? F.words[wbase + w] : 0ull;
        }
    };
    // Region r's cells into L2, a word of each line: they come from memory
    // that nothing else has read for long, further off than a region's time.
    auto touch = [&](uint32_t r) -> uint32_t {
        const uint64_t w = ((uint64_t)r << shift) + 16u * threadIdx.x;
        const bool in = kCells && 16u * threadIdx.x < S && r < P.n_regions && w < n_words;
        return in ? *reinterpret_cast<const uint32_t *>(F.words + w) : 0u;
    };
    uint32_t bs, be;  // the lane's run: its entries in the list
    const uint32_t part = wave & ((1u << B.split) - 1u);
    auto bounds = [&](uint32_t r) {
        const uint32_t b = (lane * kWaves + wave) >> B.split;
        const bool in = b < B.n_super && r < P.n_regions;
        const uint32_t *t = starts + (in ? (uint64_t)b * (P.n_regions + 1u) + r : 0ull);
        bs = t[0];
        be = in ? t[1] : bs;
    };
    struct Held {
        uint4 x[kGroups];
        uint32_t h[kGroups], which[kGroups];  // entries; run, and (from bit 28) those in the run
    };
    auto load = [&](const LaneRuns &R, uint32_t w0, Held &H) {
#pragma unroll
        for (int c = 0; c < kGroups; c++) {
            H.which[c] = 0;
            if (w0 + 64u * c < R.n) {
                uint32_t i, g;
                const uint32_t m = R.at(w0 + 64u * c, lane, i, g);
                if (m) {
                    H.x[c] = *reinterpret_cast<const uint4 *>(list + g);
                    H.h[c] = *reinterpret_cast<const uint32_t *>(list_hi + g);
                    H.which[c] = i | (m << 28);
                }
            }
        }
    };
    // visit(number, counter, position) of the entries held
    auto each = [&](const LaneRuns &R, uint32_t w0, const Held &H, auto visit) {
#pragma unroll
        for (int c = 0; c < kGroups; c++)
            if (w0 + 64u * c < R.n) {
                const uint32_t m = H.which[c];
                const uint32_t tb = ((((m & 63u) * kWaves + wave) >> B.split) * B.super) << B.pos_log;
                const uint32_t e[4] = {H.x[c].x, H.x[c].y, H.x[c].z, H.x[c].w};
#pragma unroll
                for (int q = 0; q < 4; q++)
                    if ((m >> (28 + q)) & 1u)
                        visit(4 * c + q, e[q] & ((1u << kLocalBits) - 1u),
                              tb + ((e[q] >> kLocalBits) |
                                    (((H.h[c] >> (8 * q)) & 0xFFu) << (32 - kLocalBits))));
            }
    };
    auto count = [&](int, uint32_t local, uint32_t t) {
        atomicAdd(&hits[local], 1u);
        if (t < first[local])
            atomicMin(&first[local], t);
    };
    // of a region with more entries than are held, many of them likely of one
    // counter: the lanes of the first one's counter count together
    auto count_many = [&](int, uint32_t local, uint32_t t) {
        const uint32_t l0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)local);
        const uint64_t same = __ballot(local == l0);
        const bool led = local == l0 &&
                         __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u)) != 0;
        if (!led)
            atomicAdd(&hits[local], local == l0 ? (uint32_t)__popcll(same) : 1u);
        if (t < first[local])
            atomicMin(&first[local], t);
    };
    // Whether the entry at position t is its counter's first (which then cleans
    // it: the minimum here, the hits in `taken`).
    auto is_first = [&](uint32_t local, uint32_t t) -> bool {
        if (first[local] != t)
            return false;
        // two hash functions may give one position the same counter
        if (F.k_h > 1u)
            return atomicExch(&first[local], kIdle) == t;
        first[local] = kIdle;
        return true;
    };
    auto taken = [&](uint32_t local) -> uint32_t {
        const uint32_t h = hits[local];
        hits[local] = 0;
        return h;
    };
    // The cell's update by h hits; the record's mark, or 0.  pre: the cell, as
    // far as this counter goes; the field grows without carrying out.
    auto apply = [&](unsigned long long *cell, uint64_t pre, uint32_t local,
                     uint32_t h) -> uint32_t {
        const uint32_t sh = F.alpha * (local >> shift);
        const uint32_t pf = (uint32_t)(pre >> sh) & fm;
        const uint32_t room = fm - pf, inc = h < room ? h : room;
        if (inc)
            atomicAdd(cell, (unsigned long long)inc << sh);
        return pf ? 0u : (classify && inc > tau ? 3u : 1u);
    };
    // all of it, for an entry of region r; its record's mark, or 0
    auto update = [&](uint32_t r, uint32_t local, uint32_t t) -> uint32_t {
        if (!is_first(local, t))
            return 0u;
        const uint32_t h = taken(local), w = local & (S - 1u);
        unsigned long long *cell =
            kCells ? &s_cell[w] : (unsigned long long *)F.words + ((uint64_t)r << shift) + w;
        return apply(cell, *cell, local, h);
    };
    uint32_t r = (grid & 7u) == 0 ? (blockIdx.x & 7u) * (grid >> 3) + (blockIdx.x >> 3) : blockIdx.x;
    uint64_t cell[kHold];
    Held H;
    LaneRuns R;
    load_cells(r, cell);
    bounds(r);
    share_run(bs, be, part, B.split, R);
    load(R, 0, H);
    bounds(r + grid);
    uint32_t line = touch(r + grid);
    uint32_t rec[kHeld], has = 0, at = 0, got = 0;  // records waiting for their room
    uint32_t fill = 0;                              // records in s_rec (uniform)
    auto store_records = [&](uint32_t base) {
        // (16 wavefronts share four instruction issuers: what a wavefront
        // without a record would step over lane by lane, it skips)
        if (kRecords == kFew && __ballot(has != 0) == 0)
            return;
#pragma unroll
        for (int j = 0; j < kHeld; j++)
            if ((has >> j) & 1u)
                flat[base + at + (uint32_t)__popc(has & ((1u << j) - 1u))] = rec[j];
    };
    auto flush = [&]() {  // s_rec -> flat, by all threads
        if (threadIdx.x == 0)
            s_flush = atomicAdd(cursor, fill);
        __syncthreads();
        const uint32_t base = s_flush;
        for (uint32_t i = threadIdx.x; i < fill; i += kRegionWG)
            flat[base + i] = s_rec[i];
        __syncthreads();
        fill = 0;
    };
    // kOwn: the region's record `slot`, of position t and mark or counter
    auto put = [&](uint32_t slot, uint32_t t, uint32_t half) {
        (carry_out ? C.word + (uint64_t)C.chunk * C.cap : own.word)[slot] = t;
        (carry_out ? C.half + (uint64_t)C.chunk * C.cap : own.half)[slot] = (uint16_t)half;
    };
    __syncthreads();  // counters clean
    for (uint32_t turn = 0; r < P.n_regions; r += grid, turn ^= 1u) {
        LaneRuns Rn;
        Held Hn;
        uint64_t celln[kHold];
        share_run(bs, be, part, B.split, Rn);
        load(Rn, 0, Hn);
        load_cells(r + grid, celln);
        bounds(r + 2u * grid);
#pragma unroll
        for (int k = 0; k < kCells; k++)
            s_cell[threadIdx.x + (uint32_t)k * kRegionWG] = cell[k];
        each(R, 0, H, count);
        for (uint32_t w0 = kStep; w0 < R.n; w0 += kStep) {
            Held X;
            load(R, w0, X);
            each(R, w0, X, count_many);
        }
        if constexpr (kOwn) {
            const uint32_t n = wave_inclusive(R.e - R.s);
            if (lane == 63) {
                atomicAdd(&s_total[turn], n);
                if (R.n > kStep)
                    s_over[turn] = 1;
            }
        }
        __syncthreads();  // counted
        if (threadIdx.x == 0)  // the region before's, read by every thread
            s_tally[turn ^ 1u].n = s_tally[turn ^ 1u].more = 0;
        if constexpr (kOwn) {  // room for a record of every entry
            got = 0;
            if (threadIdx.x == 0 && s_total[turn])
                got = atomicAdd(cursor, s_total[turn]);
        }
        uint32_t fresh[kHeld], halves[kHeld / 2], won = 0;
#pragma unroll
        for (int j = 0; j < kHeld; j++)
            fresh[j] = 0;
#pragma unroll
        for (int j = 0; j < kHeld / 2; j++)
            halves[j] = 0;
        // cells in memory: those of all held entries are requested together
        uint32_t marks[kHeld];
        if constexpr (kCells == 0) {
            uint64_t was[kHeld];
            unsigned long long *cells = (unsigned long long *)F.words + ((uint64_t)r << shift);
#pragma unroll
            for (int j = 0; j < kHeld; j++) {
                marks[j] = 0;
                was[j] = 0;
            }
            each(R, 0, H, [&](int j, uint32_t local, uint32_t t) {
                if (is_first(local, t)) {
                    marks[j] = taken(local);
                    was[j] = cells[local & (S - 1u)];
                }
            });
            each(R, 0, H, [&](int j, uint32_t local, uint32_t) {
                if (marks[j])
                    marks[j] = apply(&cells[local & (S - 1u)], was[j], local, marks[j]);
            });
        }
        each(R, 0, H, [&](int j, uint32_t local, uint32_t t) {
            const uint32_t mark = kCells ? update(r, local, t) : marks[j];
            if (kOwn) {
                fresh[j] = t;
                halves[j / 2] |= (carry_out ? local : mark) << (16 * (j % 2));
            } else {
                fresh[j] = t | (mark << 30);
            }
            won |= mark ? 1u << j : 0u;
        });
        if constexpr (kOwn)
            if (s_over[turn]) {
                if (threadIdx.x == 0)
                    s_tally[turn].base = got;
                __syncthreads();
            }
        for (uint32_t w0 = kStep; w0 < R.n; w0 += kStep) {
            // more than the registers hold
            load(R, w0, H);
            each(R, w0, H, [&](int, uint32_t local, uint32_t t) {
                const uint32_t mark = update(r, local, t);
                if (mark && kOwn)
                    put(s_tally[turn].base + atomicAdd(&s_tally[turn].n, 1u), t,
                        carry_out ? local : mark);
                else if (mark) {  // one atomic for the lanes that are here
                    const uint64_t m = __ballot(true);
                    const uint32_t i = __builtin_amdgcn_mbcnt_hi(
                        (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                    const uint32_t n = (uint32_t)__popcll(m), x = t | (mark << 30);
                    uint32_t at = 0;
                    if (i == 0)
                        at = atomicAdd(&s_tally[turn].more, n);
                    at = fill + (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
                    const uint32_t left = at < kRecRoom ? kRecRoom - at : 0u;
                    const uint32_t fit = n < left ? n : left;
                    if (i < fit)
                        s_rec[at + i] = x;
                    if (fit < n) {
                        if (i == 0)
                            at = atomicAdd(cursor, n - fit);
                        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
                        if (i >= fit)
                            flat[at + i - fit] = x;
                    }
                }
            });
        }
        const bool some = __ballot(won != 0) != 0;  // uniform
        uint32_t place = 0;
        if (some) {
            const uint32_t mine = (uint32_t)__popc(won), incl = wave_inclusive(mine);
            if (lane == 63)
                place = atomicAdd(&s_tally[turn].n, incl);
            place = (uint32_t)__builtin_amdgcn_readlane((int)place, 63) + incl - mine;
        }
        // every load in flight is taken in before the first store
#pragma unroll
        for (int c = 0; c < kGroups; c++)
            asm volatile(""
                         : "+v"(Hn.x[c].x), "+v"(Hn.x[c].y), "+v"(Hn.x[c].z), "+v"(Hn.x[c].w),
                           "+v"(Hn.h[c]));
#pragma unroll
        for (int k = 0; k < kCells; k++)
            asm volatile("" : "+v"(celln[k]));
        asm volatile("" : "+v"(bs), "+v"(be), "+v"(line));
        line = touch(r + 2u * grid);
        if (threadIdx.x == 0)
            s_tally[turn].base = got;
        __syncthreads();  // updated, counters clean
        const uint4 tally = *reinterpret_cast<const uint4 *>(&s_tally[turn]);
        const uint32_t base = tally.z;
        if (threadIdx.x == 0) {
            if constexpr (kOwn) {
                const uint64_t x = carry_out ? (uint64_t)C.chunk * C.stride + r : r;
                (carry_out ? C.off : own.off)[x] = base;
                (carry_out ? C.n : own.n)[x] = tally.x;
                s_total[turn] = s_over[turn] = 0;
            } else if (tally.x > (kRecords == kFew ? kBatch : 0u)) {
                got = atomicAdd(cursor, tally.x);
            }
        }
        const uint64_t wbase = (uint64_t)r << shift;
#pragma unroll
        for (int k = 0; k < kCells; k++) {
            const uint32_t w = threadIdx.x + (uint32_t)k * kRegionWG;
            const uint64_t next = s_cell[w];
            if (next != cell[k])
                F.words[wbase + w] = next;
            cell[k] = celln[k];
        }
        if constexpr (kOwn) {
            uint32_t slot = base + place;
            if (some)
#pragma unroll
                for (int j = 0; j < kHeld; j++)
                    if ((won >> j) & 1u)
                        put(slot++, fresh[j], (halves[j / 2] >> (16 * (j % 2))) & 0xFFFFu);
            if (carry_in) {
                mark_carried(F, shift, C, r, s_cell, tau);
                __syncthreads();  // the cells are rewritten by the next region
            }
        } else {
            store_records(base);
            const uint32_t more = (uint32_t)__builtin_amdgcn_readfirstlane((int)tally.y);
            fill = fill + more < kRecRoom ? fill + more : kRecRoom;
            const uint32_t n =
                kRecords == kFew ? (uint32_t)__builtin_amdgcn_readfirstlane((int)tally.x) : 0u;
            if (__builtin_expect(fill + (kRecords == kFew ? kBatch : kRecRoom / 2) > kRecRoom, 0))
                flush();
            if (kRecords == kFew && n <= kBatch) {
                has = 0;
                place += fill;
                if (some)
#pragma unroll
                    for (int j = 0; j < kHeld; j++)
                        if ((won >> j) & 1u)
                            s_rec[place++] = fresh[j];
                fill += n;
            } else {
#pragma unroll
                for (int j = 0; j < kHeld; j++)
                    rec[j] = fresh[j];
                has = won;
                at = place;
            }
        }
        R = Rn;
        H = Hn;
    }
    if constexpr (!kOwn) {
        __syncthreads();
        if (threadIdx.x == 0)
            s_tally[0].base = got;
        __syncthreads();
        store_records(s_tally[0].base);
        if (fill)
            flush();
    }
}

namespace {

using SparseKernel = void (*)(FilterArgs, BinPlan, BlockPlan, const uint32_t *, const uint8_t *,
                              const uint32_t *, int, uint32_t, uint32_t *, uint32_t *, RecordSpace,
                              Carry);
using SortKernel = void (*)(FilterArgs, ReadsArgs, uint64_t, uint64_t, uint64_t, BlockPlan, uint32_t,
                            uint32_t *, uint8_t *, uint16_t *, unsigned long long *);
using RunsKernel = void (*)(FilterArgs, uint64_t, BinPlan, BlockPlan, const uint32_t *,
                            const uint8_t *, const void *, int, uint32_t, RecordSpace, Carry);

template <int kKh, bool kFast, bool kWide, bool kTwo>
SortKernel sort_kernel_of(const BlockPlan &B) {
    if (B.wg == 1024)
        return k_hash_sort<1024, 32, kKh, kFast, kWide, kTwo>;
    if constexpr (!kTwo)
        if (B.ept == 32)
            return k_hash_sort<512, 32, kKh, kFast, kWide, false>;
    return k_hash_sort<512, 8, kKh, kFast, kWide, kTwo>;
}

template <int kKh, bool kFast>
SortKernel sort_kernel_for(const BlockPlan &B, uint32_t k) {
    if (B.two)
        return k > 32 ? sort_kernel_of<kKh, kFast, true, true>(B)
                      : sort_kernel_of<kKh, kFast, false, true>(B);
    return k > 32 ? sort_kernel_of<kKh, kFast, true, false>(B)
                  : sort_kernel_of<kKh, kFast, false, false>(B);
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

template <int kCounters, int kCells, bool kSorted>
RunsKernel runs_kernel_of(const BlockPlan &B) {
    if (B.two)
        return k_region_runs<kCounters, kCells, 1, true, kSorted>;
    if (B.turned)
        return k_region_runs<kCounters, kCells, 0, false, kSorted>;
    return B.lanes == 4 ? k_region_runs<kCounters, kCells, 4, false, kSorted>
                        : k_region_runs<kCounters, kCells, 16, false, kSorted>;
}

// The region pass's instance: counters per region, cells per thread, and
// lanes per run.
template <int kCounters, bool kSorted>
RunsKernel runs_kernel(const BinPlan &P, const BlockPlan &B) {
    switch ((1u << P.region_shift) / kRegionWG) {
    case 0:
        return runs_kernel_of<kCounters, 0, kSorted>(B);
    case 1:
        return runs_kernel_of<kCounters, 1, kSorted>(B);
    case 2:
        return runs_kernel_of<kCounters, 2, kSorted>(B);
    case 4:
        return runs_kernel_of<kCounters, 4, kSorted>(B);
    default:  // two counters a cell
        return runs_kernel_of<kCounters, 8, kSorted>(B);
    }
}

template <RecordForm kRecords>
SparseKernel sparse_kernel(const BinPlan &P) {
    return P.region_shift > 11    ? k_region_sparse<0, kRecords>
           : P.region_shift == 11 ? k_region_sparse<2, kRecords>
                                  : k_region_sparse<1, kRecords>;
}

}  // namespace

bool block_plan(const BinPlan &plan, uint32_t k_h, uint64_t len, BlockPlan &B) {
    if (len == 0)
        return false;
    B = BlockPlan{};
    B.kh = 1;
    while (B.kh < k_h)
        B.kh *= 2;
    const uint64_t entries = len * k_h;
    // (regions of half the counters: twice the regions, half the entries each)
    const uint32_t half = plan.region_counters == (uint32_t)kSmallRegionCounters ? 1u : 0u;
    B.two = plan.n_parts || plan.n_regions > kBlockRegions ||
            (plan.n_regions >= kSparseRegions << half &&
             entries <= (kSparseShort >> half) * plan.n_regions);
    // large blocks make long runs; chunks that would leave the chip idle take
    // small ones
    B.wg = B.two || plan.n_regions > kHalfRegions ? 1024u : 512u;
    B.ept = 32;
    if (len * B.kh < 512ull * 32 * 512) {
        B.wg = 512;
        B.ept = 8;
    }
    while ((1u << B.pos_log) < B.ept * B.wg / B.kh)
        B.pos_log++;
    B.cap = k_h << B.pos_log;  // a multiple of 16: blocks' lists start at 16-byte boundaries
    B.n_blocks = (uint32_t)((len + (1ull << B.pos_log) - 1) >> B.pos_log);
    if (!B.two) {
        // no power of two: the same region's runs of consecutive blocks fall
        // on different memory channels
        B.cap += kBlockPad;
        B.n_bins = plan.n_regions;
        B.row = (B.n_bins + 2u) & ~1u;
        B.turned = B.cap / B.n_bins <= kShortRun ? (B.n_blocks + 1u) & ~1u : 0u;
        B.lanes = B.cap / B.n_bins <= 64 ? 4u : 16u;
        // four wavefronts at least have blocks: a k-mer repeated over most of a
        // small call's reads is counted by as many (94% of 250 K bases over 488
        // regions 798 -> 313 us)
        B.share = B.n_blocks < 256u ? (B.n_blocks + 3u) / 4u : 64u;
        return true;
    }
    // about as many buckets as regions in a bucket, at most 512 buckets of at
    // most 2^kMaxSubLog regions (then more buckets); small forced partitions
    // (tests) make buckets of as many regions
    while (((plan.n_regions - 1u) >> B.sub_log) >= 512u && B.sub_log < kMaxSubLog)
        B.sub_log++;
    if (plan.n_parts && plan.part_log < B.sub_log)
        B.sub_log = plan.part_log;
    B.n_bins = (plan.n_regions + (1u << B.sub_log) - 1u) >> B.sub_log;
    if (B.n_bins > kMaxBins)
        return false;
    B.row = (B.n_bins + 2u) & ~1u;
    // superblocks whose buckets about fill the second level's LDS when every
    // window is valid
    const uint32_t run = B.cap / B.n_bins + 1u;
    uint32_t m = kMergeTile * 7u / 8u / run;
    // ... of at most 64 blocks for each of the second level's wavefronts
    const uint32_t most = kMergeWG < (1u << kSuperLog) >> B.pos_log ? kMergeWG
                                                                    : (1u << kSuperLog) >> B.pos_log;
    m = m < 1u ? 1u : (m > most ? most : m);
    B.super = m < B.n_blocks ? m : B.n_blocks;
    B.n_super = (B.n_blocks + B.super - 1u) / B.super;
    while ((B.n_super << (B.split + 1u)) <= (uint32_t)kRegionWG / 64u)
        B.split++;
    // sparse regions are worked by entry, up to kSparseEntries a region on
    // average (cells in memory: kSparseCells)
    B.by_entry = B.n_super <= kRegionWG &&
                 entries <= (plan.region_shift > 11 ? kSparseCells : kSparseEntries) * plan.n_regions;
    return true;
}

hipError_t launch_blocks_chunk(const FilterArgs &F, const ReadsArgs &R, uint64_t c0, uint64_t c1,
                               const BinPlan &plan, const BlockPlan &B, const Workspace &W,
                               bool classify, uint32_t tau, const Carry &carry, bool records,
                               hipStream_t s, Profiler *P) {
    const uint64_t len = c1 - c0;
    // Rooms of the workspace.  One-level form: the list in entries, the table in
    // the first matrix or in slots, the turned table in the second matrix or
    // behind the list.  Two-level form: the blocks' list and table in bucketed,
    // the superblocks' list and starts in entries (small calls: the table and
    // starts in the matrices).  Records take bucketed, which either form has
    // read by then.
    const uint64_t last = c1 - c0 - ((uint64_t)(B.n_blocks - 1) << B.pos_log);
    const uint64_t n_list = ((uint64_t)(B.n_blocks - 1) * B.cap + last * F.k_h + 15) / 16 * 16;
    const uint64_t room = 8 * W.entries_cap;  // bytes of entries, and of bucketed
    const uint64_t table_bytes = 2ull * B.n_blocks * B.row;
    const uint64_t turned_bytes = 2ull * B.turned * B.row;
    const uint64_t starts_bytes = 4ull * B.n_super * (plan.n_regions + 1u);
    if (n_list > (1ull << 32))
        return hipErrorInvalidValue;
    uint32_t *list = (uint32_t *)(B.two ? W.bucketed : W.entries), *merged = (uint32_t *)W.entries;
    uint8_t *list_hi = nullptr, *merged_hi = nullptr;
    uint16_t *table = (uint16_t *)W.matrix, *turned = (uint16_t *)W.matrix_t;
    uint32_t *starts = W.matrix;
    if (B.two) {
        if (5 * n_list > (room + 255) / 256 * 256)
            return hipErrorInvalidValue;
        list_hi = (uint8_t *)(list + n_list);
        merged_hi = (uint8_t *)(merged + n_list);
        table = (uint16_t *)(W.matrix_t + 2ull * plan.n_regions);
        if (5 * n_list + table_bytes <= room)
            table = (uint16_t *)(list_hi + n_list);
        else if (8ull * plan.n_regions + table_bytes > 4 * W.matrix_cap)
            return hipErrorInvalidValue;
        if (5 * n_list + starts_bytes <= room)
            starts = (uint32_t *)(merged_hi + n_list);
        else if (starts_bytes > 4 * W.matrix_cap)
            return hipErrorInvalidValue;
    } else {
        if (4 * n_list > (room + 255) / 256 * 256)
            return hipErrorInvalidValue;
        if (table_bytes > 4 * W.matrix_cap) {
            table = (uint16_t *)W.slots;
            if (table_bytes > 4 * W.slots_cap)
                return hipErrorInvalidValue;
        }
        if (turned_bytes > 4 * W.matrix_cap) {
            turned = (uint16_t *)(list + n_list);
            if (4 * n_list + turned_bytes > room)
                return hipErrorInvalidValue;
        }
    }
    // partitioned plans (more than kMaxRegions regions) name their phases so
    if (P)
        P->begin(plan.n_parts ? kPhBinPart : kPhBinCount, s);
    hipLaunchKernelGGL(sort_kernel(F, R.k, B), dim3(B.n_blocks), dim3(B.wg),
                       B.n_bins * sizeof(uint32_t), s, F, R, mask_words(R.n_bases), c0, c1, B,
                       plan.region_shift, list,
                       list_hi, table, (unsigned long long *)(W.totals + 5));
    if (P)
        P->end(s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    if (B.two || B.turned) {
        if (P)
            P->begin(plan.n_parts ? kPhPartCount : kPhBinRegion, s);
        if (B.two)
            hipLaunchKernelGGL(k_merge, dim3((B.n_bins + 7) / 8 * 8 * B.n_super), dim3(kMergeWG),
                               0, s, B, plan.n_regions, (const uint32_t *)list,
                               (const uint8_t *)list_hi, (const uint16_t *)table, merged,
                               merged_hi, starts);
        else
            hipLaunchKernelGGL(k_turn_table, dim3((B.row + 63) / 64, (B.n_blocks + 63) / 64),
                               dim3(256), 0, s, (const uint16_t *)table, turned, B.n_blocks, B.row,
                               B.turned);
        if (P)
            P->end(s);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    }
    RecordSpace rec{};
    while ((len + (1ull << rec.log) - 1) >> rec.log > kMarkBuckets || rec.log < 12)
        rec.log++;
    // The by-entry pass marks carried records where it writes its own to the
    // regions' room: 20 M positions in two chunks over 60 K regions 3.25 -> 2.55
    // ms, a last chunk of 461 over 316 K regions of 256 cells 19 -> 3.7, which
    // the pass by counter swept.
    records = records || (B.by_entry && carry.mode == Carry::kIn);
    const bool own = records || carry.mode == Carry::kOut;  // records in the regions' own room
    const bool sparse = B.by_entry && !own && carry.mode == Carry::kNone && 8 * len * F.k_h <= room;
    if (records || carry.mode == Carry::kOut || sparse) {
        rec.cursor = W.n_entries + 3;
        if ((e = fill_u32(rec.cursor, 1, 0u, s)) != hipSuccess)
            return e;
        if (sparse) {
            rec.room = (uint64_t)F.k_h << rec.log;
            rec.word = (uint32_t *)W.bucketed;  // the sorted records; the dense ones after them
        } else if (records) {
            uint32_t *index = B.two ? W.matrix_t : W.index;
            if (2ull * plan.n_regions > (B.two ? W.matrix_cap : W.index_cap))
                return hipErrorInvalidValue;
            rec.word = (uint32_t *)W.bucketed;
            rec.half = (uint16_t *)(rec.word + W.entries_cap);
            rec.off = index;
            rec.n = index + plan.n_regions;
        }
    } else {
        // a position can be first seen by each of its hash functions
        rec.room = (uint64_t)F.k_h << rec.log;
        rec.sorted = (uint32_t *)W.bucketed;
        rec.cursor = mark_cursors(W);
    }
    const void *runs = B.two ? (const void *)starts
                             : (const void *)(B.turned ? turned : table);
    if (P)
        P->begin(kPhRegion, s);
    // (the by-entry pass has LDS for the larger regions' counters)
    const bool whole = sparse || (B.by_entry && own);
    const uint32_t grid =
        region_grid(plan.n_regions, whole ? (uint32_t)kRegionCounters : plan.region_counters);
    if (sparse) {
        const bool few = len * F.k_h <= kFewEntries * plan.n_regions;
        hipLaunchKernelGGL((few ? sparse_kernel<kFew>(plan) : sparse_kernel<kFlat>(plan)),
                           dim3(grid), dim3(kRegionWG), 0, s, F, plan, B, (const uint32_t *)merged,
                           (const uint8_t *)merged_hi, (const uint32_t *)starts, classify ? 1 : 0,
                           tau, rec.cursor, rec.word + len * F.k_h, rec, carry);
        if (P)
            P->end(s);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
        if (P)
            P->begin(kPhWinners, s);
        e = launch_sort_records(rec.word + len * F.k_h, rec.cursor, rec.word, rec.room, rec.log,
                                mark_cursors(W), s);
        if (e == hipSuccess)
            e = launch_marks(rec.word, rec.room, rec.log, mark_cursors(W), true, c0, len, R.n_bases,
                             W, s);
        if (P)
            P->end(s);
        return e;
    }
    if (whole) {
        hipLaunchKernelGGL(sparse_kernel<kOwn>(plan),
                           dim3(grid), dim3(kRegionWG), 0, s, F, plan, B, (const uint32_t *)merged,
                           (const uint8_t *)merged_hi, (const uint32_t *)starts, classify ? 1 : 0,
                           tau, rec.cursor, nullptr, rec, carry);
    } else {
        const bool small = plan.region_counters == (uint32_t)kSmallRegionCounters;
        hipLaunchKernelGGL((rec.sorted ? (small ? runs_kernel<kSmallRegionCounters, true>(plan, B)
                                                : runs_kernel<kRegionCounters, true>(plan, B))
                                       : (small ? runs_kernel<kSmallRegionCounters, false>(plan, B)
                                                : runs_kernel<kRegionCounters, false>(plan, B))),
                           dim3(grid), dim3(kRegionWG), 0,
                           s, F, c0, plan, B, (const uint32_t *)(B.two ? merged : list),
                           (const uint8_t *)merged_hi, runs, classify ? 1 : 0, tau, rec, carry);
    }
    if (P)
        P->end(s);
    e = hipGetLastError();
    if (e == hipSuccess && records)
        return launch_record_winners(F.k_h, plan.n_regions, rec.off, rec.n, rec.word, rec.half, c0, len,
                                     R.n_bases, W, s, P);
    if (e == hipSuccess && rec.sorted) {
        if (P)
            P->begin(kPhWinners, s);
        e = launch_marks(rec.sorted, rec.room, rec.log, rec.cursor, true, c0, len, R.n_bases, W, s);
        if (P)
            P->end(s);
    }
    return e;
}

}  // namespace kc
