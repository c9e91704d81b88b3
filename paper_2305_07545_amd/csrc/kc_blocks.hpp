// Block-sorted entry lists of the binned insertion (host view).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kc_kernels.hpp"

namespace kc {

constexpr uint32_t kBlockLog = 15;  // a block holds at most 2^15 entries
constexpr uint32_t kBlockEntries = 1u << kBlockLog;
// Regions of a countBF the one-level form takes: the block's histogram fits
// beside its entries in LDS, for two hashing workgroups of 16384 entries per
// CU, or one of 32768.
constexpr uint32_t kHalfRegions = 3584;
constexpr uint32_t kBlockRegions = 7168;
constexpr uint32_t kBlockPad = 80;  // entries of a block's stride beyond its room
// Runs of up to this many entries (a block's room / regions) are short: the
// region pass takes 64 blocks' runs at a time.
constexpr uint32_t kShortRun = 16;
// Two-level form
constexpr uint32_t kMaxSubLog = 11;   // log2(regions per bucket), at most
constexpr uint32_t kMaxBins = 2048;   // buckets, at most (4M regions)
constexpr uint32_t kSuperLog = 26;    // log2(positions per superblock), at most
constexpr uint32_t kMergeWG = 1024;   // threads of the second level
// Regions of up to this many entries on average are worked by entry, which the
// pass holds in registers up to there: 150 M bases over 62 K regions (1.9 K
// entries each) 1.77 -> 1.08 ms with the records, 100 M over 16 K (5 K) 0.59 ->
// 0.52; 200 M over 16 K (10 K) 0.73 -> 0.68, but more entries than are held are
// read twice.  Regions of 256 and 512 cells, as long as these: 30 M bases over
// 20 K regions (1 K) 1.14 -> 0.58 and 0.89 -> 0.52 ms the call, 125 M (5 K)
// 2.02 -> 1.51 and 1.88 -> 1.37.
constexpr uint64_t kSparseEntries = 8192;
// The same of regions of 4096 and 8192 cells, whose first entries read a cache
// line each: 12 K regions of 1.2 K entries 0.68 -> 0.49 and 1.11 -> 0.50 ms the
// call, of 2.4 K 0.87 -> 0.73 and 1.32 -> 0.76, of 4.8 K 1.22 and 1.69 -> 1.33.
constexpr uint64_t kSparseCells = 4096;
// A countBF that the one-level form takes goes to the two-level one for that
// from this many regions on, with up to this many entries a region: the call
// (one-level against two-level) with 10 new k-mers a region over 1000 regions
// 66 and 69 us, 1500 80 and 78, 3000 115 and 95, 7000 197 and 137; with 50 over
// 7000 204 and 138; over 2000 regions with 600 entries 114 and 100, 2400 149 and
// 142, 4800 183 and 215; 4096 cells a region, 6000 regions, 300 198 and 179,
// 2400 336 and 352.
// Regions of 8192 counters: twice the one and half of the other (7000 regions
// with 10 entries 147 and 117 us, 300 204 and 167; 2000 with 1000 102 and 104;
// two-level in any case, 60 K regions with 200 new k-mers 1.40 and 0.98 ms).
constexpr uint32_t kSparseRegions = 1536;
constexpr uint64_t kSparseShort = 2048;
constexpr uint32_t kMergeTile = 12288;  // entries it stages in LDS (two workgroups per CU)

// Blocks of one chunk: block b holds the entries of positions [b << pos_log,
// (b + 1) << pos_log) of the chunk (every hash function's), sorted by bin: a
// region (one-level form) or a bucket of 2^sub_log regions, which the second
// level sorts by region, `super` blocks at a time.
struct BlockPlan {
    uint32_t pos_log;   // log2(positions per block)
    uint32_t cap;       // a block's stride in the list (entries)
    uint32_t n_blocks;
    uint32_t n_bins;
    uint32_t row;       // 16-bit offsets per block in the table (bins + 1, even)
    uint32_t kh;        // hash functions, rounded up to a power of two
    uint32_t ept;       // entries per thread of the hashing kernel
    uint32_t wg;        // threads of the hashing kernel
    uint32_t turned;    // short runs: 16-bit offsets per region of the turned table, else 0
    uint32_t lanes;     // lanes of the region pass per run
    uint32_t share;     // short runs: blocks a wavefront takes at a time (64 at most)
    uint32_t two;       // two-level form
    uint32_t sub_log;
    uint32_t super;
    uint32_t n_super;   // superblocks
    uint32_t by_entry;  // sparse regions: worked by entry
    uint32_t split;     // log2(wavefronts of the region pass that share a superblock's run)
};

// The blocks of `len` positions (false: none, or more buckets than kMaxBins).
bool block_plan(const BinPlan &plan, uint32_t k_h, uint64_t len, BlockPlan &B);

// hash + sort + region pass of chunk [c0, c1).
hipError_t launch_blocks_chunk(const FilterArgs &F, const ReadsArgs &R, uint64_t c0, uint64_t c1,
                               const BinPlan &plan, const BlockPlan &B, const Workspace &W,
                               bool classify, uint32_t tau, const Carry &carry, bool records,
                               hipStream_t s, Profiler *P);

// The winner passes of chunk [c0, c0 + len) over records, at most k_h a
// position, whose arrays lie in W.bucketed (kc_binned.hip).
hipError_t launch_record_winners(uint32_t k_h, uint32_t n_regions, const uint32_t *off, const uint32_t *n,
                                 const uint32_t *word, const uint16_t *half, uint64_t c0,
                                 uint64_t len, uint64_t n_bases, const Workspace &W, hipStream_t s,
                                 Profiler *P);
// *n records (position | mark << 30) at in, to buckets of 2^log positions:
// appended to out + g * room as position | mark << log, cursor[g] moved.
hipError_t launch_sort_records(const uint32_t *in, const uint32_t *n, uint32_t *out, uint64_t room,
                               uint32_t log, uint32_t *cursor, hipStream_t s);
// The distinct and trustworthy bits and tile counts of chunk [c0, c0 + len)
// from records sorted by bucket of 2^log positions (bucket g's cursor[g]
// records at in + g * room: position | mark << log).
hipError_t launch_marks(const uint32_t *in, uint64_t room, uint32_t log, uint32_t *cursor,
                        bool clean, uint64_t c0, uint64_t len, uint64_t n_bases,
                        const Workspace &W, hipStream_t s);

}  // namespace kc
