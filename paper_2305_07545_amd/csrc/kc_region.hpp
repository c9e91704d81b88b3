// The region pass's counter update, shared by its forms: where a first-seen
// occurrence goes, the update of one cell and the marks of carried records.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kc_device.hpp"
#include "kc_kernels.hpp"

namespace kc {

// Element at a 32-bit byte offset from a wavefront-uniform base: the address
// is the base's scalar registers plus one 32-bit vector register, not a
// 64-bit address per thread.
template <typename T>
__device__ __forceinline__ T &at_byte(T *base, uint32_t byte_off) {
    return *(T *)((char *)base + byte_off);
}

// Where the region pass puts a first-seen occurrence (chunk-relative t and
// its mark: 1 distinct, 3 distinct and trustworthy): its flag byte, or, in
// records mode, a record in the region's room of the record arrays, which the
// winner passes turn into flag bytes written in whole 16-byte groups.
struct WinnerSink {
    uint8_t *flags;
    uint64_t c0;
    uint32_t *rec_t;  // records or carry mode: the records' word array (null: flag mode)
    uint16_t *rec_m;  // ... and half array: the mark, or in carry mode the local counter
    uint64_t e0;      // the region's first record
    uint32_t *count;  // LDS: records written so far
    bool carry;       // carry mode: the half is the local counter id
};

__device__ __forceinline__ void put_winner(const WinnerSink &o, uint32_t t, uint32_t mark,
                                           uint32_t local) {
    if (!o.rec_t) {
        o.flags[o.c0 + t] = (uint8_t)mark;
        return;
    }
    const uint32_t i = atomicAdd(o.count, 1u);  // < the region's entries
    at_byte(o.rec_t + o.e0, 4u * i) = t;
    at_byte(o.rec_m + o.e0, 2u * i) = (uint16_t)(o.carry ? local : mark);
}

// Counter update of cell w of the region (pre = its value before the
// chunk); returns the cell's new value.  Leaves the cell's counters clean
// (hits 0, first kIdle) for the next region.
__device__ __forceinline__ uint64_t region_cell(const FilterArgs &F, uint32_t shift,
                                                uint64_t wbase, uint32_t w, uint64_t pre,
                                                uint32_t *hits, uint32_t *first,
                                                const WinnerSink &out, int classify,
                                                uint32_t tau) {
    // counters are at most 32 bits wide: the field arithmetic is 32-bit
    const uint32_t fm = (uint32_t)F.field_max;
    uint64_t next = pre;
    for (uint32_t l = 0; l < F.eta; l++) {
        const uint32_t idx = (l << shift) | w;
        const uint32_t h = hits[idx];
        if (h == 0)
            continue;
        const uint32_t t = first[idx];
        hits[idx] = 0;
        first[idx] = kIdle;
        const uint32_t sh = F.alpha * l;
        const uint32_t pf = (uint32_t)(pre >> sh) & fm;
        const uint32_t room = fm - pf;
        const uint32_t nf = pf + (h < room ? h : room);
        next += (uint64_t)(nf - pf) << sh;  // the field grows without carrying out
        if (pf == 0)
            put_winner(out, t, (classify && nf > tau) ? 3u : 1u, idx);
    }
    if (next != pre)
        F.words[wbase + w] = next;
    return next;
}

// The carried records of region r (chunks 0 .. n_prev - 1): trustworthy (3)
// when the counter's final value, staged in s_cell, is above tau.
__device__ __forceinline__ void mark_carried(const FilterArgs &F, uint32_t shift, const Carry &C,
                                             uint32_t r, const unsigned long long *s_cell,
                                             uint32_t tau) {
    for (uint32_t j = 0; j < C.n_prev; j++) {
        const uint64_t at = (uint64_t)j * C.stride + r;
        const uint64_t x0 = (uint64_t)j * C.cap + C.off[at];
        const uint32_t n = C.n[at];
        for (uint32_t i = threadIdx.x; i < n; i += kRegionWG) {
            const uint32_t local = C.half[x0 + i];
            const uint64_t cv = s_cell[local & ((1u << shift) - 1u)];
            const uint32_t f =
                (uint32_t)(cv >> (F.alpha * (local >> shift))) & (uint32_t)F.field_max;
            C.half[x0 + i] = f > tau ? 3u : 1u;
        }
    }
}

// Record arrays of a chunk whose regions reserve their own room: region r's
// n[r] records start at off[r] of word and half (n null: flag bytes).
struct RecordSpace {
    uint32_t *word;
    uint16_t *half;
    uint32_t *off;
    uint32_t *n;
    uint32_t *cursor;  // records reserved so far
};

// Workgroups of a persistent region pass.
uint32_t region_grid(uint32_t n_regions, uint32_t counters);

}  // namespace kc
