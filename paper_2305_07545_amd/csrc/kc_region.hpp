// What the forms of the region pass share: the marks of carried records, and
// where first-seen records go.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kc_device.hpp"
#include "kc_kernels.hpp"

namespace kc {

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

// Where a chunk's first-seen records (t, mark: 1 distinct, 3 distinct and
// trustworthy) go.  Sorted by bucket of 2^log positions (sorted non-null):
// bucket g's records, position | mark << log, are appended at sorted + g *
// room by cursor[g].  Else each region's own: its n[r] records start at off[r]
// of word (t) and half (mark), in room reserved at cursor[0].
struct RecordSpace {
    uint32_t *sorted;
    uint32_t log;
    uint64_t room;
    uint32_t *word;
    uint16_t *half;
    uint32_t *off;
    uint32_t *n;
    uint32_t *cursor;
};

// Workgroups of a persistent region pass.
uint32_t region_grid(uint32_t n_regions, uint32_t counters);

}  // namespace kc
