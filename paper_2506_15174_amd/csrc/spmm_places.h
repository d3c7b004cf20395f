// What the workgroups of a launch compute (internal): functions of the kernels that the host's tests call too.
#ifndef SPMM_PLACES_H
#define SPMM_PLACES_H

#include <stdint.h>

#ifdef __HIPCC__
#define SPMM_DEVICE __device__ __host__ __forceinline__
#else
#define SPMM_DEVICE inline
#endif

// Column tiles (strips) of all panels (groups of units), dealt in two sets: place by place the first `set` columns of every
// row, then the others; set = columns: one set.  For a place behind the last: row `rows`.
struct set_place {
    uint32_t row, column;
};
SPMM_DEVICE set_place place_in_sets(uint32_t place, uint32_t rows, uint32_t columns, uint32_t set)
{
    const uint32_t first = rows * set;
    uint32_t before = 0, width = set;
    if (__builtin_expect(place >= first, 0)) {
        if (set == columns) return set_place{rows, 0};
        before = set;
        place -= first;
        width = columns - set;
    }
    return set_place{place / width, before + place % width};
}

#endif
