// Which bytes of a statistics table a search reads through a buffer
// descriptor.  A sweep loads one plane of records a step, some planes ahead of
// its ranking and over whole runs of planes, so the last loads of a window lie
// past its planes, and near the table's end past the table.  The descriptor of
// each step therefore starts at that step's plane and holds what is left of the
// table from there: the range check of a load covers its per-lane offset alone,
// so nothing is asked of a scalar offset.  Loads past the table return 0 (the
// planes they belong to are masked).
//
// Plain arithmetic, so that it compiles for a host as well.
#pragma once

#include <cstdint>

#ifndef NRR_HOST_DEVICE
#define NRR_HOST_DEVICE __host__ __device__
#endif

namespace nrr {

struct RecordPlanes {
    const unsigned char *base;  // this step's records, from the window's corner on
    uint32_t bytes;             // readable from there (0 behind the last plane)

    // `table`: nstat records of `size` bytes; `corner`: the window's first one.
    // Offsets from the base, planes added to them included, must lie below 2^31.
    NRR_HOST_DEVICE inline void start(const void *table, int64_t nstat, int64_t corner, int size) {
        base = static_cast<const unsigned char *>(table) + corner * size;
        const int64_t left = (nstat - corner) * size;
        bytes = (uint32_t)(left < 0xffffffffll ? left : 0xffffffffll);
    }
    NRR_HOST_DEVICE inline void next(uint32_t plane_bytes) {
        const uint32_t d = bytes < plane_bytes ? bytes : plane_bytes;
        base += d;
        bytes -= d;
    }
};

}  // namespace nrr
