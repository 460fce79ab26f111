// Places of a batch's moments in their common pool (cells.hip), in rows of one (query cell,
// key chunk) pair each: arithmetic shared by the device and a test on the host.
#pragma once

#include <hip/hip_runtime.h>

namespace ct {

// Rows of one problem's buffers, from its cells and chunks of x and y and the sweeps that take
// the form (f, g, p, q): cross (f and g in turn), x-x and y-y.  A problem has up to 4096 cells
// a side, so a batch's rows go beyond 32 bits.
struct PoolRows {
    long long r[3];
    __host__ __device__ long long all() const { return r[0] + r[1] + r[2]; }
};
__host__ __device__ inline PoolRows pool_rows(int cx, int hx, int cy, int hy, const bool* on) {
    const long long f = on[0] ? (long long)cx * hy : 0, g = on[1] ? (long long)cy * hx : 0;
    return PoolRows{{f > g ? f : g, on[2] ? (long long)cx * hx : 0, on[3] ? (long long)cy * hy : 0}};
}

// First rows of n problems that need `rows` each, in problem order, each that still fits `room`;
// -1: no place, the problem sweeps directly (and takes none from those after it).
__host__ __device__ inline void pool_places(const long long* rows, int n, long long room,
                                            long long* at) {
    long long used = 0;
    for (int b = 0; b < n; ++b) {
        const bool fits = rows[b] <= room - used;
        at[b] = fits ? used : -1;
        used += fits ? rows[b] : 0;
    }
}

}  // namespace ct
