// Cell form of the Stein sum in 2-D (stein.hip): shared declarations.
#pragma once

#include "ct_internal.h"

namespace ct {

// Points from which the form is tried: below it the direct sum's rounding error is smaller (2048
// samples' flow against float64, four point sets: 24576 points 1.1 to 1.7e-7 against 1.1 to
// 2.3e-7, 32768 points 1.0 to 2.0e-7 against 1.4 to 4.0e-7), and the time is close (a call with a
// given bandwidth: 16384 points 115 us against 94, 24576 126 / 183, 32768 133 / 294, 65536
// 163 / 1076).
constexpr int kSteinCellMinT = 32768;
constexpr int kSteinCellMaxT = 92681;           // up to here the median's buffers hold the moments
constexpr int kSteinBits = 5;                    // cells per axis: at most 2^bits
constexpr int kSteinIds = 1 << (2 * kSteinBits);
constexpr int kSteinCells = 256;                 // most non-empty cells
constexpr int kSteinTerms = 64;                  // products of 8 x 8 functions
constexpr int kSteinMom = 3 * kSteinTerms;       // floats of a (query cell, key cell) pair
constexpr float kSteinSide = 1.3125f;            // of a cell, scaled: few mantissa bits (see stein.hip)
constexpr int kSteinBoxes = 64;                  // blocks of the bounding box
constexpr int kSteinTile = 64;                   // queries of a tile (one wave)

struct SteinCells {
    int n, nb, per;        // points, blocks of `per` points in the counting sort
    int kc;                // most keys of a chunk
    int chmax, tmax;       // room for chunks and tiles
    unsigned* box;         // [5][kSteinBoxes] blocks' ordered-integer minima, maxima, unusable points
    unsigned short* id;    // [n]
    unsigned* bh;          // [nb][ids] counts, then places
    unsigned* first;       // [ids]
    int* perm;             // [n] sorted place -> point
    float4* rec;           // [n] (x', score) in cell order
    float4* cen;           // [cells] centres (x, y)
    int4* chunk;           // [chmax] (first key, end, cell, 0)
    int4* tile;            // [tmax]
    int2* own;             // [cells] the cell's chunks (first, end)
    int* cnt;              // cells, chunks, tiles, mode (1: cell form, 0: direct sum)
    float* mom;            // [cells][cells][192] moments of (query cell, key cell), then
                           // [chunks][cells][192] those of a chunk for every query cell
    long long room;        // floats of mom: more cells or chunks than fit sum directly
};

// Times of both forms in us, fitted at 65536 points (direct 1085, values 27.4 and moments 33.4
// with 60 cells): a spread of points over very many cells stays direct.
struct SteinTimes {
    float cell, direct;
};
__host__ __device__ inline SteinTimes stein_times(int n, int cells, int chunks, int tiles) {
    return SteinTimes{4.6e-4f * (float)tiles * (float)cells +
                          2.5e-4f * (float)(n + 128 * chunks) * (float)((cells + 31) / 32) + 50.f,
                      2.5e-7f * (float)n * (float)n};
}
// Whether a flow is offered the form; the points then decide on the device.  The median
// bandwidth gives them some ten cells per axis; for a given bandwidth h the host takes points that
// spread over a unit box, the domain of the library: where those have too many cells, the
// partition would be made in vain (h = 1e-4: 32768 points 319 us against 284 direct, 65536 points
// 1013 against 976).
bool stein_cells_offered(int T, float h);
// Lays out the arrays after a flow's own (a no-op for sizes that the form does not take).
bool stein_cells_for(int T, int d);
// spare: a buffer of the median, no longer used when the sum runs: it holds the moments.
void stein_cells_layout(Arena& a, SteinCells& S, int T, float* spare, size_t spare_floats);
// Partition, moments and values; with mode 1 the flow phi[T][2] is written, else nothing.
// qc, krec, h: of the staged points (krec = (x', score)).
hipError_t launch_stein_cells(const SteinCells& S, const float4* krec, const float* h, float* phi,
                              float* h_used, hipStream_t s);

}  // namespace ct
