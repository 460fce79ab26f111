// Cell form of the soft-min sweep: shared declarations and device code.
//
// A sweep is  out_i = -(1/kappa) log2 sum_j 2^(h_j - |x'_i - y'_j|^2)  over scaled
// points.  Both point sets are split into the cells of a grid of side w.  With
// x'_i = A + s (A the centre of the query's cell), y'_j = C + u and d = A - C,
//     h_j - |x'_i - y'_j|^2 = (h_j - |u|^2 + 2 d.u) + (-|d|^2 - 2 d.s - |s|^2) + 2 s.u,
// so a pair couples the two points only through 2^(2 s.u), and inside a pair of cells
// |2 s_t u_t| is bounded.  In natural units, on [-1, 1]^2 per axis, that factor is
// e^(lambda s u) with lambda = ln2 w^2 / 2, and
//     e^(lambda s u) = I_0(lambda s) + 2 sum_n I_n(lambda s) T_n(u)
// (T_n Chebyshev polynomials, I_n modified Bessel functions).  The products over the
// axes with the largest coefficients, 64 of them in 2-D at lambda = 1 and 192 in 3-D at
// lambda = 0.46, leave out terms that add up to less than 9e-8, whatever the points: of the
// factor, which is smallest at opposite corners of the cells, at most 1.4e-7 (2.2e-8 in 3-D),
// about the rounding of float32.  A sweep becomes
//     moments   M[a][c][n] = sum_{j in c} 2^(h_j - |u_j|^2 + 2 d.u_j - mu_ac) T_n(u_j)
//     values    sum_c 2^(mu_ac - |d|^2 - 2 d.s_i - |s_i|^2 - sh_i) sum_n phi_n(s_i) M[a][c][n]
// for every pair (a, c) of query and key cell, two matrix products of float32 in the
// matrix cores (v_mfma_f32_32x32x2), with mu_ac the largest exponent of the cell's keys, so
// that nothing leaves float32's range however far apart the cells are and however much
// the potentials vary.  Per point and cell it costs 64 (192) multiply-adds; per point
// pair the direct sweep costs 5 (6) instructions, one of them an exponential.  Measured on
// an MI355X, d = 2, T = 65536, M = 262144, eps = 0.002, 200 iterations: 1142 ms with direct
// sweeps (94 % of their issue roof), 83 to 84 ms in this form; T = 4096, M = 16384, eps = 0.005,
// 200 iterations: 16.0 against 8.7 to 9.4 ms, by the points' spread.
#pragma once

#include "ct_internal.h"

namespace ct {

template <int D>
struct CellDim;
template <>
struct CellDim<2> {
    static constexpr int N = 64;     // products kept
    static constexpr int F = 9;      // one-dimensional functions n = 0..8
    static constexpr int bits = 5;   // cells per axis: at most 2^bits
    static constexpr double side = 435.0 / 256;
    static constexpr double lambda = 1.00067730;
};
template <>
struct CellDim<3> {
    static constexpr int N = 192;
    static constexpr int F = 8;
    static constexpr int bits = 4;
    static constexpr double side = 295.0 / 256;
    static constexpr double lambda = 0.46021373;
};
template <int D>
constexpr bool lambda_is_of_side() {
    const double e = CellDim<D>::lambda - 0.34657359027997264 * CellDim<D>::side * CellDim<D>::side;
    return e < 1e-7 && e > -1e-7;
}
static_assert(lambda_is_of_side<2>() && lambda_is_of_side<3>(), "lambda = ln2 w^2 / 2");
constexpr int kCellIds = 4096;       // most cell codes of either dimension (1024 in 2-D)
constexpr int kCellTile = 32;        // queries per evaluation tile, cells per moment tile
constexpr int kCellChunkMax = 1024;  // most keys of one chunk

// One point set's partition, in the workspace.
struct CellSide {
    int off, n;            // the set's first point in the caller's array, points
    int nb, per;           // blocks of `per` points in the counting sort
    int kc;                // most keys of a chunk
    int cmax, chmax, tmax; // room for cells, chunks and tiles
    unsigned* box;         // [8] ordered-integer minima and maxima, [6] unusable points
    unsigned short* id;    // [n] cell code
    unsigned* bh;          // [nb][ids] counts, then offsets within the code
    unsigned* first;       // [ids] first sorted place of the code
    int* perm;             // [n] sorted place -> caller's index
    float4* cen;           // [cmax] cell centres (scaled coordinates)
    int4* chunk;           // [chmax] (first key, end, cell, 0)
    float4* chcen;         // [chmax] centre of the chunk's cell
    int4* tile;            // [tmax] (first query, end, cell, 0)
    float4* phi;           // [tmax][N / 8][64] a tile's functions: products 4 i.. (lanes < 32: of
                           // the first half of the products) of query lane % 32
    int* cnt;              // [4] cells, chunks, tiles, 1: does not fit
};

struct CellPrep {
    CellSide side[2];      // x, y
    const float* origin;   // [3] subtracted before scaling
    int d, ids, bits;
    float cell;            // side of a cell, scaled
    size_t mom_cap[3];     // room for moments: cross, x-x, y-y (floats)
    int* mode;             // out: [5] of the f, g, p, q sweeps: 1 the cell form pays and fits,
                           // 0 the direct sweep; then 0
    float *xs, *ys, *ws;   // out: points and weights in cell order
    float* pot_s;          // out: the starting potentials in cell order (when given)
};

// What a call passes to the partition beside it.
struct CellInputs {
    const float *x, *y;    // caller's points
    const float* w;        // caller's reference weights or null
    const float* pot;      // [2T+2M] starting potentials or null (one problem only)
    float sqrt_kappa;
};

// A soft-min job in the cell form, beside its direct form (Job).
struct CellJob {
    const int* mode;       // 1: cell form
    const int* ncq;        // query cells (device)
    const float4* qcen;
    const int4* tile;      // query tiles
    const int* ntile;
    const float4* phi;
    int tmax;              // room of the tile array
    const int* nch;        // key chunks
    const int4* chunk;
    const float4* chcen;
    float* mom;            // [ncq][nch][N]
    float* mu;             // [ncq][nch]  mu_ac - |d|^2
};

struct CellLaunch {
    CellJob job[2];
    const int* never;      // a zero mode
    int R, WS;             // the direct sweep's schedule
    float inv_cell;        // 1 / w
};

// Side w of a cell in scaled coordinates.
inline double cell_side(int d) { return d == 2 ? CellDim<2>::side : CellDim<3>::side; }

// What a sweep's time in the cell form depends on, of one point set.
struct CellCounts {
    double n, cells, chunks, tiles;
};
// Times of one sweep in us from a model of both forms in clocks of one compute unit, fitted to
// launches of 4096 to 262144 points (d = 2: T = 4096, M = 16384, f: 18 us measured, 16 modelled,
// direct 20 and 19; T = 65536, M = 262144, g: 166 and 150, direct 2290 and 2900; d = 3, M =
// 65521: the q sweep 450 and 446, direct 800 and 884).
//   moments  the keys' products for 32 query cells at a time at 73 % of the matrix cores'
//            128 multiply-adds per clock, and a fixed part per (chunk, 32 cells)
//   values   twice the products' clocks, and a fixed part per tile
//   direct   the pairs' instructions at 75 % of their issue rate
struct CellTimes {
    double cell, direct;
};
__host__ __device__ inline CellTimes cell_times(const CellCounts& q, const CellCounts& k, int d) {
    const double N = d == 2 ? CellDim<2>::N : CellDim<3>::N;
    const double pair = d == 2 ? 2.0 / 128 + 2.0 / 64 + 1.0 / 32 : 2.0 / 128 + 3.0 / 64 + 1.0 / 32;
    const double at = ceil(q.cells / kCellTile), ct = ceil(k.chunks / kCellTile);
    const double moments = at * (kCellTile * N / 128.0 / 0.73 * k.n + (d == 2 ? 9e3 : 18e3) * k.chunks);
    const double values = q.tiles * (ct * 2.0 * kCellTile * kCellTile * N / 128.0 + 1e3);
    const double direct = q.n * k.n * pair / 0.75;
    const double per_us = 256.0 * 2400.0;
    return CellTimes{(moments + values) / per_us, direct / per_us};
}
// A sweep's launches in us (a batch shares them), and the modelled gain below which the device
// leaves a sweep direct in a single problem; a batch's launch is slower the more of its jobs are
// direct (their units wait behind the moments, three blocks to a compute unit), so there the
// form is taken unless the model puts it at twice the direct time (24 ragged problems of other
// seeds than the timed case's, 150 iterations: 0.9 53.2 ms, 1.2 50.8, 1.6 46.0, 2.5 45.9, 4 45.1).
constexpr double kCellLaunch = 8.0;
constexpr double kGain = 0.9, kBatchGain = 2.0;
__host__ __device__ inline bool cell_gains(const CellTimes& t, double launch, double gain) {
    return t.cell + 0.6 * launch < gain * (t.direct + launch);
}
// Sizes of a problem's partition and its arrays from the arena (all but the function tables,
// the sorted inputs and the moments).
void cell_prep_layout(Arena& a, CellPrep& P, int d, int T, int M, int xo, int yo, int kcx, int kcy);
// Mean points of a cell below which the form cannot pay: bounds the room for cells.
constexpr int kCellMinPoints = 24;
// Largest number of keys in a chunk for a set of n points.
int cell_chunk(int n);

hipError_t launch_cell_prep(const CellPrep& P, const CellInputs& in, hipStream_t s);
// Calls too small for the cell form; the environment variable CT_CELL_MIN_PAIRS (a test and
// tuning hook) replaces `pairs` and `pairs3` and drops `work` and CellOffer's question.
constexpr int kCellMinIters = 8;
constexpr int kCellMaxPoints = 1 << 22;
struct CellLimits {
    // Pairs of one iteration below which the two forms' launches take the same time (150
    // iterations: 4.7e7 pairs 5.4 against 5.0 ms, 1.04e8 pairs 5.0 against 5.7).
    double pairs = 1e8;
    // Pairs of all iterations below which splitting the points (0.1 ms) costs more than it
    // saves: 40 iterations at T = 3174, M = 12915 (3.7e9 pairs) 1.69 against 1.54 ms.
    double work = 1e10;
    // Pairs of a 3-D sweep below which it stays direct, from whole calls at eps = 0.01 (40
    // iterations at T = 16355, M = 22674 lose 2 %, at T = 10246, M = 35898 win 26 %).  The points
    // per cell would be the truer rule; the model that knows them is fitted to larger sweeps.
    double pairs3 = 1.2e9;
    bool expect = true;   // ask CellOffer
};
CellLimits cell_limits();
bool cell_candidate(int d, int nq, int nk);

// Whether a call is offered the form at all, before the device sees its points.  A call that is
// offered it and does not take it pays for the partition, for a launch or two more per sweep and,
// in 2-D, for direct sweeps at the registers and LDS of the moments (three blocks to a compute
// unit instead of five or six): 5 to 10 % of a single problem (T = 4096, M = 16384, eps = 0.001,
// 120 iterations: 10.3 ms against 9.7), 18 to 31 % of a batch (16 problems below 4000 x 9000,
// eps = 0.001: 8.3 against 6.8 ms; 300 below 1000 x 1500: 5.7 against 3.9).  The host knows eps
// and the sizes, not the extent, so it takes the library's domain, the unit box: a side of it has
// c = sqrt(log2(e) / eps) / w cells, and points that spread over it lie in about (c + 1/2)^d of
// them (counted on random walks and mixtures: 0.55 to 1.2 of that in 2-D, where 0.8 is taken, 0.2
// to 1.1 in 3-D, where 0.3 is taken, since the form's launches there leave direct sweeps at
// their own speed: 0 to 2 %).  The same model as on the device then says whether the form is
// likely to pay.  Of 105 calls around the crossover (single problems of 2500 x 10000 to 20000 x
// 20000 points and batches of 4 to 300, eps 0.0001 to 0.1) none that it offers the form is slower than
// its direct sweeps, and those that it refuses could have gained 7 % at most.
class CellOffer {
public:
    // d, eps of a call; launch, gain: as for the device's choice; slow: time of a direct sweep
    // within the form's launches over that of a launch of its own.
    CellOffer(int d, double eps, double launch, double gain, double slow);
    CellCounts expect(int n, int chunk_keys, bool* fits) const;
    void sweep(int nq, int nk, int chunk_q, int chunk_k);   // one more sweep of every iteration
    // prep_us: the partition.
    bool pays(int iters, double prep_us) const;

private:
    int d_;
    double side_cells_, launch_, gain_, slow_, form_ = 0.0, direct_ = 0.0;
    bool any_ = false;
};
// One sweep of one or two jobs (nblocks direct work units): moments then values, or the
// direct sweep then its merge.
hipError_t launch_cell_sweep(int d, const Schedule& sc, bool lagged, const Launch& L,
                             const CellLaunch& C, int nblocks, hipStream_t s);

// The batched path: the same over tables in device memory.  Kind k of the lockstep
// launches has njobs jobs; every job of the direct table has a cell job beside it.
constexpr int kCellBatchJobs = 1024;   // most jobs of a launch (their prefix sums sit in LDS)
struct CellBatch {
    CellPrep* prep;        // [B]
    CellJob* jobs;         // [kinds][3B]
    int* uend;             // [kinds][2][3B] ends of the jobs' units: moments, values
    int* info;             // [kinds] 1: some job takes the direct sweep
    int* njobs;            // [kinds]
    float* mom;            // pool of moments and of their exponents
    float* mu;
    long long rows;        // (query cell, chunk) pairs that the pool holds
    int B, kinds, stride;  // stride = 3B
    int self_x, self_y;    // 1: the batch has sweeps of x (y) against itself
};
// Partitions of every problem, then the jobs' modes, places in the pool and units.
hipError_t launch_cell_prep_batch(int d, const CellBatch& C, const CellInputs& in, int max_n,
                                  int max_nb, hipStream_t s);
// One lockstep launch of kind k: the cell form's jobs and the direct ones of L.
hipError_t launch_cell_tab(int d, const Schedule& sc, bool lagged, const TabLaunch& L,
                           const CellBatch& C, int k, hipStream_t s);
}  // namespace ct
