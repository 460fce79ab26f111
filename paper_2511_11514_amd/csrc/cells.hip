// Kernels of the cell form of the soft-min sweep (see cells.h): the partition of a
// point set into cells, the moments of the keys, the values at the queries.
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>

#include "cell_pool.h"
#include "cells.h"
#include "sweep_device.h"

namespace ct {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// Kept products, by decreasing coefficient: one hexadecimal digit per axis (x lowest), the
// order of that axis's function.
__device__ constexpr unsigned short kTerms2[CellDim<2>::N] = {
    0x00, 0x10, 0x01, 0x11, 0x20, 0x02, 0x21, 0x12, 0x22, 0x30, 0x03, 0x31, 0x13, 0x32, 0x23, 0x40,
    0x04, 0x41, 0x14, 0x33, 0x42, 0x24, 0x50, 0x05, 0x51, 0x15, 0x43, 0x34, 0x52, 0x25, 0x60, 0x06,
    0x61, 0x16, 0x44, 0x53, 0x35, 0x62, 0x26, 0x70, 0x07, 0x71, 0x17, 0x54, 0x45, 0x63, 0x36, 0x72,
    0x27, 0x55, 0x80, 0x08, 0x64, 0x46, 0x81, 0x18, 0x73, 0x37, 0x82, 0x28, 0x65, 0x56, 0x74, 0x47,
};
__device__ constexpr unsigned short kTerms3[CellDim<3>::N] = {
    0x000, 0x010, 0x001, 0x100, 0x110, 0x101, 0x011, 0x111, 0x020, 0x002, 0x200, 0x210,
    0x120, 0x201, 0x021, 0x102, 0x012, 0x211, 0x121, 0x112, 0x300, 0x030, 0x003, 0x022,
    0x220, 0x202, 0x310, 0x130, 0x301, 0x031, 0x103, 0x013, 0x221, 0x212, 0x122, 0x311,
    0x131, 0x113, 0x400, 0x040, 0x004, 0x320, 0x230, 0x302, 0x032, 0x203, 0x023, 0x222,
    0x410, 0x401, 0x140, 0x041, 0x104, 0x014, 0x321, 0x231, 0x312, 0x132, 0x213, 0x123,
    0x411, 0x141, 0x114, 0x033, 0x330, 0x303, 0x420, 0x402, 0x042, 0x024, 0x240, 0x204,
    0x050, 0x005, 0x500, 0x322, 0x232, 0x223, 0x133, 0x331, 0x313, 0x421, 0x412, 0x142,
    0x124, 0x241, 0x214, 0x051, 0x015, 0x510, 0x150, 0x501, 0x105, 0x511, 0x151, 0x115,
    0x430, 0x340, 0x403, 0x043, 0x304, 0x034, 0x233, 0x332, 0x323, 0x422, 0x242, 0x224,
    0x520, 0x502, 0x052, 0x025, 0x250, 0x205, 0x060, 0x006, 0x600, 0x431, 0x341, 0x413,
    0x143, 0x314, 0x134, 0x521, 0x251, 0x512, 0x152, 0x215, 0x125, 0x160, 0x106, 0x610,
    0x601, 0x061, 0x016, 0x611, 0x161, 0x116, 0x333, 0x440, 0x404, 0x044, 0x432, 0x342,
    0x423, 0x243, 0x324, 0x234, 0x530, 0x350, 0x503, 0x053, 0x305, 0x035, 0x522, 0x252,
    0x225, 0x441, 0x414, 0x144, 0x620, 0x260, 0x602, 0x062, 0x206, 0x026, 0x531, 0x351,
    0x513, 0x153, 0x315, 0x135, 0x700, 0x070, 0x007, 0x621, 0x261, 0x612, 0x162, 0x216,
    0x126, 0x710, 0x170, 0x701, 0x071, 0x107, 0x017, 0x433, 0x343, 0x334, 0x711, 0x171,
};
template <int D>
__device__ __forceinline__ constexpr int term(int i, int axis) {
    return ((D == 2 ? kTerms2[i] : kTerms3[i]) >> (4 * axis)) & 15;
}

// ------------------------------------------------------------------ partition

// Floats as unsigned integers in the same order.
__device__ __forceinline__ unsigned ordered(float v) {
    const unsigned u = __float_as_uint(v);
    return (u & 0x80000000u) ? ~u : u | 0x80000000u;
}
__device__ __forceinline__ float from_ordered(unsigned u) {
    return __uint_as_float((u & 0x80000000u) ? u & 0x7fffffffu : ~u);
}

// Lower corner of the grid: a multiple of 1/128 at or below the smallest coordinate.  The sides of
// cells have few mantissa bits too, so that centres, their differences and a point's offset from
// its centre are exact: their rounding is common to all keys of a pair of cells (gradient's error
// against float64 over that of the direct sweeps, single problems, eps = 0.002 / 0.005 / 0.01 /
// 0.02: 1.03 / 0.99 / 1.06 / 1.01 with rounded differences, 0.95 / 0.97 / 1.04 / 0.99 with exact ones).
__device__ __forceinline__ float corner(unsigned u) {
    return floorf(from_ordered(u) * 128.f) * (1.f / 128.f);
}

// The partition kernels take one problem by value, or (TAB) blockIdx.z's of a table.
template <bool TAB>
__global__ __launch_bounds__(64) void k_cell_init(CellPrep one, const CellPrep* tab) {
    const CellPrep& P = TAB ? tab[blockIdx.z] : one;
    const int i = (int)threadIdx.x;
    if (i < 16) {
        const CellSide& S = P.side[i >> 3];
        S.box[i & 7] = (i & 7) < 3 ? 0xffffffffu : 0u;
    }
}

// Bounding box of the scaled points (minima and maxima do not depend on the order of the
// atomics), and the number of points that no cell can take: non-finite coordinates, or
// weights that are not positive and finite.
template <bool TAB>
__global__ __launch_bounds__(256) void k_cell_box(CellPrep one, const CellPrep* tab, CellInputs in) {
    const CellPrep& P = TAB ? tab[blockIdx.z] : one;
    const CellSide& S = P.side[blockIdx.y];
    const float* pts = (blockIdx.y ? in.y : in.x) + (size_t)S.off * P.d;
    const int d = P.d;
    unsigned lo[3] = {0xffffffffu, 0xffffffffu, 0xffffffffu}, hi[3] = {0u, 0u, 0u}, bad = 0u;
    for (int i = (int)(blockIdx.x * 256 + threadIdx.x); i < S.n; i += (int)gridDim.x * 256) {
        bool ok = true;
        for (int t = 0; t < d; ++t) {
            const float c = (pts[(size_t)i * d + t] - P.origin[t]) * in.sqrt_kappa;
            ok = ok && isfinite(c);
            if (isfinite(c)) {
                lo[t] = min(lo[t], ordered(c));
                hi[t] = max(hi[t], ordered(c));
            }
        }
        if (blockIdx.y == 1 && in.w) {
            const float w = in.w[S.off + i];
            ok = ok && w > 0.f && isfinite(w);
        }
        bad += ok ? 0u : 1u;
    }
    for (int m = 1; m < 64; m <<= 1) {
        for (int t = 0; t < 3; ++t) {
            lo[t] = min(lo[t], __shfl_xor(lo[t], m));
            hi[t] = max(hi[t], __shfl_xor(hi[t], m));
        }
        bad += __shfl_xor(bad, m);
    }
    if ((threadIdx.x & 63) == 0) {
        for (int t = 0; t < d; ++t) {
            atomicMin(&S.box[t], lo[t]);
            atomicMax(&S.box[3 + t], hi[t]);
        }
        if (bad) atomicAdd(&S.box[6], bad);
    }
}

// Cell code of a point: its cell's coordinates, bits interleaved, so that cells of
// neighbouring codes are neighbours.  Points outside the coded box take its border cells
// (the partition is then marked as not fitting, see k_cell_lists).
__device__ __forceinline__ int cell_code(const float* c, const float* lo, float inv, int d,
                                         int bits) {
    int code = 0;
    for (int t = 0; t < d; ++t) {
        const float v = (c[t] - lo[t]) * inv;
        int k = v > 0.f ? (int)fminf(v, 65535.f) : 0;   // NaN: 0
        k = min(k, (1 << bits) - 1);
        for (int b = 0; b < bits; ++b) code |= ((k >> b) & 1) << (b * d + t);
    }
    return code;
}

// Counts per block of `per` points and code.
template <bool TAB>
__global__ __launch_bounds__(256) void k_cell_hist(CellPrep one, const CellPrep* tab, CellInputs in) {
    __shared__ unsigned h[kCellIds];
    const CellPrep& P = TAB ? tab[blockIdx.z] : one;
    const CellSide& S = P.side[blockIdx.y];
    const float* pts = (blockIdx.y ? in.y : in.x) + (size_t)S.off * P.d;
    const int b = (int)blockIdx.x;
    if (b >= S.nb) return;
    for (int i = (int)threadIdx.x; i < P.ids; i += 256) h[i] = 0u;
    __syncthreads();
    float lo[3];
    for (int t = 0; t < 3; ++t) lo[t] = corner(S.box[t]);
    const int i1 = min(S.n, (b + 1) * S.per);
    for (int i = b * S.per + (int)threadIdx.x; i < i1; i += 256) {
        float c[3];
        for (int t = 0; t < P.d; ++t)
            c[t] = (pts[(size_t)i * P.d + t] - P.origin[t]) * in.sqrt_kappa;
        const int id = cell_code(c, lo, 1.f / P.cell, P.d, P.bits);
        S.id[i] = (unsigned short)id;
        atomicAdd(&h[id], 1u);
    }
    __syncthreads();
    for (int i = (int)threadIdx.x; i < P.ids; i += 256) S.bh[(size_t)b * P.ids + i] = h[i];
}

// Per code: exclusive sums of its counts over the blocks, and its total.  The four waves of a
// block take a quarter of the blocks each for 64 codes: first their sums, then the places.
template <bool TAB>
__global__ __launch_bounds__(256) void k_cell_scan(CellPrep one, const CellPrep* tab) {
    __shared__ unsigned part[4][64];
    const CellPrep& P = TAB ? tab[blockIdx.z] : one;
    const CellSide& S = P.side[blockIdx.y];
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    const int id = (int)blockIdx.x * 64 + lane;
    const int per = (S.nb + 3) / 4, b0 = min(S.nb, wave * per), b1 = min(S.nb, b0 + per);
    unsigned sum = 0u;
#pragma unroll 8
    for (int b = b0; b < b1; ++b) sum += S.bh[(size_t)b * P.ids + id];
    part[wave][lane] = sum;
    __syncthreads();
    unsigned run = 0u;
    for (int w = 0; w < wave; ++w) run += part[w][lane];
#pragma unroll 8
    for (int b = b0; b < b1; ++b) {
        const size_t at = (size_t)b * P.ids + id;
        const unsigned v = S.bh[at];
        S.bh[at] = run;
        run += v;
    }
    if (wave == 3) S.first[id] = run;   // the total; k_cell_lists turns it into the first place
}

// Inclusive block scan of one int per thread (1024 threads); returns the exclusive sum
// and the total.
__device__ __forceinline__ int block_scan(int v, int* sh, int* total) {
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    int s = v;
    for (int m = 1; m < 64; m <<= 1) {
        const int o = __shfl_up(s, m);
        if (lane >= m) s += o;
    }
    __syncthreads();
    if (lane == 63) sh[wave] = s;
    __syncthreads();
    int before = 0, all = 0;
    for (int w = 0; w < 16; ++w) {
        if (w < wave) before += sh[w];
        all += sh[w];
    }
    *total = all;
    return before + s - v;
}

// Sorted places, the non-empty cells, their chunks of at most kc keys and their tiles of
// 32 queries (one block per side; four codes per thread count, all threads write the lists).
template <bool TAB>
__global__ __launch_bounds__(1024) void k_cell_lists(CellPrep one, const CellPrep* tab) {
    __shared__ int sh[16];
    __shared__ int at0[kCellIds + 1], ih0[kCellIds], it0[kCellIds];   // per non-empty cell
    const CellPrep& P = TAB ? tab[blockIdx.z] : one;
    const CellSide& S = P.side[blockIdx.x];
    constexpr int per = kCellIds / 1024;
    int n[per], pts = 0, cells = 0, chunks = 0, tiles = 0;
    for (int k = 0; k < per; ++k) {
        const int id = (int)threadIdx.x * per + k;
        n[k] = id < P.ids ? (int)S.first[id] : 0;
        pts += n[k];
        cells += n[k] > 0;
        chunks += (n[k] + S.kc - 1) / S.kc;
        tiles += (n[k] + kCellTile - 1) / kCellTile;
    }
    int tp, tc, th, tt;
    int at = block_scan(pts, sh, &tp);
    int ic = block_scan(cells, sh, &tc);
    int ih = block_scan(chunks, sh, &th);
    int it = block_scan(tiles, sh, &tt);
    bool fits = tc <= S.cmax && th <= S.chmax && tt <= S.tmax && S.box[6] == 0u;
    float lo[3] = {0.f, 0.f, 0.f};
    for (int t = 0; t < P.d; ++t) {
        lo[t] = corner(S.box[t]);
        // every point in the cell of its code
        fits = fits && (from_ordered(S.box[3 + t]) - lo[t]) <= P.cell * (float)(1 << P.bits);
    }
    if (threadIdx.x == 0) {
        S.cnt[0] = tc;
        S.cnt[1] = th;
        S.cnt[2] = tt;
        S.cnt[3] = fits ? 0 : 1;
    }
    for (int k = 0; k < per; ++k) {
        const int id = (int)threadIdx.x * per + k;
        if (id >= P.ids) break;
        S.first[id] = (unsigned)at;
        if (n[k] > 0) {
            at0[ic] = at;
            ih0[ic] = ih;
            it0[ic] = it;
            if (fits) {
                float c[3] = {0.f, 0.f, 0.f};
                for (int t = 0; t < P.d; ++t) {
                    int g = 0;
                    for (int b = 0; b < P.bits; ++b) g |= ((id >> (b * P.d + t)) & 1) << b;
                    c[t] = lo[t] + ((float)g + 0.5f) * P.cell;
                }
                S.cen[ic] = make_float4(c[0], c[1], c[2], 0.f);
            }
            ++ic;
            ih += (n[k] + S.kc - 1) / S.kc;
            it += (n[k] + kCellTile - 1) / kCellTile;
        }
        at += n[k];
    }
    if (threadIdx.x == 0) at0[tc] = tp;
    if (!fits) return;   // the same in every thread
    __syncthreads();
    // the cell of entry e: the last one whose entries start at or before e
    auto cell_of = [&](const int* first, int e) {
        int a = 0, b = tc - 1;
        while (a < b) {
            const int mid = (a + b + 1) >> 1;
            if (first[mid] <= e) a = mid;
            else b = mid - 1;
        }
        return a;
    };
    for (int e = (int)threadIdx.x; e < th; e += 1024) {
        const int c = cell_of(ih0, e), q = at0[c] + (e - ih0[c]) * S.kc;
        S.chunk[e] = make_int4(q, min(at0[c + 1], q + S.kc), c, 0);
        S.chcen[e] = S.cen[c];
    }
    for (int e = (int)threadIdx.x; e < tt; e += 1024) {
        const int c = cell_of(it0, e), q = at0[c] + (e - it0[c]) * kCellTile;
        S.tile[e] = make_int4(q, min(at0[c + 1], q + kCellTile), c, 0);
    }
}

// Stable scatter: one wave per block of points walks them in order, 64 at a time; the
// lanes of one code rank themselves by ballots over the code's bits.
template <bool TAB>
__global__ __launch_bounds__(64) void k_cell_scatter(CellPrep one, const CellPrep* tab) {
    __shared__ unsigned cur[kCellIds];
    const CellPrep& P = TAB ? tab[blockIdx.z] : one;
    const CellSide& S = P.side[blockIdx.y];
    const int b = (int)blockIdx.x, lane = (int)threadIdx.x;
    if (b >= S.nb) return;
    for (int i = lane; i < P.ids; i += 64) cur[i] = S.first[i] + S.bh[(size_t)b * P.ids + i];
    __syncthreads();
    const int i1 = min(S.n, (b + 1) * S.per);
    const int nbit = P.bits * P.d;
    for (int i0 = b * S.per; i0 < i1; i0 += 64) {
        const int i = i0 + lane;
        const bool on = i < i1;
        const int id = on ? (int)S.id[i] : 0;
        unsigned long long same = __ballot(on);
        for (int k = 0; k < nbit; ++k) {
            const unsigned long long m = __ballot((id >> k) & 1);
            same &= ((id >> k) & 1) ? m : ~m;
        }
        const int rank = __popcll(same & ((1ull << lane) - 1ull));
        unsigned base = 0u;
        if (on) base = cur[id];
        __syncthreads();
        if (on) {
            S.perm[base + rank] = i;
            if (rank == 0) cur[id] = base + (unsigned)__popcll(same);
        }
        __syncthreads();
    }
}

// Whether a sweep pays in the cell form (and fits).
__device__ bool cell_pays(const CellSide& q, const CellSide& k, int d, double launch, double gain) {
    if (q.cnt[3] || k.cnt[3]) return false;
    const CellCounts Q{(double)q.n, (double)q.cnt[0], (double)q.cnt[1], (double)q.cnt[2]};
    const CellCounts K{(double)k.n, (double)k.cnt[0], (double)k.cnt[1], (double)k.cnt[2]};
    return cell_gains(cell_times(Q, K, d), launch, gain);
}

// Points, weights and starting potentials in cell order.
template <bool TAB>
__global__ __launch_bounds__(256) void k_cell_gather(CellPrep one, const CellPrep* tab,
                                                     CellInputs in) {
    const CellPrep& P = TAB ? tab[blockIdx.z] : one;
    const CellSide& X = P.side[0];
    const CellSide& Y = P.side[1];
    const int d = P.d;
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    if (!TAB && i == 0) {
        const size_t N = d == 2 ? CellDim<2>::N : CellDim<3>::N;
        const CellSide* q[4] = {&X, &Y, &X, &Y};
        const CellSide* k[4] = {&Y, &X, &X, &Y};
        for (int j = 0; j < 4; ++j) {
            const size_t need = (size_t)q[j]->cnt[0] * k[j]->cnt[1] * N;
            P.mode[j] = need <= P.mom_cap[j < 2 ? 0 : j - 1] && cell_pays(*q[j], *k[j], d, kCellLaunch, kGain) ? 1 : 0;
        }
        P.mode[4] = 0;
    }
    if (i < X.n) {
        const int s = X.perm[i];
        const float* pts = in.x + (size_t)X.off * d;
        for (int t = 0; t < d; ++t) P.xs[(size_t)i * d + t] = pts[(size_t)s * d + t];
        if (in.pot) {
            P.pot_s[i] = in.pot[s];
            P.pot_s[(size_t)X.n + Y.n + i] = in.pot[(size_t)X.n + Y.n + s];
        }
    }
    if (i < Y.n) {
        const int s = Y.perm[i];
        const float* pts = in.y + (size_t)Y.off * d;
        for (int t = 0; t < d; ++t) P.ys[(size_t)i * d + t] = pts[(size_t)s * d + t];
        if (in.w) P.ws[i] = in.w[Y.off + s];
        if (in.pot) {
            P.pot_s[(size_t)X.n + i] = in.pot[(size_t)X.n + s];
            P.pot_s[2 * (size_t)X.n + Y.n + i] = in.pot[2 * (size_t)X.n + Y.n + s];
        }
    }
}

// A batch's modes, places in the pool and units (one block).  A problem's three buffers
// (cross, x-x, y-y) are taken in problem order while they fit; the rest of the batch sweeps
// directly.
__global__ __launch_bounds__(1024) void k_cell_plan(CellBatch C, int d) {
    __shared__ int sh[16];
    const int N = d == 2 ? CellDim<2>::N : CellDim<3>::N;
    __shared__ long long rows[kCellBatchJobs / 3], at[kCellBatchJobs / 3];
    const int b = (int)threadIdx.x;   // the batch's problems are fewer than the threads
    PoolRows mine{{0, 0, 0}};
    bool pays[4] = {false, false, false, false};
    if (b < C.B) {
        const CellSide& X = C.prep[b].side[0];
        const CellSide& Y = C.prep[b].side[1];
        pays[0] = cell_pays(X, Y, d, 0.0, kBatchGain);
        pays[1] = cell_pays(Y, X, d, 0.0, kBatchGain);
        pays[2] = C.self_x && cell_pays(X, X, d, 0.0, kBatchGain);
        pays[3] = C.self_y && cell_pays(Y, Y, d, 0.0, kBatchGain);
        mine = pool_rows(X.cnt[0], X.cnt[1], Y.cnt[0], Y.cnt[1], pays);
        rows[b] = mine.all();
    }
    __syncthreads();
    if (threadIdx.x == 0) pool_places(rows, C.B, C.rows, at);
    __syncthreads();
    if (b < C.B) {
        const bool fits = at[b] >= 0;
        for (int j = 0; j < 4; ++j) C.prep[b].mode[j] = fits && pays[j] ? 1 : 0;
        const long long r[3] = {at[b], at[b] + mine.r[0], at[b] + mine.r[0] + mine.r[1]};
        for (int k = 0; k < C.kinds; ++k) {
            const int per = C.njobs[k] / C.B;
            for (int i = 0; i < per; ++i) {
                CellJob& J = C.jobs[(size_t)k * C.stride + (size_t)b * per + i];
                const int m = (int)(J.mode - C.prep[b].mode);   // 0 f, 1 g, 2 p, 3 q
                const long long row = fits ? r[m < 2 ? 0 : m - 1] : 0;
                J.mom = C.mom + row * N;
                J.mu = C.mu + row;
            }
        }
    }
    __syncthreads();
    __threadfence_block();
    for (int k = 0; k < C.kinds; ++k) {
        int before[2] = {0, 0}, direct = 0;
        for (int j0 = 0; j0 < C.njobs[k]; j0 += 1024) {
            const int j = j0 + (int)threadIdx.x;
            int n[2] = {0, 0}, dir = 0;
            if (j < C.njobs[k]) {
                const CellJob& J = C.jobs[(size_t)k * C.stride + j];
                if (*J.mode) {
                    n[0] = *J.nch * ((*J.ncq + kCellTile - 1) / kCellTile);
                    n[1] = (*J.ntile + 3) / 4;
                } else {
                    dir = 1;
                }
            }
            for (int v = 0; v < 2; ++v) {
                int total;
                const int e = before[v] + block_scan(n[v], sh, &total) + n[v];
                if (j < C.njobs[k]) C.uend[((size_t)k * 2 + v) * C.stride + j] = e;
                before[v] += total;
            }
            int total;
            block_scan(dir, sh, &total);
            direct += total;
        }
        if (threadIdx.x == 0) C.info[k] = direct;
    }
}

// (n ? 2 : 1) I_n(z) for n < F by the ascending series, |z| <= 1 or so.
template <int F>
__device__ __forceinline__ void bessel(float z, float* out, int stride) {
    const float q = 0.25f * z * z;
    float lead = 1.f;   // (z/2)^n / n!
#pragma unroll
    for (int n = 0; n < F; ++n) {
        float s = 1.f;
#pragma unroll
        for (int m = 5; m >= 1; --m) s = __builtin_fmaf(s * (1.f / (float)(m * (n + m))), q, 1.f);
        out[n * stride] = (n ? 2.f : 1.f) * lead * s;
        lead *= 0.5f * z * (1.f / (float)(n + 1));
    }
}

// The functions phi_n(s) of every tile's queries, laid out as the values kernel takes them.
// They depend on the points alone: made once per call, read by every sweep (making them
// in each sweep took as long as a whole tile's matrix products).
template <int D>
__global__ __launch_bounds__(256) void k_cell_functions(CellPrep P, CellInputs in) {
    constexpr int N = CellDim<D>::N, F = CellDim<D>::F, H = N / 2;
    __shared__ float fn[D * F * 33];
    const CellSide& S = P.side[blockIdx.y];
    const float* pts = blockIdx.y ? P.ys : P.xs;
    if (S.cnt[3] || !S.phi) return;   // (null: no sweep of the set takes the form)
    const int nt = S.cnt[2], tid = (int)threadIdx.x, col = tid & 31;
    const float inv = 2.f / P.cell;
    for (int t = (int)blockIdx.x; t < nt; t += (int)gridDim.x) {
        const int4 tl = S.tile[t];
        if ((tid >> 5) < D) {
            const int x = tid >> 5;
            const float4 c = S.cen[tl.z];
            const int q = min(tl.x + col, tl.y - 1);
            const float v = (pts[(size_t)q * D + x] - P.origin[x]) * in.sqrt_kappa;
            const float s = (v - (x == 0 ? c.x : x == 1 ? c.y : c.z)) * inv;   // on [-1, 1]
            bessel<F>((float)CellDim<D>::lambda * s, fn + x * F * 33 + col, 33);
        }
        __syncthreads();
        for (int e = tid; e < H * 16; e += 256) {
            const int lane = e & 63, i = e >> 6;
            float p[4];
            for (int k = 0; k < 4; ++k) {
                const int n = (lane >> 5) * H + 4 * i + k;
                p[k] = 1.f;
                for (int x = 0; x < D; ++x) p[k] *= fn[(x * F + term<D>(n, x)) * 33 + (lane & 31)];
            }
            S.phi[(size_t)t * (H * 16) + e] = make_float4(p[0], p[1], p[2], p[3]);
        }
        __syncthreads();
    }
}

// -------------------------------------------------------------------- moments

template <int D>
struct MomentSmem {
    float4 key[kCellChunkMax];                    // (2u, [..], h - |u|^2), .z (2-D) or .w (3-D)
    float tab[4][D * CellDim<D>::F * 65];         // T_n(u) of 64 keys per wave, rows of 65
    float mu[4][kCellTile];
};

// Moments of chunk `c` for 32 query cells.  The four waves take a quarter of the chunk's
// keys each; an MFMA multiplies the weights of 2 keys for 32 query cells (A: lane = cell,
// half wave = key) with 32 of the keys' products of Chebyshev polynomials (B: lane =
// product), and the waves' sums meet in LDS.
template <int D>
__device__ __forceinline__ void cell_moments(const CellJob& C, const Job& J, int c, int at, int nch,
                                             int ncq, float inv_cell, MomentSmem<D>& sm) {
    constexpr int N = CellDim<D>::N, F = CellDim<D>::F, CT = N / 32;
    const int tid = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, col = lane & 31, half = lane >> 5;
    const int4 ch = C.chunk[c];
    const float4 cc = C.chcen[c];
    const int nk = ch.y - ch.x, nkp = (nk + 7) & ~7;
    for (int i = tid; i < nkp; i += kBlock) {
        float4 k = make_float4(0.f, 0.f, D == 2 ? kNegInf : 0.f, kNegInf);
        if (i < nk) {
            const float4 r = J.krec[ch.x + i];
            const float ux = r.x - cc.x, uy = r.y - cc.y;
            if (D == 2) {
                k = make_float4(2.f * ux, 2.f * uy, r.z - __builtin_fmaf(ux, ux, uy * uy), 0.f);
            } else {
                const float uz = r.z - cc.z;
                k = make_float4(2.f * ux, 2.f * uy, 2.f * uz,
                                r.w - __builtin_fmaf(ux, ux, __builtin_fmaf(uy, uy, uz * uz)));
            }
        }
        sm.key[i] = k;
    }
    const int a = min(at * kCellTile + col, ncq - 1);
    const float4 qc = C.qcen[a];
    const float dx = qc.x - cc.x, dy = qc.y - cc.y, dz = D == 3 ? qc.z - cc.z : 0.f;
    auto expo = [&](const float4& k) {
        if (D == 2) return __builtin_fmaf(dx, k.x, __builtin_fmaf(dy, k.y, k.z));
        return __builtin_fmaf(dx, k.x, __builtin_fmaf(dy, k.y, __builtin_fmaf(dz, k.z, k.w)));
    };
    // products of this lane's columns: rows of the table
    int row[CT][D];
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int x = 0; x < D; ++x) row[t][x] = (x * F + term<D>(t * 32 + col, x)) * 65;
    __syncthreads();
    const int kw = nkp >> 2, kb = wave * kw;   // even, this wave's keys [kb, kb + kw)
    float mx = kNegInf;
    int k1 = 0;
    for (; k1 + 8 <= kw; k1 += 8) {
        float e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = expo(sm.key[kb + k1 + 2 * i + half]);
        mx = fmaxf(mx, fmaxf(fmaxf(e[0], e[1]), fmaxf(e[2], e[3])));
    }
    for (; k1 < kw; k1 += 2) mx = fmaxf(mx, expo(sm.key[kb + k1 + half]));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    if (half == 0) sm.mu[wave][col] = mx;
    __syncthreads();
    float mu = fmaxf(fmaxf(sm.mu[0][col], sm.mu[1][col]), fmaxf(sm.mu[2][col], sm.mu[3][col]));
    const float shift = mu == kNegInf ? 0.f : mu;
    f32x16 acc[CT];
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
    float* tab = sm.tab[wave];
    for (int k0 = 0; k0 < kw; k0 += 64) {
        const int nn = min(64, kw - k0);
        __builtin_amdgcn_wave_barrier();
        if (lane < nn) {
            const float4 k = sm.key[kb + k0 + lane];
#pragma unroll
            for (int x = 0; x < D; ++x) {
                const float u = (x == 0 ? k.x : x == 1 ? k.y : k.z) * inv_cell;   // on [-1, 1]
                float t0 = 1.f, t1 = u;
#pragma unroll
                for (int n = 0; n < F; ++n) {
                    tab[(x * F + n) * 65 + lane] = t0;
                    const float t2 = __builtin_fmaf(2.f * u, t1, -t0);
                    t0 = t1;
                    t1 = t2;
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        auto step = [&](int k, float W) {
#pragma unroll
            for (int t = 0; t < CT; ++t) {
                float b = tab[row[t][0] + k] * tab[row[t][1] + k];
                if (D == 3) b *= tab[row[t][D - 1] + k];
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(W, b, acc[t], 0, 0, 0);
            }
        };
        // four steps' LDS reads in flight together
        int p = 0;
        for (; p + 8 <= nn; p += 8) {
            float W[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) W[i] = ex2(expo(sm.key[kb + k0 + p + 2 * i + half]) - shift);
#pragma unroll
            for (int i = 0; i < 4; ++i) step(p + 2 * i + half, W[i]);
        }
        for (; p < nn; p += 2) step(p + half, ex2(expo(sm.key[kb + k0 + p + half]) - shift));
    }
    // the four waves' sums, 32 products at a time (4 KB per wave in the keys' place)
    float* red = reinterpret_cast<float*>(sm.key);
    static_assert(sizeof(sm.key) >= 4 * 1024 * sizeof(float), "room for four waves' tiles");
#pragma unroll
    for (int t = 0; t < CT; ++t) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r)
            red[wave * 1024 + (8 * (r >> 2) + 4 * half + (r & 3)) * 32 + col] = acc[t][r];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = i * 256 + tid, aa = at * kCellTile + (e >> 5);
            const float v = (red[e] + red[1024 + e]) + (red[2048 + e] + red[3072 + e]);
            if (aa < ncq) C.mom[((size_t)aa * nch + c) * N + t * 32 + (e & 31)] = v;
        }
    }
    if (wave == 0 && half == 0 && at * kCellTile + col < ncq)
        C.mu[(size_t)a * nch + c] =
            mu - __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz));
    __syncthreads();
}

// --------------------------------------------------------------------- values

template <int D, bool PHI>
struct ValueSmem {
    float fn[PHI ? 1 : 4][PHI ? 1 : D * CellDim<D>::F * 33];   // per wave: phi_n per axis
    float4 cd[4][kCellTile];            // per wave: (-2d, mu - |d|^2) of 32 chunks
    float red[4][kCellTile];
    int flist[4 * kCellTile];
    int nflag;
};

// Values of tiles of 32 queries: WS waves of a block share a tile (each takes every WS-th
// tile of 32 chunks), 4 / WS tiles per block.  An MFMA multiplies the chunks' moments (A:
// lane = chunk) with the queries' functions (B: lane = query), so that a lane holds 16
// chunks' sums of its own query.  The functions come from the table, or (PHI false: many
// problems, whose tables would take gigabytes) are made here, about a tenth of a tile's work.
template <int D, bool LAGGED, int WS, bool PHI>
__device__ __forceinline__ void cell_values(const CellJob& C, const Job& J, int u, int nt, int nch,
                                            float inv_cell, float kappa, float inv_kappa,
                                            float inv_sqrt_kappa, ValueSmem<D, PHI>& sm) {
    constexpr int N = CellDim<D>::N, F = CellDim<D>::F, H = N / 2;
    static_assert(PHI || WS == 1, "the functions are made by the wave that owns the tile");
    const int tid = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, col = lane & 31, half = lane >> 5;
    const int part = wave % WS, ti = min(u * (4 / WS) + wave / WS, C.tmax - 1);
    const int4 t0 = C.tile[ti];   // in its array whatever nt is, so the load need not wait for it
    const bool on = ti < nt;
    const int4 tl = on ? t0 : make_int4(0, 1, 0, 0);
    const int ntc = on ? (nch + kCellTile - 1) / kCellTile : 0;
    // 4 V products of a chunk's moments per step, read one step ahead
    constexpr int V = D == 2 ? 8 : 4, G = H / (4 * V);
    auto load = [&](int ct, int g, float4 (&A)[V]) {
        const int c = min(ct * kCellTile + col, nch - 1);
        const float4* M = reinterpret_cast<const float4*>(
            C.mom + ((size_t)tl.z * nch + c) * N + half * H) + g * V;
#pragma unroll
        for (int i = 0; i < V; ++i) A[i] = M[i];
    };
    float4 A[V];
    if (part < ntc) load(part, 0, A);
    float4 b[H / 4];
    if constexpr (PHI) {
#pragma unroll
        for (int i = 0; i < H / 4; ++i) b[i] = C.phi[((size_t)ti * (H / 4) + i) * 64 + lane];
    }
    const float4 qc = C.qcen[tl.z];
    const int q = min(tl.x + col, tl.y - 1);
    const float4 v = J.qrec[q];
    const float sx = v.x - qc.x, sy = v.y - qc.y, sz = D == 3 ? v.z - qc.z : 0.f;
    const float sq = __builtin_fmaf(sx, sx, __builtin_fmaf(sy, sy, sz * sz));
    if constexpr (!PHI) {
        float* fn = sm.fn[wave];
        __builtin_amdgcn_wave_barrier();
        // half a wave per axis; the third axis by the first half
#pragma unroll
        for (int x0 = 0; x0 < D; x0 += 2) {
            const int x = x0 + half;
            const float s = (x == 0 ? sx : x == 1 ? sy : sz) * 2.f * inv_cell;   // on [-1, 1]
            if (x < D) bessel<F>((float)CellDim<D>::lambda * s, fn + x * F * 33 + col, 33);
        }
        __builtin_amdgcn_wave_barrier();
        // the empty asm keeps the places' addresses from living in registers across tiles
        int sel = half, at = col;
#pragma unroll
        for (int n = 0; n < H; ++n) {
            if (n % 8 == 0) asm volatile("" : "+v"(sel), "+v"(at));
            float p = 1.f;
#pragma unroll
            for (int x = 0; x < D; ++x) {
                const int r0 = (x * F + term<D>(n, x)) * 33, r1 = (x * F + term<D>(n + H, x)) * 33;
                const float f = fn[(sel ? r1 : r0) + at];
                p = x == 0 ? f : p * f;
            }
            asm volatile("" : "+v"(p));
            if (n % 4 == 0) b[n / 4].x = p;
            else if (n % 4 == 1) b[n / 4].y = p;
            else if (n % 4 == 2) b[n / 4].z = p;
            else b[n / 4].w = p;
        }
    }
    const float old = J.qpot[q], lw = J.qlog2w ? J.qlog2w[q] : J.qlog2w_s;
    if (tid == 0) sm.nflag = 0;
    float4* cd = sm.cd[wave];
    auto load_cd = [&](int ct) {
        // (-2d, mu - |d|^2) of the tile's chunks; past the last one mu = -inf
        __builtin_amdgcn_wave_barrier();
        if (half == 0) {
            const int c = min(ct * kCellTile + col, nch - 1);
            const float4 kc = C.chcen[c];
            const float m = ct * kCellTile + col < nch ? C.mu[(size_t)tl.z * nch + c] : kNegInf;
            cd[col] = make_float4(-2.f * (qc.x - kc.x), -2.f * (qc.y - kc.y),
                                  D == 3 ? -2.f * (qc.z - kc.z) : 0.f, m);
        }
        __builtin_amdgcn_wave_barrier();
    };
    auto expo = [&](int r, float base) {
        const float4 k = cd[8 * (r >> 2) + 4 * half + (r & 3)];
        float e = __builtin_fmaf(sy, k.y, k.w);
        if (D == 3) e = __builtin_fmaf(sz, k.z, e);
        return __builtin_fmaf(sx, k.x, e) + base;
    };
    float m;
    if (LAGGED) {
        m = -old * kappa;
    } else {
        m = kNegInf;
        for (int ct = part; ct < ntc; ct += WS) {
            load_cd(ct);
#pragma unroll
            for (int r = 0; r < 16; ++r) m = fmaxf(m, expo(r, -sq));
        }
        m = fmaxf(m, __shfl_xor(m, 32));
        if (WS > 1) {
            if (half == 0) sm.red[wave][col] = m;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < WS; ++w) m = fmaxf(m, sm.red[wave - part + w][col]);
            __syncthreads();
        }
        if (m == kNegInf) m = 0.f;
    }
    const float base = -sq - m;
    float sum = 0.f;
#pragma unroll 1
    for (int ct = part; ct < ntc; ct += WS) {
        load_cd(ct);
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float4 nx[V];
            if (g + 1 < G) load(ct, g + 1, nx);
            else load(min(ct + WS, ntc - 1), 0, nx);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < V; ++i) {
                const float4 f = b[g * V + i];
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(A[i].x, f.x, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(A[i].y, f.y, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(A[i].z, f.z, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(A[i].w, f.w, acc, 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < V; ++i) A[i] = nx[i];
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) sum = __builtin_fmaf(acc[r], ex2(expo(r, base)), sum);
    }
    sum += __shfl_xor(sum, 32);
    if (WS > 1 && half == 0) sm.red[wave][col] = sum;
    __syncthreads();
    if (part == 0 && half == 0 && on && tl.x + col < tl.y) {
        float s = sum;
#pragma unroll
        for (int w = 1; w < WS; ++w) s += sm.red[wave + w][col];
        if (LAGGED && !(s >= kSumLo && s <= kSumHi)) {
            sm.flist[atomicAdd(&sm.nflag, 1)] = q;
        } else {
            // as finish_row, with the loads already there
            const float t = -(m + __log2f(s)) * inv_kappa;
            const float nv = J.self_avg ? 0.5f * (old + t) : t;
            J.out_pot[q] = nv;
            if (J.out_rec)
                reinterpret_cast<float*>(J.out_rec + q)[D == 2 ? 2 : 3] = __builtin_fmaf(nv, kappa, lw);
        }
    }
    __syncthreads();
    if (LAGGED) {
        const int n = sm.nflag;
        if (n > 0) rescue_rows<D, false>(J, sm.flist, n, kappa, inv_kappa, inv_sqrt_kappa);
        __syncthreads();
    }
}

// --------------------------------------------------------------- launch kernels

// In 2-D a launch carries a job's direct sweep too, for the points that the device leaves to
// it.  In 3-D the moments need twice the registers, which cost such a sweep 6 to 20 %: there
// the direct sweeps keep their own launch and leave it where the cell form is on
// (launch_sweep's skip); their merges ride in the values' launch.
template <int D>
constexpr bool kBoth = D == 2;

template <int D, int R>
union StepSmem {
    MomentSmem<D> m;
    SweepSmem<D, R> s;
};
template <int R>
union StepSmem<3, R> {
    MomentSmem<3> m;
};

// First launch of a sweep: of each job the moments of every (chunk, 32 query cells), or the
// direct sweep's work units.  The units are walked with the grid as the stride: how many
// there are is known on the device only.
template <int D, int R, int WS, bool LAGGED>
__global__ __launch_bounds__(kBlock, 2) void k_cell_moments(Launch L, CellLaunch C) {
    __shared__ StepSmem<D, R> sm;
    const int grid = (int)gridDim.x;
    int u = (int)blockIdx.x;
    // both jobs' counts at once (job[1] repeats job[0] where there is one)
    const int mode[2] = {*C.job[0].mode, *C.job[1].mode};
    const int nchs[2] = {*C.job[0].nch, *C.job[1].nch}, ncqs[2] = {*C.job[0].ncq, *C.job[1].ncq};
    for (int j = 0; j < L.njobs; ++j) {
        const Job& J = L.job[j];
        const CellJob& K = C.job[j];
        int nu;
        if (j ? mode[1] : mode[0]) {
            const int nch = j ? nchs[1] : nchs[0], ncq = j ? ncqs[1] : ncqs[0];
            nu = nch * ((ncq + kCellTile - 1) / kCellTile);
            for (; u < nu; u += grid)
                cell_moments<D>(K, J, u % nch, u / nch, nch, ncq, C.inv_cell, sm.m);
        } else if constexpr (!kBoth<D>) {
            nu = 0;
        } else {
            nu = J.nqb * J.splits;
            for (; u < nu; u += grid) {
                sweep_unit<D, R, WS, LAGGED, false, true, LAGGED>(
                    J, u % J.nqb, u / J.nqb, L.kappa, L.inv_kappa, L.inv_sqrt_kappa, sm.s);
                __syncthreads();
            }
        }
        u -= nu;
    }
}

// Second launch: the values of every query tile, or the direct sweep's merge.
template <int D, bool LAGGED, int VS>
__global__ __launch_bounds__(kBlock, 2) void k_cell_values(Launch L, CellLaunch C) {
    __shared__ ValueSmem<D, true> sm;
    const int grid = (int)gridDim.x;
    int u = (int)blockIdx.x;
    const int mode[2] = {*C.job[0].mode, *C.job[1].mode};
    const int nchs[2] = {*C.job[0].nch, *C.job[1].nch}, nts[2] = {*C.job[0].ntile, *C.job[1].ntile};
    for (int j = 0; j < L.njobs; ++j) {
        const Job& J = L.job[j];
        const CellJob& K = C.job[j];
        int nu;
        if (j ? mode[1] : mode[0]) {
            const int nch = j ? nchs[1] : nchs[0], nt = j ? nts[1] : nts[0];
            nu = (nt + 4 / VS - 1) / (4 / VS);
            // workgroup b runs on die b mod 8, each with its own L2: a die takes a run of tiles,
            // which share their cells' moments
            const int per = (nu + 7) >> 3;
            for (; u < 8 * per; u += grid) {
                const int v = (u & 7) * per + (u >> 3);
                if (v < nu)
                    cell_values<D, LAGGED, VS, true>(K, J, v, nt, nch, C.inv_cell, L.kappa,
                                                     L.inv_kappa, L.inv_sqrt_kappa, sm);
            }
            nu = 8 * per;
        } else {
            nu = J.splits > 1 ? (J.nq + kMergeRows - 1) / kMergeRows : 0;
            for (; u < nu; u += grid) {
                merge_block<D, LAGGED, false>(J, u * kMergeRows, J.nqb * 64 * C.R * (4 / C.WS),
                                              L.kappa, L.inv_kappa, L.inv_sqrt_kappa);
                __syncthreads();
            }
        }
        u -= nu;
    }
}

// The same launches over job tables (the batched path).  A block keeps the ends of the jobs'
// units in LDS and finds each unit's job by bisection; where some job takes the direct
// sweep, its work units follow.
__device__ __forceinline__ int unit_owner(const int* end, int n, int u) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (end[mid] > u) hi = mid;
        else lo = mid + 1;
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

template <int D, int R, int WS, bool LAGGED>
__global__ __launch_bounds__(kBlock, 2) void k_cell_tab_moments(TabLaunch L, CellBatch C, int k,
                                                               float inv_cell) {
    __shared__ StepSmem<D, R> sm;
    __shared__ int end[kCellBatchJobs];
    const int grid = (int)gridDim.x;
    const CellJob* jobs = C.jobs + (size_t)k * C.stride;
    const int* ends = C.uend + (size_t)k * 2 * C.stride;
    const int direct = C.info[k];
    for (int i = (int)threadIdx.x; i < L.njobs; i += kBlock) end[i] = ends[i];
    __syncthreads();
    const int total = end[L.njobs - 1];
    for (int u = (int)blockIdx.x; u < total; u += grid) {
        const int j = unit_owner(end, L.njobs, u);
        const CellJob& K = jobs[j];
        const int v = u - (j ? end[j - 1] : 0), nch = *K.nch;
        cell_moments<D>(K, L.jobs[j], v % nch, v / nch, nch, *K.ncq, inv_cell, sm.m);
    }
    if constexpr (kBoth<D>) {
        if (direct == 0) return;
        __syncthreads();
        for (int i = (int)threadIdx.x; i < L.njobs; i += kBlock) end[i] = L.blk_end[i];
        __syncthreads();
        for (int u = (int)blockIdx.x; u < L.nblocks; u += grid) {
            const int j = unit_owner(end, L.njobs, u);
            if (*jobs[j].mode) continue;
            const Job& J = L.jobs[j];
            const int v = u - (j ? end[j - 1] : 0);
            sweep_unit<D, R, WS, LAGGED, false, true, LAGGED>(J, v % J.nqb, v / J.nqb, L.kappa,
                                                              L.inv_kappa, L.inv_sqrt_kappa, sm.s);
            __syncthreads();
        }
    }
}

template <int D, bool LAGGED>
__global__ __launch_bounds__(kBlock, 2) void k_cell_tab_values(TabLaunch L, CellBatch C, int k,
                                                              float inv_cell, int qpb) {
    __shared__ ValueSmem<D, false> sm;
    __shared__ int end[kCellBatchJobs];
    const int grid = (int)gridDim.x;
    const CellJob* jobs = C.jobs + (size_t)k * C.stride;
    const int* ends = C.uend + (size_t)(k * 2 + 1) * C.stride;
    const int direct = C.info[k];
    for (int i = (int)threadIdx.x; i < L.njobs; i += kBlock) end[i] = ends[i];
    __syncthreads();
    const int total = end[L.njobs - 1], per = (total + 7) >> 3;
    for (int u = (int)blockIdx.x; u < 8 * per; u += grid) {
        const int w = (u & 7) * per + (u >> 3);   // runs of tiles per die, as in k_cell_values
        if (w >= total) continue;
        const int j = unit_owner(end, L.njobs, w);
        const CellJob& K = jobs[j];
        cell_values<D, LAGGED, 1, false>(K, L.jobs[j], w - (j ? end[j - 1] : 0), *K.ntile, *K.nch,
                                         inv_cell, L.kappa, L.inv_kappa, L.inv_sqrt_kappa, sm);
    }
    if (!kBoth<D> || direct == 0 || L.nmerge == 0) return;
    __syncthreads();
    for (int i = (int)threadIdx.x; i < L.njobs; i += kBlock) end[i] = L.mrg_end[i];
    __syncthreads();
    for (int u = (int)blockIdx.x; u < L.nmerge; u += grid) {
        const int j = unit_owner(end, L.njobs, u);
        if (*jobs[j].mode) continue;
        const Job& J = L.jobs[j];
        merge_block<D, LAGGED, false>(J, (u - (j ? end[j - 1] : 0)) * kMergeRows, J.nqb * qpb,
                                      L.kappa, L.inv_kappa, L.inv_sqrt_kappa);
        __syncthreads();
    }
}

template <int D, int R, int WS>
void tab_moments(bool lagged, const TabLaunch& L, const CellBatch& C, int k, float inv_cell, int nb,
                 hipStream_t s) {
    if (lagged)
        hipLaunchKernelGGL((k_cell_tab_moments<D, R, WS, true>), dim3(nb), dim3(kBlock), 0, s, L, C,
                           k, inv_cell);
    else
        hipLaunchKernelGGL((k_cell_tab_moments<D, R, WS, false>), dim3(nb), dim3(kBlock), 0, s, L, C,
                           k, inv_cell);
}

template <int D>
hipError_t tab_launch(const Schedule& sc, bool lagged, const TabLaunch& L, const CellBatch& C, int k,
                      hipStream_t s) {
    const float inv_cell = (float)(1.0 / cell_side(D));
    const int nm = 4096, nv = 2048, qpb = 64 * sc.R * (4 / sc.WS);
    if constexpr (!kBoth<D>) {
        tab_moments<D, 4, 4>(lagged, L, C, k, inv_cell, nm, s);
    } else if (sc.WS == 2) {
        if (sc.R == 1) tab_moments<D, 1, 2>(lagged, L, C, k, inv_cell, nm, s);
        else if (sc.R == 2) tab_moments<D, 2, 2>(lagged, L, C, k, inv_cell, nm, s);
        else tab_moments<D, 4, 2>(lagged, L, C, k, inv_cell, nm, s);
    } else {
        if (sc.R == 1) tab_moments<D, 1, 4>(lagged, L, C, k, inv_cell, nm, s);
        else if (sc.R == 2) tab_moments<D, 2, 4>(lagged, L, C, k, inv_cell, nm, s);
        else tab_moments<D, 4, 4>(lagged, L, C, k, inv_cell, nm, s);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (lagged)
        hipLaunchKernelGGL((k_cell_tab_values<D, true>), dim3(nv), dim3(kBlock), 0, s, L, C, k,
                           inv_cell, qpb);
    else
        hipLaunchKernelGGL((k_cell_tab_values<D, false>), dim3(nv), dim3(kBlock), 0, s, L, C, k,
                           inv_cell, qpb);
    return hipGetLastError();
}

template <int D, int R, int WS>
hipError_t moments_drw(bool lagged, const Launch& L, const CellLaunch& C, int nb, hipStream_t s,
                       hipEvent_t e0, hipEvent_t e1) {
    auto go = [&](auto kernel) {
        if (e0) hipExtLaunchKernelGGL(kernel, dim3(nb), dim3(kBlock), 0, s, e0, e1, 0, L, C);
        else hipLaunchKernelGGL(kernel, dim3(nb), dim3(kBlock), 0, s, L, C);
    };
    if (lagged) go(k_cell_moments<D, R, WS, true>);
    else go(k_cell_moments<D, R, WS, false>);
    return hipGetLastError();
}

template <int D, int R>
hipError_t moments_dr(bool lagged, const Launch& L, const CellLaunch& C, int nb, hipStream_t s,
                      hipEvent_t e0, hipEvent_t e1) {
    switch (C.WS) {
        case 1: return moments_drw<D, R, 1>(lagged, L, C, nb, s, e0, e1);
        case 2: return moments_drw<D, R, 2>(lagged, L, C, nb, s, e0, e1);
        default: return moments_drw<D, R, 4>(lagged, L, C, nb, s, e0, e1);
    }
}

template <int D>
hipError_t moments_d(bool lagged, const Launch& L, const CellLaunch& C, int nb, hipStream_t s,
                     hipEvent_t e0, hipEvent_t e1) {
    if constexpr (!kBoth<D>) {
        return moments_drw<D, 4, 4>(lagged, L, C, nb, s, e0, e1);
    } else {
        switch (C.R) {
            case 1: return moments_dr<D, 1>(lagged, L, C, nb, s, e0, e1);
            case 2: return moments_dr<D, 2>(lagged, L, C, nb, s, e0, e1);
            case 4: return moments_dr<D, 4>(lagged, L, C, nb, s, e0, e1);
            default: return moments_dr<D, 8>(lagged, L, C, nb, s, e0, e1);
        }
    }
}

template <int D, int VS>
hipError_t values_d(bool lagged, const Launch& L, const CellLaunch& C, int nb, hipStream_t s,
                    hipEvent_t e0, hipEvent_t e1) {
    auto go = [&](auto kernel) {
        if (e0) hipExtLaunchKernelGGL(kernel, dim3(nb), dim3(kBlock), 0, s, e0, e1, 0, L, C);
        else hipLaunchKernelGGL(kernel, dim3(nb), dim3(kBlock), 0, s, L, C);
    };
    if (lagged) go(k_cell_values<D, true, VS>);
    else go(k_cell_values<D, false, VS>);
    return hipGetLastError();
}

}  // namespace

// Smaller chunks make more, evener work of the moments and more chunks for the values (one
// iteration with 256 / 512 / 1024 keys: 46 / 48 / 55 us at M = 16384, 68 / 65 / 75 at 30001,
// 537 / 407 / 385 at 262144).
int cell_chunk(int n) { return n <= 24576 ? 256 : n <= 131072 ? 512 : kCellChunkMax; }

void cell_prep_layout(Arena& a, CellPrep& P, int d, int T, int M, int xo, int yo, int kcx, int kcy) {
    P.d = d;
    P.bits = d == 2 ? CellDim<2>::bits : CellDim<3>::bits;
    P.ids = 1 << (P.bits * d);
    P.cell = (float)cell_side(d);
    for (int s = 0; s < 2; ++s) {
        CellSide& S = P.side[s];
        S.off = s ? yo : xo;
        S.n = s ? M : T;
        // points per block of the sort: few, since one wave scatters them in order, but at most
        // 256 blocks up to 2^18 points, since every code's counts are summed over the blocks
        S.per = std::max(256, ((S.n + 255) / 256 + 63) / 64 * 64);
        S.nb = (S.n + S.per - 1) / S.per;
        S.kc = s ? kcy : kcx;
        S.cmax = std::min(P.ids, S.n / kCellMinPoints + 1);
        S.chmax = S.cmax + S.n / S.kc;
        S.tmax = S.cmax + S.n / kCellTile;
        S.box = a.take<unsigned>(8);
        S.id = a.take<unsigned short>(S.n);
        S.bh = a.take<unsigned>((size_t)S.nb * P.ids);
        S.first = a.take<unsigned>(P.ids);
        S.perm = a.take<int>(S.n);
        S.cen = a.take<float4>(S.cmax);
        S.chunk = a.take<int4>(S.chmax);
        S.chcen = a.take<float4>(S.chmax);
        S.tile = a.take<int4>(S.tmax);
        S.cnt = a.take<int>(4);
    }
    P.mode = a.take<int>(5);
}

// The partition's launches; TAB: of nprob problems of at most n points and nb sort blocks.
template <bool TAB>
static void partition(const CellPrep& P, const CellPrep* tab, const CellInputs& in, int ids, int n,
                      int nb, int nprob, hipStream_t s) {
    hipLaunchKernelGGL(k_cell_init<TAB>, dim3(1, 1, nprob), dim3(64), 0, s, P, tab);
    hipLaunchKernelGGL(k_cell_box<TAB>, dim3(std::min(512, (n + 1023) / 1024), 2, nprob), dim3(256),
                       0, s, P, tab, in);
    hipLaunchKernelGGL(k_cell_hist<TAB>, dim3(nb, 2, nprob), dim3(256), 0, s, P, tab, in);
    hipLaunchKernelGGL(k_cell_scan<TAB>, dim3(ids / 64, 2, nprob), dim3(256), 0, s, P, tab);
    hipLaunchKernelGGL(k_cell_lists<TAB>, dim3(2, 1, nprob), dim3(1024), 0, s, P, tab);
    hipLaunchKernelGGL(k_cell_scatter<TAB>, dim3(nb, 2, nprob), dim3(64), 0, s, P, tab);
    hipLaunchKernelGGL(k_cell_gather<TAB>, dim3((n + 255) / 256, 1, nprob), dim3(256), 0, s, P, tab,
                       in);
}

hipError_t launch_cell_prep(const CellPrep& P, const CellInputs& in, hipStream_t s) {
    const int n = std::max(P.side[0].n, P.side[1].n);
    partition<false>(P, nullptr, in, P.ids, n, std::max(P.side[0].nb, P.side[1].nb), 1, s);
    const dim3 gf(std::min(2048, n / kCellTile + 128), 2);
    if (P.d == 2) hipLaunchKernelGGL(k_cell_functions<2>, gf, dim3(256), 0, s, P, in);
    else hipLaunchKernelGGL(k_cell_functions<3>, gf, dim3(256), 0, s, P, in);
    return hipGetLastError();
}

hipError_t launch_cell_prep_batch(int d, const CellBatch& C, const CellInputs& in, int max_n,
                                  int max_nb, hipStream_t s) {
    CellPrep none;
    std::memset(&none, 0, sizeof(none));
    const int bits = d == 2 ? CellDim<2>::bits : CellDim<3>::bits;
    partition<true>(none, C.prep, in, 1 << (bits * d), max_n, max_nb, C.B, s);
    hipLaunchKernelGGL(k_cell_plan, dim3(1), dim3(1024), 0, s, C, d);
    return hipGetLastError();
}

hipError_t launch_cell_tab(int d, const Schedule& sc, bool lagged, const TabLaunch& L,
                           const CellBatch& C, int k, hipStream_t s) {
    if (d == 2) return tab_launch<2>(sc, lagged, L, C, k, s);
    TabLaunch T = L;
    T.cell = C.jobs + (size_t)k * C.stride;
    const hipError_t e = launch_tab(d, sc, lagged, false, T, s);
    return e != hipSuccess ? e : tab_launch<3>(sc, lagged, L, C, k, s);
}

CellLimits cell_limits() {
    CellLimits l;
    if (const char* e = std::getenv("CT_CELL_MIN_PAIRS")) {
        l.pairs = l.pairs3 = std::atof(e);
        l.work = 0.0;
        l.expect = false;
    }
    return l;
}

bool cell_candidate(int d, int nq, int nk) {
    return d == 2 || (double)nq * nk >= cell_limits().pairs3;
}

CellOffer::CellOffer(int d, double eps, double launch, double gain, double slow)
    : d_(d), side_cells_(std::sqrt(1.4426950408889634 / eps) / cell_side(d)), launch_(launch),
      gain_(gain), slow_(slow) {}

CellCounts CellOffer::expect(int n, int chunk_keys, bool* fits) const {
    const int bits = d_ == 2 ? CellDim<2>::bits : CellDim<3>::bits;
    const double box = std::pow(side_cells_ + 0.5, d_) * (d_ == 2 ? 0.8 : 0.3);
    const double cells = std::max(1.0, box * -std::expm1(-n / box));   // n points at random
    *fits = side_cells_ <= (1 << bits) && cells <= n / kCellMinPoints + 1;
    // parts of `most` points of a cell, the cells' sizes spread exponentially
    auto parts = [&](int most) { return cells / -std::expm1(-most * cells / n); };
    return CellCounts{(double)n, cells, parts(chunk_keys), parts(kCellTile)};
}

void CellOffer::sweep(int nq, int nk, int chunk_q, int chunk_k) {
    bool fq, fk;
    const CellTimes t = cell_times(expect(nq, chunk_q, &fq), expect(nk, chunk_k, &fk), d_);
    direct_ += t.direct + launch_;
    if (fq && fk && cell_gains(t, launch_, gain_)) {
        any_ = true;
        form_ += t.cell + 0.6 * launch_;
    } else {
        form_ += slow_ * t.direct + launch_;
    }
}

bool CellOffer::pays(int iters, double prep_us) const {
    return any_ && iters * form_ + prep_us < iters * direct_;
}

hipError_t launch_cell_sweep(int d, const Schedule& sc, bool lagged, const Launch& L0,
                             const CellLaunch& C0, int nblocks, hipStream_t s) {
    Launch L = L0;
    CellLaunch C = C0;
    if (d == 3) {
        bool any = false;
        const int* skip[kMaxJobs] = {};
        for (int j = 0; j < L.njobs; ++j) {
            if (cell_candidate(d, L.job[j].nq, L.job[j].nk)) any = true;
            else C.job[j].mode = C.never;
            skip[j] = C.job[j].mode;
        }
        if (L.njobs == 1) C.job[1] = C.job[0];
        if (!any) return launch_sweep(d, sc, lagged, false, L0, nblocks, s);
        const hipError_t e = launch_sweep(d, Schedule{sc.R, sc.WS, sc.blocks_per_cu, 1}, lagged,
                                          false, L, nblocks, s, skip);
        if (e != hipSuccess) return e;
    }
    // grids for the units one can expect, up to the blocks that are resident at once (both
    // kernels walk whatever there is; blocks beyond that only queue)
    int units = 0, tiles = 0, direct = 0, merges = 0;
    double pairs = 0.0;
    for (int j = 0; j < L.njobs; ++j) {
        const Job& J = L.job[j];
        units += (J.nk / cell_chunk(J.nk) + 64) * 4;
        tiles += J.nq / kCellTile + 64;
        direct += J.nqb * J.splits;
        if (J.splits > 1) merges += (J.nq + kMergeRows - 1) / kMergeRows;
        pairs += (double)J.nq * J.nk;
    }
    // Waves per tile of the values: few tiles leave the GPU idle unless several waves share one,
    // many repeat the tile's loads (one iteration at T = 4096, M = 16384: 46 us with 4 waves, 48
    // with 2, 52 with 1; T = 9001, M = 30001: 68, 63, 69; T = 65536, M = 262144: 438, 406, 405).
    const int vs = tiles < 900 ? 4 : tiles < 3000 ? 2 : 1;
    // In 3-D a launch can mix a direct sweep, which prefers resident blocks only.
    const int nm = std::min(d == 2 ? 4096 : 768, std::max(units, std::min(direct, 768)));
    const int nv = std::min(1024, std::max((tiles * vs + 3) / 4, merges));
    const int code = sc.R * 100 + sc.WS * 10 + sc.sep + (lagged && L.expanded ? 1000 : 0);
    hipEvent_t e0, e1;
    void* tok = profile_kernel_begin(&e0, &e1);
    hipError_t e = d == 2 ? moments_d<2>(lagged, L, C, nm, s, e0, e1)
                          : moments_d<3>(lagged, L, C, nm, s, e0, e1);
    // kind 50/51: moments (or a direct sweep) of a safe/lagged sweep; 60/61: its values
    profile_kernel_end(tok, 50 + lagged, 0, code, nm, pairs);
    if (e != hipSuccess) return e;
    tok = profile_kernel_begin(&e0, &e1);
    if (vs == 4)
        e = d == 2 ? values_d<2, 4>(lagged, L, C, nv, s, e0, e1) : values_d<3, 4>(lagged, L, C, nv, s, e0, e1);
    else if (vs == 2)
        e = d == 2 ? values_d<2, 2>(lagged, L, C, nv, s, e0, e1) : values_d<3, 2>(lagged, L, C, nv, s, e0, e1);
    else
        e = d == 2 ? values_d<2, 1>(lagged, L, C, nv, s, e0, e1) : values_d<3, 1>(lagged, L, C, nv, s, e0, e1);
    profile_kernel_end(tok, 60 + lagged, 0, code, nv, 0.0);
    return e;
}

}  // namespace ct
