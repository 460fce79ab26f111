// Cell form of the Stein sum in 2-D.
//
//   phi_i = 1/T sum_j k_ij [score_j + cb (x'_i - x'_j)],  k_ij = 2^-|x'_i - x'_j|^2
//
// over scaled points x'.  The points are split into the cells of a grid of side w.  With
// x'_j = C + u in cell c, x'_i = A + s in cell a and d = A - C,
//     -|x'_i - x'_j|^2 = -|x'_i - C|^2 + (2 d.u - |u|^2) + 2 s.u
// holds exactly, and on each axis, in units of half a cell, 2^(2 s u) is e^(lambda s u) with
// lambda = ln2 w^2 / 2 = 0.597, expanded as in the cell form of the soft-min sweep:
// I_0(lambda s) + 2 sum_n I_n(lambda s) T_n(u).  Eight functions per axis leave out
// 2 I_8(lambda) < 4e-9 per axis, of a pair's term at most 1.2e-8 (at opposite corners).  The moments of a cell's keys, for query cell a,
//     M[a][c][r][n] = sum_{j in c} 2^(2 d.u - |u|^2) v_rj T_nx(u_x) T_ny(u_y)
// with v = (1, score_x - cb u_x, score_y - cb u_y), are a product of two matrices over the keys
// (float32 in the matrix cores, v_mfma_f32_32x32x2); a query then costs 192 multiply-adds per
// key cell, in a chain over axes that reads its moments as scalars.
//
// The bandwidth is the squared median distance over ln T, so the samples span some ten cells per
// axis whatever their scale: the sum falls from T^2 pairs to T times 50 to 100 cells.  A side of
// 21/16 and grid corners that are multiples of 1/64 make centres and their differences exact,
// and the exponent of a (query, cell), whose rounding would be common to all of the cell's keys,
// is formed in float64; the other roundings are float32's, as in the direct sum.
// Measured on an MI355X, d = 2, T = 65536, median bandwidth: the sum 1085 us directly, 105 us
// in this form (moments 33, values 27, the partition's six launches 40, the two launches of the
// direct sum that end at once 9), and an error against float64 of 1.6e-7 where the direct sum's
// longer chains of additions have 7.9e-7.
#include <algorithm>
#include <cmath>

#include "stein.h"

namespace ct {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr double kLambda = 0.5 * 0.69314718055994531 * (double)kSteinSide * kSteinSide;
constexpr float kInvHalf = 2.f / kSteinSide;

__device__ __forceinline__ unsigned ordered(float v) {
    const unsigned u = __float_as_uint(v);
    return (u & 0x80000000u) ? ~u : u | 0x80000000u;
}
__device__ __forceinline__ float from_ordered(unsigned u) {
    return __uint_as_float((u & 0x80000000u) ? u & 0x7fffffffu : ~u);
}
// Lower corner of the grid: a multiple of 1/64 at or below the smallest coordinate.
__device__ __forceinline__ float corner(unsigned u) {
    return floorf(from_ordered(u) * 64.f) * (1.f / 64.f);
}
__device__ __forceinline__ int cell_of_point(float x, float y, float lx, float ly) {
    const int n = (1 << kSteinBits) - 1;
    const float vx = (x - lx) * (1.f / kSteinSide), vy = (y - ly) * (1.f / kSteinSide);
    const int kx = vx > 0.f ? min(n, (int)fminf(vx, 65535.f)) : 0;
    const int ky = vy > 0.f ? min(n, (int)fminf(vy, 65535.f)) : 0;
    return kx | ky << kSteinBits;
}

// Bounding box of each block's share of the points, and the points that the form cannot take: coordinates or scores that are not
// finite, or scores whose sums could leave float32's range where the direct sum's do not.
__global__ __launch_bounds__(256) void k_st_box(SteinCells S, const float4* __restrict__ krec) {
    __shared__ unsigned w[5][4];
    unsigned lo[2] = {0xffffffffu, 0xffffffffu}, hi[2] = {0u, 0u}, bad = 0u;
    for (int i = (int)(blockIdx.x * 256 + threadIdx.x); i < S.n; i += (int)gridDim.x * 256) {
        const float4 r = krec[i];
        lo[0] = min(lo[0], ordered(r.x));
        hi[0] = max(hi[0], ordered(r.x));
        lo[1] = min(lo[1], ordered(r.y));
        hi[1] = max(hi[1], ordered(r.y));
        const bool ok = fabsf(r.x) < 16384.f && fabsf(r.y) < 16384.f && fabsf(r.z) < 1e20f &&
                        fabsf(r.w) < 1e20f;
        bad += ok ? 0u : 1u;
    }
    for (int m = 1; m < 64; m <<= 1) {
        for (int t = 0; t < 2; ++t) {
            lo[t] = min(lo[t], __shfl_xor(lo[t], m));
            hi[t] = max(hi[t], __shfl_xor(hi[t], m));
        }
        bad += __shfl_xor(bad, m);
    }
    if ((threadIdx.x & 63) == 0) {
        const int k = (int)threadIdx.x >> 6;
        w[0][k] = lo[0];
        w[1][k] = lo[1];
        w[2][k] = hi[0];
        w[3][k] = hi[1];
        w[4][k] = bad;
    }
    __syncthreads();
    if (threadIdx.x < 5) {
        const unsigned* v = w[threadIdx.x];
        unsigned r = v[0];
        for (int k = 1; k < 4; ++k) r = threadIdx.x < 2 ? min(r, v[k]) : threadIdx.x < 4 ? max(r, v[k]) : r + v[k];
        S.box[threadIdx.x * kSteinBoxes + blockIdx.x] = r;
    }
}

// The whole box from the blocks' (the first wave; atomics on one box from every wave took
// 48 us at 65536 points).
__device__ __forceinline__ void read_box(const SteinCells& S, unsigned* sh) {
    if (threadIdx.x < 64) {
        for (int t = 0; t < 5; ++t) {
            unsigned v = S.box[t * kSteinBoxes + threadIdx.x];
            for (int m = 1; m < 64; m <<= 1) {
                const unsigned o = __shfl_xor(v, m);
                v = t < 2 ? min(v, o) : t < 4 ? max(v, o) : v + o;
            }
            if (threadIdx.x == 0) sh[t] = v;
        }
    }
    __syncthreads();
}

// Counts per block of `per` points and cell code.
__global__ __launch_bounds__(256) void k_st_hist(SteinCells S, const float4* __restrict__ krec) {
    __shared__ unsigned h[kSteinIds], box[5];
    for (int i = (int)threadIdx.x; i < kSteinIds; i += 256) h[i] = 0u;
    read_box(S, box);
    const float lx = corner(box[0]), ly = corner(box[1]);
    const int b = (int)blockIdx.x, i1 = min(S.n, (b + 1) * S.per);
    for (int i = b * S.per + (int)threadIdx.x; i < i1; i += 256) {
        const float4 r = krec[i];
        const int id = cell_of_point(r.x, r.y, lx, ly);
        S.id[i] = (unsigned short)id;
        atomicAdd(&h[id], 1u);
    }
    __syncthreads();
    for (int i = (int)threadIdx.x; i < kSteinIds; i += 256) S.bh[(size_t)b * kSteinIds + i] = h[i];
}

// Per code: exclusive sums of its counts over the blocks, and its total (four waves share 64
// codes, a quarter of the blocks each).
__global__ __launch_bounds__(256) void k_st_scan(SteinCells S) {
    __shared__ unsigned part[4][64];
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    const int id = (int)blockIdx.x * 64 + lane;
    const int per = (S.nb + 3) / 4, b0 = min(S.nb, wave * per), b1 = min(S.nb, b0 + per);
    unsigned sum = 0u;
#pragma unroll 8
    for (int b = b0; b < b1; ++b) sum += S.bh[(size_t)b * kSteinIds + id];
    part[wave][lane] = sum;
    __syncthreads();
    unsigned run = 0u;
    for (int w = 0; w < wave; ++w) run += part[w][lane];
#pragma unroll 4
    for (int b = b0; b < b1; ++b) {
        const size_t at = (size_t)b * kSteinIds + id;
        const unsigned v = S.bh[at];
        S.bh[at] = run;
        run += v;
    }
    if (wave == 3) S.first[id] = run;
}

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

// Places, cells, chunks of at most kc keys, tiles of 64 queries, and the mode (one thread per
// code).
__global__ __launch_bounds__(kSteinIds) void k_st_lists(SteinCells S) {
    __shared__ int sh[16];
    __shared__ unsigned box[5];
    read_box(S, box);
    const int id = (int)threadIdx.x, n = (int)S.first[id];
    int tp, tc, th, tt;
    const int at = block_scan(n, sh, &tp);
    const int ic = block_scan(n > 0 ? 1 : 0, sh, &tc);
    const int nh = (n + S.kc - 1) / S.kc, nt = (n + kSteinTile - 1) / kSteinTile;
    const int ih = block_scan(nh, sh, &th);
    const int it = block_scan(nt, sh, &tt);
    const float lx = corner(box[0]), ly = corner(box[1]);
    const float ext = kSteinSide * (float)(1 << kSteinBits);
    const SteinTimes t = stein_times(S.n, tc, th, tt);
    // every point in the cell of its code: nothing outside the coded box
    const bool ok = box[4] == 0u && tc <= kSteinCells && th <= S.chmax && tt <= S.tmax && t.cell < t.direct &&
                    (long long)(th + tc) * tc * kSteinMom <= S.room &&
                    from_ordered(box[2]) - lx < ext && from_ordered(box[3]) - ly < ext;
    if (id == 0) {
        S.cnt[0] = tc;
        S.cnt[1] = th;
        S.cnt[2] = tt;
        S.cnt[3] = ok ? 1 : 0;
    }
    S.first[id] = (unsigned)at;
    if (!ok || n == 0) return;
    const int kx = id & ((1 << kSteinBits) - 1), ky = id >> kSteinBits;
    S.cen[ic] = make_float4(lx + ((float)kx + 0.5f) * kSteinSide, ly + ((float)ky + 0.5f) * kSteinSide, 0.f, 0.f);
    S.own[ic] = make_int2(ih, ih + nh);
    for (int e = 0; e < nh; ++e)
        S.chunk[ih + e] = make_int4(at + e * S.kc, min(at + n, at + (e + 1) * S.kc), ic, 0);
    for (int e = 0; e < nt; ++e)
        S.tile[it + e] = make_int4(at + e * kSteinTile, min(at + n, at + (e + 1) * kSteinTile), ic, 0);
}

// Stable scatter: one wave per block of points, 64 at a time; the lanes of one code rank
// themselves by ballots over the code's bits.
__global__ __launch_bounds__(64) void k_st_scatter(SteinCells S, const float4* __restrict__ krec) {
    __shared__ unsigned cur[kSteinIds];
    if (S.cnt[3] == 0) return;
    const int b = (int)blockIdx.x, lane = (int)threadIdx.x;
    for (int i = lane; i < kSteinIds; i += 64) cur[i] = S.first[i] + S.bh[(size_t)b * kSteinIds + i];
    __syncthreads();
    const int i1 = min(S.n, (b + 1) * S.per);
    for (int i0 = b * S.per; i0 < i1; i0 += 64) {
        const int i = i0 + lane;
        const bool on = i < i1;
        const int id = on ? (int)S.id[i] : 0;
        unsigned long long same = __ballot(on);
        for (int k = 0; k < 2 * kSteinBits; ++k) {
            const unsigned long long m = __ballot((id >> k) & 1);
            same &= ((id >> k) & 1) ? m : ~m;
        }
        const int rank = __popcll(same & ((1ull << lane) - 1ull));
        unsigned base = 0u;
        if (on) base = cur[id];
        __syncthreads();
        if (on) {
            S.perm[base + rank] = i;
            S.rec[base + rank] = krec[i];
            if (rank == 0) cur[id] = base + (unsigned)__popcll(same);
        }
        __syncthreads();
    }
}

__device__ __forceinline__ float bandwidth_cb(float h) {
    const double s = sqrt(1.4426950408889634 / (double)h);
    return (float)(2.0 / ((double)h * s));
}

// A bound of 2 d.u within a cell, taken off the keys' exponents and added to the query's, so that
// neither leaves float32's range where the pair counts.  Exact: d is a multiple of the side.
__device__ __forceinline__ float exponent_bound(float dx, float dy) {
    return (fabsf(dx) + fabsf(dy)) * kSteinSide;
}

// Moments of one chunk of keys (blockIdx.x) for 32 query cells (blockIdx.y): the four waves
// take every fourth batch of 64 keys, products 32 x 32 x 2 at a time.  A wave's accumulators are
// three right-hand sides by two halves of the 64 products, 96 registers; the waves' sums meet
// in LDS in a fixed order.
constexpr int kStWaves = 4;
__global__ __launch_bounds__(kStWaves * 64, 2) void k_st_moments(SteinCells S, const float* __restrict__ h) {
    __shared__ float tx[kStWaves][64][9], ty[kStWaves][64][9];     // T_n(u), odd pitch
    __shared__ float4 ku[kStWaves][64];                            // (2 u, |u|^2, 0)
    __shared__ float2 kv[kStWaves][64];
    __shared__ float red[2][6 * 16][64];
    const int ncell = S.cnt[0], nch = S.cnt[1], a0 = (int)blockIdx.y * 32;
    if (S.cnt[3] == 0 || (int)blockIdx.x >= nch || a0 >= ncell) return;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
    const int4 ch = S.chunk[blockIdx.x];
    const float4 C = S.cen[ch.z], A = S.cen[min(ncell - 1, a0 + (lane & 31))];
    const float dx = A.x - C.x, dy = A.y - C.y;
    const float mu = exponent_bound(dx, dy);
    const float cb = bandwidth_cb(*h);
    const int col = lane & 31, hi = lane >> 5;
    const int nx = col & 7, ny = col >> 3;                         // product of half 0; half 1: ny + 4
    f32x16 acc[6];
#pragma unroll
    for (int t = 0; t < 6; ++t)
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
    for (int k0 = ch.x + wave * 64; k0 < ch.y; k0 += kStWaves * 64) {
        const int k = k0 + lane;
        const bool on = k < ch.y;
        const float4 r = S.rec[min(k, ch.y - 1)];
        const float ux = r.x - C.x, uy = r.y - C.y;
        // a lane past the end takes an exponent that underflows
        ku[wave][lane] = make_float4(2.f * ux, 2.f * uy, on ? __builtin_fmaf(ux, ux, uy * uy) : 1e30f, 0.f);
        kv[wave][lane] = make_float2(__builtin_fmaf(-cb, ux, r.z), __builtin_fmaf(-cb, uy, r.w));
        float c0 = 1.f, c1 = ux * kInvHalf, e0 = 1.f, e1 = uy * kInvHalf;
        const float ax = 2.f * c1, ay = 2.f * e1;
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            tx[wave][lane][n] = c0;
            ty[wave][lane][n] = e0;
            const float c2 = __builtin_fmaf(ax, c1, -c0), e2 = __builtin_fmaf(ay, e1, -e0);
            c0 = c1; c1 = c2; e0 = e1; e1 = e2;
        }
        __builtin_amdgcn_wave_barrier();
        const int pairs = (min(64, ch.y - k0) + 1) / 2;
#pragma unroll 2
        for (int p = 0; p < pairs; ++p) {
            const int key = 2 * p + hi;
            const float4 u = ku[wave][key];
            const float2 v = kv[wave][key];
            const float w = __builtin_amdgcn_exp2f(__builtin_fmaf(dx, u.x, __builtin_fmaf(dy, u.y, -u.z - mu)));
            const float w1 = w * v.x, w2 = w * v.y;
            const float f = tx[wave][key][nx];
            const float b0 = f * ty[wave][key][ny], b1 = f * ty[wave][key][ny + 4];
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(w, b0, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(w, b1, acc[1], 0, 0, 0);
            acc[2] = __builtin_amdgcn_mfma_f32_32x32x2f32(w1, b0, acc[2], 0, 0, 0);
            acc[3] = __builtin_amdgcn_mfma_f32_32x32x2f32(w1, b1, acc[3], 0, 0, 0);
            acc[4] = __builtin_amdgcn_mfma_f32_32x32x2f32(w2, b0, acc[4], 0, 0, 0);
            acc[5] = __builtin_amdgcn_mfma_f32_32x32x2f32(w2, b1, acc[5], 0, 0, 0);
        }
        __builtin_amdgcn_wave_barrier();
    }
    // waves 2, 3 to 0, 1, then 1 to 0
    for (int half = 2; half > 0; half >>= 1) {
        __syncthreads();
        if (wave >= half && wave < 2 * half) {
#pragma unroll
            for (int t = 0; t < 6; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) red[wave - half][t * 16 + r][lane] = acc[t][r];
        }
        __syncthreads();
        if (wave < half) {
#pragma unroll
            for (int t = 0; t < 6; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[t][r] += red[wave][t * 16 + r][lane];
        }
    }
    if (wave != 0) return;
    // register r of a lane: row (query cell) 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int a = a0 + 8 * (r >> 2) + 4 * hi + (r & 3);
        if (a >= ncell) continue;
        float* out = S.mom + ((size_t)(ncell + (int)blockIdx.x) * ncell + a) * kSteinMom;
#pragma unroll
        for (int t = 0; t < 6; ++t) out[(t >> 1) * kSteinTerms + (t & 1) * 32 + col] = acc[t][r];
    }
}

// Sums over a key cell's chunks, in chunk order: a wave per pair (query cell, key cell).
__global__ __launch_bounds__(256) void k_st_reduce(SteinCells S) {
    const int ncell = S.cnt[0], lane = (int)threadIdx.x & 63;
    if (S.cnt[3] == 0 || lane >= kSteinMom / 4) return;
    const int w0 = (int)blockIdx.x * 4 + ((int)threadIdx.x >> 6);
    for (int w = w0; w < ncell * ncell; w += (int)gridDim.x * 4) {
        const int c = w / ncell, a = w - c * ncell;
        const int2 own = S.own[c];
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
        for (int e = own.x; e < own.y; ++e) {
            const float4 v = reinterpret_cast<const float4*>(S.mom + ((size_t)(ncell + e) * ncell + a) * kSteinMom)[lane];
            s.x += v.x;
            s.y += v.y;
            s.z += v.z;
            s.w += v.w;
        }
        reinterpret_cast<float4*>(S.mom + ((size_t)a * ncell + c) * kSteinMom)[lane] = s;
    }
}

// I_n(lambda t), n = 0..7 (n > 0 doubled), by their power series: |lambda t| <= 0.6, so the
// terms beyond the sixth are below 1e-13 of the first.
__device__ __forceinline__ void bessel(float t, float* f) {
    const float z = (float)(0.5 * kLambda) * t, q = z * z;
    float lead = 1.f;
#pragma unroll
    for (int n = 0; n < 8; ++n) {
        float s = 1.f;
#pragma unroll
        for (int k = 5; k >= 1; --k) s = __builtin_fmaf(s * q, 1.f / (float)(k * (n + k)), 1.f);
        f[n] = (n ? 2.f : 1.f) * lead * s;
        lead *= z * (1.f / (float)(n + 1));
    }
}

// 2^f for |f| <= 1/2 to 5e-9, by its power series.
__device__ __forceinline__ double exp2_half(double f) {
    double s = 1.5252733804059841e-05;   // ln2^k / k!, k = 7..0
    s = __builtin_fma(s, f, 1.5403530393381610e-04);
    s = __builtin_fma(s, f, 1.3333558146428443e-03);
    s = __builtin_fma(s, f, 9.6181291076284772e-03);
    s = __builtin_fma(s, f, 5.5504108664821580e-02);
    s = __builtin_fma(s, f, 2.4022650695910071e-01);
    s = __builtin_fma(s, f, 6.9314718055994531e-01);
    return __builtin_fma(s, f, 1.0);
}

// Values: a block takes a tile of 64 queries of one cell; its four waves take every fourth key
// cell and meet in LDS in wave order.  The moments of (a, c) are the same for the wave, so they
// are read as scalars.
__global__ __launch_bounds__(256) void k_st_values(SteinCells S, const float* __restrict__ mom,
                                                   const float* __restrict__ h, float* __restrict__ phi,
                                                   float* __restrict__ h_used) {
    __shared__ float red[3][2][64];
    if (S.cnt[3] == 0) return;
    const int tile = (int)blockIdx.x;
    if (tile == 0 && threadIdx.x == 0 && h_used) *h_used = *h;
    if (tile >= S.cnt[2]) return;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
    const int4 tl = S.tile[tile];
    const int a = __builtin_amdgcn_readfirstlane(tl.z), ncell = __builtin_amdgcn_readfirstlane(S.cnt[0]);
    const int q = min(tl.x + lane, tl.y - 1);
    const float4 r = S.rec[q];
    const float4 A = S.cen[a];
    const float cb = bandwidth_cb(*h);
    float fx[8], fy[8];
    bessel((r.x - A.x) * kInvHalf, fx);
    bessel((r.y - A.y) * kInvHalf, fy);
    float o0 = 0.f, o1 = 0.f;
    for (int c = wave; c < ncell; c += 4) {
        const float4 C = S.cen[c];
        const double dx = (double)r.x - (double)C.x, dy = (double)r.y - (double)C.y;
        const double e = (double)exponent_bound(A.x - C.x, A.y - C.y) - __builtin_fma(dx, dx, dy * dy);
        const double n = rint(e);
        const float w = (float)ldexp(exp2_half(e - n), (int)fmax(n, -1000.0));
        const float* M = mom + ((size_t)a * ncell + c) * kSteinMom;
        float F[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            float s = 0.f;
#pragma unroll
            for (int j = 7; j >= 0; --j) {
                float g = 0.f;
#pragma unroll
                for (int i = 7; i >= 0; --i) g = __builtin_fmaf(fx[i], M[k * kSteinTerms + j * 8 + i], g);
                s = __builtin_fmaf(fy[j], g, s);
            }
            F[k] = s;
        }
        o0 = __builtin_fmaf(w, __builtin_fmaf(cb * (float)dx, F[0], F[1]), o0);
        o1 = __builtin_fmaf(w, __builtin_fmaf(cb * (float)dy, F[0], F[2]), o1);
    }
    if (wave > 0) {
        red[wave - 1][0][lane] = o0;
        red[wave - 1][1][lane] = o1;
    }
    __syncthreads();
    if (wave != 0 || tl.x + lane >= tl.y) return;
    for (int w = 0; w < 3; ++w) {
        o0 += red[w][0][lane];
        o1 += red[w][1][lane];
    }
    const int i = S.perm[q];
    const float invT = 1.0f / (float)S.n;
    phi[2 * (size_t)i] = o0 * invT;
    phi[2 * (size_t)i + 1] = o1 * invT;
}

}  // namespace

bool stein_cells_offered(int T, float h) {
    if (h <= 0.f) return true;
    const double side = std::sqrt(1.4426950408889634 / (double)h) / kSteinSide;
    const double cells = (side + 0.5) * (side + 0.5);   // random walks lie in 0.96 of these
    if (side > (1 << kSteinBits) || cells > kSteinCells) return false;
    const int c = std::max(1, (int)cells), chunks = c + T / std::max(512, (T / 128 + 255) / 256 * 256);
    const SteinTimes t = stein_times(T, c, chunks, c / 2 + T / kSteinTile);
    // (the model is a fifth too kind to many cells of few points: 32768 points, h = 0.004, 225
    // cells, 316 us against 283 direct)
    return t.cell < 0.8f * t.direct;
}

bool stein_cells_for(int T, int d) { return d == 2 && T >= kSteinCellMinT && T <= kSteinCellMaxT; }

void stein_cells_layout(Arena& a, SteinCells& S, int T, float* spare, size_t spare_floats) {
    S.n = T;
    S.per = std::max(256, (T + 1023) / 1024);
    S.per = (S.per + 63) / 64 * 64;
    S.nb = (T + S.per - 1) / S.per;
    S.kc = std::max(512, (T / 128 + 255) / 256 * 256);
    S.chmax = T / S.kc + kSteinCells;
    S.tmax = T / kSteinTile + kSteinCells;
    S.box = a.take<unsigned>(5 * kSteinBoxes);
    S.id = a.take<unsigned short>(T);
    S.bh = a.take<unsigned>((size_t)S.nb * kSteinIds);
    S.first = a.take<unsigned>(kSteinIds);
    S.perm = a.take<int>(T);
    S.rec = a.take<float4>(T);
    S.cen = a.take<float4>(kSteinCells);
    S.chunk = a.take<int4>(S.chmax);
    S.tile = a.take<int4>(S.tmax);
    S.own = a.take<int2>(kSteinCells);
    S.cnt = a.take<int>(4);
    S.room = (long long)spare_floats;
    S.mom = spare;
}

hipError_t launch_stein_cells(const SteinCells& S, const float4* krec, const float* h, float* phi,
                              float* h_used, hipStream_t s) {
    hipLaunchKernelGGL(k_st_box, dim3(kSteinBoxes), dim3(256), 0, s, S, krec);
    hipLaunchKernelGGL(k_st_hist, dim3(S.nb), dim3(256), 0, s, S, krec);
    hipLaunchKernelGGL(k_st_scan, dim3(kSteinIds / 64), dim3(256), 0, s, S);
    hipLaunchKernelGGL(k_st_lists, dim3(1), dim3(kSteinIds), 0, s, S);
    hipLaunchKernelGGL(k_st_scatter, dim3(S.nb), dim3(64), 0, s, S, krec);
    hipLaunchKernelGGL(k_st_moments, dim3(S.chmax, kSteinCells / 32), dim3(kStWaves * 64), 0, s, S, h);
    hipLaunchKernelGGL(k_st_reduce, dim3(4 * kNumCU), dim3(256), 0, s, S);
    hipLaunchKernelGGL(k_st_values, dim3(S.tmax), dim3(256), 0, s, S, S.mom, h, phi, h_used);
    return hipGetLastError();
}

}  // namespace ct
