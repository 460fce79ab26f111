// Multi-workgroup LDS-resident solve of a small Sinkhorn problem: the K
// iterations of the cross and self sweeps (Sec. II-B, eq. 5 solved by
// Sinkhorn's algorithm; eq. 6's self terms) in one launch of G workgroups
// without grid barriers.
//
// Every block holds all points (their records) in LDS and owns some rows (8 to 64) of
// each point set: rows [b*xr, (b+1)*xr) of x (the f and p updates) and [b*yr,
// (b+1)*yr) of y (the g and q updates).  An iteration k of a block:
//   gather g and p of version k; finish and publish q(k); sweep f;
//   finish and publish f(k+1); sweep p; gather f(k+1) and q(k);
//   finish and publish p(k+1); sweep g; finish and publish g(k+1); sweep q.
// A sweep gives each thread two own rows and a subset of the keys: the lanes of a wave
// split over row pairs first and keys for the rest (all of them where a block owns two
// rows), the waves split over the remaining row pairs and key ranges.  Two rows per
// thread read each key record once for two terms: one row per thread is bound by LDS
// reads.  Lane sums go through DPP and permlane swaps, waves' partials through LDS.
// What bounds an iteration of a small problem is the chain of two exchanges (a
// published word takes about a microsecond to be seen), which is why the self sweeps
// (p, q) run while the cross potentials travel and are finished half an iteration
// late by other waves than the cross rows.  At 1000 points the sweeps' own issue time
// is the larger part, hence as few rows per block as the device has room for.
// LOCAL (one block, at most 128 points a side): the finished rows write their records
// directly and nothing is exchanged; its registers are not bound to two blocks per
// compute unit.  A self sweep's rows write theirs only after the next barrier (put_rows):
// its records are those that a rescued row walks again, and more than 64 rows are finished
// by two waves that do not wait for each other.  That costs 0.06 us an iteration of 3.39 at
// T = M = 100; two copies of the self records by the iteration's parity cost 0.65 (their
// addresses are no longer the same in every iteration), one wave for all self rows 0.27.  Measured, us per iteration (d = 3, cached reference; before: 64 rows
// per block, one row per lane, f and p published together): T = M = 100 3.5 (4.9 in
// the one-workgroup solve), 300 5.3 (7.9), 500 5.6 (10.0), 1000 8.0 (14.5), 2000 12.1
// (24.9).  Launching a block per compute unit at 1024 threads (no two resident) was
// 0.3 us faster at 8 rows, but leaves room for one solve less on each hardware queue.
//
// Potentials travel as 64-bit words (version << 32 | float bits), stored and
// polled with relaxed device-scope atomics: a reader waits until a word carries
// the version it needs, so each value brings its own synchronisation and no
// block writes back or invalidates a cache (a grid barrier's release and
// acquire fences do, and cost several microseconds at every half-iteration).
// Words of version v live in buffer v mod 2.  No word is overwritten before every
// reader has taken it: version v + 2 of f (p) is published after the gather of g at
// version v + 1 (of f at v + 2), which waits on every block with y (x) rows, and each
// of them publishes those only after its own reads of version v; the same holds for g
// and q with x and y exchanged, and a block without rows of one set is waited on
// through its rows of the other, which every block has.  The buffers are filled with a
// never-matching version before each launch.
//
// All G blocks must be resident together (the plan keeps G at or below what
// fits).  Every wait is bounded; a wait that gives up sets a flag that makes
// every later wait pass at once, marks the outputs invalid and makes the status
// query report it, so even a broken launch finishes.
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>

#include "ct_internal.h"
#include "lds_solve.h"

namespace ct {

namespace {

using namespace lds_solve;

__device__ __forceinline__ unsigned long long ldx(const unsigned long long* w) {
    return __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// |v'|^2 from a record's (2v'): a power-of-two scaling of the same FMA chain, so
// the same float as when formed from v' itself.
__device__ __forceinline__ float rec_norm(float x2, float y2, float z2) {
    return 0.25f * __builtin_fmaf(x2, x2, __builtin_fmaf(y2, y2, z2 * z2));
}

// Gather one or two potentials (the second: null xch for none) into the key records.  A thread
// takes up to kMeshGatherPerThread words: their first loads are issued together, then each
// word not yet at the awaited version is polled on its own.
struct Gather {
    const unsigned long long* xch;   // [2][n]
    int n;                           // points
    int rec;                         // record array that takes H = h - |v'|^2
    int lw;                          // log2 mass, or -1: the constant log2a
    unsigned version;                // awaited
};
template <int NT>
__device__ __forceinline__ void gather(const MeshArgs& A, const Gather& G0, const Gather& G1,
                                       float* lds) {
    const int tid = (int)threadIdx.x;
    const int n0 = G0.n, ntot = n0 + G1.n;
    const unsigned long long* X0 = G0.xch + (size_t)(G0.version & 1u) * G0.n;
    const unsigned long long* X1 = G1.xch + (size_t)(G1.version & 1u) * G1.n;
    for (int e0 = tid; e0 < ntot; e0 += NT * kMeshGatherPerThread) {
        unsigned long long w[kMeshGatherPerThread];
#pragma unroll
        for (int s = 0; s < kMeshGatherPerThread; ++s) {
            const int e = e0 + s * NT;
            if (e < ntot) w[s] = e < n0 ? ldx(X0 + e) : ldx(X1 + (e - n0));
        }
#pragma unroll
        for (int s = 0; s < kMeshGatherPerThread; ++s) {
            const int e = e0 + s * NT;
            if (e >= ntot) break;
            const bool sec = e >= n0;
            const int i = sec ? e - n0 : e;
            const unsigned long long* a = sec ? X1 + i : X0 + i;
            const unsigned want = (sec ? G1.version : G0.version) + A.version_extra;
            unsigned spins = 0;
            while ((unsigned)(w[s] >> 32) != want) {
                if (spins >= A.polls ||
                    __hip_atomic_load(A.expired, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) {
                    atomicOr(A.expired, 1u);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
                ++spins;
                w[s] = ldx(a);
            }
            const float v = __uint_as_float((unsigned)w[s]);
            const int lw = sec ? G1.lw : G0.lw;
            const float l = lw >= 0 ? lds[lw + i] : A.log2a;
            float* rec = lds + 4 * ((sec ? G1.rec : G0.rec) + i);
            rec[3] = __builtin_fmaf(v, A.kappa, l) - rec_norm(rec[0], rec[1], rec[2]);
        }
    }
}

__device__ __forceinline__ void publish(unsigned long long* xch, int n, int row, unsigned version,
                                        float v) {
    const unsigned long long word = ((unsigned long long)version << 32) | __float_as_uint(v);
    __hip_atomic_store(xch + (size_t)(version & 1u) * n + row, word, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// One point set's own rows as a thread sees them: two rows (slots r and r + 2^(lg-1) of
// 2^lg), swept over every 2^(11-lg)-th key.  Lanes of a wave that share rows sit 2^(lg-1)
// apart, so a wave reads 2^(7-lg) adjacent records at a time.
struct Rows {
    int first, n, lg, sub, nsub, slot;
    float q[2][3], nrm[2];
};
template <int D, int NT>
__device__ __forceinline__ Rows rows_of(const MeshArgs& A, bool yside, int b, const float4* lds4) {
    Rows R;
    const int tid = (int)threadIdx.x, N = yside ? A.M : A.T, per = yside ? A.yr : A.xr;
    R.first = min(N, b * per);
    R.n = min(N, R.first + per) - R.first;
    R.lg = yside ? A.ly : A.lx;
    const int half = 1 << (R.lg - 1);
    R.slot = tid & (half - 1);
    R.sub = tid >> (R.lg - 1);
    R.nsub = NT >> (R.lg - 1);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        // slots past the last row repeat it; nothing reads their sums
        const int i = R.first + max(0, min(R.n - 1, R.slot + r * half));
        const float4 v = lds4[(yside ? A.o_rg : A.o_rf) + min(i, N - 1)];
        R.q[r][0] = 0.5f * v.x;
        R.q[r][1] = 0.5f * v.y;
        R.q[r][2] = 0.5f * v.z;
        R.nrm[r] = rec_norm(v.x, v.y, v.z);
    }
    return R;
}

// Sum over the lanes whose numbers agree modulo `step` (a power of two), the same in each of
// them.  Rotations inside rows of 16 lanes, then swaps of rows and halves: register moves, a
// tenth of the latency of shuffles through LDS.
template <int CTRL>
__device__ __forceinline__ float rot(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float swap16(float v) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
__device__ __forceinline__ float swap32(float v) {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
__device__ __forceinline__ float lane_sum(float v, int step) {
    if (step >= 64) return v;
    if (step == 32) return swap32(v);
    if (step == 16) return swap32(swap16(v));
    v += rot<0x128>(v);   // row_ror:8
    if (step < 8) {
        v += rot<0x124>(v);
        if (step < 4) {
            v += rot<0x122>(v);
            if (step < 2) v += rot<0x121>(v);
        }
    }
    return swap32(swap16(v));
}

// (m, s) and (m2, s2): a sum of 2^(e - m) each.
__device__ __forceinline__ void join(float& m, float& s, float m2, float s2) {
    const float t = fmaxf(m, m2);
    const float u = t == -__builtin_huge_valf() ? 0.f : t;
    s = s * tex2(m - u) + s2 * tex2(m2 - u);
    m = t;
}

// Sums of the own rows over all keys with a tracked maximum, left as the waves' partials
// part[0][wave][row] (sums) and part[1][wave][row] (maxima).  Out of line: only a cold first
// iteration and CT_SAFE_LSE run it, and the loop's code should stay in the instruction cache.
template <int D, int NT>
__device__ __attribute__((noinline)) void sweep_tracked(const Rows R, const float4* kr, int keys,
                                                        int prows, float* part) {
    const int half = 1 << (R.lg - 1), tid = (int)threadIdx.x, st = R.nsub;
    float C[2], m[2], s[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        m[r] = -__builtin_huge_valf();
        C[r] = -R.nrm[r];
        s[r] = 0.f;
    }
    for (int j = R.sub; j < keys; j += st) {
        const float4 k = kr[j];
#pragma unroll
        for (int r = 0; r < 2; ++r) m[r] = fmaxf(m[r], kdot<D>(k, R.q[r]) + C[r]);
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) C[r] -= m[r] == -__builtin_huge_valf() ? 0.f : m[r];
    for (int j = R.sub; j < keys; j += st) {
        const float4 k = kr[j];
#pragma unroll
        for (int r = 0; r < 2; ++r) s[r] += tex2(kdot<D>(k, R.q[r]) + C[r]);
    }
    for (int x = half; x < 64; x <<= 1) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const float s2 = __shfl_xor(s[r], x), m2 = __shfl_xor(m[r], x);
            // the same order of the pair in both lanes
            float ma = (tid & x) ? m2 : m[r], sa = (tid & x) ? s2 : s[r];
            join(ma, sa, (tid & x) ? m[r] : m2, (tid & x) ? s[r] : s2);
            m[r] = ma;
            s[r] = sa;
        }
    }
    if ((tid & 63) < half) {
        float* P = part + (tid >> 6) * prows + R.slot;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            P[r * half] = s[r];
            P[(NT / 64) * prows + r * half] = m[r];
        }
    }
}

// The same with the rows' own potentials as shifts: sums only.
template <int D, int NT>
__device__ __forceinline__ void sweep_rows(const MeshArgs& A, const Rows& R, const float4* kr,
                                           int keys, const float* pot, bool lagged, float* part) {
    if (R.n <= 0) return;
    if (!lagged) {
        sweep_tracked<D, NT>(R, kr, keys, A.rows, part);
        return;
    }
    const int half = 1 << (R.lg - 1), tid = (int)threadIdx.x, st = R.nsub;
    float C[2], acc[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
#pragma unroll
    for (int r = 0; r < 2; ++r)
        C[r] = __builtin_fmaf(pot[min(R.n - 1, R.slot + r * half)], A.kappa, -R.nrm[r]);
    int j = R.sub;
    // four keys' records in flight together
    for (; j + 3 * st < keys; j += 4 * st) {
        float4 k[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) k[u] = kr[j + u * st];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int r = 0; r < 2; ++r) acc[r][u & 1] += tex2(kdot<D>(k[u], R.q[r]) + C[r]);
    }
    for (; j < keys; j += st) {
        const float4 k = kr[j];
#pragma unroll
        for (int r = 0; r < 2; ++r) acc[r][0] += tex2(kdot<D>(k, R.q[r]) + C[r]);
    }
    const float s0 = lane_sum(acc[0][0] + acc[0][1], half), s1 = lane_sum(acc[1][0] + acc[1][1], half);
    if ((tid & 63) < half) {
        float* P = part + (tid >> 6) * A.rows + R.slot;
        P[0] = s0;
        P[half] = s1;
    }
}

// A row whose lagged sum left [2^-64, 2^64], with a tracked maximum over every key.
template <int D>
__device__ __attribute__((noinline)) float tracked_row(const float4 c, const float4* kr, int keys) {
    const float q[1][3] = {{c.x, c.y, D == 3 ? c.z : 0.f}};
    const float C[1] = {-norm2<D>(c)};
    float m[1], s[1];
    sum_safe<D, 1>(kr, 0, keys, q, C, m, s);
    return m[0] + __log2f(s[0]);
}

// Finish the own rows from the waves' partials: their new potentials, kept and published
// (or, one block, written into the key records; of a self sweep by put_rows).  By the threads from wave `w0` on, one wave
// or (more than 64 rows) two.
template <int D, int NT, bool LOCAL>
__device__ __forceinline__ void finish_rows(const MeshArgs& A, const Rows& R, int w0, bool yside,
                                            bool avg, const float4* kr, int keys, float* pot,
                                            bool lagged, const float* part, unsigned long long* xch,
                                            float* rec, const float* lw, unsigned version) {
    const int rows = 1 << R.lg, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (R.n <= 0 || wave < w0 || wave >= w0 + max(1, rows >> 6)) return;
    // opaque, so that what follows from it is formed here and not kept across iterations (70
    // registers, the difference between one and two blocks per compute unit)
    int t = (int)threadIdx.x - w0 * 64;
    if (!LOCAL) asm volatile("" : "+v"(t));
    const int row = t & (rows - 1);
    const int groups = rows >= 64 ? 1 : 64 >> R.lg;   // lanes that share a row
    const int row_c = min(row, R.n - 1);
    const float old = pot[row_c];
    const float* P = part + row;
    const int g = (t >> R.lg) & (groups - 1);
    float m, s = 0.f;
    if (lagged) {
        m = -old * A.kappa;
        // a uniform count of reads per lane, four in flight (lanes beyond the waves add nothing)
        const int n = max(1, NT / 64 / groups), st = groups * A.rows;
        const float* Q = P + min(g, NT / 64 - 1) * A.rows;
        if (n >= 4) {
            for (int i = 0; i < n; i += 4) s += (Q[i * st] + Q[(i + 1) * st]) + (Q[(i + 2) * st] + Q[(i + 3) * st]);
        } else {
            for (int i = 0; i < n; ++i) s += Q[i * st];
        }
        s = lane_sum(g < NT / 64 ? s : 0.f, rows);
    } else {
        m = -__builtin_huge_valf();
        for (int w = g; w < NT / 64; w += groups) join(m, s, P[(NT / 64 + w) * A.rows], P[w * A.rows]);
        for (int x = rows; x < 64; x <<= 1) join(m, s, __shfl_xor(m, x), __shfl_xor(s, x));
    }
    if (t >= rows || row >= R.n) return;
    float lse = m + __log2f(s);
    if (lagged && !(s >= kLo && s <= kHi)) {
        lse = tracked_row<D>((yside ? A.cy : A.cx)[R.first + row], kr, keys);
        atomicAdd(A.rescued, 1u);
    }
    const float tn = -lse * A.inv_kappa;
    const float nv = avg ? 0.5f * (old + tn) : tn;
    pot[row] = nv;
    if (LOCAL) {
        float* r = rec + 4 * row;
        if (!avg) r[3] = __builtin_fmaf(nv, A.kappa, lw ? lw[row] : A.log2a) - rec_norm(r[0], r[1], r[2]);
    } else {
        publish(xch, yside ? A.M : A.T, R.first + row, version, nv);
    }
}

// One block: the records of self rows that finish_rows has finished before the last barrier, by
// the same threads.
__device__ __forceinline__ void put_rows(const MeshArgs& A, const Rows& R, int w0, float* rec,
                                         const float* pot, const float* lw) {
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (wave < w0 || wave >= w0 + max(1, (1 << R.lg) >> 6)) return;
    const int row = (int)threadIdx.x - w0 * 64;
    if (row < R.n) {
        float* r = rec + 4 * row;
        r[3] = __builtin_fmaf(pot[row], A.kappa, lw ? lw[row] : A.log2a) - rec_norm(r[0], r[1], r[2]);
    }
}

extern __shared__ float4 mesh_lds4[];

// Block b of one problem's exchange solve.
template <int D, int NT, bool LOCAL>
__device__ __forceinline__ void mesh_solve(const MeshArgs& A, const int b) {
    float4* lds4 = mesh_lds4;
    float* lds = reinterpret_cast<float*>(lds4);
    const int tid = (int)threadIdx.x;
    const float kap = A.kappa;
    const int x0 = min(A.T, b * A.xr), x1 = min(A.T, x0 + A.xr);
    const int y0 = min(A.M, b * A.yr), y1 = min(A.M, y0 + A.yr);

    // load: every point's record (2v', .w filled by the gathers) and log2 b; the own rows'
    // potentials (indexed from the block's first own row), published as version 0
    for (int i = tid; i < A.T; i += NT) {
        const float4 c = A.cx[i];
        const float4 r = make_float4(2.f * c.x, 2.f * c.y, D == 3 ? 2.f * c.z : 0.f, 0.f);
        lds4[A.o_rf + i] = r;
        if (A.debias) {
            const float p = LOCAL ? A.p[i] : 0.f;
            lds4[A.o_rp + i] = make_float4(r.x, r.y, r.z, __builtin_fmaf(p, kap, A.log2a) -
                                                              rec_norm(r.x, r.y, r.z));
        }
    }
    for (int j = tid; j < A.M; j += NT) {
        const float4 c = A.cy[j];
        const float4 r = make_float4(2.f * c.x, 2.f * c.y, D == 3 ? 2.f * c.z : 0.f, 0.f);
        const float lb = A.log2b[j], n = rec_norm(r.x, r.y, r.z);
        const float g = LOCAL ? A.g[j] : 0.f, q = LOCAL ? A.q[j] : 0.f;
        lds4[A.o_rg + j] = make_float4(r.x, r.y, r.z, __builtin_fmaf(g, kap, lb) - n);
        if (A.ref_iter) lds4[A.o_rq + j] = make_float4(r.x, r.y, r.z, __builtin_fmaf(q, kap, lb) - n);
        lds[A.o_lb + j] = lb;
    }
    for (int i = x0 + tid; i < x1; i += NT) {
        lds[A.o_f + i - x0] = A.f[i];   // f's version 0 is never awaited: iteration 0 reads version 1
        if (A.debias) {
            const float p = A.p[i];
            lds[A.o_p + i - x0] = p;
            if (!LOCAL) publish(A.xch_p, A.T, i, 0u, p);
        }
    }
    for (int j = y0 + tid; j < y1; j += NT) {
        const float g = A.g[j];
        lds[A.o_g + j - y0] = g;
        if (!LOCAL) publish(A.xch_g, A.M, j, 0u, g);
        if (A.ref_iter) {
            const float q = A.q[j];
            lds[A.o_q + j - y0] = q;
            if (!LOCAL) publish(A.xch_q, A.M, j, 0u, q);
        }
    }
    __syncthreads();
    const Rows X = rows_of<D, NT>(A, false, b, lds4), Y = rows_of<D, NT>(A, true, b, lds4);
    const float4 *rf = lds4 + A.o_rf, *rg = lds4 + A.o_rg, *rp = lds4 + A.o_rp, *rq = lds4 + A.o_rq;
    float *pf = lds + A.o_f, *pg = lds + A.o_g, *pp = lds + A.o_p, *pq = lds + A.o_q;
    float *cross = lds + A.o_cross, *self = lds + A.o_self;
    const Gather none{A.xch_f, 0, 0, -1, 0u};

    // An iteration: f over the keys of g, p while the new f travels, g over the keys of f, q
    // while the new g travels (and before the next f).  p is finished and published after the
    // wait for f, q after the next wait for g: each arrives half an iteration before it is
    // read.  Waves 0 (1) finish the cross rows, waves 2 (3) the self rows, beside the sweep
    // that the others have begun.
    bool lag_q = false;   // mode of the sweep of q that waits to be finished
    for (int k = 0; k < A.iters; ++k) {
        const bool lagged = !A.safe_only && (A.lagged0 || k > 0);
        const unsigned v = (unsigned)k;
        if (!LOCAL)
            gather<NT>(A, Gather{A.xch_g, A.M, A.o_rg, A.o_lb, v},
                   A.debias ? Gather{A.xch_p, A.T, A.o_rp, -1, v} : none, lds);
        __syncthreads();
        if (A.ref_iter && k > 0)
            finish_rows<D, NT, LOCAL>(A, Y, 2, true, true, rq, A.M, pq, lag_q, self, A.xch_q,
                           lds + 4 * A.o_rq, lds + A.o_lb, v);
        sweep_rows<D, NT>(A, X, rg, A.M, pf, lagged, cross);
        __syncthreads();
        if (LOCAL && A.ref_iter && k > 0) put_rows(A, Y, 2, lds + 4 * A.o_rq, pq, lds + A.o_lb);
        finish_rows<D, NT, LOCAL>(A, X, 0, false, false, rg, A.M, pf, lagged, cross, A.xch_f,
                       lds + 4 * A.o_rf, nullptr, v + 1u);
        if (A.debias) sweep_rows<D, NT>(A, X, rp, A.T, pp, lagged, self);
        if (!LOCAL)
            gather<NT>(A, Gather{A.xch_f, A.T, A.o_rf, -1, v + 1u},
                   A.ref_iter ? Gather{A.xch_q, A.M, A.o_rq, A.o_lb, v} : none, lds);
        __syncthreads();
        if (A.debias)
            finish_rows<D, NT, LOCAL>(A, X, 2, false, true, rp, A.T, pp, lagged, self, A.xch_p,
                           lds + 4 * A.o_rp, nullptr, v + 1u);
        sweep_rows<D, NT>(A, Y, rf, A.T, pg, lagged, cross);
        __syncthreads();
        if (LOCAL && A.debias) put_rows(A, X, 2, lds + 4 * A.o_rp, pp, nullptr);
        finish_rows<D, NT, LOCAL>(A, Y, 0, true, false, rf, A.T, pg, lagged, cross, A.xch_g,
                       lds + 4 * A.o_rg, lds + A.o_lb, v + 1u);
        if (A.ref_iter) {
            sweep_rows<D, NT>(A, Y, rq, A.M, pq, lagged, self);
            lag_q = lagged;
        }
    }
    __syncthreads();
    if (A.ref_iter && A.iters > 0)
        finish_rows<D, NT, LOCAL>(A, Y, 2, true, true, rq, A.M, pq, lag_q, self, A.xch_q, lds + 4 * A.o_rq,
                       lds + A.o_lb, (unsigned)A.iters);
    __syncthreads();

    // store the own rows: potentials and the key terms the final pass reads
    const int hofs = D == 2 ? 2 : 3;
    for (int i = x0 + tid; i < x1; i += NT) {
        const float f = lds[A.o_f + i - x0];
        A.f[i] = f;
        reinterpret_cast<float*>(A.xrec_f + i)[hofs] = __builtin_fmaf(f, kap, A.log2a);
        if (A.debias) {
            const float p = lds[A.o_p + i - x0];
            A.p[i] = p;
            reinterpret_cast<float*>(A.xrec_p + i)[hofs] = __builtin_fmaf(p, kap, A.log2a);
        }
    }
    for (int j = y0 + tid; j < y1; j += NT) {
        const float g = lds[A.o_g + j - y0], lb = lds[A.o_lb + j];
        A.g[j] = g;
        reinterpret_cast<float*>(A.yrec_g + j)[hofs] = __builtin_fmaf(g, kap, lb);
        if (A.ref_iter) {
            const float q = lds[A.o_q + j - y0];
            A.q[j] = q;
            reinterpret_cast<float*>(A.yrec_q + j)[hofs] = __builtin_fmaf(q, kap, lb);
        }
    }
}

// NT threads per block: 512 (two blocks to a compute unit) or 1024; one block (LOCAL) 512.
template <int D, int NT, bool LOCAL>
__global__ __launch_bounds__(NT, LOCAL ? 2 : 4) void k_mesh(MeshArgs A) {
    mesh_solve<D, NT, LOCAL>(A, (int)blockIdx.x);
}

// Many problems in one launch: blk_end[p] is the end of problem p's blocks.  A
// block finds its problem, copies the problem's arguments into LDS and runs that
// problem's exchange solve as its block (blockIdx.x - start).  Every problem
// exchanges only among its own blocks.
template <int D>
__global__ __launch_bounds__(kMeshBatchThreads, 4) void k_mesh_batch(const MeshArgs* __restrict__ tab,
                                                             const int* __restrict__ blk_end,
                                                             int nprob) {
    __shared__ MeshArgs sA;
    const int bid = (int)blockIdx.x;
    int lo = 0, hi = nprob - 1;   // first problem whose blocks end after bid
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (blk_end[mid] > bid) hi = mid;
        else lo = mid + 1;
    }
    const int start = lo ? blk_end[lo - 1] : 0;
    const unsigned* src = reinterpret_cast<const unsigned*>(tab + lo);
    unsigned* dst = reinterpret_cast<unsigned*>(&sA);
    for (int i = (int)threadIdx.x; i < (int)(sizeof(MeshArgs) / 4); i += kMeshBatchThreads) dst[i] = src[i];
    __syncthreads();
    mesh_solve<D, kMeshBatchThreads, false>(sA, bid - start);
}

// A batch of problems of one block each: the one-block form, problem blockIdx.x.  (Exchanging
// with itself through device memory such a batch took longer than in blocks of 1024 threads: 250
// problems of 64 x 64 with values, 40 iterations, 314 us against 276; in this form 258.)
template <int D>
__global__ __launch_bounds__(kMeshBatchThreads, 2) void k_mesh_batch_local(const MeshArgs* __restrict__ tab) {
    const MeshArgs A = tab[blockIdx.x];
    mesh_solve<D, kMeshBatchThreads, true>(A, 0);
}

}  // namespace

bool mesh_plan(int T, int M, int d, bool debias, bool ref_iter, size_t lds_cap, bool allow_single,
               int rows, int threads, MeshArgs& A, size_t& lds_bytes, int* blocks) {
    std::memset(&A, 0, sizeof(A));
    lds_bytes = 0;
    *blocks = 0;
    const int most = std::max(T, M);
    const int need = (most + kMeshRows - 1) / kMeshRows;
    if (need < (allow_single ? 1 : 2) || need > kMeshMaxBlocks) return false;
    if (rows > kMeshRows && most > rows) return false;
    const int G = (most + rows - 1) / rows;
    A.T = T;
    A.M = M;
    A.debias = debias;
    A.ref_iter = ref_iter;
    A.threads = threads;
    A.local = G == 1 && rows > kMeshRows;
    A.xr = (T + G - 1) / G;
    A.yr = (M + G - 1) / G;
    // row slots: at least two (a thread has two rows), so that a wave's lanes split keys too
    auto lg = [](int n) {
        int l = 1;
        while ((1 << l) < n) ++l;
        return l;
    };
    A.lx = lg(A.xr);
    A.ly = lg(A.yr);
    A.rows = 1 << std::max(A.lx, A.ly);
    int r4 = 0;
    A.o_rf = r4; r4 += T;
    A.o_rg = r4; r4 += M;
    A.o_rp = r4; r4 += debias ? T : 0;
    A.o_rq = r4; r4 += ref_iter ? M : 0;
    int off = 4 * r4;
    auto take = [&](int n) {
        const int o = off;
        off += n;
        return o;
    };
    // own rows only
    A.o_f = take(A.xr);
    A.o_g = take(A.yr);
    A.o_p = take(debias ? A.xr : 0);
    A.o_q = take(ref_iter ? A.yr : 0);
    A.o_lb = take(M);
    A.o_cross = take(2 * (threads / 64) * A.rows);
    A.o_self = take(debias || ref_iter ? 2 * (threads / 64) * A.rows : 0);
    lds_bytes = (size_t)off * sizeof(float);
    if (lds_bytes > lds_cap) return false;
    *blocks = G;
    return true;
}

hipError_t ensure_dynamic_lds(const void* fn, size_t bytes) {
    if (bytes <= (size_t(64) << 10)) return hipSuccess;
    static std::mutex mu;
    static std::map<std::pair<int, const void*>, size_t> set;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lk(mu);
    size_t& cur = set[std::make_pair(dev, fn)];
    if (bytes <= cur) return hipSuccess;
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) cur = bytes;
    return e;
}

enum MeshKernel { kOne512, kOne1024, kOneLocal, kBatch };
static const void* mesh_kernel(int d, int which) {
    switch (which) {
        case kOne512:
            return d == 2 ? reinterpret_cast<const void*>(&k_mesh<2, 512, false>)
                          : reinterpret_cast<const void*>(&k_mesh<3, 512, false>);
        case kOne1024:
            return d == 2 ? reinterpret_cast<const void*>(&k_mesh<2, 1024, false>)
                          : reinterpret_cast<const void*>(&k_mesh<3, 1024, false>);
        case kOneLocal:
            return d == 2 ? reinterpret_cast<const void*>(&k_mesh<2, 512, true>)
                          : reinterpret_cast<const void*>(&k_mesh<3, 512, true>);
        default:
            return d == 2 ? reinterpret_cast<const void*>(&k_mesh_batch<2>)
                          : reinterpret_cast<const void*>(&k_mesh_batch<3>);
    }
}
static int mesh_which(const MeshArgs& A) {
    return A.local ? kOneLocal : A.threads == 1024 ? kOne1024 : kOne512;
}

static int resident_blocks(int d, size_t lds_bytes, int which, int threads) {
    static std::mutex mu;
    static std::map<std::pair<int, std::pair<int, size_t>>, int> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    const auto key = std::make_pair(dev * 4 + which, std::make_pair(d, lds_bytes));
    std::lock_guard<std::mutex> lk(mu);
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    int per_cu = 0, cus = 0;
    const void* fn = mesh_kernel(d, which);
    if (ensure_dynamic_lds(fn, lds_bytes) != hipSuccess)
        per_cu = 0;
    else if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, lds_bytes) != hipSuccess)
        per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 0;
    const int n = std::max(0, per_cu) * std::max(0, cus);
    cache.emplace(key, n);
    return n;
}

int mesh_resident_blocks(int d, size_t lds_bytes, const MeshArgs* one) {
    return one ? resident_blocks(d, lds_bytes, mesh_which(*one), one->threads)
               : resident_blocks(d, lds_bytes, kBatch, kMeshBatchThreads);
}

bool mesh_choose(int T, int M, int d, bool debias, bool ref_iter, size_t lds_cap, bool allow_single,
                 MeshArgs& A, size_t& lds_bytes, int* blocks) {
    // test and tuning hook: at most so many own rows per block
    int force = 0;
    if (const char* e = std::getenv("CT_MESH_ROWS")) force = std::atoi(e);
    auto plan = [&](int rows, int threads, int share) {
        return mesh_plan(T, M, d, debias, ref_iter, lds_cap, allow_single, rows, threads, A,
                         lds_bytes, blocks) &&
               *blocks * share <= mesh_resident_blocks(d, lds_bytes, &A);
    };
    if ((force == 0 || force == kMeshLocalRows) && plan(kMeshLocalRows, 512, 1)) return true;
    for (int rows = 8; rows <= 16; rows *= 2)
        if ((force == 0 || force == rows) && plan(rows, 512, 4)) return true;
    if ((force == 0 || force == 32) && plan(32, 1024, 4)) return true;
    return plan(kMeshRows, 1024, 1) || plan(kMeshRows, 512, 1);   // (512 threads: less LDS)
}

hipError_t launch_mesh(int d, const MeshArgs& A, size_t lds_bytes, int blocks, hipStream_t s) {
    hipEvent_t e0, e1;
    void* tok = profile_kernel_begin(&e0, &e1);
    const double pairs = (double)A.iters * ((double)A.T * A.M * 2 + (A.debias ? (double)A.T * A.T : 0.0) +
                                            (A.ref_iter ? (double)A.M * A.M : 0.0));
    {
        const hipError_t e = ensure_dynamic_lds(mesh_kernel(d, mesh_which(A)), lds_bytes);
        if (e != hipSuccess) return e;
    }
    auto go = [&](auto kernel) {
        if (e0) hipExtLaunchKernelGGL(kernel, dim3(blocks), dim3(A.threads), lds_bytes, s, e0, e1, 0, A);
        else hipLaunchKernelGGL(kernel, dim3(blocks), dim3(A.threads), lds_bytes, s, A);
    };
    const int which = mesh_which(A);
    if (which == kOneLocal) d == 2 ? go(k_mesh<2, 512, true>) : go(k_mesh<3, 512, true>);
    else if (which == kOne512) d == 2 ? go(k_mesh<2, 512, false>) : go(k_mesh<3, 512, false>);
    else d == 2 ? go(k_mesh<2, 1024, false>) : go(k_mesh<3, 1024, false>);
    const hipError_t e = hipGetLastError();
    // kind 40/41: a multi-workgroup exchange solve (safe / lagged from its first iteration)
    profile_kernel_end(tok, 40 + A.lagged0, 0, 0, blocks, pairs);
    return e;
}

hipError_t launch_mesh_batch(int d, const MeshArgs* tab, const int* blk_end, int nprob, bool local,
                             size_t lds_bytes, int blocks, double pairs, hipStream_t s) {
    hipEvent_t e0, e1;
    void* tok = profile_kernel_begin(&e0, &e1);
    {
        // set when the batch was planned (so not during a graph capture of the run)
        const hipError_t e = local ? hipSuccess : ensure_dynamic_lds(mesh_kernel(d, kBatch), lds_bytes);
        if (e != hipSuccess) return e;
    }
    auto go = [&](auto kernel, auto... args) {
        if (e0) hipExtLaunchKernelGGL(kernel, dim3(blocks), dim3(kMeshBatchThreads), lds_bytes, s, e0, e1, 0, args...);
        else hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kMeshBatchThreads), lds_bytes, s, args...);
    };
    if (local) d == 2 ? go(k_mesh_batch_local<2>, tab) : go(k_mesh_batch_local<3>, tab);
    else d == 2 ? go(k_mesh_batch<2>, tab, blk_end, nprob) : go(k_mesh_batch<3>, tab, blk_end, nprob);
    const hipError_t e = hipGetLastError();
    // kind 42: the exchange solve of a whole batch in one launch
    profile_kernel_end(tok, 42, 0, 0, blocks, pairs);
    return e;
}

}  // namespace ct
