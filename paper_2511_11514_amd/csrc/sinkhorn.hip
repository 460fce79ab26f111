// ct_sinkhorn_grad: debiased Sinkhorn divergence gradient for one problem
// (Sec. II-B, eqs. 5-7).  Staging, the iteration schedule, the final
// extrapolation pass and the reductions; the sweeps themselves are in sweep.hip.
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>

#include "cells.h"
#include "ct_internal.h"

namespace ct {

constexpr double kLog2e = 1.4426950408889634;
constexpr int kCounters = 8;   // words of a call's device-side conditions (see OutArgs)

// ------------------------------------------------------------------ kernels

__global__ __launch_bounds__(256) void k_zero3(unsigned* a, int na, unsigned* b, int nb,
                                               unsigned* c, int nc) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (a && i < na) a[i] = 0u;
    if (b && i < nb) b[i] = 0u;
    if (c && i < nc) c[i] = 0u;
}

// A fixed-order sum over blocks' partial sums part[b][NV], b < nb <= 64, by the first wave; every
// lane of it gets the totals.
constexpr int kSumBlocks = 64;
template <int NV>
__device__ __forceinline__ void total(const double* __restrict__ part, int nb, double* v) {
    const int lane = (int)threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        double s = lane < nb ? part[(size_t)lane * NV + k] : 0.0;
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) s += __shfl_xor(s, m);
        v[k] = s;
    }
}
// The block's sums of each thread's v[NV] (256 threads) into out[NV].
template <int NV>
__device__ __forceinline__ void block_total(const double* v, double* __restrict__ out) {
    __shared__ double red[4][NV];
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        double s = v[k];
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) s += __shfl_xor(s, m);
        if (lane == 0) red[wave][k] = s;
    }
    __syncthreads();
    if ((int)threadIdx.x < NV)
        out[threadIdx.x] = (red[0][threadIdx.x] + red[1][threadIdx.x]) +
                           (red[2][threadIdx.x] + red[3][threadIdx.x]);
}

// What every call begins with, in one launch (six before: with k_out and k_value a flow call at
// T = M = 100 takes 383 us instead of 393; at 65536 + 262144 points the two sums took 255 and
// 72 us in one block each): partial sums of the points'
// coordinates and of the reference weights, cleared arrival tickets and counters, and the
// exchange solve's words filled with ones (a version that no exchange awaits).
//
// The common origin of both point sets is the mean of every coordinate (double, fixed order,
// non-finite values skipped).  The soft-min is translation invariant, but the float32 prescale
// x * sqrt(kappa) is not: far from the coordinate origin it would round away the low bits of
// every difference x_i - y_j.  Subtracting the origin first (exact for nearby float32 values)
// keeps them.
constexpr int kBeginSums = 5;    // sums of x, y, z, the points counted, the weights
struct BeginArgs {
    const float *x, *y, *w;
    int T, M, d, nt, nx;
    double* part;            // [blocks][kBeginSums]
    unsigned* tick[3];       // [nt] each
    unsigned* counters;
    unsigned long long* xch; // [nx]
};
__global__ __launch_bounds__(256) void k_begin(BeginArgs A) {
    const int tid = (int)(blockIdx.x * 256 + threadIdx.x), nthr = (int)gridDim.x * 256;
    for (int i = tid; i < A.nt; i += nthr)
        for (int k = 0; k < 3; ++k) A.tick[k][i] = 0u;
    if (tid < kCounters) A.counters[tid] = 0u;
    for (int i = tid; i < A.nx; i += nthr) A.xch[i] = ~0ull;
    double s[kBeginSums] = {0.0, 0.0, 0.0, 0.0, 0.0};
    const long long n = (long long)A.T + A.M, chunk = (n + gridDim.x - 1) / gridDim.x;
    const long long i0 = min(n, (long long)blockIdx.x * chunk), i1 = min(n, i0 + chunk);
    // a skipped point adds zeros (no branch), so eight loads can be in flight
#pragma unroll 8
    for (long long i = i0 + (int)threadIdx.x; i < i1; i += 256) {
        const float* p = i < A.T ? A.x + (size_t)i * A.d : A.y + (size_t)(i - A.T) * A.d;
        float v[3] = {0.f, 0.f, 0.f};
        bool ok = true;
        for (int t = 0; t < A.d; ++t) {
            v[t] = p[t];
            ok = ok && isfinite(v[t]);
        }
        for (int t = 0; t < A.d; ++t) s[t] += ok ? (double)v[t] : 0.0;
        s[3] += ok ? 1.0 : 0.0;
    }
    if (A.w) {
#pragma unroll 8
        for (int j = tid; j < A.M; j += nthr) s[4] += (double)A.w[j];
    } else if (tid == 0) {
        s[4] = (double)A.M;
    }
    block_total<kBeginSums>(s, A.part + (size_t)blockIdx.x * kBeginSums);
}

// The origin and the weights' sum from k_begin's partials, by the first wave.
__device__ __forceinline__ void begin_totals(const double* __restrict__ part, int nb, int d,
                                             float* origin, double* wsum) {
    double v[kBeginSums];
    total<kBeginSums>(part, nb, v);
    if (threadIdx.x == 0) {
        const double c = v[3] > 0.0 ? v[3] : 1.0;
        for (int t = 0; t < 3; ++t) origin[t] = t < d ? (float)(v[t] / c) : 0.f;
        *wsum = v[4];
    }
}
// The same into the workspace, for the partition into cells, which precedes k_stage.
__global__ __launch_bounds__(64) void k_totals(const double* __restrict__ part, int nb, int d,
                                               float* __restrict__ origin, double* __restrict__ wsum) {
    begin_totals(part, nb, d, origin, wsum);
}

struct StageArgs {
    const float* x;
    const float* y;
    const float* w;
    const float* pot_in;     // [2T+2M] warm start (f, g, p, q) or null
    int warm, ref_cached;
    int T, M, d, Tpad, Mpad;
    float sqrt_kappa, kappa, log2a;
    const double* part;      // k_begin's partial sums
    int nb;                  // of so many blocks
    double* wsum;            // out
    float4* cx;              // query coordinates of x
    float4* cy;              // query coordinates of y
    float4* xrec[4];         // key records of x: f (g-sweeps), f+ (g+ sweep), p ping-pong
    float4* yrec[3];         // key records of y: g (f-sweeps), q ping-pong
    float* b;
    float* log2b;
    float *f, *g, *p, *q;
    float *fp, *gp, *pp, *qp; // extrapolated potentials, zeroed here
    unsigned* nonfinite;
};

__device__ __forceinline__ float4 make_rec(const float* c, int d, float h) {
    return d == 2 ? make_float4(c[0], c[1], h, 0.f) : make_float4(c[0], c[1], c[2], h);
}

// Pre-scale coordinates, form the reference masses and the initial key records
// (h = log2 mass + kappa * potential; padding records get h = -inf).
__global__ __launch_bounds__(256) void k_stage(StageArgs A) {
    __shared__ float origin[3];      // subtracted before scaling
    __shared__ double wsum;
    if (threadIdx.x < 64) {
        begin_totals(A.part, A.nb, A.d, origin, &wsum);
        if (blockIdx.x == 0 && threadIdx.x == 0) *A.wsum = wsum;
    }
    __syncthreads();
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const float ninf = -__builtin_huge_valf();
    if (i < A.Tpad) {
        float c[3] = {0.f, 0.f, 0.f};
        if (i < A.T) {
            bool bad = false;
            for (int t = 0; t < A.d; ++t) {
                const float v = A.x[(size_t)i * A.d + t];
                bad |= !isfinite(v);
                c[t] = (v - origin[t]) * A.sqrt_kappa;
            }
            A.cx[i] = make_float4(c[0], c[1], c[2], 0.f);
            const float f0 = A.warm ? A.pot_in[i] : 0.f;
            const float p0 = A.warm ? A.pot_in[(size_t)A.T + A.M + i] : 0.f;
            A.f[i] = f0;
            A.p[i] = p0;
            A.fp[i] = 0.f;
            A.pp[i] = 0.f;
            A.xrec[0][i] = make_rec(c, A.d, ninf);
            A.xrec[1][i] = make_rec(c, A.d, ninf);
            A.xrec[2][i] = make_rec(c, A.d, __builtin_fmaf(p0, A.kappa, A.log2a));
            A.xrec[3][i] = make_rec(c, A.d, ninf);
            if (bad) atomicAdd(A.nonfinite, 1u);
        } else {
            for (int r = 0; r < 4; ++r) A.xrec[r][i] = make_rec(c, A.d, ninf);
        }
    }
    if (i < A.Mpad) {
        float c[3] = {0.f, 0.f, 0.f};
        if (i < A.M) {
            bool bad = false;
            for (int t = 0; t < A.d; ++t) {
                const float v = A.y[(size_t)i * A.d + t];
                bad |= !isfinite(v);
                c[t] = (v - origin[t]) * A.sqrt_kappa;
            }
            A.cy[i] = make_float4(c[0], c[1], c[2], 0.f);
            const float wj = A.w ? A.w[i] : 1.f;
            bad |= !(wj > 0.f) || !isfinite(wj);
            const float bj = (float)((double)wj / wsum);
            const float lb = __log2f(bj);
            A.b[i] = bj;
            A.log2b[i] = lb;
            const float g0 = A.warm ? A.pot_in[(size_t)A.T + i] : 0.f;
            const float q0 = (A.warm || A.ref_cached) ? A.pot_in[2 * (size_t)A.T + A.M + i] : 0.f;
            A.g[i] = g0;
            A.q[i] = q0;
            A.gp[i] = 0.f;
            A.qp[i] = 0.f;
            A.yrec[0][i] = make_rec(c, A.d, __builtin_fmaf(g0, A.kappa, lb));
            A.yrec[1][i] = make_rec(c, A.d, __builtin_fmaf(q0, A.kappa, lb));
            A.yrec[2][i] = make_rec(c, A.d, ninf);
            if (bad) atomicAdd(A.nonfinite, 1u);
        } else {
            for (int r = 0; r < 3; ++r) A.yrec[r][i] = make_rec(c, A.d, ninf);
        }
    }
}

// What every call ends with, in two launches (k_out and, with a value or grad_w, k_value; up to
// eleven before, and at 65536 + 262144 points 233 us in one block for the sums).
struct OutArgs {
    int T, M, d, debias, need_ref, want_v;
    int nb;                     // blocks that sum (k_out's first)
    float kappa, two_a;
    const float *dy, *ds;       // ds: null unless debiased
    const float *f, *g, *p, *q, *fp, *gp, *pp, *qp, *b;
    const double* wsum;
    unsigned* counters;         // [0] non-finite inputs, [1] rescued rows, [2] residual (float
                                // bits), [3] 1 once the residual is written, [4] a wait of a
                                // one-launch solve gave up
    const int *perm_x, *perm_y; // the caller's index of each row, or null
    double* part;               // [nb][kOutSums]
    float *grad_x, *grad_w, *value, *pot, *pot_plus, *aux;
};
constexpr int kOutSums = 8;

__device__ __forceinline__ void aux_counters(const OutArgs& A) {
    A.aux[4] = (float)A.counters[1];
    A.aux[5] = (float)A.counters[0];
    A.aux[6] = A.counters[4] ? 1.f : 0.f;
    A.aux[7] = 0.f;
}

// grad_x = 2 a (Ds - Dy)  (debiased) or -2 a Dy, NaN after a one-launch solve gave up; the
// potentials pot = (f [T], g [M], p [T], q [M]) and pot_plus; partial sums of the dual
// objectives, <b,G> and the column residual (double, fixed order).
__global__ __launch_bounds__(256) void k_out(OutArgs A) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    const int T = A.T, M = A.M;
    if (i < (long long)T * A.d) {
        const float v = A.ds ? A.ds[i] - A.dy[i] : -A.dy[i];
        const size_t at = A.perm_x ? (size_t)A.perm_x[i / A.d] * A.d + i % A.d : (size_t)i;
        A.grad_x[at] = A.counters[4] ? __builtin_nanf("") : A.two_a * v;
    }
    if (A.pot || A.pot_plus) {
        if (i < T) {
            const size_t x = A.perm_x ? (size_t)A.perm_x[i] : (size_t)i, p = (size_t)T + M + x;
            if (A.pot) {
                A.pot[x] = A.f[i];
                A.pot[p] = A.p[i];
            }
            if (A.pot_plus) {
                A.pot_plus[x] = A.fp[i];
                A.pot_plus[p] = A.pp[i];
            }
        }
        if (i < M) {
            const size_t y = (size_t)T + (A.perm_y ? (size_t)A.perm_y[i] : (size_t)i), q = (size_t)T + M + y;
            if (A.pot) {
                A.pot[y] = A.g[i];
                A.pot[q] = A.q[i];
            }
            if (A.pot_plus) {
                A.pot_plus[y] = A.gp[i];
                A.pot_plus[q] = A.qp[i];
            }
        }
    }
    if (!A.want_v) {
        if (A.aux && blockIdx.x == 0 && threadIdx.x == 0) {
            for (int k = 0; k < 4; ++k) A.aux[k] = 0.f;
            aux_counters(A);
        }
        return;
    }
    if ((int)blockIdx.x >= A.nb) return;
    double acc[kOutSums] = {0, 0, 0, 0, 0, 0, 0, 0};
    const double invT = 1.0 / T;
    const int stride = A.nb * 256;
    for (long long k = i; k < T; k += stride) {
        acc[0] += A.fp[k] * invT;
        if (A.debias) {
            acc[1] += A.pp[k] * invT;
            acc[2] += A.p[k] * invT;
        }
    }
    for (long long j = i; j < M; j += stride) {
        const double bj = A.b[j];
        acc[3] += bj * A.g[j];
        if (A.need_ref) {
            acc[4] += bj * A.qp[j];
            acc[5] += bj * A.q[j];
        }
        const double G = A.need_ref ? (double)A.gp[j] - (double)A.qp[j] : (double)A.gp[j];
        acc[6] += bj * G;
        acc[7] += bj * fabs(exp2(((double)A.g[j] - (double)A.gp[j]) * (double)A.kappa) - 1.0);
    }
    block_total<kOutSums>(acc, A.part + (size_t)blockIdx.x * kOutSums);
}

// Dual objectives, value and residual (block 0), and grad_w = (G - <b,G>) / sum w.
__global__ __launch_bounds__(256) void k_value(OutArgs A) {
    __shared__ double bG;
    if (threadIdx.x < 64) {
        double r[kOutSums];
        total<kOutSums>(A.part, A.nb, r);
        if (threadIdx.x == 0) {
            bG = r[6];
            if (blockIdx.x == 0) {
                const double ot_ab = r[0] + r[3], ot_aa = r[1] + r[2], ot_bb = r[4] + r[5];
                const double S = A.debias ? ot_ab - 0.5 * ot_aa - 0.5 * ot_bb : ot_ab;
                if (A.value) *A.value = A.counters[4] ? __builtin_nanf("") : (float)S;
                if (A.aux) {
                    A.aux[0] = (float)ot_ab;
                    A.aux[1] = A.debias ? (float)ot_aa : 0.f;
                    A.aux[2] = A.need_ref ? (float)ot_bb : 0.f;
                    A.aux[3] = (float)r[7];
                    aux_counters(A);
                }
                A.counters[2] = __float_as_uint((float)r[7]);
                A.counters[3] = 1u;
            }
        }
    }
    __syncthreads();
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (!A.grad_w || j >= A.M) return;
    const double G = A.need_ref ? (double)A.gp[j] - (double)A.qp[j] : (double)A.gp[j];
    A.grad_w[A.perm_y ? A.perm_y[j] : j] = A.counters[4] ? __builtin_nanf("") : (float)((G - bG) / *A.wsum);
}

// --------------------------------------------------------------- layout

struct SkLayout {
    double* wsum;
    unsigned* counters;      // [8]: see OutArgs
    float4* cx;
    float4* cy;
    float4* xrec[4];         // 0: h from f (keys of g-sweeps), 1: from f+, 2/3: from p (ping-pong)
    float4* yrec[3];         // 0: h from g (keys of f-sweeps), 1/2: from q (ping-pong)
    float* origin;           // [4] common origin subtracted before scaling
    float* b;
    float* log2b;
    float *f, *g, *p, *q;
    float *fp, *gp, *pp, *qp;
    float *dy, *ds;
    float* part[3];          // partial buffers: cross jobs, x self jobs, y self jobs
    unsigned* tick[3];
    size_t ntick;
    unsigned* bar;           // [kFusedBarWords] barrier words of the fused solve
    unsigned long long* xch; // [2 (2T + 2M)] versioned potential words of the exchange solve
    bool cells;              // the cell form's arrays are there:
    CellPrep prep;           //   partitions, sorted inputs, mode
    float* mom[3];           //   moments: cross, x self, y self
    float* mu[3];
    size_t bytes;
};


// Cell form of the sweeps (see cells.h): by default where the library would launch one
// direct sweep at a time and the call is large enough (cell_limits), up to kCellMaxPoints
// points a side (cell codes sorted by at most 256 blocks).  Whether it pays and fits
// for the points at hand, k_cell_gather settles on the device.  CT_UNFUSED, CT_DIFFERENCE,
// CT_SAFE_LSE and the flags of the other executions rule it out, and so does a workspace
// without its arrays.  The workspace's size, its layout and the dispatch ask the same question.
constexpr size_t kCellMomentsMax = size_t(96) << 20;   // floats of one moments buffer
constexpr double kMeshAutoPairs = 1.5e7;

struct CellSweeps {
    bool cross = false, x = false, y = false;   // f and g, x against itself, y against itself
    bool any() const { return cross || x || y; }
};

// The sweeps of a call that are offered the cell form.
static CellSweeps cell_sweeps(int T, int M, const ct_sinkhorn_opts* o) {
    CellSweeps s;
    const bool debias = o->flags & CT_DEBIAS;
    const bool need_ref = debias && (o->flags & (CT_VALUE | CT_GRAD_W));
    const double pairs = 2.0 * T * M + (debias ? (double)T * T : 0.0) +
                         (need_ref && !(o->flags & CT_REF_CACHED) ? (double)M * M : 0.0);
    const CellLimits lim = cell_limits();
    if ((o->flags & (CT_UNFUSED | CT_DIFFERENCE | CT_SAFE_LSE | CT_FUSED | CT_TINY | CT_MESH)) ||
        o->iters < kCellMinIters || T > kCellMaxPoints || M > kCellMaxPoints ||
        pairs <= std::max(lim.pairs, kMeshAutoPairs) || o->iters * pairs <= lim.work)
        return s;
    s.cross = cell_candidate(o->d, T, M);
    s.x = debias && cell_candidate(o->d, T, T);
    s.y = need_ref && cell_candidate(o->d, M, M);
    if (!lim.expect) return s;
    const int kx = cell_chunk(T), ky = cell_chunk(M);
    CellOffer offer(o->d, o->eps, kCellLaunch, kGain, o->d == 2 ? 1.06 : 1.0);
    if (s.cross) {
        offer.sweep(T, M, kx, ky);
        offer.sweep(M, T, ky, kx);
    }
    if (s.x) offer.sweep(T, T, kx, kx);
    if (s.y && !(o->flags & CT_REF_CACHED)) offer.sweep(M, M, ky, ky);
    return offer.pays(o->iters, 150.0) ? s : CellSweeps();
}

static void cell_layout(Arena& a, SkLayout& L, int T, int M, int d, const CellSweeps& sweeps) {
    CellPrep& P = L.prep;
    std::memset(&P, 0, sizeof(P));
    cell_prep_layout(a, P, d, T, M, 0, 0, cell_chunk(T), cell_chunk(M));
    const int N = d == 2 ? CellDim<2>::N : CellDim<3>::N;
    for (int s = 0; s < 2; ++s)
        if (sweeps.cross || (s ? sweeps.y : sweeps.x))
            P.side[s].phi = a.take<float4>((size_t)P.side[s].tmax * N * 8);
    P.xs = a.take<float>((size_t)T * d);
    P.ys = a.take<float>((size_t)M * d);
    P.ws = a.take<float>(M);
    P.pot_s = a.take<float>(2 * ((size_t)T + M));
    const CellSide &X = P.side[0], &Y = P.side[1];
    const size_t rows[3] = {std::max((size_t)X.cmax * Y.chmax, (size_t)Y.cmax * X.chmax),
                            (size_t)X.cmax * X.chmax, (size_t)Y.cmax * Y.chmax};
    const bool on[3] = {sweeps.cross, sweeps.x, sweeps.y};
    for (int i = 0; i < 3; ++i) {
        L.mom[i] = L.mu[i] = nullptr;   // mom_cap 0: k_cell_gather leaves the sweep direct
        if (!on[i]) continue;
        const size_t r = std::min(rows[i], kCellMomentsMax / N);
        P.mom_cap[i] = r * N;
        L.mom[i] = a.take<float>(r * N);
        L.mu[i] = a.take<float>(r);
    }
}

// o: the call's options, or null for the layout without the cell form.
static SkLayout sk_layout(void* ws, int T, int M, int d, const ct_sinkhorn_opts* o) {
    Arena a(ws);
    SkLayout L;
    const int Tp = pad_keys(T), Mp = pad_keys(M);
    L.wsum = a.take<double>(1);
    L.counters = a.take<unsigned>(kCounters);
    L.cx = a.take<float4>(T);
    L.cy = a.take<float4>(M);
    for (int r = 0; r < 4; ++r) L.xrec[r] = a.take<float4>(Tp);
    for (int r = 0; r < 3; ++r) L.yrec[r] = a.take<float4>(Mp);
    L.origin = a.take<float>(4);
    L.b = a.take<float>(M);
    L.log2b = a.take<float>(M);
    L.f = a.take<float>(T);
    L.g = a.take<float>(M);
    L.p = a.take<float>(T);
    L.q = a.take<float>(M);
    L.fp = a.take<float>(T);
    L.gp = a.take<float>(M);
    L.pp = a.take<float>(T);
    L.qp = a.take<float>(M);
    L.dy = a.take<float>((size_t)T * d);
    L.ds = a.take<float>((size_t)T * d);
    L.part[0] = a.take<float>(std::max(job_part_floats_max(d, T, M), job_part_floats_max(d, M, T)));
    L.part[1] = a.take<float>(job_part_floats_max(d, T, T));
    L.part[2] = a.take<float>(job_part_floats_max(d, M, M));
    L.ntick = std::max(job_tickets_max(T), job_tickets_max(M));
    for (int i = 0; i < 3; ++i) L.tick[i] = a.take<unsigned>(L.ntick);
    L.bar = a.take<unsigned>(kFusedBarWords);
    L.xch = a.take<unsigned long long>(4 * ((size_t)T + M));
    const CellSweeps sweeps = o ? cell_sweeps(T, M, o) : CellSweeps();
    L.cells = sweeps.any();
    if (L.cells) cell_layout(a, L, T, M, d, sweeps);
    L.bytes = a.off + 256;
    return L;
}

static const uint32_t kKnownFlags = CT_DEBIAS | CT_GRAD_W | CT_VALUE | CT_WARM_START |
                                    CT_REF_CACHED | CT_SAFE_LSE | CT_ONE_STREAM | CT_FUSED |
                                    CT_UNFUSED | CT_DIFFERENCE | CT_TINY | CT_MESH;

static ct_status validate(const float* x, int64_t T, const float* y, int64_t M,
                          const ct_sinkhorn_opts* o) {
    if (!o) return fail(CT_E_ARG, "opts is null");
    if (o->d != 2 && o->d != 3) return fail(CT_E_SHAPE, "d must be 2 or 3 (got %d)", o->d);
    if (T < 1 || M < 1) return fail(CT_E_SHAPE, "T and M must be >= 1 (T=%lld, M=%lld)",
                                    (long long)T, (long long)M);
    if (T > (int64_t(1) << 30) || M > (int64_t(1) << 30))
        return fail(CT_E_SHAPE, "T and M must be <= 2^30");
    if (!(o->eps > 0.f) || !std::isfinite(o->eps))
        return fail(CT_E_ARG, "eps must be finite and > 0");
    if (o->iters < 0) return fail(CT_E_ARG, "iters must be >= 0");
    if (o->flags & ~kKnownFlags) return fail(CT_E_ARG, "unknown flag bits 0x%x", o->flags & ~kKnownFlags);
    {
        const uint32_t ex = o->flags & (CT_FUSED | CT_UNFUSED | CT_TINY | CT_MESH);
        if (ex & (ex - 1))
            return fail(CT_E_ARG, "CT_FUSED, CT_UNFUSED, CT_TINY and CT_MESH exclude each other");
    }
    if (!x || !y) return fail(CT_E_ARG, "x and y must be non-null");
    return CT_OK;
}

// Launch-time constants of one problem.
struct SkConsts {
    int d, T, M;
    int expanded;   // lagged sweeps without offsets in the expanded form (unless CT_DIFFERENCE)
    float kappa, inv_kappa, inv_sqrt_kappa, log2a;
};

static SkConsts sk_consts(int T, int M, const ct_sinkhorn_opts* o) {
    const double kappa_d = kLog2e / (double)o->eps;
    SkConsts c;
    c.d = o->d;
    c.T = T;
    c.M = M;
    c.expanded = (o->flags & CT_DIFFERENCE) ? 0 : 1;
    c.kappa = (float)kappa_d;
    c.inv_kappa = (float)(1.0 / kappa_d);
    c.inv_sqrt_kappa = (float)(1.0 / std::sqrt(kappa_d));
    c.log2a = (float)(-std::log2((double)T));
    return c;
}

struct JobSet {
    Job j[kMaxJobs];
    CellJob cell[kMaxJobs];
    int n = 0;
    void add(const Job& x, const CellJob& y = CellJob()) {
        if (x.nq > 0) {
            j[n] = x;
            cell[n++] = y;
        }
    }
};

// Sweep the jobs: in the cell form where `cells` has their arrays (else null).
static ct_status launch_set(const JobSet& js, const SkConsts& c, const Schedule& sc, bool lagged,
                            bool bary, const SkLayout* cells, hipStream_t st) {
    if (js.n == 0) return CT_OK;
    Launch Lc;
    std::memset(&Lc, 0, sizeof(Lc));
    Lc.kappa = c.kappa;
    Lc.inv_kappa = c.inv_kappa;
    Lc.inv_sqrt_kappa = c.inv_sqrt_kappa;
    Lc.expanded = c.expanded;
    int nb = 0;
    for (int i = 0; i < js.n; ++i) {
        Lc.job[i] = js.j[i];
        nb += plan_job(Lc.job[i], sc);
        Lc.blk_end[i] = nb;
    }
    Lc.njobs = js.n;
    if (cells) {
        CellLaunch C;
        std::memset(&C, 0, sizeof(C));
        for (int i = 0; i < 2; ++i) C.job[i] = js.cell[std::min(i, js.n - 1)];
        C.never = cells->prep.mode + 4;
        C.R = sc.R;
        C.WS = sc.WS;
        C.inv_cell = (float)(1.0 / cell_side(c.d));
        CT_CHECK_HIP(launch_cell_sweep(c.d, sc, lagged, Lc, C, nb, st));
        return CT_OK;
    }
    CT_CHECK_HIP(launch_sweep(c.d, sc, lagged, bary, Lc, nb, st));
    return CT_OK;
}

// Job builders: queries x against keys y (f-type) or x (p-type); queries y
// against keys x (g-type) or y (q-type).
struct SkJobs {
    const SkLayout& L;
    const SkConsts& c;
    Job base() const {
        Job j;
        std::memset(&j, 0, sizeof(Job));
        j.rescued = L.counters + 1;
        return j;
    }
    Job f(float* out_pot, float4* out_rec, float* out_bary) const {
        Job j = base();
        j.qrec = L.cx; j.qpot = L.f; j.qlog2w_s = c.log2a;
        j.krec = L.yrec[0]; j.nq = c.T; j.nk = c.M;
        j.part = L.part[0]; j.ticket = L.tick[0];
        j.out_pot = out_pot; j.out_rec = out_rec; j.out_bary = out_bary;
        return j;
    }
    Job p(int cur, bool avg, float* out_pot, float4* out_rec, float* out_bary) const {
        Job j = base();
        j.qrec = L.cx; j.qpot = L.p; j.qlog2w_s = c.log2a; j.self_avg = avg;
        j.krec = L.xrec[2 + cur]; j.nq = c.T; j.nk = c.T;
        j.part = L.part[1]; j.ticket = L.tick[1];
        j.out_pot = out_pot; j.out_rec = out_rec; j.out_bary = out_bary;
        return j;
    }
    Job g(const float4* krec, float* out_pot, float4* out_rec) const {
        Job j = base();
        j.qrec = L.cy; j.qpot = L.g; j.qlog2w = L.log2b;
        j.krec = krec; j.nq = c.M; j.nk = c.T;
        j.part = L.part[0]; j.ticket = L.tick[0];
        j.out_pot = out_pot; j.out_rec = out_rec;
        return j;
    }
    Job q(int cur, bool avg, float* out_pot, float4* out_rec) const {
        Job j = base();
        j.qrec = L.cy; j.qpot = L.q; j.qlog2w = L.log2b; j.self_avg = avg;
        j.krec = L.yrec[1 + cur]; j.nq = c.M; j.nk = c.M;
        j.part = L.part[2]; j.ticket = L.tick[2];
        j.out_pot = out_pot; j.out_rec = out_rec;
        return j;
    }
    // queries of side qs against keys of side ks (0: x, 1: y)
    CellJob cell(int qs, int ks) const {
        CellJob C;
        std::memset(&C, 0, sizeof(C));
        if (!L.cells) return C;
        const CellSide &Q = L.prep.side[qs], &K = L.prep.side[ks];
        const int b = qs != ks ? 0 : 1 + qs;   // the moments' buffer
        C.mode = L.prep.mode + (qs != ks ? qs : 2 + qs);
        C.ncq = Q.cnt;
        C.qcen = Q.cen;
        C.tile = Q.tile;
        C.ntile = Q.cnt + 2;
        C.phi = Q.phi;
        C.tmax = Q.tmax;
        C.nch = K.cnt + 1;
        C.chunk = K.chunk;
        C.chcen = K.chcen;
        C.mom = L.mom[b];
        C.mu = L.mu[b];
        return C;
    }
};

// One auxiliary stream per device (default priority, non-blocking), created on first use.
static ct_status aux_stream(hipStream_t* out) {
    static std::mutex mu;
    static std::map<int, hipStream_t> streams;
    int dev = 0;
    CT_CHECK_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(mu);
    auto it = streams.find(dev);
    if (it == streams.end()) {
        hipStream_t s;
        CT_CHECK_HIP(hipStreamCreateWithFlags(&s, hipStreamNonBlocking));
        it = streams.emplace(dev, s).first;
    }
    *out = it->second;
    return CT_OK;
}

// Auxiliary stream and fork/join events of the two-stream schedule, made once and
// reused by every call (the allocation-free entry point); null members: made and
// destroyed by each call.
struct ForkJoin {
    hipStream_t aux = nullptr;
    hipEvent_t fork = nullptr, join = nullptr;
};

// Fused solve (all K iterations in one launch; see fused.hip).  By default it is
// taken when one iteration has at most kFusedAutoPairs point pairs: there the
// per-sweep launches are bound by launch latency, and two grid barriers per
// iteration cost less than the four or five kernel boundaries they replace
// (measured on an MI355X, K = 100, d = 3, T = M: 1.2x at 200-300 samples per side,
// 1.04x at 500; at 1000, 3*10^6 pairs per iteration, the barriers' cross-die
// cache write-backs cost more than the launches, 4.3 against 2.7 ms).  CT_FUSED
// forces it and CT_UNFUSED rules it out.  The grid has at most kFusedMaxBlocks
// blocks and never more than can be resident at once.
constexpr double kFusedAutoPairs = 1048576.0;
constexpr int kFusedMaxBlocks = 512;
constexpr unsigned kFusedWaitPolls = 1u << 20;

static ct_status run_fused(const SkLayout& L, const SkConsts& c, const SkJobs& J,
                           const ct_sinkhorn_opts* o, bool debias, bool ref_iter, bool warm,
                           bool safe_only, hipStream_t st, bool* ran) {
    *ran = false;
    const int T = c.T, M = c.M, d = c.d;
    const bool forced = o->flags & CT_FUSED;
    const double pa = (double)T * M + (debias ? (double)T * T : 0.0);
    const double pb = (double)M * T + (ref_iter ? (double)M * M : 0.0);
    if (!forced && pa + pb > kFusedAutoPairs) return CT_OK;
    int gmax = std::min(fused_resident_blocks(d), kFusedMaxBlocks);
    // test and tuning hook: a cap on the grid
    if (const char* e = std::getenv("CT_FUSED_GRID"))
        gmax = std::min(std::min(fused_resident_blocks(d), kFusedMaxGrid),
                        std::max(1, std::atoi(e)));
    if (gmax < 1) {
        if (forced) return fail(CT_E_UNSUPPORTED, "the fused solve cannot place a block on this device");
        return CT_OK;
    }
    // partial buffers of the layout: cross jobs, trajectory self, reference self
    const size_t cap_cross = std::max(job_part_floats_max(d, T, M), job_part_floats_max(d, M, T));
    const size_t cap_p = job_part_floats_max(d, T, T), cap_q = job_part_floats_max(d, M, M);
    const Schedule fs{kFusedR, kFusedWS, 0, 0};
    FusedLaunch F;
    std::memset(&F, 0, sizeof(F));
    // plan every job for about the same pairs per unit, so that one half-iteration
    // is about one unit per block; coarser units if a job's partials would not fit
    double ppb = std::max(pa, pb) / gmax;
    int units_max = 0;
    for (int attempt = 0;; ++attempt) {
        bool fits = true;
        units_max = 0;
        auto add = [&](FusedPhase& P, Job j, size_t cap) {
            const int u = plan_job_target(j, fs, ppb);
            const size_t need = j.splits > 1 ? (size_t)(2 + d) * j.splits * (size_t)j.nqb * 64 *
                                                   kFusedR * (4 / kFusedWS)
                                             : 0;
            if (need > cap) fits = false;
            P.job[P.njobs] = j;
            P.unit_end[P.njobs] = (P.njobs ? P.unit_end[P.njobs - 1] : 0) + u;
            ++P.njobs;
            units_max = std::max(units_max, P.unit_end[P.njobs - 1]);
        };
        for (int par = 0; par < 2; ++par) {
            FusedPhase& A = F.ph[par][0];
            FusedPhase& B = F.ph[par][1];
            A.njobs = B.njobs = 0;
            add(A, J.f(L.f, L.xrec[0], nullptr), cap_cross);
            if (debias) add(A, J.p(par, true, L.p, L.xrec[2 + (par ^ 1)], nullptr), cap_p);
            add(B, J.g(L.xrec[0], L.g, L.yrec[0]), cap_cross);
            if (ref_iter) add(B, J.q(par, true, L.q, L.yrec[1 + (par ^ 1)]), cap_q);
        }
        if (fits) break;
        if (attempt >= 30) {
            if (forced) return fail(CT_E_UNSUPPORTED, "the fused solve found no plan for T=%d, M=%d", T, M);
            return CT_OK;
        }
        ppb *= 2.0;
    }
    F.iters = o->iters;
    F.lagged0 = warm ? 1 : 0;
    F.safe_only = safe_only ? 1 : 0;
    F.bar = L.bar;
    F.expired = L.counters + 4;
    F.wait_polls = kFusedWaitPolls;
    // test hooks of the give-up path: a poll bound, and waits that no arrival count satisfies
    if (const char* e = std::getenv("CT_FUSED_WAIT_POLLS")) F.wait_polls = (unsigned)std::strtoul(e, nullptr, 10);
    if (const char* e = std::getenv("CT_FUSED_UNSATISFIABLE_WAITS")) F.target_extra = std::atoi(e) ? 1u : 0u;
    F.kappa = c.kappa;
    F.inv_kappa = c.inv_kappa;
    F.inv_sqrt_kappa = c.inv_sqrt_kappa;
    hipLaunchKernelGGL(k_zero3, dim3((kFusedBarWords + 255) / 256), dim3(256), 0, st, L.bar,
                       kFusedBarWords, nullptr, 0, nullptr, 0);
    CT_CHECK_HIP(hipGetLastError());
    CT_CHECK_HIP(launch_fused(d, F, std::min(gmax, units_max), st));
    *ran = true;
    return CT_OK;
}

// One-workgroup solve (all K iterations in one workgroup, everything in LDS; see
// tiny.hip).  By default it is taken, where the exchange solve is not, when one
// iteration has at most kTinyAutoPairs point pairs and the problem fits in the
// LDS a workgroup may take: one compute unit evaluates such an iteration faster
// than the GPU can synchronise across its dies (measured on an MI355X, K = 100,
// d = 3, whole call: 0.59 ms at T = M = 100 against 1.34 for the fused solve and
// 1.41 for per-sweep launches).  CT_TINY forces it (CT_E_UNSUPPORTED when the
// problem does not fit); CT_FUSED, CT_UNFUSED and CT_MESH rule it out.
constexpr double kTinyAutoPairs = 150000.0;

static size_t device_max_lds() {
    static std::mutex mu;
    static std::map<int, size_t> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    std::lock_guard<std::mutex> lk(mu);
    auto it = cache.find(dev);
    if (it != cache.end()) return it->second;
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) v = 0;
    cache.emplace(dev, (size_t)std::max(0, v));
    return (size_t)std::max(0, v);
}

static ct_status run_tiny(const SkLayout& L, const SkConsts& c, const ct_sinkhorn_opts* o,
                          bool debias, bool ref_iter, bool warm, bool safe_only, hipStream_t st,
                          bool* ran) {
    *ran = false;
    const int T = c.T, M = c.M, d = c.d;
    const bool forced = o->flags & CT_TINY;
    const double pairs = 2.0 * T * M + (debias ? (double)T * T : 0.0) +
                         (ref_iter ? (double)M * M : 0.0);
    if (!forced && pairs > kTinyAutoPairs) return CT_OK;
    TinyArgs A;
    size_t lds = 0;
    const size_t cap = std::min(kTinyMaxLds, device_max_lds());
    // test and tuning hook: query rows per lane (1, 2 or 4) instead of the cost model's choice
    int r_force = 0;
    if (const char* e = std::getenv("CT_TINY_R")) {
        r_force = std::atoi(e);
        if (r_force != 1 && r_force != 2 && r_force != 4) r_force = 0;
    }
    if (!tiny_plan(T, M, d, debias, ref_iter, cap, r_force, A, lds)) {
        if (forced)
            return fail(CT_E_UNSUPPORTED, "T=%d, M=%d needs %zu bytes of LDS; the one-workgroup "
                                          "solve may take %zu", T, M, lds, cap);
        return CT_OK;
    }
    const int cur = o->iters & 1;   // the self record arrays current after K iterations
    A.cx = L.cx;
    A.cy = L.cy;
    A.log2b = L.log2b;
    A.f = L.f;
    A.g = L.g;
    A.p = L.p;
    A.q = L.q;
    A.xrec_f = L.xrec[0];
    A.yrec_g = L.yrec[0];
    A.xrec_p = L.xrec[2 + cur];
    A.yrec_q = L.yrec[1 + cur];
    A.rescued = L.counters + 1;
    A.d = d;
    A.iters = o->iters;
    A.lagged0 = warm ? 1 : 0;
    A.safe_only = safe_only ? 1 : 0;
    A.kappa = c.kappa;
    A.inv_kappa = c.inv_kappa;
    A.log2a = c.log2a;
    CT_CHECK_HIP(launch_tiny(d, A, lds, st));
    *ran = true;
    return CT_OK;
}

// Exchange solve (all K iterations in one launch of blocks that each hold every point
// in LDS; see mesh.hip and mesh_choose).  By default it is taken when it plans (every
// point in one block's LDS, all blocks resident at once) and one iteration has at most
// kMeshAutoPairs point pairs and more than kMeshMinPairs, or both sides fit its
// one-block form and one has more than kMeshMinPoints points (kMeshMinPointsRef where the
// reference is solved too): elsewhere the one-workgroup
// solve is as fast or faster (130 x 20 points: 490 us against 531; 20 x 400: 516 / 591;
// 130 x 60: 518 / 515).  Measured on an MI355X, K = 100, d = 3, T = M, whole call (exchange /
// one-workgroup), without a reference solve: T = 17: 295 / 289 us; 24: 295 / 302; 40: 329 /
// 341; 64: 327 / 346; 72: 354 / 479; with it: 17: 379 / 304; 40: 424 / 371; 64: 418 / 381; 66:
// 435 / 515; 20 x 65: 398 / 410; cached reference (exchange / fused / per-sweep
// launches): T = 300: 0.60 / 1.87 / 2.26 ms; 500: 0.64 / 2.63 / 2.66; 1000: 0.9 / 7.0 /
// 2.70; 2000: 1.3 / 23.5 / 3.13.  CT_MESH forces it (CT_E_UNSUPPORTED when it cannot
// plan); CT_FUSED, CT_UNFUSED and CT_TINY rule it out.
constexpr double kMeshMinPairs = 40000.0;
constexpr int kMeshMinPoints = 20, kMeshMinPointsRef = 64;
constexpr unsigned kMeshWaitPolls = 1u << 18;

static ct_status run_mesh(const SkLayout& L, const SkConsts& c, const ct_sinkhorn_opts* o,
                          bool debias, bool ref_iter, bool warm, bool safe_only, hipStream_t st,
                          bool* ran) {
    *ran = false;
    const int T = c.T, M = c.M, d = c.d;
    const bool forced = o->flags & CT_MESH;
    const double pairs = 2.0 * T * M + (debias ? (double)T * T : 0.0) +
                         (ref_iter ? (double)M * M : 0.0);
    if (!forced && (pairs > kMeshAutoPairs ||
                    (pairs <= kMeshMinPairs && (std::max(T, M) > kMeshLocalRows ||
                                                std::max(T, M) <= (ref_iter ? kMeshMinPointsRef
                                                                            : kMeshMinPoints)))))
        return CT_OK;
    MeshArgs A;
    size_t lds = 0;
    int blocks = 0;
    const size_t cap = std::min(kTinyMaxLds, device_max_lds());
    if (!mesh_choose(T, M, d, debias, ref_iter, cap, !forced, A, lds, &blocks)) {
        if (forced)
            return fail(CT_E_UNSUPPORTED, "the exchange solve has no plan for T=%d, M=%d (it needs "
                                          "a side of more than 64 points, at most %d blocks of at most %d rows and every point in "
                                          "%zu bytes of LDS)", T, M, kMeshMaxBlocks, kMeshRows, cap);
        return CT_OK;
    }
    const int cur = o->iters & 1;   // the self record arrays current after K iterations
    A.cx = L.cx;
    A.cy = L.cy;
    A.log2b = L.log2b;
    A.f = L.f;
    A.g = L.g;
    A.p = L.p;
    A.q = L.q;
    A.xrec_f = L.xrec[0];
    A.yrec_g = L.yrec[0];
    A.xrec_p = L.xrec[2 + cur];
    A.yrec_q = L.yrec[1 + cur];
    A.xch_f = L.xch;
    A.xch_p = L.xch + 2 * (size_t)T;
    A.xch_g = L.xch + 4 * (size_t)T;
    A.xch_q = L.xch + 4 * (size_t)T + 2 * (size_t)M;
    A.rescued = L.counters + 1;
    A.expired = L.counters + 4;
    A.polls = kMeshWaitPolls;
    // test hooks of the give-up path: a poll bound, and waits that no version satisfies
    if (const char* e = std::getenv("CT_MESH_WAIT_POLLS")) A.polls = (unsigned)std::strtoul(e, nullptr, 10);
    if (const char* e = std::getenv("CT_MESH_UNSATISFIABLE_WAITS")) A.version_extra = std::atoi(e) ? (1u << 20) : 0u;
    A.d = d;
    A.iters = o->iters;
    A.lagged0 = warm ? 1 : 0;
    A.safe_only = safe_only ? 1 : 0;
    A.kappa = c.kappa;
    A.inv_kappa = c.inv_kappa;
    A.log2a = c.log2a;
    CT_CHECK_HIP(launch_mesh(d, A, lds, blocks, st));
    *ran = true;
    return CT_OK;
}

// Iterate-and-extrapolate for one problem whose arrays are staged in L.
static ct_status run_problem(const SkLayout& L, int T, int M, const ct_sinkhorn_opts* o,
                             hipStream_t st, const ForkJoin* fj) {
    const int d = o->d;
    const SkLayout* cl = L.cells ? &L : nullptr;
    const bool debias = o->flags & CT_DEBIAS;
    const bool want_v = o->flags & (CT_VALUE | CT_GRAD_W);
    const bool need_ref = debias && want_v;
    const bool ref_iter = need_ref && !(o->flags & CT_REF_CACHED);
    const bool warm = o->flags & CT_WARM_START;
    const bool safe_only = o->flags & CT_SAFE_LSE;
    const SkConsts c = sk_consts(T, M, o);
    const SkJobs J{L, c};
    const Schedule sA = schedule_for(d, T, M);
    const Schedule sB = schedule_for(d, M, T);

    int cur = 0;  // which ping-pong self record array is current
    bool fused = false;
    if (o->iters > 0 && !(o->flags & CT_UNFUSED)) {
        if (!(o->flags & (CT_FUSED | CT_TINY))) {
            ct_status rc = run_mesh(L, c, o, debias, ref_iter, warm, safe_only, st, &fused);
            if (rc) return rc;
        }
        if (!fused && !(o->flags & (CT_FUSED | CT_MESH))) {
            ct_status rc = run_tiny(L, c, o, debias, ref_iter, warm, safe_only, st, &fused);
            if (rc) return rc;
        }
        if (!fused && !(o->flags & (CT_TINY | CT_MESH))) {
            ct_status rc = run_fused(L, c, J, o, debias, ref_iter, warm, safe_only, st, &fused);
            if (rc) return rc;
        }
        if (fused) cur = o->iters & 1;
    }

    // The self problems do not depend on f and g: their K sweeps run on the
    // auxiliary stream (forked from / joined back into `st` with events) while the
    // cross sweeps run on `st`; with CT_ONE_STREAM the same launches are serialised
    // on `st`.
    const bool any_self = !fused && (debias || ref_iter);
    const bool two_streams = any_self && o->iters > 0 && !(o->flags & CT_ONE_STREAM);
    hipStream_t sst = st;
    hipEvent_t fork = nullptr, join = nullptr;
    const bool own_events = !(fj && fj->fork);
    if (two_streams) {
        if (own_events) {
            ct_status rc = aux_stream(&sst);
            if (rc) return rc;
            CT_CHECK_HIP(hipEventCreateWithFlags(&fork, hipEventDisableTiming));
            CT_CHECK_HIP(hipEventCreateWithFlags(&join, hipEventDisableTiming));
        } else {
            sst = fj->aux;
            fork = fj->fork;
            join = fj->join;
        }
        CT_CHECK_HIP(hipEventRecord(fork, st));
        CT_CHECK_HIP(hipStreamWaitEvent(sst, fork, 0));
    }
    if (any_self) {
        const Schedule sS = schedule_for(d, ref_iter ? M : T, ref_iter ? M : T);
        for (int k = 0; k < o->iters; ++k) {
            const bool lagged = !safe_only && (warm || k > 0);
            JobSet Sf;
            if (debias) Sf.add(J.p(cur, true, L.p, L.xrec[2 + (cur ^ 1)], nullptr), J.cell(0, 0));
            if (ref_iter) Sf.add(J.q(cur, true, L.q, L.yrec[1 + (cur ^ 1)]), J.cell(1, 1));
            ct_status rc = launch_set(Sf, c, sS, lagged, false, cl, sst);
            if (rc) return rc;
            cur ^= 1;
        }
    }
    for (int k = 0; k < (fused ? 0 : o->iters); ++k) {
        const bool lagged = !safe_only && (warm || k > 0);
        JobSet A, B;
        A.add(J.f(L.f, L.xrec[0], nullptr), J.cell(0, 1));
        B.add(J.g(L.xrec[0], L.g, L.yrec[0]), J.cell(1, 0));
        ct_status rc = launch_set(A, c, sA, lagged, false, cl, st);
        if (rc) return rc;
        rc = launch_set(B, c, sB, lagged, false, cl, st);
        if (rc) return rc;
    }
    if (two_streams) {
        CT_CHECK_HIP(hipEventRecord(join, sst));
        CT_CHECK_HIP(hipStreamWaitEvent(st, join, 0));
        if (own_events) {
            CT_CHECK_HIP(hipEventDestroy(fork));
            CT_CHECK_HIP(hipEventDestroy(join));
        }
    }
    const bool lagged_final = !safe_only && (warm || o->iters > 0);
    {
        JobSet F;
        F.add(J.f(L.fp, L.xrec[1], L.dy));
        if (debias) F.add(J.p(cur, false, L.pp, nullptr, L.ds));
        ct_status rc = launch_set(F, c, sA, lagged_final, true, nullptr, st);
        if (rc) return rc;
    }
    if (want_v) {
        JobSet F;
        F.add(J.g(L.xrec[1], L.gp, nullptr), J.cell(1, 0));
        if (need_ref) F.add(J.q(ref_iter ? cur : 0, false, L.qp, nullptr), J.cell(1, 1));
        ct_status rc = launch_set(F, c, sB, lagged_final, false, cl, st);
        if (rc) return rc;
    }
    return CT_OK;
}

}  // namespace ct

using namespace ct;

extern "C" size_t ct_sinkhorn_workspace_size(int64_t T, int64_t M, const ct_sinkhorn_opts* o) {
    if (!o || (o->d != 2 && o->d != 3) || T < 1 || M < 1 || T > (int64_t(1) << 30) ||
        M > (int64_t(1) << 30))
        return 0;
    return sk_layout(nullptr, (int)T, (int)M, o->d, o).bytes;
}

namespace ct {

// Host checks of one gradient call's arguments (everything but the workspace).
static ct_status validate_call(const float* x, int64_t T64, const float* y, int64_t M64,
                               const ct_sinkhorn_opts* o, const float* grad_x,
                               const float* grad_w, const float* value, const float* pot) {
    ct_status rc = validate(x, T64, y, M64, o);
    if (rc) return rc;
    if (!grad_x) return fail(CT_E_ARG, "grad_x must be non-null");
    if (grad_w && !(o->flags & CT_GRAD_W)) return fail(CT_E_ARG, "grad_w given without CT_GRAD_W");
    if (!grad_w && (o->flags & CT_GRAD_W)) return fail(CT_E_ARG, "CT_GRAD_W needs grad_w");
    if (value && !(o->flags & CT_VALUE)) return fail(CT_E_ARG, "value given without CT_VALUE");
    if (!value && (o->flags & CT_VALUE)) return fail(CT_E_ARG, "CT_VALUE needs value");
    if (!pot && (o->flags & (CT_WARM_START | CT_REF_CACHED)))
        return fail(CT_E_ARG, "CT_WARM_START / CT_REF_CACHED need pot");
    return CT_OK;
}

// The whole gradient call on the workspace `ws` (both entry points).
static ct_status sinkhorn_grad_impl(const float* x, int64_t T64, const float* y, const float* w,
                                    int64_t M64, const ct_sinkhorn_opts* o, float* grad_x,
                                    float* grad_w, float* value, float* pot, float* pot_plus,
                                    float* aux, void* ws, size_t ws_bytes, void* stream,
                                    const ForkJoin* fj) {
    ct_status rc = validate_call(x, T64, y, M64, o, grad_x, grad_w, value, pot);
    if (rc) return rc;
    const int T = (int)T64, M = (int)M64, d = o->d;
    if (!ws) return fail(CT_E_ARG, "workspace is null");
    if (reinterpret_cast<uintptr_t>(ws) % 256) return fail(CT_E_WORKSPACE, "workspace not 256-byte aligned");
    // a workspace without room for the cell form's arrays serves the direct sweeps
    SkLayout L = sk_layout(ws, T, M, d, o);
    if (L.cells && ws_bytes < L.bytes) L = sk_layout(ws, T, M, d, nullptr);
    if (ws_bytes < L.bytes)
        return fail(CT_E_WORKSPACE, "workspace too small: %zu < %zu bytes", ws_bytes, L.bytes);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool debias = o->flags & CT_DEBIAS;
    const bool want_v = o->flags & (CT_VALUE | CT_GRAD_W);
    const bool need_ref = debias && want_v;
    const double kappa_d = kLog2e / (double)o->eps;

    // (fills by a kernel, no memset nodes, so the sequence can be captured into a graph; the
    // sums' partials use the words that the fused solve clears for its barrier)
    static_assert(kFusedBarWords * sizeof(unsigned) >= kSumBlocks * kOutSums * sizeof(double), "partials");
    BeginArgs B;
    B.x = x; B.y = y; B.w = w;
    B.T = T; B.M = M; B.d = d;
    B.nt = (int)L.ntick;
    for (int k = 0; k < 3; ++k) B.tick[k] = L.tick[k];
    B.counters = L.counters;
    B.xch = L.xch;
    const bool may_exchange = std::max(T, M) <= kMeshRows * kMeshMaxBlocks &&
                              !(o->flags & (CT_FUSED | CT_UNFUSED | CT_TINY));
    B.nx = may_exchange ? 4 * (T + M) : 0;
    B.part = reinterpret_cast<double*>(L.bar);
    const int nsum = (int)std::min<int64_t>(kSumBlocks, (T64 + M64 + 1023) / 1024);
    hipLaunchKernelGGL(k_begin, dim3(nsum), dim3(256), 0, st, B);
    CT_CHECK_HIP(hipGetLastError());
    const bool pot_given = o->flags & (CT_WARM_START | CT_REF_CACHED);
    const int* perm_x = nullptr;
    const int* perm_y = nullptr;
    StageArgs A;
    A.x = x; A.y = y; A.w = w; A.pot_in = pot;
    if (L.cells) {
        // everything below works on the points in cell order; the outputs go back through
        // the permutations
        CellPrep& P = L.prep;
        P.origin = L.origin;
        hipLaunchKernelGGL(k_totals, dim3(1), dim3(64), 0, st, B.part, nsum, d, L.origin, L.wsum);
        CT_CHECK_HIP(hipGetLastError());
        CT_CHECK_HIP(launch_cell_prep(P, CellInputs{x, y, w, pot_given ? pot : nullptr,
                                                    (float)std::sqrt(kappa_d)}, st));
        A.x = P.xs;
        A.y = P.ys;
        A.w = w ? P.ws : nullptr;
        A.pot_in = pot_given ? P.pot_s : nullptr;
        perm_x = P.side[0].perm;
        perm_y = P.side[1].perm;
    }
    A.warm = (o->flags & CT_WARM_START) ? 1 : 0;
    A.ref_cached = (o->flags & CT_REF_CACHED) ? 1 : 0;
    A.T = T; A.M = M; A.d = d; A.Tpad = pad_keys(T); A.Mpad = pad_keys(M);
    A.sqrt_kappa = (float)std::sqrt(kappa_d);
    A.kappa = (float)kappa_d;
    A.log2a = (float)(-std::log2((double)T));
    A.part = B.part; A.nb = nsum; A.wsum = L.wsum; A.cx = L.cx; A.cy = L.cy; A.b = L.b; A.log2b = L.log2b;
    A.f = L.f; A.g = L.g; A.p = L.p; A.q = L.q;
    for (int r = 0; r < 4; ++r) A.xrec[r] = L.xrec[r];
    for (int r = 0; r < 3; ++r) A.yrec[r] = L.yrec[r];
    A.fp = L.fp; A.gp = L.gp; A.pp = L.pp; A.qp = L.qp;
    A.nonfinite = L.counters;
    const int n = std::max(pad_keys(T), pad_keys(M));
    hipLaunchKernelGGL(k_stage, dim3((n + 255) / 256), dim3(256), 0, st, A);
    CT_CHECK_HIP(hipGetLastError());

    rc = run_problem(L, T, M, o, st, fj);
    if (rc) return rc;

    OutArgs R;
    R.T = T; R.M = M; R.d = d; R.debias = debias; R.need_ref = need_ref; R.want_v = want_v;
    R.kappa = (float)kappa_d;
    R.two_a = (float)(2.0 / T);
    R.dy = L.dy; R.ds = debias ? L.ds : nullptr;
    R.f = L.f; R.g = L.g; R.p = L.p; R.q = L.q;
    R.fp = L.fp; R.gp = L.gp; R.pp = L.pp; R.qp = L.qp;
    R.b = L.b; R.wsum = L.wsum; R.counters = L.counters;
    R.perm_x = perm_x; R.perm_y = perm_y;
    R.part = B.part;
    R.grad_x = grad_x; R.grad_w = grad_w; R.value = value;
    R.pot = pot; R.pot_plus = pot_plus; R.aux = aux;
    const int64_t rows = std::max<int64_t>((int64_t)T * d, M);
    const int nout = (int)((rows + 255) / 256);
    R.nb = std::min(nsum, nout);
    hipLaunchKernelGGL(k_out, dim3(nout), dim3(256), 0, st, R);
    CT_CHECK_HIP(hipGetLastError());
    if (want_v) {
        hipLaunchKernelGGL(k_value, dim3(grad_w ? (M + 255) / 256 : 1), dim3(256), 0, st, R);
        CT_CHECK_HIP(hipGetLastError());
    }
    return CT_OK;
}

// ------------------------------------------------- allocation-free variant
// Scratch of ct_sinkhorn_grad_static: one array per device, held until the process
// ends.  Host code never passes `scratch` itself (its host name is a stand-in, not
// a device address): each device's address comes from hipGetSymbolAddress once,
// with that device current, and is kept in g_static below.
constexpr size_t kStaticScratchBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

struct StaticDevice {
    void* ptr = nullptr;   // device address of `scratch` on this device
    ForkJoin fj;           // auxiliary stream and events made at set-up
};

// Per-device set-up on the first call on that device: the scratch address, the
// auxiliary stream and the fork/join events.  Later calls only look them up.
static ct_status static_device(StaticDevice* out) {
    static std::mutex mu;
    static std::map<int, StaticDevice> devs;
    int dev = 0;
    CT_CHECK_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(mu);
    auto it = devs.find(dev);
    if (it == devs.end()) {
        StaticDevice sd;
        CT_CHECK_HIP(hipGetSymbolAddress(&sd.ptr, HIP_SYMBOL(scratch)));
        if (!sd.ptr || reinterpret_cast<uintptr_t>(sd.ptr) % 256)
            return fail(CT_E_HIP, "static scratch has no usable device address on device %d", dev);
        ct_status rc = aux_stream(&sd.fj.aux);
        if (rc) return rc;
        CT_CHECK_HIP(hipEventCreateWithFlags(&sd.fj.fork, hipEventDisableTiming));
        CT_CHECK_HIP(hipEventCreateWithFlags(&sd.fj.join, hipEventDisableTiming));
        it = devs.emplace(dev, sd).first;
    }
    *out = it->second;
    return CT_OK;
}

}  // namespace ct

extern "C" ct_status ct_sinkhorn_grad(const float* x, int64_t T64, const float* y, const float* w,
                                      int64_t M64, const ct_sinkhorn_opts* o, float* grad_x,
                                      float* grad_w, float* value, float* pot, float* pot_plus,
                                      float* aux, void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    return sinkhorn_grad_impl(x, T64, y, w, M64, o, grad_x, grad_w, value, pot, pot_plus, aux, ws,
                              ws_bytes, stream, nullptr);
}

extern "C" size_t ct_sinkhorn_static_scratch_bytes(void) { return kStaticScratchBytes; }

extern "C" ct_status ct_sinkhorn_grad_static(const float* x, int64_t T64, const float* y,
                                             const float* w, int64_t M64,
                                             const ct_sinkhorn_opts* o, float* grad_x,
                                             float* grad_w, float* value, float* pot,
                                             float* pot_plus, float* aux, void* stream) {
    clear_error();
    ct_status rc = validate_call(x, T64, y, M64, o, grad_x, grad_w, value, pot);
    if (rc) return rc;
    const size_t need = sk_layout(nullptr, (int)T64, (int)M64, o->d, nullptr).bytes;
    if (need > kStaticScratchBytes)
        return fail(CT_E_WORKSPACE,
                    "problem needs %zu bytes of scratch; the static scratch holds %zu "
                    "(T=%lld, M=%lld, d=%d): use ct_sinkhorn_grad with a workspace",
                    need, kStaticScratchBytes, (long long)T64, (long long)M64, o->d);
    if (profiling())
        return fail(CT_E_UNSUPPORTED, "launch profiling creates events; disable it for this entry point");
    StaticDevice sd;
    rc = static_device(&sd);
    if (rc) return rc;
    return sinkhorn_grad_impl(x, T64, y, w, M64, o, grad_x, grad_w, value, pot, pot_plus, aux,
                              sd.ptr, kStaticScratchBytes, stream, &sd.fj);
}

// ------------------------------------------------------------- autotuning

namespace ct {

// Synthetic staged problem for timing: points from a hash in [0,1]^d, equal
// masses, zero potentials (the timing of a sweep does not depend on the data
// beyond its size).
__device__ __forceinline__ float hash01(unsigned v) {
    v ^= v >> 16;
    v *= 0x7feb352du;
    v ^= v >> 15;
    v *= 0x846ca68bu;
    v ^= v >> 16;
    return (float)(v >> 8) * (1.0f / 16777216.0f);
}

__global__ __launch_bounds__(256) void k_synth(int T, int M, int d, int Tpad, int Mpad,
                                               float sqrt_kappa, float log2a, float log2b,
                                               float4* cx, float4* cy, float4* x0, float4* x1,
                                               float4* x2, float4* x3, float4* y0, float4* y1,
                                               float4* y2, float* f, float* g, float* p, float* q,
                                               float* b, float* lb) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const float ninf = -__builtin_huge_valf();
    if (i < Tpad) {
        float c[3];
        for (int t = 0; t < 3; ++t) c[t] = hash01(2654435761u * (unsigned)i + 97u * t + 1u) * sqrt_kappa;
        const float h = i < T ? log2a : ninf;
        float4 r = d == 2 ? make_float4(c[0], c[1], h, 0.f) : make_float4(c[0], c[1], c[2], h);
        x0[i] = r; x1[i] = r; x2[i] = r; x3[i] = r;
        if (i < T) {
            cx[i] = make_float4(c[0], c[1], c[2], 0.f);
            f[i] = 0.f;
            p[i] = 0.f;
        }
    }
    if (i < Mpad) {
        float c[3];
        for (int t = 0; t < 3; ++t) c[t] = hash01(40503u * (unsigned)i + 131u * t + 7u) * sqrt_kappa;
        const float h = i < M ? log2b : ninf;
        float4 r = d == 2 ? make_float4(c[0], c[1], h, 0.f) : make_float4(c[0], c[1], c[2], h);
        y0[i] = r; y1[i] = r; y2[i] = r;
        if (i < M) {
            cy[i] = make_float4(c[0], c[1], c[2], 0.f);
            g[i] = 0.f;
            q[i] = 0.f;
            b[i] = exp2f(log2b);
            lb[i] = log2b;
        }
    }
}

}  // namespace ct

extern "C" ct_status ct_autotune_sinkhorn(int64_t T64, int64_t M64, const ct_sinkhorn_opts* o,
                                          void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    static const float dummy = 0.f;
    ct_status rc = validate(&dummy, T64, &dummy, M64, o);
    if (rc) return rc;
    if (!ws) return fail(CT_E_ARG, "workspace is null");
    const int T = (int)T64, M = (int)M64, d = o->d;
    SkLayout L = sk_layout(ws, T, M, d, nullptr);
    if (ws_bytes < L.bytes) return fail(CT_E_WORKSPACE, "workspace too small: %zu < %zu", ws_bytes, L.bytes);
    hipStream_t st = static_cast<hipStream_t>(stream);
    rc = refuse_capture(st, "ct_autotune_sinkhorn");
    if (rc) return rc;
    const double kappa_d = kLog2e / (double)o->eps;
    const int n = std::max(pad_keys(T), pad_keys(M));
    hipLaunchKernelGGL(k_zero3, dim3(((int)L.ntick + 255) / 256), dim3(256), 0, st, L.tick[0],
                       (int)L.ntick, L.tick[1], (int)L.ntick, L.tick[2], (int)L.ntick);
    hipLaunchKernelGGL(k_zero3, dim3(1), dim3(256), 0, st, L.counters, kCounters, nullptr, 0, nullptr, 0);
    hipLaunchKernelGGL(k_synth, dim3((n + 255) / 256), dim3(256), 0, st, T, M, d, pad_keys(T),
                       pad_keys(M), (float)std::sqrt(kappa_d), (float)(-std::log2((double)T)),
                       (float)(-std::log2((double)M)), L.cx, L.cy, L.xrec[0], L.xrec[1], L.xrec[2],
                       L.xrec[3], L.yrec[0], L.yrec[1], L.yrec[2], L.f, L.g, L.p, L.q, L.b, L.log2b);
    CT_CHECK_HIP(hipGetLastError());
    hipEvent_t e0, e1;
    CT_CHECK_HIP(hipEventCreate(&e0));
    CT_CHECK_HIP(hipEventCreate(&e1));
    Schedule cand[kMaxCandidates];
    const int nc = schedule_candidates(cand, kMaxCandidates);
    const SkConsts c = sk_consts(T, M, o);
    const SkJobs J{L, c};
    const bool debias = o->flags & CT_DEBIAS;
    const bool ref_iter = debias && (o->flags & (CT_VALUE | CT_GRAD_W));
    // the launches of the default (two-stream) schedule: cross f, cross g, self p + q
    JobSet sets[3];
    sets[0].add(J.f(L.f, L.xrec[0], nullptr));
    sets[1].add(J.g(L.xrec[0], L.g, L.yrec[0]));
    if (debias) sets[2].add(J.p(0, true, L.p, L.xrec[3], nullptr));
    if (ref_iter) sets[2].add(J.q(0, true, L.q, L.yrec[2]));
    const int keys[3][2] = {{T, M}, {M, T}, {ref_iter ? M : T, ref_iter ? M : T}};
    for (int side = 0; side < 3; ++side) {
        const JobSet& S = sets[side];
        if (S.n == 0) continue;
        float best = 1e30f;
        Schedule bs = cand[0];
        for (int ci = 0; ci < nc; ++ci) {
            ct_status rc2 = launch_set(S, c, cand[ci], true, false, nullptr, st);  // warm-up
            if (rc2) return rc2;
            CT_CHECK_HIP(hipEventRecord(e0, st));
            const int reps = 3;
            for (int r = 0; r < reps; ++r) {
                rc2 = launch_set(S, c, cand[ci], true, false, nullptr, st);
                if (rc2) return rc2;
            }
            CT_CHECK_HIP(hipEventRecord(e1, st));
            CT_CHECK_HIP(hipEventSynchronize(e1));
            float ms = 0.f;
            CT_CHECK_HIP(hipEventElapsedTime(&ms, e0, e1));
            ms /= reps;
            if (ms < best) {
                best = ms;
                bs = cand[ci];
            }
        }
        tuning_record(d, keys[side][0], keys[side][1], bs, (int)(best * 1000.f + 0.5f));
    }
    CT_CHECK_HIP(hipEventDestroy(e0));
    CT_CHECK_HIP(hipEventDestroy(e1));
    return CT_OK;
}

extern "C" ct_status ct_status_sync(const void* ws, float resid_tol, uint32_t* nonfinite,
                                    uint32_t* rescued, float* resid, void* stream) {
    clear_error();
    if (!ws) return fail(CT_E_ARG, "workspace is null");
    if (reinterpret_cast<uintptr_t>(ws) % 256) return fail(CT_E_WORKSPACE, "workspace not 256-byte aligned");
    if (!(resid_tol >= 0.f)) return fail(CT_E_ARG, "resid_tol must be >= 0 (0: no convergence check)");
    hipStream_t st = static_cast<hipStream_t>(stream);
    ct_status rc = refuse_capture(st, "ct_status_sync");
    if (rc) return rc;
    // the counters come before every size-dependent buffer of the layout; a stand-in
    // base (never dereferenced) gives their offset
    char* const probe = reinterpret_cast<char*>(uintptr_t(1) << 20);
    const size_t off = static_cast<size_t>(reinterpret_cast<char*>(sk_layout(probe, 1, 1, 2, nullptr).counters) - probe);
    unsigned c[kCounters] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
    CT_CHECK_HIP(hipMemcpyAsync(c, static_cast<const char*>(ws) + off, sizeof(c),
                                hipMemcpyDeviceToHost, st));
    CT_CHECK_HIP(hipStreamSynchronize(st));
    float r;
    std::memcpy(&r, &c[2], sizeof(r));
    if (!c[3]) r = __builtin_nanf("");
    if (nonfinite) *nonfinite = c[0];
    if (rescued) *rescued = c[1];
    if (resid) *resid = r;
    if (c[4])
        return fail(CT_E_DEVICE, "a wait of the last call's fused or exchange solve gave up: "
                                 "its outputs are not valid");
    if (c[0])
        return fail(CT_E_NONFINITE, "the last gradient call saw %u non-finite coordinates or "
                                    "non-positive weights: its outputs are not valid", c[0]);
    if (resid_tol > 0.f && c[3] && !(r <= resid_tol))
        return fail(CT_WARN_NOT_CONVERGED, "column residual %.3g above the tolerance %.3g", r,
                    resid_tol);
    return CT_OK;
}
