// Simulated annealing over D-subsets of a subspace, the stochastic search
// the paper names for the sparsifying step (Software Description) when the
// exhaustive L0 of Eq. (1) (Core Optimization Objective) is out of reach:
// D > 3, or subspaces too large for every subset.
//
// Chains are independent, and a chain's steps are a dependent sequence of
// gathers from the correlation matrix and a small Cholesky; a group of
// lanes evaluates a chain's next proposals at once (k_sa_run).  The rules,
// which an implementation elsewhere can follow to reproduce a trajectory
// bit for bit:
//
//   energy   E(a) = 1 - c_a^T C_aa^{-1} c_a for the subset array a, by a
//            Cholesky of C_aa in array order (pivot <= 1e-10: singular,
//            E = +inf), C and c the correlations of the rows and target;
//   move     position p = draw mod D, row r = draw mod S; a row already in
//            the subset leaves the state unchanged;
//   accept   E' <= E, or u < exp(-(E' - E) / T), u = (draw >> 11) 2^-53;
//            T = T0 alpha^k, formed by one multiplication per proposal;
//   best     per chain the smallest E seen (ties: the smaller sorted
//            candidate-ID tuple); per problem the best over chains.
//
// Random numbers are SplitMix64 (Steele, Lea and Flood, OOPSLA 2014) used
// counter-based: chain q's key is output q + 1 of the stream with state
// seed, its draw c is output c + 1 of the stream with state key.  Random
// starts use draws 0, 1, ... (repeats skipped); proposal k uses draws
// 2^40 + 3k (position), + 1 (row), + 2 (uniform).
//
// Every operation that decides a move is one IEEE double operation with
// one rounding: this file is compiled with -ffp-contract=off, correlations
// are left-to-right sums over samples, and exp(-x) is the range reduction
// x = k ln 2 + r with the degree-18 Taylor series of exp(-r) in Horner form.
#include "dsc_internal.h"

#include <string>

namespace dsc {
namespace {

constexpr uint64_t SM_GAMMA = 0x9E3779B97F4A7C15ull;

__device__ __forceinline__ uint64_t sm_mix(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Output i (i >= 1) of the SplitMix64 stream with state x0.
__device__ __forceinline__ uint64_t sm_at(uint64_t x0, uint64_t i) { return sm_mix(x0 + i * SM_GAMMA); }

__device__ __forceinline__ double exp_neg(double x) {
    if (!(x < 700.0)) return 0.0;
    if (x <= 0.0) return 1.0;
    const double LN2 = 0.6931471805599453;
    const double INV_LN2 = 1.4426950408889634;
    const int k = (int)(x * INV_LN2);
    const double t = (double)k * LN2;
    const double r = x - t;
    double p = 1.0;
#pragma unroll
    for (int i = 18; i >= 1; i--) {
        double q = p * -r;
        q = q / (double)i;
        p = 1.0 + q;
    }
    return ldexp(p, -k);
}

struct SaArgs {
    int n, S, ldz;
    const double* F;
    int64_t ldf;
    const double* y;
    const int64_t* ids;
    double* Zt;               // [n][ldz] centred values, sample-major (S rows + the target)
    double* nrm;              // [S + 1]
    double* C;                // [S][S]
    double* c;                // [S]
    const int32_t* init;      // [D] or NULL
    int32_t* chain_rows;      // [chains][D] best rows per chain, ascending
    double* chain_e;          // [chains]
    int32_t* out_rows;        // [D]
    double* out_e;
};

// Rows i of the problem (i = S: the target): mean and centred values as
// left-to-right sums, norm = sqrt(sum of squares).  A row's sum is one
// dependent chain of additions, so a block takes PR rows: its 256 threads
// stage PT samples of them at a time in LDS (coalesced, the next tile's
// loads issued before the sums of this one), PR of its lanes walk a row
// each, and the centred values are written sample-major, PR rows together.
// Bound by the addition chains (2 n of them per row).  One thread per row
// reading its own row took 660 us for 3001 rows of 2000 samples (S = 3000);
// this form takes 78 us.
constexpr int PR = 16, PT = 128;

__global__ __launch_bounds__(256) void k_sa_prep(ctab<SaArgs> A) {
    const SaArgs& a = tab(A, blockIdx.y);
    DSC_GLOBAL(a.F); DSC_GLOBAL(a.y); DSC_GLOBAL(a.Zt); DSC_GLOBAL(a.nrm);
    __shared__ double tile[PR][PT + 1];
    __shared__ double mean[PR];
    const int i0 = blockIdx.x * PR, tid = threadIdx.x;
    if (i0 > a.S) return;
    const int lr = tid / 16, lt = tid % 16;              // this thread loads samples lt, lt + 16, ... of row lr
    const int li = min(i0 + lr, a.S);
    const double* f = li < a.S ? a.F + (int64_t)li * a.ldf : a.y;
    const int n = a.n;
    constexpr int PV = PT / 16;
    double v[PV];
    auto load = [&](int t0) {
#pragma unroll
        for (int u = 0; u < PV; u++) v[u] = t0 + lt + 16 * u < n ? f[t0 + lt + 16 * u] : 0.0;
    };
    auto stage = [&]() {
#pragma unroll
        for (int u = 0; u < PV; u++) tile[lr][lt + 16 * u] = v[u];
    };
    double s = 0.0;
    load(0);
    for (int t0 = 0; t0 < n; t0 += PT) {
        stage();
        __syncthreads();
        if (t0 + PT < n) load(t0 + PT);
        if (tid < PR) {
            const int m = min(PT, n - t0);
#pragma unroll 16
            for (int t = 0; t < m; t++) s = s + tile[tid][t];
        }
        __syncthreads();
    }
    if (tid < PR) mean[tid] = s / (double)n;
    __syncthreads();
    double q = 0.0;
    load(0);
    for (int t0 = 0; t0 < n; t0 += PT) {
        const double mr = mean[lr];
#pragma unroll
        for (int u = 0; u < PV; u++) tile[lr][lt + 16 * u] = v[u] - mr;
        __syncthreads();
        if (t0 + PT < n) load(t0 + PT);
        const int m = min(PT, n - t0);
        if (i0 + lt <= a.S)
            for (int t = lr; t < m; t += 16) a.Zt[(int64_t)(t0 + t) * a.ldz + i0 + lt] = tile[lt][t];
        if (tid < PR) {
#pragma unroll 16
            for (int t = 0; t < m; t++) q = q + tile[tid][t] * tile[tid][t];
        }
        __syncthreads();
    }
    if (tid < PR && i0 + tid <= a.S) a.nrm[i0 + tid] = sqrt(q);
}

// C[i][j] = (left-to-right sum of z_i z_j) / (nrm_i nrm_j), and c[i] for
// j = S.  A block takes CI consecutive rows i and 256 columns j; each thread
// keeps CI independent sequential sums, so every entry is summed in sample
// order while the rows' values are read once per block (scalar loads of CI
// consecutive values: Zt's rows are padded past i0 + CI).  A product and a
// sum rounded apart rule out fused and matrix instructions, so the floor is
// 2 FP64 instructions per entry and sample.  C is symmetric bit for bit
// (products and norms commute): blocks below the diagonal are left out and
// each entry is written to both places.  Full square with clamped scalar
// addresses: 2.9 ms at S = 3000, n = 2000; this form: 1.4 ms.
constexpr int CI = 16;

__global__ __launch_bounds__(256) void k_sa_corr(ctab<SaArgs> A) {
    const SaArgs& a = tab(A, blockIdx.z);
    DSC_GLOBAL(a.Zt); DSC_GLOBAL(a.nrm); DSC_GLOBAL(a.C); DSC_GLOBAL(a.c);
    const int i0 = blockIdx.y * CI;
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (i0 >= a.S || blockIdx.x * 256 > a.S || (int)blockIdx.x * 256 + 255 < i0) return;
    const int jj = min(j, a.S);
    const int64_t ldz = a.ldz;
    double d[CI];
#pragma unroll
    for (int k = 0; k < CI; k++) d[k] = 0.0;
    const double* zi = a.Zt + i0;
    const double* zj = a.Zt + jj;
    const int n = a.n;
    int t = 0;
    for (; t + 4 <= n; t += 4) {
        double y[4];
#pragma unroll
        for (int u = 0; u < 4; u++) y[u] = zj[(t + u) * ldz];
#pragma unroll
        for (int u = 0; u < 4; u++)
#pragma unroll
            for (int k = 0; k < CI; k++) d[k] = d[k] + zi[(t + u) * ldz + k] * y[u];
    }
    for (; t < n; t++) {
        const double y = zj[t * ldz];
#pragma unroll
        for (int k = 0; k < CI; k++) d[k] = d[k] + zi[t * ldz + k] * y;
    }
    if (j > a.S) return;
    const double nj = a.nrm[j];
#pragma unroll
    for (int k = 0; k < CI; k++) {
        const int i = i0 + k;
        if (i >= a.S) break;
        const double ni = a.nrm[i];
        const double v = ni > 0.0 && nj > 0.0 ? d[k] / (ni * nj) : 0.0;
        if (j == a.S) {
            a.c[i] = v;
        } else {
            a.C[(int64_t)i * a.S + j] = v;
            if (j > i) a.C[(int64_t)j * a.S + i] = v;
        }
    }
}

// v / b correctly rounded, given r = 1 / b correctly rounded: with q within
// an ulp of the quotient, q + r (v - q b) rounds to it (Markstein, IBM J.
// Res. Dev. 34, 1990; the remainder is exact in one fused operation).  The
// first correction brings q there, the second rounds it.  Holds while
// nothing under- or overflows, which the caller checks (out_of_range).
__device__ __forceinline__ double div_by(double v, double b, double r) {
    double q = v * r;
    q = __builtin_fma(__builtin_fma(-b, q, v), r, q);
    return __builtin_fma(__builtin_fma(-b, q, v), r, q);
}

// Whether |v| lies outside [2^-700, 2^700) (zero among it): the quotient is
// then left to the plain division.  Divisors here are square roots of
// pivots in (1e-10, 1 + rounding].
__device__ __forceinline__ bool out_of_range(double v) {
    const uint32_t e = ((uint32_t)__double2hiint(v) >> 20) & 0x7FFu;
    return e - 323u >= 1400u;
}

// Energy of the subset with correlations M[i][j] (i >= j) among its rows
// and c[i] with the target.  EXACT_DIV: every quotient by the plain
// division; else by the shared reciprocal of its column's pivot, and *odd
// is set where that would not be certain (the result is then not used).
template <int D, bool EXACT_DIV>
__device__ __forceinline__ double energy(const double (&M)[D][D], const double (&c)[D], bool* odd) {
    double L[D][D], r[D], w[D];
    bool good = true, o = false;
    auto quot = [&](double v, int j) {
        if (EXACT_DIV) return v / L[j][j];
        o |= out_of_range(v);
        return div_by(v, L[j][j], r[j]);
    };
#pragma unroll
    for (int j = 0; j < D; j++) {
        double d = M[j][j];
#pragma unroll
        for (int k = 0; k < j; k++) d = d - L[j][k] * L[j][k];
        const bool ok = d > 1e-10;
        good = good && ok;
        L[j][j] = sqrt(ok ? d : 1.0);      // past a singular pivot the values are not used
        if (!EXACT_DIV) r[j] = 1.0 / L[j][j];
#pragma unroll
        for (int i = j + 1; i < D; i++) {
            double v = M[i][j];
#pragma unroll
            for (int k = 0; k < j; k++) v = v - L[i][k] * L[j][k];
            L[i][j] = quot(v, j);
        }
    }
    double ex = 0.0;
#pragma unroll
    for (int j = 0; j < D; j++) {
        double v = c[j];
#pragma unroll
        for (int k = 0; k < j; k++) v = v - L[j][k] * w[k];
        w[j] = quot(v, j);
        ex = ex + w[j] * w[j];
    }
    if (odd) *odd = o;
    return good ? 1.0 - ex : INFINITY;
}

template <int D>
__device__ __forceinline__ void sort_rows(int* s) {
#pragma unroll
    for (int i = 1; i < D; i++)
#pragma unroll
        for (int j = i; j > 0; j--)
            if (s[j] < s[j - 1]) { const int t = s[j]; s[j] = s[j - 1]; s[j - 1] = t; }
}

// Sorted candidate-ID tuple of rows a before that of rows b.
template <int D>
__device__ __forceinline__ bool ids_before(const int* a, const int* b, const int64_t* __restrict__ ids) {
    int64_t ia[D], ib[D];
#pragma unroll
    for (int i = 0; i < D; i++) { ia[i] = ids[a[i]]; ib[i] = ids[b[i]]; }
#pragma unroll
    for (int i = 1; i < D; i++)
#pragma unroll
        for (int j = i; j > 0; j--) {
            if (ia[j] < ia[j - 1]) { const int64_t t = ia[j]; ia[j] = ia[j - 1]; ia[j - 1] = t; }
            if (ib[j] < ib[j - 1]) { const int64_t t = ib[j]; ib[j] = ib[j - 1]; ib[j - 1] = t; }
        }
#pragma unroll
    for (int i = 0; i < D; i++)
        if (ia[i] != ib[i]) return ia[i] < ib[i];
    return false;
}

struct SaRun {
    int Q;
    int64_t K;
    double T0, alpha;
    uint64_t seed;
    int lanes;                // lanes per chain, a power of two <= 64
};

// x mod S by a multiplication: m = floor((2^64 - 1) / S), so the estimated
// quotient is at most one below the true one.
__device__ __forceinline__ int mod_s(uint64_t x, uint32_t S, uint64_t m) {
    uint32_t r = (uint32_t)x - (uint32_t)__umul64hi(x, m) * S;
    if (r >= S) r -= S;
    return (int)r;
}

// u < exp(-x) for x = dE / T as the exact form decides it, from a rough
// estimate of exp(-x) where that is clear: the estimate (x and exp(-x) to
// about 5e-6 relative) decides outside 1e-4 of itself, u = 0 beyond x = 40
// (u is a multiple of 2^-53 > exp(-40)), and the exact form in between.
__device__ __forceinline__ bool metropolis(double dE, double T, uint64_t u53) {
    const double x = dE * __builtin_amdgcn_rcp(T);
    const double u = (double)u53 * 0x1.0p-53;
    if (x < 40.0) {
        const float e = __expf(-(float)x), uf = (float)u;
        if (uf > e * 1.0001f) return false;
        if (uf < e * 0.9999f) return true;
    } else if (x < 699.0) {
        return u53 == 0;
    } else if (x > 701.0) {
        return false;
    }
    return u < exp_neg(dE / T);
}

// The annealing.  R.lanes consecutive lanes hold one chain's state, each a
// copy, and lane l evaluates proposal k + l as if none of those before it
// were accepted (proposals come from counters, not from the state); the
// first accepted one becomes the state and the walk goes on after it, so
// the trajectory is that of one proposal at a time.  Most proposals are
// rejected once the walk has cooled, and a chain's own steps are a chain of
// dependent loads and FP64 operations, so lanes fill the SIMDs that few
// chains leave idle.  Everything is indexed statically (a proposal's row
// and column replace the old ones by selects) and stays in registers: a
// form with one lane per chain that indexed its factor by the position
// spilled 808 bytes per lane.  The next proposals' correlations are loaded
// a turn ahead.  Bound by the latency of a proposal's own chain (pivot, square root,
// reciprocal, column, and the gathers after an accepted move).  16,384 chains x 2,000 proposals, D = 6, S = 3000: 41.8 ms in
// that form, 4.6 ms in this one (two lanes per chain).
template <int D>
__global__ __launch_bounds__(256) void k_sa_run(ctab<SaArgs> A, SaRun R) {
    const SaArgs& g = tab(A, blockIdx.y);
    DSC_GLOBAL(g.C); DSC_GLOBAL(g.c); DSC_GLOBAL(g.ids); DSC_GLOBAL(g.init); DSC_GLOBAL(g.chain_rows); DSC_GLOBAL(g.chain_e);
    const int G = R.lanes, l = threadIdx.x & (G - 1);
    const int64_t q = ((int64_t)blockIdx.x * 256 + threadIdx.x) / G;
    if (q >= R.Q) return;
    const int lane = threadIdx.x & 63, first_lane = lane - l;
    const uint64_t group = (G == 64 ? ~0ull : (1ull << G) - 1ull) << first_lane;
    const int S = g.S;
    const uint64_t ms = ~0ull / (uint64_t)S;
    const uint64_t key = sm_at(R.seed, (uint64_t)q + 1);
    int a[D], bs[D];
    bool use_init = g.init != nullptr;
    if (use_init) {                          // distinct rows in 0..S-1, else a random start
#pragma unroll
        for (int j = 0; j < D; j++) {
            a[j] = g.init[j];
            use_init = use_init && a[j] >= 0 && a[j] < S;
#pragma unroll
            for (int i = 0; i < j; i++) use_init = use_init && a[i] != a[j];
        }
    }
    if (!use_init) {
        uint64_t ctr = 0;
#pragma unroll
        for (int j = 0; j < D; j++) {
            for (;;) {
                const int r = mod_s(sm_at(key, ++ctr), (uint32_t)S, ms);
                bool dup = false;
#pragma unroll
                for (int i = 0; i < j; i++) dup |= a[i] == r;
                if (!dup) { a[j] = r; break; }
            }
        }
    }
    // correlations of the current subset, among its rows (lower half) and with the target
    double M[D][D], c[D];
#pragma unroll
    for (int i = 0; i < D; i++) {
        c[i] = g.c[a[i]];
#pragma unroll
        for (int j = 0; j <= i; j++) M[i][j] = g.C[(int64_t)a[i] * S + a[j]];
    }
    double E = energy<D, true>(M, c, nullptr);
    double bE = E;
#pragma unroll
    for (int j = 0; j < D; j++) bs[j] = a[j];
    sort_rows<D>(bs);
    double T = R.T0;                         // of this lane's proposal
    for (int i = 0; i < l; i++) T = T * R.alpha;
    const uint64_t base = (uint64_t)1 << 40;
    // this lane's proposal: position, row, 53 random bits, the row's correlations
    int p, r;
    uint64_t u;
    double x[D], xr, xc;
    auto propose = [&](int64_t kk) {
        const uint64_t c0 = base + 3 * (uint64_t)kk;
        p = (int)(sm_at(key, c0 + 1) % (uint64_t)D);
        r = mod_s(sm_at(key, c0 + 2), (uint32_t)S, ms);
        u = sm_at(key, c0 + 3) >> 11;
        const double* row = g.C + (int64_t)r * S;
#pragma unroll
        for (int j = 0; j < D; j++) x[j] = row[a[j]];
        xr = row[r];
        xc = g.c[r];
    };
    int64_t k = 0;                           // proposal of the group's first lane
    if (k < R.K) propose(k + l);
    while (k < R.K) {
        const int p0 = p, r0 = r;
        const uint64_t u0 = u;
        double x0[D];
        const double xr0 = xr, xc0 = xc;
#pragma unroll
        for (int j = 0; j < D; j++) x0[j] = x[j];
        propose(k + G + l);                  // the next turn's, should nothing be accepted
        bool in = false;
#pragma unroll
        for (int j = 0; j < D; j++) in |= a[j] == r0;
        double N[D][D], cn[D];
#pragma unroll
        for (int i = 0; i < D; i++) {
            cn[i] = i == p0 ? xc0 : c[i];
#pragma unroll
            for (int j = 0; j < i; j++) N[i][j] = i == p0 ? x0[j] : j == p0 ? x0[i] : M[i][j];
            N[i][i] = i == p0 ? xr0 : M[i][i];
        }
        bool odd = false;
        double En = energy<D, false>(N, cn, &odd);
        if (odd) En = energy<D, true>(N, cn, nullptr);
        bool acc = En <= E;
        if (!acc && En < INFINITY) acc = metropolis(En - E, T, u0);
        acc = acc && !in && k + l < R.K;
        const uint64_t won = __ballot(acc) & group;
        if (won == 0) {
            k += G;
            for (int i = 0; i < G; i++) T = T * R.alpha;
        } else {
            const int w = __ffsll((unsigned long long)won) - 1;
            const int pw = __shfl(p0, w), rw = __shfl(r0, w);
            E = __shfl(En, w);
            const double xrw = __shfl(xr0, w), xcw = __shfl(xc0, w);
            double xw[D];
#pragma unroll
            for (int j = 0; j < D; j++) xw[j] = __shfl(x0[j], w);
#pragma unroll
            for (int i = 0; i < D; i++) {
                c[i] = i == pw ? xcw : c[i];
#pragma unroll
                for (int j = 0; j < i; j++) M[i][j] = i == pw ? xw[j] : j == pw ? xw[i] : M[i][j];
                M[i][i] = i == pw ? xrw : M[i][i];
                a[i] = i == pw ? rw : a[i];
            }
            int sa[D];
#pragma unroll
            for (int j = 0; j < D; j++) sa[j] = a[j];
            sort_rows<D>(sa);
            if (E < bE || (E == bE && ids_before<D>(sa, bs, g.ids))) {
                bE = E;
#pragma unroll
                for (int j = 0; j < D; j++) bs[j] = sa[j];
            }
            k += w - first_lane + 1;
            T = __shfl(T, w) * R.alpha;      // the next proposal's, then this lane's
            for (int i = 0; i < l; i++) T = T * R.alpha;
            if (k < R.K) propose(k + l);
        }
    }
    if (l == 0) {
#pragma unroll
        for (int j = 0; j < D; j++) g.chain_rows[q * D + j] = bs[j];
        g.chain_e[q] = bE;
    }
}

// The best chain of each problem, as a walk in chain order that replaces
// its choice by a smaller energy, or an equal one of a smaller sorted ID
// tuple, finds it (a chain whose energy is not a number is never taken, or
// never replaced if it is the first).  One block per problem: each thread
// walks every 256th chain, then the threads' choices are combined in
// pairs, the earlier chain kept on a full tie.  One thread for everything
// took 2.3 ms for 16,384 chains; this takes 26 us.
template <int D>
__global__ __launch_bounds__(256) void k_sa_pick(ctab<SaArgs> A, int Q) {
    const SaArgs& g = tab(A, blockIdx.x);
    DSC_GLOBAL(g.chain_rows); DSC_GLOBAL(g.chain_e); DSC_GLOBAL(g.out_rows); DSC_GLOBAL(g.out_e); DSC_GLOBAL(g.ids);
    __shared__ int best[256];
    __shared__ double en[256];
    // whether chain q comes before chain w (-1: none)
    auto before = [&](int q, double eq, int w, double ew) {
        if (q < 0 || eq != eq) return false;
        if (w < 0) return true;
        if (eq != ew) return eq < ew;
        const int32_t* rq = g.chain_rows + (int64_t)q * D;
        const int32_t* rw = g.chain_rows + (int64_t)w * D;
        if (ids_before<D>(rq, rw, g.ids)) return true;
        return q < w && !ids_before<D>(rw, rq, g.ids);
    };
    const int tid = threadIdx.x;
    int w = -1;
    double ew = INFINITY;
    for (int q = tid; q < Q; q += 256) {
        const double eq = g.chain_e[q];
        if (before(q, eq, w, ew)) { w = q; ew = eq; }
    }
    best[tid] = w;
    en[tid] = ew;
    __syncthreads();
    for (int h = 128; h >= 1; h >>= 1) {
        if (tid < h && before(best[tid + h], en[tid + h], best[tid], en[tid])) {
            best[tid] = best[tid + h];
            en[tid] = en[tid + h];
        }
        __syncthreads();
    }
    if (tid != 0) return;
    const double e0 = g.chain_e[0];
    w = e0 != e0 || best[0] < 0 ? 0 : best[0];
    for (int j = 0; j < D; j++) g.out_rows[j] = g.chain_rows[(int64_t)w * D + j];
    *g.out_e = g.chain_e[w];
}

template <int D>
void launch_run(ctab<SaArgs> A, int nb, const SaRun& R, hipStream_t st) {
    k_sa_run<D><<<dim3((unsigned)cdiv((int64_t)R.Q * R.lanes, 256), nb), 256, 0, st>>>(A, R);
    k_sa_pick<D><<<nb, 256, 0, st>>>(A, R.Q);
}

}  // namespace
}  // namespace dsc

extern "C" discover_status discover_l0_anneal(discover_ctx* ctx, const discover_l0_problem* probs,
                                              int32_t n_problems, int32_t D,
                                              const discover_anneal_params* prm,
                                              const int32_t* init_active, int32_t* out_subsets,
                                              double* out_rmse, double* out_coef, double* out_energy,
                                              int32_t* out_chain_subsets, double* out_chain_energy,
                                              double* out_resid, int64_t ldr, void* stream) {
    using namespace dsc;
    return guarded([&] {
        DSC_REQUIRE(ctx && probs && prm && n_problems >= 1 && n_problems <= 65535, "ctx/probs/prm/n_problems");
        DSC_REQUIRE(D >= 1 && D <= DISCOVER_MAX_D, "D = %d outside 1..%d", D, DISCOVER_MAX_D);
        DSC_REQUIRE(prm->chains >= 1 && prm->chains <= (1 << 20), "chains = %d outside 1..2^20", prm->chains);
        DSC_REQUIRE(prm->steps >= 0, "steps < 0");
        DSC_REQUIRE(prm->T0 >= 0.0 && prm->T0 < INFINITY, "T0 must be finite and >= 0");
        DSC_REQUIRE(prm->alpha > 0.0 && prm->alpha <= 1.0, "alpha outside (0, 1]");
        DSC_REQUIRE(out_subsets && out_rmse && out_coef && out_energy, "outputs required");
        for (int b = 0; b < n_problems; b++) {
            const discover_l0_problem& p = probs[b];
            DSC_REQUIRE(p.S >= D && p.S <= 16384, "problem %d: S = %d outside D..16384", b, p.S);
            DSC_REQUIRE(p.n >= D + 2, "problem %d: n = %d < D + 2", b, p.n);
            DSC_REQUIRE(p.F && p.ids && p.y && p.ldf >= p.n, "problem %d: F/ids/y/ldf", b);
            DSC_REQUIRE(!out_resid || ldr >= p.n, "problem %d: ldr < n", b);
        }
        DSC_HIP(hipSetDevice(ctx->device));
        const hipStream_t st = (hipStream_t)stream;
        CallMode mode(ctx, stream_capturing(st), false);
        const int Q = prm->chains;
        std::vector<SaArgs> sa(n_problems);
        int Smax = 0, nmax = 0;
        for (int b = 0; b < n_problems; b++) {
            const discover_l0_problem& p = probs[b];
            const std::string sfx = std::to_string(b) + ctx->tag;
            SaArgs& a = sa[b];
            a = SaArgs{};
            a.n = p.n; a.S = p.S; a.ldz = (int)cdiv(p.S + 1, 64) * 64;
            a.F = p.F; a.ldf = p.ldf; a.y = p.y; a.ids = p.ids;
            a.Zt = ctx->buf<double>("sa_Zt" + sfx, (size_t)p.n * a.ldz);
            a.nrm = ctx->buf<double>("sa_nrm" + sfx, (size_t)p.S + 1);
            a.C = ctx->buf<double>("sa_C" + sfx, (size_t)p.S * p.S);
            a.c = ctx->buf<double>("sa_c" + sfx, (size_t)p.S);
            a.init = init_active ? init_active + (int64_t)b * D : nullptr;
            a.chain_rows = out_chain_subsets ? out_chain_subsets + (int64_t)b * Q * D
                                             : ctx->buf<int32_t>("sa_rows" + sfx, (size_t)Q * D);
            a.chain_e = out_chain_energy ? out_chain_energy + (int64_t)b * Q
                                         : ctx->buf<double>("sa_e" + sfx, (size_t)Q);
            a.out_rows = out_subsets + (int64_t)b * D;
            a.out_e = out_energy + b;
            Smax = std::max(Smax, p.S);
            nmax = std::max(nmax, p.n);
        }
        const ctab<SaArgs> dA = ct(ctx->upload("sa_args", sa, st));
        {
            KTimer kt(ctx, st, "anneal_corr");
            k_sa_prep<<<dim3((unsigned)cdiv(Smax + 1, PR), n_problems), 256, 0, st>>>(dA);
            k_sa_corr<<<dim3((unsigned)cdiv(Smax + 1, 256), (unsigned)cdiv(Smax, CI), n_problems), 256, 0, st>>>(dA);
            check_launch("k_sa_corr");
        }
        // Lanes per chain: as many as keep the launch within 512 waves (32,768
        // lanes), a wave on every second SIMD; more look further ahead than the
        // walk goes between two accepted proposals.  Measured for 1, 2, 4, 8, 16,
        // 32, 64 lanes, ms per call: 16,384 chains, D = 6, S = 3000: 9.2, 6.1, 6.4,
        // 8.4, 12, 20, 37; 4096 chains, D = 8: 5.8, 4.2, 3.4, 3.5, 5.1, 9.0, 17;
        // 2048 chains, D = 4: 2.8, 1.8, 1.4, 1.3, 1.3, 1.4, 1.9; 512 chains, D = 2:
        // 0.53, 0.34, 0.24, 0.20, 0.18, 0.17, 0.19; 65,536 chains, D = 6: 15, 17, 20, ...
        int lanes = 1;
        while (lanes < 64 && (int64_t)Q * n_problems * lanes * 2 <= 32768) lanes *= 2;
        const SaRun R{Q, prm->steps, prm->T0, prm->alpha, prm->seed, lanes};
        {
            KTimer kt(ctx, st, "anneal");
            switch (D) {
            case 1: launch_run<1>(dA, n_problems, R, st); break;
            case 2: launch_run<2>(dA, n_problems, R, st); break;
            case 3: launch_run<3>(dA, n_problems, R, st); break;
            case 4: launch_run<4>(dA, n_problems, R, st); break;
            case 5: launch_run<5>(dA, n_problems, R, st); break;
            case 6: launch_run<6>(dA, n_problems, R, st); break;
            case 7: launch_run<7>(dA, n_problems, R, st); break;
            default: launch_run<8>(dA, n_problems, R, st); break;
            }
            check_launch("k_sa_run");
        }
        fit_rows(ctx, probs, n_problems, D, out_subsets, D, out_coef, D + 1, out_rmse, out_resid, ldr, st);
    });
}
