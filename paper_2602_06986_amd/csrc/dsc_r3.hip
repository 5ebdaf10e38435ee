// Operator-limited rung 3 on gfx950: screening of op3(f_i, g) for every
// partner f_i of the pool and every rung-2 feature g, without storing g
// (candidate generation by operators, Software Description; screening, the
// SIS step of the cited SISSO method, Summary).
//
// mul / div / rdiv: the per-candidate sums are matrix products over samples.
// A wave holds GT blocks of 16 rung-2 features (rows, regenerated in
// registers from their two rung-1 operands, 4 consecutive samples per lane)
// and one tile of 16 partner columns.  For every target t, the products
// sum_s a_s (x_s y_ts) give P_t, sum_s a_s x_s gives S1 and sum_s a_s^2 x_s^2
// gives S2, where a = g (mul, and rdiv with x replaced by 1/x) or a = 1/g
// (div).  The right-hand operands [x y_t | x | x^2] of every column tile are
// laid out once per call by k_r3_bmat, in the lane order of
// v_mfma_f64_16x16x4f64 (B[k][j] from lane j + 16k, four samples per lane),
// so a wave reads each as one 32-byte load per lane.
//
// The one-pass moments are unshifted: with kappa = S2 / (S2 - S1^2/n) the
// rounding error of every score is below 2.5 n u kappa (u = 2^-53; n sums
// of rounded products, plus the variance's cancellation), inside the
// selection margin 4 n u KAPPA_MAX for kappa <= KAPPA_MAX.  Candidates with
// a larger kappa, or whose values might overflow, are listed for the exact
// two-pass fix-up; candidates whose values are certainly not finite (a
// division by an exact zero) are left invalid.
#include "dsc_pairs.h"
#include "dsc_r3.h"

#include <algorithm>
#include <map>
#include <string>
#include <type_traits>

namespace dsc {

namespace {

constexpr double R3_KAPPA_MAX = 64.0;   // same bound as the other fast screens
constexpr double R3_BIG = 1e150;        // |f| below this: f and n f^2 stay finite
constexpr double R3_TINY = 1e-300;      // |g| above this: 1/g is finite
constexpr double R3_TAU_CONST = 1e-8;
constexpr double R3_TAU_CANCEL_FAST = 1e-12;

typedef double r3_v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int r3_wave() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// Workgroups are dealt to the 8 XCDs in turn (block b to XCD b % 8); this
// numbering gives each XCD a contiguous range of the grid's logical blocks,
// so that the row tiles one XCD works on at a time are neighbours in the
// record order and share their operand rows in that XCD's L2.
__device__ __forceinline__ int r3_xcd_block() {
    const int nb = (int)gridDim.x, b = (int)blockIdx.x;
    const int per = nb >> 3, rem = nb & 7, x = b & 7, pos = b >> 3;
    return x < rem ? x * (per + 1) + pos : rem * (per + 1) + (x - rem) * per + pos;
}

// Slot of each active lane in a list (lane order), one atomic per wave.
__device__ __forceinline__ unsigned long long r3_slot(unsigned long long* ctr) {
    const uint64_t m = __builtin_amdgcn_ballot_w64(true);
    const int lane = threadIdx.x & 63;
    const int leader = __ffsll((long long)m) - 1;
    unsigned long long base = 0;
    if (lane == leader) base = atomicAdd(ctr, (unsigned long long)__popcll(m));
    base = __shfl(base, leader, 64);
    return base + (unsigned long long)__popcll(m & ((1ull << lane) - 1ull));
}

__device__ __forceinline__ double r3_un(int op, double a) {
    switch (op) {
    case OP_EXP: return exp(a);
    case OP_LOG: return log(a);
    case OP_SQRT: return sqrt(a);
    default: return a * a;               // OP_SQ (OP_INV reads the reciprocal row)
    }
}

// Rung-2 operator applied to operands already loaded: x from row p1, y from
// row p2 of r3_rows (reciprocal rows where the operator divides).
__device__ __forceinline__ r3_v4d r3_combine(int op2, r3_v4d x, r3_v4d y) {
    switch (op2) {
    case OP_EXP: return r3_v4d{exp(x.x), exp(x.y), exp(x.z), exp(x.w)};
    case OP_LOG: return r3_v4d{log(x.x), log(x.y), log(x.z), log(x.w)};
    case OP_SQRT: return r3_v4d{sqrt(x.x), sqrt(x.y), sqrt(x.z), sqrt(x.w)};
    case OP_SQ: return x * x;
    case OP_INV: return x;
    case OP_ADD: return x + y;
    case OP_SUB: return x - y;
    default: return x * y;               // OP_MUL, OP_DIV, OP_RDIV
    }
}

// Operand rows of rung-2 feature (k, l, op2): the combine above of rows p1
// and p2 gives its values (the formulas of the rung-2 screen: a division
// multiplies by the stored reciprocal).
__device__ __forceinline__ void r3_rows(const double* Vf, const double* Rf, int64_t ldn, int k, int l,
                                        int op2, const double*& p1, const double*& p2) {
    const int64_t kk = k < 0 ? 0 : k;
    if (op2 < OP_ADD) {
        p1 = (op2 == OP_INV ? Rf : Vf) + (int64_t)l * ldn;
        p2 = p1;
    } else if (op2 == OP_RDIV) {
        p1 = Vf + (int64_t)l * ldn;
        p2 = Rf + kk * ldn;
    } else {
        p1 = Vf + kk * ldn;
        p2 = (op2 == OP_DIV ? Rf : Vf) + (int64_t)l * ldn;
    }
}

// How a row's values come from its two operand rows in the precision form:
// kinds with loops of their own, so that a loop holds no branch.
enum { RK_PROD, RK_ADD, RK_SUB, RK_OTHER };

// Kind and operand rows (row i of a table b: Vf or Rf, the same for the rows
// of a tile) for the values g, or (recip) for 1/g: where g is a product or
// quotient, 1/g is one of the operands' reciprocals and values, which are
// stored; elsewhere the reciprocal is taken of g.
__device__ __forceinline__ int r3_rows_lp(const double* Vf, const double* Rf, int k, int l, int op2, bool recip,
                                          const double*& b1, const double*& b2, int& i1, int& i2) {
    i1 = op2 < OP_ADD ? l : op2 == OP_RDIV ? l : k;
    i2 = op2 < OP_ADD ? l : op2 == OP_RDIV ? k : l;
    b1 = op2 == OP_INV ? Rf : Vf;
    b2 = op2 == OP_INV || op2 == OP_DIV || op2 == OP_RDIV ? Rf : Vf;
    switch (op2) {
    case OP_MUL:
    case OP_SQ:
        if (recip) b1 = b2 = Rf;
        return RK_PROD;
    case OP_DIV:
    case OP_RDIV:
        if (recip) {
            b1 = Rf;
            b2 = Vf;
        }
        return RK_PROD;
    case OP_ADD: return RK_ADD;
    case OP_SUB: return RK_SUB;
    default: return RK_OTHER;
    }
}

__device__ __forceinline__ double r3_regen1(const double* __restrict__ Vf, const double* __restrict__ Rf,
                                            int64_t ldn, int k, int l, int op2, int s) {
    const double b = Vf[(int64_t)l * ldn + s];
    if (k < 0) return op2 == OP_INV ? Rf[(int64_t)l * ldn + s] : r3_un(op2, b);
    const double a = Vf[(int64_t)k * ldn + s];
    switch (op2) {
    case OP_ADD: return a + b;
    case OP_SUB: return a - b;
    case OP_MUL: return a * b;
    case OP_DIV: return a * Rf[(int64_t)l * ldn + s];
    default: return b * Rf[(int64_t)k * ldn + s];
    }
}

__device__ __forceinline__ double r3_rcp(double g) {
    double r = __builtin_amdgcn_rcp(g);
    r = fma(r, fma(-g, r, 1.0), r);
    return fma(r, fma(-g, r, 1.0), r);
}

__device__ __forceinline__ void r3_rec(int2 rc, int& k, int& l, int& op2) {
    k = rc.x;
    l = rc.y & 0x0FFFFFFF;
    op2 = (int)((unsigned)rc.y >> 28);
}

__device__ __forceinline__ int64_t r3_j2(const SpaceDev& sd, const int64_t* mat_raw, int k, int l, int op2) {
    return k < 0 ? unary_id(sd, 2, op2, mat_raw[l]) : pair_id(sd, 2, op2, mat_raw[k], mat_raw[l]);
}

// ------------------------------------------------------------ set-up
// max |x| and min |x| of every partner over the n samples.
__global__ __launch_bounds__(256) void k_r3_pstat(int n, int64_t ldn, int pe, const double* __restrict__ Vf,
                                                  double* __restrict__ pstat) {
    const int p = blockIdx.x;
    double mx = 0.0, mn = INFINITY;
    for (int s = threadIdx.x; s < n; s += 256) {
        const double v = fabs(Vf[(int64_t)p * ldn + s]);
        mx = fmax(mx, v);
        mn = fmin(mn, v);
    }
    __shared__ double smx[256], smn[256];
    smx[threadIdx.x] = mx;
    smn[threadIdx.x] = mn;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            smx[threadIdx.x] = fmax(smx[threadIdx.x], smx[threadIdx.x + o]);
            smn[threadIdx.x] = fmin(smn[threadIdx.x], smn[threadIdx.x + o]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        pstat[p] = smx[0];
        pstat[pe + p] = smn[0];
    }
}

// Per-partner sums for add / sub: pc[p (TP + 2) + t] = sum_s x_s y_ts (t <
// TP), sum x (t = TP), sum x^2 (t = TP + 1); one block per partner, a fixed
// reduction order.
__global__ __launch_bounds__(256) void k_r3_pconst(int n, int64_t ldn, int TP, const double* __restrict__ Vf,
                                                   const double* __restrict__ Yn, double* __restrict__ pc) {
    const int p = blockIdx.x;
    __shared__ double part[256];
    for (int t = 0; t < TP + 2; t++) {
        double a = 0.0;
        for (int s = threadIdx.x; s < n; s += 256) {
            const double x = Vf[(int64_t)p * ldn + s];
            a += t < TP ? x * Yn[(int64_t)t * ldn + s] : t == TP ? x : x * x;
        }
        part[threadIdx.x] = a;
        __syncthreads();
        for (int o = 128; o > 0; o >>= 1) {
            if ((int)threadIdx.x < o) part[threadIdx.x] += part[threadIdx.x + o];
            __syncthreads();
        }
        if (threadIdx.x == 0) pc[(int64_t)p * (TP + 2) + t] = part[0];
        __syncthreads();
    }
}

// Right-hand operands: bmat[((c TK + t) NQ + q) 64 + 4 j + e] = column j of
// tile c, kind t, sample 4q + e; kinds t < TP: x y_t, t = TP: x, TP+1: x^2,
// with x = f_p (mul, div and add/sub columns), 1/f_p (rdiv columns) or 1
// (the column of ones of an add/sub tile); zero for padding columns and
// samples >= n.
__global__ __launch_bounds__(256) void k_r3_bmat(int n, int64_t ldn, int TP, int NQ, int nct,
                                                 const int32_t* __restrict__ coldesc,
                                                 const double* __restrict__ Vf, const double* __restrict__ Rf,
                                                 const double* __restrict__ Yn, double* __restrict__ bmat) {
    const int TK = TP + 2;
    const int64_t total = (int64_t)nct * TK * NQ * 64;
    for (int64_t f = (int64_t)blockIdx.x * 256 + threadIdx.x; f < total; f += (int64_t)gridDim.x * 256) {
        const int e = (int)(f & 3), j = (int)((f >> 2) & 15);
        const int64_t r = f >> 6;
        const int q = (int)(r % NQ);
        const int64_t ct_t = r / NQ;
        const int t = (int)(ct_t % TK), c = (int)(ct_t / TK);
        const int s = 4 * q + e;
        const int32_t d = coldesc[c * 16 + j];
        double v = 0.0;
        if (d >= 0 && s < n) {
            const int p = d & 0xFFFF, kind = d >> 16;
            const double x = kind == 3 ? 1.0 : kind == 1 ? Rf[(int64_t)p * ldn + s] : Vf[(int64_t)p * ldn + s];
            v = t < TP ? x * Yn[(int64_t)t * ldn + s] : t == TP ? x : x * x;
        }
        bmat[f] = v;
    }
}

// The targets in the B lane order: yb[q 64 + 4 j + e] = y_j at sample 4q + e
// (0 for j >= TP and samples >= n).
__global__ __launch_bounds__(256) void k_r3_ybmat(int n, int64_t ldn, int TP, int NQ,
                                                  const double* __restrict__ Yn, double* __restrict__ yb) {
    const int64_t total = (int64_t)NQ * 64;
    for (int64_t f = (int64_t)blockIdx.x * 256 + threadIdx.x; f < total; f += (int64_t)gridDim.x * 256) {
        const int e = (int)(f & 3), j = (int)((f >> 2) & 15);
        const int s = 4 * (int)(f >> 6) + e;
        yb[f] = j < TP && s < n ? Yn[(int64_t)j * ldn + s] : 0.0;
    }
}

// ------------------------------------------------------------ MFMA screen
struct R3mArgs {
    const int2* grec;
    int64_t n_grec;
    const int2* work;         // add / sub: (row tile, column tile) per wave
    int64_t n_work;
    const double* pconst;     // add / sub: per-partner sums (k_r3_pconst)
    const int32_t* coldesc;
    int n_gct, n_gblk, NQ, n, T, mode;
    int64_t ldn;
    const double* bmat;
    const double* ybmat;      // add / sub: the targets (k_r3_ybmat)
    const double *Vf, *Rf;
    const double* pstat;
    int pe;
    uint32_t ops;
    const uint8_t *valid, *cls;
    const int64_t* mat_raw;
    const uint8_t* r2v;
    const double* ysum;
    SpaceDev sd;
    SlotMap sm;
    int64_t N;
    double* scores;
    unsigned long long* nscored;
    int64_t* fix_ids;         // score slots
    unsigned long long* fix_cnt;
    int64_t fix_cap;
};

template <int TP, int GT, bool AS>
__global__ __launch_bounds__(256) void k_r3_mm(R3mArgs g) {
    constexpr int TK = TP + 2;
    static_assert(!AS || GT == 1, "add/sub tiles come one per wave");
    const int lane = threadIdx.x & 63;
    const int r16 = lane & 15, kq = lane >> 4;
    int ct;
    int64_t tile0;
    const int64_t w = (int64_t)blockIdx.x * 4 + r3_wave();   // add / sub: the work item
    if (AS) {                                          // explicit (row tile, column tile) list
        if (w >= g.n_work) return;
        const int2 wk = g.work[w];
        tile0 = wk.x;
        ct = wk.y;
    } else {
        const int lb = r3_xcd_block();
        ct = lb / g.n_gblk;                            // column tile (slowest: its operands stay in L2)
        const int gb = lb - ct * g.n_gblk;
        tile0 = ((int64_t)gb * 4 + r3_wave()) * GT;
        if (tile0 * 16 >= g.n_grec) return;
    }
    const bool hk = !AS && ct >= g.n_gct;              // rows hold 1/g (div columns)
    const double* __restrict__ Vf = g.Vf;
    const double* __restrict__ Rf = g.Rf;

    // every tile's records share one operator (runs are padded to 16), so
    // the regeneration's branches are uniform; absent rows read feature 0
    int kk[GT], ll[GT], oo[GT];
    bool rok[GT];
    int64_t j2[GT];
#pragma unroll
    for (int u = 0; u < GT; u++) {
        const int64_t t16 = min(tile0 + u, (g.n_grec >> 4) - 1) * 16;
        const int64_t rec = (tile0 + u) * 16 + r16;
        int k = -2, l = 0, op2;
        r3_rec(g.grec[rec < g.n_grec ? rec : t16], k, l, op2);
        oo[u] = __builtin_amdgcn_readfirstlane(op2);
        rok[u] = rec < g.n_grec && k != -2;
        j2[u] = rok[u] ? r3_j2(g.sd, g.mat_raw, k, l, op2) : 0;
        rok[u] = rok[u] && g.r2v[j2[u] - g.sd.off[2]];
        kk[u] = oo[u] < OP_ADD ? -1 : (rok[u] ? k : 0);
        ll[u] = rok[u] ? l : 0;
    }
    const double* p1[GT];
    const double* p2[GT];
#pragma unroll
    for (int u = 0; u < GT; u++) r3_rows(Vf, Rf, g.ldn, kk[u], ll[u], oo[u], p1[u], p2[u]);
    r3_v4d acc[GT][TK];
#pragma unroll
    for (int u = 0; u < GT; u++)
#pragma unroll
        for (int t = 0; t < TK; t++) acc[u][t] = r3_v4d{0.0, 0.0, 0.0, 0.0};
    double gmx[GT], gmn[GT];
#pragma unroll
    for (int u = 0; u < GT; u++) { gmx[u] = 0.0; gmn[u] = INFINITY; }

    const double* bp = g.bmat + (int64_t)ct * TK * g.NQ * 64 + lane * 4;
    const int nm = g.NQ >> 2;
    if constexpr (AS) {
        // add / sub need per row only sum g y_t, sum g, sum g^2 and per pair
        // sum x g: three product streams, g against [x | 1] (acc[0][TP]),
        // against the targets (acc[0][0], column t = target t) and g^2
        // against [x^2 | 1] (acc[0][TP + 1], its column of ones)
        const double* yp = g.ybmat + lane * 4;
        for (int m = 0; m < nm; m++) {
            const int s = 16 * m + 4 * kq;
            r3_v4d v = r3_combine(oo[0], *(const r3_v4d*)(p1[0] + s), *(const r3_v4d*)(p2[0] + s));
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const bool in = rok[0] && s + e < g.n;
                v[e] = in ? v[e] : 0.0;
            }
            const r3_v4d v2 = v * v;
            const r3_v4d bx = *(const r3_v4d*)(bp + ((int64_t)TP * g.NQ + 4 * m) * 64);
            const r3_v4d bq = *(const r3_v4d*)(bp + ((int64_t)(TP + 1) * g.NQ + 4 * m) * 64);
            const r3_v4d by = *(const r3_v4d*)(yp + (int64_t)(4 * m) * 64);
#pragma unroll
            for (int e = 0; e < 4; e++) {
                acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[e], by[e], acc[0][0], 0, 0, 0);
                acc[0][TP] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[e], bx[e], acc[0][TP], 0, 0, 0);
                acc[0][TP + 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(v2[e], bq[e], acc[0][TP + 1], 0, 0, 0);
            }
        }
    } else {
    for (int m = 0; m < nm; m++) {
        const int s = 16 * m + 4 * kq;
        r3_v4d A[GT], A2[GT];
#pragma unroll
        for (int u = 0; u < GT; u++) {
            r3_v4d v = r3_combine(oo[u], *(const r3_v4d*)(p1[u] + s), *(const r3_v4d*)(p2[u] + s));
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const bool in = rok[u] && s + e < g.n;
                const double x = in ? v[e] : 0.0;
                v[e] = x;
                if (in) {
                    gmx[u] = fmax(gmx[u], fabs(x));
                    gmn[u] = fmin(gmn[u], fabs(x));
                }
                if (hk) v[e] = in ? r3_rcp(x) : 0.0;
            }
            A[u] = v;
            A2[u] = v * v;
        }
#pragma unroll
        for (int t = 0; t < TK; t++) {
            const r3_v4d b = *(const r3_v4d*)(bp + ((int64_t)t * g.NQ + 4 * m) * 64);
#pragma unroll
            for (int u = 0; u < GT; u++) {
                const r3_v4d a = t == TK - 1 ? A2[u] : A[u];
                acc[u][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, acc[u][t], 0, 0, 0);
                acc[u][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.y, acc[u][t], 0, 0, 0);
                acc[u][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.z, b.z, acc[u][t], 0, 0, 0);
                acc[u][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.w, b.w, acc[u][t], 0, 0, 0);
            }
        }
    }
    }
    // row ranges over the four sample groups of each row
#pragma unroll
    for (int u = 0; u < GT; u++) {
        gmx[u] = fmax(gmx[u], __shfl_xor(gmx[u], 16, 64));
        gmx[u] = fmax(gmx[u], __shfl_xor(gmx[u], 32, 64));
        gmn[u] = fmin(gmn[u], __shfl_xor(gmn[u], 16, 64));
        gmn[u] = fmin(gmn[u], __shfl_xor(gmn[u], 32, 64));
    }
    // this lane's column: D[i][j] sits in lane j + 16 (i mod 4), register i / 4
    const double nn = (double)g.n;
    unsigned cnt = 0;
    if (AS) {
        // column 15 holds the ones: sum g y_t, sum g, sum g^2 of each row; a
        // partner column holds sum x g.  The add / sub moments follow from
        // these and the partner's own sums:
        //   S1 = Sx +- Sg, S2 = Sx2 +- 2 Sxg + Sg2, P_t = Sxy_t +- Sgy_t.
        // Their rounding error is below 3.2 n u kappa' with kappa' =
        // (Sx2 + Sg2) / (S2 - S1^2/n), so kappa' <= KAPPA_MAX keeps every
        // score inside the selection margin; other pairs go to the fix-up.
        const int32_t cd = g.coldesc[ct * 16 + r16];
        const int p = cd & 0xFFFF;
        const bool colok = cd >= 0 && (cd >> 16) == 0 && g.valid[p];
        const int src = (lane & 48) | 15;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int i = kq + 4 * r;
            double gs[TK];                             // sum g y_t, sum g, sum g^2 of row i
#pragma unroll
            for (int t = 0; t < TP; t++) gs[t] = __shfl(acc[0][0][r], (lane & 48) | t, 64);
            gs[TP] = __shfl(acc[0][TP][r], src, 64);
            gs[TP + 1] = __shfl(acc[0][TP + 1][r], src, 64);
            const bool ok = __shfl((int)rok[0], i, 64) != 0 && colok;
            if (!ok) continue;
            const double* pc = g.pconst + (int64_t)p * TK;
            const double Sxg = acc[0][TP][r];
            const double A = pc[TP + 1] + gs[TP + 1];
#pragma unroll
            for (int o = 0; o < 2; o++) {
                if (!((g.ops >> o) & 1u)) continue;
                const double sg = o == 0 ? 1.0 : -1.0;
                const int64_t id = slot3as(g.sm, OP_ADD + o, w, i, r16);   // score slot
                const double S1 = pc[TP] + sg * gs[TP];
                const double S2 = pc[TP + 1] + 2.0 * sg * Sxg + gs[TP + 1];
                const double varn = S2 - S1 * (S1 / nn);
                const double kappa = varn > 0.0 ? A / varn : INFINITY;
                if (!(S2 < INFINITY) || !(kappa <= R3_KAPPA_MAX) || S2 <= R3_TAU_CANCEL_FAST * A) {
                    const unsigned long long slot = r3_slot(g.fix_cnt);
                    if ((int64_t)slot < g.fix_cap) g.fix_ids[slot] = id;
                    continue;
                }
                const double isd = 1.0 / sqrt(varn);
                cnt++;
                if (g.mode == DISCOVER_SCORE_MAX) {
                    double best = 0.0;
#pragma unroll
                    for (int t = 0; t < TP; t++)
                        if (t < g.T) best = fmax(best, fabs((pc[t] + sg * gs[t] - S1 * (g.ysum[t] / nn)) * isd));
                    g.scores[id] = best;
                } else {
#pragma unroll
                    for (int t = 0; t < TP; t++)
                        if (t < g.T)
                            g.scores[(int64_t)t * g.N + id] = fabs((pc[t] + sg * gs[t] - S1 * (g.ysum[t] / nn)) * isd);
                }
            }
        }
    } else {
        const int32_t cd = g.coldesc[ct * 16 + r16];
        const int p = cd & 0xFFFF, kind = cd >> 16;
        const int op3 = kind == 0 ? OP_MUL : kind == 1 ? OP_RDIV : OP_DIV;
        const bool colok = cd >= 0 && ((g.ops >> (op3 - OP_ADD)) & 1u) && g.valid[p];
        const double xmx = colok ? g.pstat[p] : 0.0, xmn = colok ? g.pstat[g.pe + p] : 1.0;
    #pragma unroll
        for (int u = 0; u < GT; u++) {
    #pragma unroll
            for (int r = 0; r < 4; r++) {
                const int i = kq + 4 * r;                      // row of this register
                const bool ok = __shfl((int)rok[u], i, 64) != 0 && colok;
                const double rmx = __shfl(gmx[u], i, 64), rmn = __shfl(gmn[u], i, 64);
                if (!ok) continue;
                const int64_t id = slot3(g.sm, op3, (tile0 + u) * 16 + i, p);   // score slot
                // finiteness of the candidate's values
                bool sure = true;
                if (op3 == OP_MUL) {
                    sure = rmx * xmx < R3_BIG;
                } else if (op3 == OP_DIV) {
                    if (rmn == 0.0) continue;                  // x / 0: not finite
                    sure = rmn >= R3_TINY && xmx < R3_BIG * rmn;
                } else {
                    if (xmn == 0.0) continue;                  // g / 0: not finite
                    sure = xmn >= R3_TINY && rmx < R3_BIG * xmn;
                }
                const double S1 = acc[u][TP][r], S2 = acc[u][TP + 1][r];
                const double varn = S2 - S1 * (S1 / nn);
                const double kappa = varn > 0.0 ? S2 / varn : INFINITY;
                if (!sure || !(kappa <= R3_KAPPA_MAX)) {
                    const unsigned long long slot = r3_slot(g.fix_cnt);
                    if ((int64_t)slot < g.fix_cap) g.fix_ids[slot] = id;
                    continue;
                }
                const double isd = 1.0 / sqrt(varn);
                cnt++;
                if (g.mode == DISCOVER_SCORE_MAX) {
                    double best = 0.0;
    #pragma unroll
                    for (int t = 0; t < TP; t++)
                        if (t < g.T) best = fmax(best, fabs((acc[u][t][r] - S1 * (g.ysum[t] / nn)) * isd));
                    g.scores[id] = best;
                } else {
    #pragma unroll
                    for (int t = 0; t < TP; t++)
                        if (t < g.T)
                            g.scores[(int64_t)t * g.N + id] = fabs((acc[u][t][r] - S1 * (g.ysum[t] / nn)) * isd);
                }
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor((int)cnt, o, 64);
    if (lane == 0 && cnt) atomicAdd(g.nscored, (unsigned long long)cnt);
}

// ------------------------------------------------------------ precision form
// BF16 numerators, split-BF16 moments.  Per 32-sample chunk a wave
// regenerates its 16 rows (rung-2 features, as above) in FP64 and rounds
// them to FP32 (a) and BF16 (a_h).  Every product
// is a v_mfma_f32_16x16x32_bf16 (lane l supplies row l%16 at samples
// 8(l/16)..+7 of the chunk and column l%16 at the same samples, and
// receives D[4(l/16)+e][l%16] in slot e): the T numerators against x y_t
// rounded to BF16, and the moments S1 = sum a x and S2 = sum a^2 x^2 each
// from three products of two-term splits a = a_h + a_l (a_h = BF16(a), a_l
// = BF16(a - a_h)): a_h x_h + (a_h x_l + a_l x_h), the cross terms in an
// accumulator of their own.
//
// Error: with u = 2^-8 (plus the FP64 -> FP32 -> BF16 double rounding) the
// product of two rounded values is within 2u + u^2 of the true product and
// the FP32 sum adds gamma_n, so |P_lp - P| <= delta ||f|| ||y_t|| and
// |r_lp - r| <= delta sqrt(kappa) with kappa = S2 / (S2 - S1^2/n): delta is
// the precision form's BF16 bound.  A split product misses a_l x_l and the
// splits' own rounding: within 3 2^-16 of a x (plus the FP32 roundings of a,
// x, a^2 and x^2, 8 v, v = 2^-24); the FP32 accumulation adds at most
// (n + 42) v of the summed magnitudes (at most 31 roundings inside one
// product's 32-term sum, one per accumulation).  So |dS1| <= e sqrt(n)
// ||f|| and |dS2| <= e S2 with e = (n + 50) v + 3 2^-16, the variance moves
// by at most 3 e kappa of itself and the score (targets centred, unit norm)
// by at most cm kappa with cm = 3 e (r3_moment_err); kappa itself is then
// known within a factor 1 +- 4/3 cm kappa, which the bound below absorbs.
// Scores with kappa <= LP_KAPPA are stored (error within the selection
// margin 1.1 delta + 1.5 cm); others store the upper bound -(s + delta
// sqrt(kappa)(1 + cm kappa) + 1.1 cm kappa) and are rescored exactly when
// they can reach the pool.  Rows or partners whose values leave a safe FP32
// range (products above LP_BIG, squares above LP_BIG2, a norm below
// LP_SMALL2 where subnormals would matter) or whose kappa makes cm kappa
// exceed 0.05 go to the exact fix-up.
constexpr double LP_BIG = 1e30;
constexpr double LP_BIG2 = 1e16;        // |f|, |g|, |x| below this: n f^2 stays finite in FP32
constexpr double LP_SMALL2 = 1e-10;     // ||f|| above this: FP32 subnormals are negligible
constexpr double LP_KAPPA = 1.21;

typedef double r3_v2d __attribute__((ext_vector_type(2)));
typedef __attribute__((ext_vector_type(8))) __bf16 r3_bf16x8;
typedef __attribute__((ext_vector_type(4))) float r3_f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned r3_u32x4;

// Two FP32 values rounded to BF16 (nearest, ties to even: gfx950's packed
// conversion) and packed, lo in bits 0..15, hi in bits 16..31; the layout
// kernel and the screen round the same way.
__device__ __forceinline__ unsigned r3_bf16_pack(float lo, float hi) {
    typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
    bf2 v;
    v[0] = (__bf16)lo;
    v[1] = (__bf16)hi;
    return __builtin_bit_cast(unsigned, v);
}

// Two-term BF16 splits of two FP32 values: hi = their BF16 roundings
// (packed as r3_bf16_pack), lo = the BF16 roundings of the exact remainders
// v - hi.
__device__ __forceinline__ void r3_split(float v0, float v1, unsigned& hi, unsigned& lo) {
    hi = r3_bf16_pack(v0, v1);
    __asm__("" : "+v"(hi));              // (the compiler would otherwise convert v0 twice)
    const float h0 = __uint_as_float(hi << 16), h1 = __uint_as_float(hi & 0xFFFF0000u);
    lo = r3_bf16_pack(v0 - h0, v1 - h1);
}

// Right-hand operands of the precision form, per column tile c and 32-sample
// chunk ch 4 + TP blocks of 512 BF16, lane-major (entry 8 l + e belongs to
// column l%16 at sample 32 ch + 8(l/16) + e): the splits x_h, x_l, (x^2)_h,
// (x^2)_l of FP32(x) and its square, then x y_t rounded, t < TP.  This is
// the layout the screen's blocks copy into LDS.
__global__ __launch_bounds__(256) void k_r3_bmat_lp(int n, int64_t ldn, int TP, int NC, int nct,
                                                    const int32_t* __restrict__ coldesc,
                                                    const double* __restrict__ Vf, const double* __restrict__ Rf,
                                                    const double* __restrict__ Yn, __bf16* __restrict__ blp) {
    const int TB = 4 + TP;
    const int64_t total = (int64_t)nct * NC * 512;
    for (int64_t f = (int64_t)blockIdx.x * 256 + threadIdx.x; f < total; f += (int64_t)gridDim.x * 256) {
        const int w = (int)(f % 512);
        const int64_t cc = f / 512;
        const int ch = (int)(cc % NC), c = (int)(cc / NC);
        const int l = w >> 3, e = w & 7;
        const int j = l & 15, s = 32 * ch + 8 * (l >> 4) + e;
        const int32_t d = coldesc[c * 16 + j];
        double x = 0.0;
        if (d >= 0 && s < n) {
            const int p = d & 0xFFFF, kind = d >> 16;
            x = kind == 3 ? 1.0 : kind == 1 ? Rf[(int64_t)p * ldn + s] : Vf[(int64_t)p * ldn + s];
        }
        unsigned short* o = (unsigned short*)blp + cc * TB * 512 + w;
        const float x32 = (float)x;
        unsigned hi, lo;
        r3_split(x32, x32 * x32, hi, lo);
        o[0] = (unsigned short)hi;
        o[512] = (unsigned short)lo;
        o[1024] = (unsigned short)(hi >> 16);
        o[1536] = (unsigned short)(lo >> 16);
        for (int t = 0; t < TP; t++) {
            const double yv = s < n ? Yn[(int64_t)t * ldn + s] : 0.0;
            o[(4 + t) * 512] = (unsigned short)r3_bf16_pack((float)(x * yv), 0.0f);
        }
    }
}

struct R3lpArgs {
    R3mArgs m;
    const __bf16* blp;
    const double* r2q;        // mean square of each rung-2 feature (by id - off[2])
    int NC;
    int ct0, ct1;             // column tiles of the launch
    double delta;
    double cm;                // FP32-moment error coefficient (r3_moment_err)
};

typedef float r3_f32x2 __attribute__((ext_vector_type(2)));

// A block's four waves take four row tiles (16 rung-2 features each)
// against CT column tiles (16 partner columns each): a wave regenerates its
// row values once per chunk and issues the products of every column tile
// from them.  The column tiles' operands of a chunk (4 + TP KB per tile) are
// copied from memory into LDS once per block, double-buffered, and each wave
// reads them there (16 contiguous bytes per lane per read).
// The row operands are loaded with the samples across the lanes (16 lanes
// read 256 contiguous bytes of a row), combined and rounded to FP32 in that
// order and turned to the products' order (a lane's 8 samples of one row)
// through 2 KB of the wave's own LDS: loaded in the products' order, each
// load would touch 64 cache lines.
// Bound: no unit by itself.  At 8 targets the mul / rdiv tiles keep vector
// instructions busy for 37 % of the cycles, LDS for 32 % and the matrix cores
// for 30 %, in two waves per SIMD (all that the accumulators leave) that wait
// on memory or LDS for a third of theirs.  Measured with 24 partners, 8
// targets and 2000 samples, all rung-2 features: mul / rdiv tiles 6.6 ms, div
// tiles 5.2 ms (with operands through registers, two column tiles per wave
// and rows in the products' order 11.9 and 7.1; with three tiles and copies
// to LDS, rows in the products' order, 8.4 and 6.5).
// HK: the launch's column tiles multiply 1/g (div), else g (mul, rdiv);
// the two kinds are separate launches, so that neither carries the
// other's per-sample work.  Column tiles past the launch's range (the last
// group may be short) repeat its last tile and store nothing.
template <int TP, int CT, bool HK>
__global__ __launch_bounds__(256, 2) void k_r3_lp(R3lpArgs a) {
    const R3mArgs& g = a.m;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int r16 = lane & 15, kq = lane >> 4;
    const int lb = r3_xcd_block();
    const int cb = lb / g.n_gblk;
    const int ctb = a.ct0 + cb * CT;                     // first column tile of the block
    const int64_t tile0 = (int64_t)(lb - cb * g.n_gblk) * 4 + r3_wave();
    constexpr bool hk = HK;
    bool rok;
    int64_t j2;
    int oo, rkind;                                       // of every row of the block (build_r3_plan)
    bool rzero;                                          // 1/g is infinite through a zero operand
    const double* b1;
    const double* b2;
    unsigned ri1[4], ri2[4];
    {
        int k = -2, l = 0, op2;
        r3_rec(g.grec[tile0 * 16 + r16], k, l, op2);
        op2 = __builtin_amdgcn_readfirstlane(op2);
        oo = op2;
        rok = k != -2;
        j2 = rok ? r3_j2(g.sd, g.mat_raw, k, l, op2) : 0;
        rok = rok && g.r2v[j2 - g.sd.off[2]];
        int i1, i2;
        rkind = r3_rows_lp(g.Vf, g.Rf, rok ? k : 0, rok ? l : 0, op2, hk, b1, b2, i1, i2);
        rzero = hk && rkind == RK_PROD && (((b1 == g.Rf ? g.cls[i1] : 0) | (b2 == g.Rf ? g.cls[i2] : 0)) & PC_ZERO);
#pragma unroll
        for (int h = 0; h < 4; h++) {
            ri1[h] = (unsigned)__shfl(i1, 4 * h + kq, 64);
            ri2[h] = (unsigned)__shfl(i2, 4 * h + kq, 64);
        }
    }
    r3_f32x4 s1[CT], s2[CT], c1[CT], c2[CT];              // moments: a_h x_h and cross terms
    r3_f32x4 pa[CT][TP];
    float hmx = 0.0f;                                    // div tiles: max |1/g| of the lane's samples, rounded
#pragma unroll
    for (int c = 0; c < CT; c++) {
        s1[c] = r3_f32x4{0.f, 0.f, 0.f, 0.f};
        s2[c] = r3_f32x4{0.f, 0.f, 0.f, 0.f};
        c1[c] = r3_f32x4{0.f, 0.f, 0.f, 0.f};
        c2[c] = r3_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < TP; t++) pa[c][t] = r3_f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // LDS buffer: per column tile the 4 + TP blocks of a chunk, copied
    // straight from memory (1 KB per wave instruction)
    constexpr int TB = (4 + TP) * 1024;
    constexpr int BUF = CT * TB;
    __shared__ __attribute__((aligned(16))) char smem[2 * BUF];
    __shared__ __attribute__((aligned(16))) char trow[4 * 2048];
    const int wv = r3_wave();
    auto stage = [&](int ch, int buf) {
#pragma unroll
        for (int c = 0; c < CT; c++) {
            const int ctc = min(ctb + c, a.ct1 - 1);
            const char* src = (const char*)a.blp + ((int64_t)ctc * a.NC + ch) * TB + wv * 1024;
            __asm__("" : "+s"(src));                     // (uniform base, lane offset: no address registers)
            char* dst = smem + buf * BUF + c * TB;
#pragma unroll
            for (int v = 0; v < (4 + TP + 3) / 4; v++) {
                const int b = 4 * v + wv;
                if ((4 + TP) % 4 == 0 || b < 4 + TP)
                    __builtin_amdgcn_global_load_lds(
                        (const __attribute__((address_space(1))) void*)(src + v * 4096 + (unsigned)(lane * 16)),
                        (__attribute__((address_space(3))) void*)(dst + b * 1024), 16, 0, 0);
            }
        }
    };
    // row operands of chunk ch: lane l loads samples 2(l%16), +1 of rows
    // l/16 + 4h
    struct Ld {
        r3_v2d x1[4], x2[4];
    };
    auto load_rows = [&](int ch, Ld& L) {
        unsigned ldb = (unsigned)(g.ldn * 8);
        __asm__("" : "+s"(ldb));                         // (addresses formed here, not kept)
        const char* q1 = (const char*)b1 + (int64_t)ch * 256 + r16 * 16;
        const char* q2 = (const char*)b2 + (int64_t)ch * 256 + r16 * 16;
#pragma unroll
        for (int h = 0; h < 4; h++) {
            L.x1[h] = *(const r3_v2d*)(q1 + (uint64_t)ri1[h] * ldb);
            L.x2[h] = *(const r3_v2d*)(q2 + (uint64_t)ri2[h] * ldb);
        }
    };
    char* const tw = trow + wv * 2048 + kq * 128 + (r16 & 1) * 8;
    const int tws = ((r16 >> 1) ^ (kq >> 1)) * 16;
    const char* const tr = trow + wv * 2048 + r16 * 128;
    const int trs = ((2 * kq) ^ (r16 >> 1)) * 16;
    // a chunk's left-hand operands: a_h (also the numerators'), a_l and the
    // splits of a^2
    struct Lhs {
        r3_u32x4 ah, al, qh, ql;
    };
    // Row values of a chunk, in FP32, to the wave's LDS (row r: 32 values in
    // eight 16-byte pieces, piece q at q ^ (r / 2): writes and reads touch
    // every bank once).  Only the last chunk holds samples >= n: there the
    // values are set to 0 (the right-hand operands are 0 too, but a row value
    // there may be inf or NaN).  A row whose feature is invalid only reaches
    // its own row of the products, whose scores are never stored, so it is
    // not masked.  FP64 -> FP32 here and FP32 -> BF16 in prepare are two
    // hardware roundings (the error bound counts both).
    auto combine = [&](const Ld& L, auto kind_c, double (&v)[8]) {
        constexpr int kind = decltype(kind_c)::value;
        if constexpr (kind == RK_OTHER) {
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const r3_v4d w = r3_combine(oo, r3_v4d{L.x1[2 * h].x, L.x1[2 * h].y, L.x1[2 * h + 1].x, L.x1[2 * h + 1].y},
                                            r3_v4d{0.0, 0.0, 0.0, 0.0});
#pragma unroll
                for (int e = 0; e < 4; e++) v[4 * h + e] = w[e];
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; e++) {
                const double x = L.x1[e >> 1][e & 1], y = L.x2[e >> 1][e & 1];
                v[e] = kind == RK_PROD ? x * y : kind == RK_ADD ? x + y : x - y;
            }
        }
    };
    auto form = [&](int ch, const Ld& L, auto kind_c, auto tail_c) {
        constexpr int kind = decltype(kind_c)::value;
        constexpr bool tail = decltype(tail_c)::value;
        double v[8];
        combine(L, kind_c, v);
#pragma unroll
        for (int h = 0; h < 4; h++) {
            r3_f32x2 w;
#pragma unroll
            for (int e = 0; e < 2; e++) {
                double x = v[2 * h + e];
                if (hk && kind != RK_PROD) x = r3_rcp(x);
                if (tail && 32 * ch + 2 * r16 + e >= g.n) x = 0.0;
                w[e] = (float)x;
            }
            *(r3_f32x2*)(tw + h * 512 + (tws ^ (32 * h))) = w;
        }
    };
    auto prepare = [&](Lhs& A) {
        float vf[8];
        *(r3_f32x4*)vf = *(const r3_f32x4*)(tr + trs);
        *(r3_f32x4*)(vf + 4) = *(const r3_f32x4*)(tr + (trs ^ 16));
#pragma unroll
        for (int e = 0; e < 8; e++)
            if (hk) hmx = fmaxf(hmx, fabsf(vf[e]));      // NaN leaves it unchanged
#pragma unroll
        for (int e = 0; e < 4; e++) {
            unsigned h, l;
            r3_split(vf[2 * e], vf[2 * e + 1], h, l);
            A.ah[e] = h;
            A.al[e] = l;
            r3_split(vf[2 * e] * vf[2 * e], vf[2 * e + 1] * vf[2 * e + 1], h, l);
            A.qh[e] = h;
            A.ql[e] = l;
        }
    };
    // The products of a chunk in groups of up to 4 right-hand operands: per
    // column tile the moments (x_h, x_l, (x^2)_h, (x^2)_l; 6 products), then
    // the targets by fours.  A group's operands are read from LDS while the
    // products of the group before it run (the scheduling barriers keep the
    // reads there: the compiler would move each to its product and wait out
    // the LDS latency every time).
    constexpr int GT = (TP + 3) / 4, NG = CT * (1 + GT);
    struct Rhs {
        r3_bf16x8 v[4];
    };
    auto read_group = [&](int buf, auto gi_c, Rhs& R) {
        constexpr int gi = decltype(gi_c)::value, c = gi / (1 + GT), q = gi % (1 + GT);
        const char* xs = smem + buf * BUF + c * TB + 16 * lane;
        constexpr int n = q == 0 || TP >= 4 * q ? 4 : TP - 4 * (q - 1);
#pragma unroll
        for (int i = 0; i < n; i++) R.v[i] = *(const r3_bf16x8*)(xs + (q * 4 + i) * 1024);
    };
    auto mul_group = [&](const Lhs& A, auto gi_c, const Rhs& R) {
        constexpr int gi = decltype(gi_c)::value, c = gi / (1 + GT), q = gi % (1 + GT);
        const r3_bf16x8 av = __builtin_bit_cast(r3_bf16x8, A.ah);
        if constexpr (q == 0) {
            const r3_bf16x8 avl = __builtin_bit_cast(r3_bf16x8, A.al);
            const r3_bf16x8 aq = __builtin_bit_cast(r3_bf16x8, A.qh);
            const r3_bf16x8 aql = __builtin_bit_cast(r3_bf16x8, A.ql);
            s1[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, R.v[0], s1[c], 0, 0, 0);
            s2[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq, R.v[2], s2[c], 0, 0, 0);
            c1[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(avl, R.v[0], c1[c], 0, 0, 0);
            c2[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aql, R.v[2], c2[c], 0, 0, 0);
            c1[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, R.v[1], c1[c], 0, 0, 0);
            c2[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq, R.v[3], c2[c], 0, 0, 0);
        } else {
            constexpr int t0 = 4 * (q - 1), n = TP - t0 < 4 ? TP - t0 : 4;
#pragma unroll
            for (int i = 0; i < n; i++)
                pa[c][t0 + i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, R.v[i], pa[c][t0 + i], 0, 0, 0);
        }
    };
    Rhs R[2];
    auto products = [&](int buf, const Lhs& A) {             // (group 0 has been read)
        auto step = [&](auto self, auto gi_c) -> void {
            constexpr int gi = decltype(gi_c)::value;
            if constexpr (gi + 1 < NG) read_group(buf, std::integral_constant<int, gi + 1>{}, R[(gi + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            mul_group(A, gi_c, R[gi & 1]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (gi + 1 < NG) self(self, std::integral_constant<int, gi + 1>{});
        };
        step(step, std::integral_constant<int, 0>{});
    };
    // Per chunk: the loads of the next chunk's row operands and the copies of
    // its right-hand operands start, this chunk's left-hand operands and
    // products are formed, then the next chunk's row values, and the block
    // meets once the copies are in LDS.
    auto run = [&](auto kind_c) {
        const int NC = a.NC;
        Ld L;
        Lhs A;
        stage(0, 0);
        load_rows(0, L);
        if (NC > 1)
            form(0, L, kind_c, std::false_type{});
        else
            form(0, L, kind_c, std::true_type{});
        __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        for (int ch = 0; ch < NC; ch++) {
            const bool more = ch + 1 < NC;
            if (more) {
                load_rows(ch + 1, L);
                stage(ch + 1, (ch + 1) & 1);
            }
            prepare(A);
            read_group(ch & 1, std::integral_constant<int, 0>{}, R[0]);
            products(ch & 1, A);
            if (!more) break;
            if (ch + 2 < NC)
                form(ch + 1, L, kind_c, std::false_type{});
            else
                form(ch + 1, L, kind_c, std::true_type{});
            __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
        }
    };
    // (block-uniform: every wave takes the same loop and its barriers)
    switch (rkind) {
    case RK_PROD: run(std::integral_constant<int, RK_PROD>{}); break;
    case RK_ADD: run(std::integral_constant<int, RK_ADD>{}); break;
    case RK_SUB: run(std::integral_constant<int, RK_SUB>{}); break;
    default: run(std::integral_constant<int, RK_OTHER>{}); break;
    }
    // of rows 4 kq + e: max |1/g| or a bound of it, and whether g has a zero
    double hx4[4] = {0.0, 0.0, 0.0, 0.0};
    bool gz4[4] = {false, false, false, false};
    if constexpr (hk) {
        hmx = fmaxf(hmx, __shfl_xor(hmx, 16, 64));
        hmx = fmaxf(hmx, __shfl_xor(hmx, 32, 64));
        // the largest rounded value, rounded up (from the FP32 subnormals too)
        const double hb = fmax((double)hmx * (1.0 + 0x1p-22), 0x1p-125);
        bool far = false;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            hx4[e] = __shfl(hb, 4 * kq + e, 64);
            gz4[e] = __shfl((int)rzero, 4 * kq + e, 64) != 0;
            const bool ok = __shfl((int)rok, 4 * kq + e, 64) != 0 && !gz4[e];
            const double rmn = 1.0 / hx4[e];
#pragma unroll
            for (int c = 0; c < CT; c++) {
                const int32_t cd = g.coldesc[min(ctb + c, a.ct1 - 1) * 16 + r16];
                if (!ok || cd < 0 || !g.valid[cd & 0xFFFF]) continue;
                const double xmx = g.pstat[cd & 0xFFFF];
                const bool in = rmn >= R3_TINY && xmx < R3_BIG * rmn && hx4[e] < LP_BIG2 && xmx * hx4[e] < LP_BIG2;
                far = far || !in || !(s2[c][e] + c2[c][e] < INFINITY);
            }
        }
        // where that does not settle a candidate's range, or its sums are not
        // finite (a zero of g gives no reciprocal): the largest |1/g| in FP64
        // and the zeros, from the rows again
        if (__any(far)) {
            double hm[4] = {0.0, 0.0, 0.0, 0.0};         // of row l/16 + 4h
            unsigned hz = 0;                             // bit h: zero
            auto scan = [&](auto kind_c) {
                constexpr int kind = decltype(kind_c)::value;
                for (int ch = 0; ch < a.NC; ch++) {
                    Ld L;
                    load_rows(ch, L);
                    double v[8];
                    combine(L, kind_c, v);
#pragma unroll
                    for (int e = 0; e < 8; e++) {
                        if (32 * ch + 2 * r16 + (e & 1) >= g.n) continue;
                        if (kind != RK_PROD && v[e] == 0.0) hz |= 1u << (e >> 1);
                        hm[e >> 1] = fmax(hm[e >> 1], fabs(kind == RK_PROD ? v[e] : r3_rcp(v[e])));
                    }
                }
            };
            switch (rkind) {
            case RK_PROD: scan(std::integral_constant<int, RK_PROD>{}); break;
            case RK_ADD: scan(std::integral_constant<int, RK_ADD>{}); break;
            case RK_SUB: scan(std::integral_constant<int, RK_SUB>{}); break;
            default: scan(std::integral_constant<int, RK_OTHER>{}); break;
            }
            uint64_t z = 0;                              // of rows 4 kq .. 4 kq + 3: 16 bits each
#pragma unroll
            for (int h = 0; h < 4; h++) {
                for (int o = 8; o > 0; o >>= 1) hm[h] = fmax(hm[h], __shfl_xor(hm[h], o, 64));
                const uint64_t m = __builtin_amdgcn_ballot_w64((hz >> h) & 1u);
                z = kq == h ? m : z;
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const double x = __shfl(hm[h], 16 * e, 64);      // row 4 h + e
                    hx4[e] = kq == h ? x : hx4[e];
                }
            }
#pragma unroll
            for (int e = 0; e < 4; e++) gz4[e] = gz4[e] || ((z >> (16 * e)) & 0xFFFFu) != 0;
        }
    }
    const double nn = (double)g.n;
    unsigned cnt = 0;
#pragma unroll
    for (int c = 0; c < CT; c++) {
        if (ctb + c >= a.ct1) continue;                  // repeated tile: stores nothing
        const int ct = ctb + c;
        const int32_t cd = g.coldesc[ct * 16 + r16];
        const int p = cd & 0xFFFF, kind = cd >> 16;
        const int op3 = kind == 0 ? OP_MUL : kind == 1 ? OP_RDIV : OP_DIV;
        const bool colok = cd >= 0 && ((g.ops >> (op3 - OP_ADD)) & 1u) && g.valid[p];
        const double xmx = colok ? g.pstat[p] : 0.0, xmn = colok ? g.pstat[g.pe + p] : 1.0;
        double S1[4], S2[4];                             // row 4 kq + e in slot e
#pragma unroll
        for (int e = 0; e < 4; e++) {
            S1[e] = (double)s1[c][e] + (double)c1[c][e];
            S2[e] = (double)s2[c][e] + (double)c2[c][e];
        }
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const int i = 4 * kq + e;                      // row of slot e
            const bool ok = __shfl((int)rok, i, 64) != 0 && colok;
            const int64_t gj = __shfl(j2, i, 64);
            const double hx = hx4[e];
            if (!ok) continue;
            // max |g| <= sqrt(sum g^2) = sqrt(n E[g^2]) (E[g^2] recorded by the
            // rung-2 screen; 1 % margin for its rounding): only compared with
            // range limits many orders of magnitude away; min |g| = 1 / max
            // |1/g| (div tiles only)
            const double rmx = sqrt(nn * a.r2q[gj - g.sd.off[2]]) * 1.01;
            const double rmn = hk ? 1.0 / hx : 0.0;
            const int64_t id = slot3(g.sm, op3, tile0 * 16 + i, p);   // score slot
            bool sure;
            double amx, fmx, bmx;                          // largest |A|, |f|, |B| of the products
            if (op3 == OP_MUL) {
                sure = rmx * xmx < R3_BIG;
                amx = rmx; fmx = rmx * xmx; bmx = xmx;
            } else if (op3 == OP_DIV) {
                if (gz4[e]) continue;                      // x / 0: not finite
                sure = rmn >= R3_TINY && xmx < R3_BIG * rmn;
                amx = hx; fmx = xmx * hx; bmx = xmx;
            } else {
                if (xmn == 0.0) continue;                  // g / 0: not finite
                sure = xmn >= R3_TINY && rmx < R3_BIG * xmn;
                amx = rmx; fmx = rmx / xmn; bmx = 1.0 / xmn;
            }
            const double varn = S2[e] - S1[e] * (S1[e] / nn);
            const double kappa = varn > 0.0 ? S2[e] / varn : INFINITY;
            const bool lp_ok = amx < LP_BIG2 && fmx < LP_BIG2 && bmx < LP_BIG2 &&
                               S2[e] > LP_SMALL2 * LP_SMALL2 && a.cm * kappa <= 0.05;
            if (!sure || !lp_ok || !(kappa <= R3_KAPPA_MAX)) {
                const unsigned long long slot = r3_slot(g.fix_cnt);
                if ((int64_t)slot < g.fix_cap) g.fix_ids[slot] = id;
                continue;
            }
            const double isd = 1.0 / sqrt(varn);
            const bool precise = kappa <= LP_KAPPA;
            const double ub = a.delta * sqrt(kappa) * (1.0 + a.cm * kappa) + 1.1 * a.cm * kappa;
            cnt++;
            if (g.mode == DISCOVER_SCORE_MAX) {
                double best = 0.0;
#pragma unroll
                for (int t = 0; t < TP; t++)
                    if (t < g.T) best = fmax(best, fabs(((double)pa[c][t][e] - S1[e] * (g.ysum[t] / nn)) * isd));
                g.scores[id] = precise ? best : -(best + ub);
            } else {
#pragma unroll
                for (int t = 0; t < TP; t++)
                    if (t < g.T) {
                        const double r = fabs(((double)pa[c][t][e] - S1[e] * (g.ysum[t] / nn)) * isd);
                        g.scores[(int64_t)t * g.N + id] = precise ? r : -(r + ub);
                    }
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor((int)cnt, o, 64);
    if (lane == 0 && cnt) atomicAdd(g.nscored, (unsigned long long)cnt);
}

// One launch over the mul / rdiv column tiles [0, n_gct), one over the div
// tiles [n_gct, nct); each in groups of CT tiles per block.
template <int TP, int CT, bool HK>
void launch_lp_range(R3lpArgs l, int ct0, int ct1, hipStream_t st) {
    if (ct1 <= ct0) return;
    l.ct0 = ct0;
    l.ct1 = ct1;
    const int64_t groups = (ct1 - ct0 + CT - 1) / CT;
    DSC_REQUIRE((int64_t)l.m.n_gblk * groups < ((int64_t)1 << 31), "rung-3 grid too large");
    k_r3_lp<TP, CT, HK><<<(unsigned)((int64_t)l.m.n_gblk * groups), 256, 0, st>>>(l);
}

// Column tiles per wave: as many as the range holds, up to the most whose
// accumulators leave two waves per SIMD (256 registers): 3 up to 8 targets
// (2 for the div tiles at 8, which would spill), 1 at 16; the rest in
// smaller groups.
template <int TP>
void launch_lp(R3lpArgs l, int n_gct, int nct, int64_t n_grec, hipStream_t st) {
    DSC_REQUIRE(n_grec % 64 == 0, "rung-3 records come in blocks of 64");
    l.m.n_gblk = (int)(n_grec / 64);
    auto range = [&](int c0, int c1, auto hk) {
        constexpr bool HK = decltype(hk)::value;
        constexpr int CMAX = TP <= 4 || (TP <= 8 && !HK) ? 3 : TP <= 8 ? 2 : 1;
        int c = c0;
        if constexpr (CMAX >= 3) {
            const int m = (c1 - c) / 3 * 3;
            launch_lp_range<TP, 3, HK>(l, c, c + m, st);
            c += m;
        }
        if constexpr (CMAX >= 2) {
            const int m = (c1 - c) / 2 * 2;
            launch_lp_range<TP, 2, HK>(l, c, c + m, st);
            c += m;
        }
        launch_lp_range<TP, 1, HK>(l, c, c1, st);
    };
    range(0, n_gct, std::false_type{});
    range(n_gct, nct, std::true_type{});
}

template <class T>
T* r3_up(R3Plan& P, const std::vector<T>& v) {
    void* p = nullptr;
    const size_t bytes = std::max<size_t>(v.size() * sizeof(T), 16);
    if (hipMalloc(&p, bytes) != hipSuccess) DSC_FAIL(DISCOVER_E_NOMEM, "rung-3 plan allocation failed");
    P.allocs.push_back(p);
    if (!v.empty()) DSC_HIP(hipMemcpy(p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice));
    return (T*)p;
}

template <int TP, int GT>
void launch_mm(R3mArgs a, int nct, hipStream_t st) {
    const int64_t ntl = (a.n_grec + 15) / 16;
    a.n_gblk = (int)((ntl + 4 * GT - 1) / (4 * GT));
    const int64_t blocks = (int64_t)a.n_gblk * nct;
    DSC_REQUIRE(blocks < ((int64_t)1 << 31), "rung-3 grid too large");
    k_r3_mm<TP, GT, false><<<(unsigned)blocks, 256, 0, st>>>(a);
}

template <int TP>
void launch_as(const R3mArgs& a, hipStream_t st) {
    const int64_t blocks = (a.n_work + 3) / 4;
    DSC_REQUIRE(blocks < ((int64_t)1 << 31), "rung-3 add/sub grid too large");
    k_r3_mm<TP, 1, true><<<(unsigned)blocks, 256, 0, st>>>(a);
}

}  // namespace

std::shared_ptr<R3Plan> build_r3_plan(const Space& sp, uint32_t r3_ops) {
    auto P = std::make_shared<R3Plan>();
    const SpaceDev& d = sp.d;
    const int B = sp.B, Bq = B > 0 ? B : 1;
    P->ops = r3_ops;
    P->pe = sp.rung_start[d.pool[3] + 1];
    DSC_REQUIRE(P->pe < 65536, "rung-3 partner pool too large");
    const int32_t c0 = sp.rung_start[1], c1 = sp.rung_start[2];
    DSC_REQUIRE(c1 < (1 << 28), "rung-1 operand count too large");
    const int pool2 = d.pool[2];
    const bool addsub = (r3_ops & 3u) != 0;
    // every unit-legal rung-2 feature with its unit vector (unary operators
    // in ID order, binary ones in windows of operands, below)
    std::vector<int2> rec;
    std::vector<int32_t> gunit;
    std::vector<int32_t> u2(Bq, 0);
    auto push = [&](int k, int l, int o) {
        rec.push_back(make_int2(k, l | (o << 28)));
        if (addsub) gunit.insert(gunit.end(), u2.begin(), u2.end());
    };
    // each operator's run is padded to a multiple of 64 records (k = -2:
    // no feature), so that the four 16-row tiles of a block share one
    // operator (k_r3_lp branches on its kind around a loop with barriers)
    auto pad64 = [&](int o) {
        while (rec.size() % 64) {
            rec.push_back(make_int2(-2, o << 28));
            if (addsub) gunit.insert(gunit.end(), Bq, INT32_MIN);
        }
    };
    for (int o = 0; o < OP_ADD; o++) {
        if (d.block[2][o] < 0) continue;
        for (int32_t l = c0; l < c1; l++)
            if (unit_rule(o, B, &sp.mat_unit[(size_t)l * Bq], nullptr, u2.data())) push(-1, l, o);
        pad64(o);
    }
    // binary records in windows of R3_SW operands l by R3_SW operands k: the
    // tiles of a window need 2 R3_SW operand rows, which stay in L2 while
    // its tiles run (the kernels keep neighbouring blocks on one XCD)
    constexpr int32_t R3_SW = 64;
    const int32_t kend = pool2 == 1 ? c1 : sp.rung_start[pool2 + 1];
    for (int o = OP_ADD; o <= OP_RDIV; o++) {
        if (d.block[2][o] < 0) continue;
        for (int32_t l0 = c0; l0 < c1; l0 += R3_SW)
            for (int32_t k0 = 0; k0 < kend; k0 += R3_SW)
                for (int32_t l = l0; l < std::min(l0 + R3_SW, c1); l++) {
                    const int32_t kmax = std::min(pool2 == 1 ? l : sp.rung_start[pool2 + 1], k0 + R3_SW);
                    for (int32_t k = k0; k < kmax; k++)
                        if (unit_rule(o, B, &sp.mat_unit[(size_t)k * Bq], &sp.mat_unit[(size_t)l * Bq], u2.data()))
                            push(k, l, o);
                }
        pad64(o);
    }
    P->n_grec = (int64_t)rec.size();
    DSC_REQUIRE(P->n_grec < ((int64_t)1 << 31), "rung-3 record list too large");
    // partner column tiles: per group of 8 partners, 8 mul then 8 rdiv
    // columns (both against g); then the div columns (against 1/g)
    const bool mul = (r3_ops >> (OP_MUL - OP_ADD)) & 1u, div = (r3_ops >> (OP_DIV - OP_ADD)) & 1u,
               rdiv = (r3_ops >> (OP_RDIV - OP_ADD)) & 1u;
    std::vector<int32_t> cols;
    for (int g8 = 0; g8 < (P->pe + 7) / 8; g8++)
        for (int kind = 0; kind < 2; kind++) {
            if (kind == 0 ? !mul : !rdiv) continue;
            for (int q = 0; q < 8; q++) {
                const int p = 8 * g8 + q;
                cols.push_back(p < P->pe ? (p | (kind << 16)) : -1);
            }
        }
    while (cols.size() % 16) cols.push_back(-1);
    P->n_gct = (int)(cols.size() / 16);
    if (div) {
        for (int p = 0; p < P->pe; p++) cols.push_back(p | (2 << 16));
        while (cols.size() % 16) cols.push_back(-1);
    }
    P->n_ctiles = (int)(cols.size() / 16);
    P->h_coldesc = cols;
    if (P->n_grec) P->grec = r3_up(*P, rec);            // also what the score slots decode
    if (P->n_grec && P->n_ctiles) P->coldesc = r3_up(*P, cols);
    // add / sub: records grouped by unit vector and operator, against
    // column tiles of the partners with the same unit vector (15 at most)
    // and a column of ones
    if (addsub && P->n_grec) {
        auto key = [&](const int32_t* u) { return std::string((const char*)u, sizeof(int32_t) * Bq); };
        std::map<std::string, std::vector<int32_t>> pg;
        for (int p = 0; p < P->pe; p++) pg[key(&sp.mat_unit[(size_t)p * Bq])].push_back(p);
        std::map<std::string, std::map<int, std::vector<int64_t>>> byk;
        for (int64_t r = 0; r < P->n_grec; r++) {
            if (rec[r].x == -2) continue;
            const std::string kk = B > 0 ? key(&gunit[(size_t)r * Bq]) : key(u2.data());
            if (pg.count(kk)) byk[kk][(int)((unsigned)rec[r].y >> 28)].push_back(r);
        }
        std::vector<int2> arec, work;
        std::vector<int32_t> acols;
        for (auto& e : byk) {
            const std::vector<int32_t>& pl = pg[e.first];
            const int ct0 = (int)(acols.size() / 16);
            for (size_t q = 0; q < pl.size(); q += 15) {
                for (size_t z = 0; z < 15; z++) acols.push_back(q + z < pl.size() ? pl[q + z] : -1);
                acols.push_back(3 << 16);                        // the ones
            }
            const int ct1 = (int)(acols.size() / 16);
            for (auto& ro : e.second) {
                const int64_t rt0 = (int64_t)arec.size() / 16;
                for (int64_t r : ro.second) arec.push_back(rec[r]);
                while (arec.size() % 16) arec.push_back(make_int2(-2, ro.first << 28));
                const int64_t rt1 = (int64_t)arec.size() / 16;
                for (int64_t rt = rt0; rt < rt1; rt++)
                    for (int c = ct0; c < ct1; c++) work.push_back(make_int2((int)rt, c));
            }
        }
        DSC_REQUIRE(arec.size() < ((size_t)1 << 35), "rung-3 add/sub list too large");
        P->n_as_grec = (int64_t)arec.size();
        P->n_as_ctiles = (int)(acols.size() / 16);
        P->n_as_work = (int64_t)work.size();
        if (P->n_as_work) {
            P->as_grec = r3_up(*P, arec);
            P->as_coldesc = r3_up(*P, acols);
            P->as_work = r3_up(*P, work);
        }
    }
    return P;
}

void launch_r3(discover_ctx* ctx, const R3Launch& a, hipStream_t st) {
    const R3Plan& P = *a.plan;
    const int NQ = r3_quads(a.n);
    if (P.n_grec && P.n_ctiles && a.precision == DISCOVER_BF16_GUARD) {
        k_r3_pstat<<<(unsigned)P.pe, 256, 0, st>>>(a.n, a.ldn, P.pe, a.Vf, a.pstat);
        check_launch("k_r3_pstat");
        const int NC = r3_chunks(a.n);
        __bf16* blp = (__bf16*)a.bmat;
        const int64_t tot = (int64_t)P.n_ctiles * NC * 512;
        k_r3_bmat_lp<<<(unsigned)std::min<int64_t>(cdiv(tot, 256), 16384), 256, 0, st>>>(
            a.n, a.ldn, a.TP, NC, P.n_ctiles, P.coldesc, a.Vf, a.Rf, a.Yn, blp);
        check_launch("k_r3_bmat_lp");
        R3lpArgs l{};
        R3mArgs& m = l.m;
        m.grec = P.grec; m.n_grec = P.n_grec; m.coldesc = P.coldesc; m.n_gct = P.n_gct;
        m.NQ = NQ; m.n = a.n; m.T = a.T; m.mode = a.mode; m.ldn = a.ldn; m.bmat = a.bmat;
        m.Vf = a.Vf; m.Rf = a.Rf; m.pstat = a.pstat; m.pe = P.pe; m.ops = P.ops;
        m.valid = a.valid; m.cls = a.cls; m.mat_raw = a.mat_raw; m.r2v = a.r2v; m.ysum = a.ysum; m.sd = a.sd;
        m.sm = a.sm; m.N = a.N; m.scores = a.scores; m.nscored = a.nscored; m.fix_ids = a.fix_ids;
        m.fix_cnt = a.fix_cnt; m.fix_cap = a.fix_cap;
        l.blp = blp; l.r2q = a.r2q; l.NC = NC; l.delta = a.delta; l.cm = r3_moment_err(a.n);
        KTimer kt(ctx, st, "screen_r3");
        switch (a.TP) {
        case 1: launch_lp<1>(l, P.n_gct, P.n_ctiles, P.n_grec, st); break;
        case 2: launch_lp<2>(l, P.n_gct, P.n_ctiles, P.n_grec, st); break;
        case 4: launch_lp<4>(l, P.n_gct, P.n_ctiles, P.n_grec, st); break;
        case 8: launch_lp<8>(l, P.n_gct, P.n_ctiles, P.n_grec, st); break;
        default: launch_lp<16>(l, P.n_gct, P.n_ctiles, P.n_grec, st); break;
        }
        check_launch("k_r3_lp");
    } else if (P.n_grec && P.n_ctiles) {
        k_r3_pstat<<<(unsigned)P.pe, 256, 0, st>>>(a.n, a.ldn, P.pe, a.Vf, a.pstat);
        check_launch("k_r3_pstat");
        const int64_t tot = (int64_t)P.n_ctiles * (a.TP + 2) * NQ * 64;
        k_r3_bmat<<<(unsigned)std::min<int64_t>(cdiv(tot, 256), 16384), 256, 0, st>>>(
            a.n, a.ldn, a.TP, NQ, P.n_ctiles, P.coldesc, a.Vf, a.Rf, a.Yn, a.bmat);
        check_launch("k_r3_bmat");
        R3mArgs m{};
        m.grec = P.grec; m.n_grec = P.n_grec; m.coldesc = P.coldesc; m.n_gct = P.n_gct;
        m.NQ = NQ; m.n = a.n; m.T = a.T; m.mode = a.mode; m.ldn = a.ldn; m.bmat = a.bmat;
        m.Vf = a.Vf; m.Rf = a.Rf; m.pstat = a.pstat; m.pe = P.pe; m.ops = P.ops;
        m.valid = a.valid; m.mat_raw = a.mat_raw; m.r2v = a.r2v; m.ysum = a.ysum; m.sd = a.sd;
        m.sm = a.sm; m.N = a.N; m.scores = a.scores; m.nscored = a.nscored; m.fix_ids = a.fix_ids;
        m.fix_cnt = a.fix_cnt; m.fix_cap = a.fix_cap;
        KTimer kt(ctx, st, "screen_r3");
        switch (a.TP) {
        // row tiles per wave: as many as keep two or three waves per SIMD
        // with the accumulators in VGPRs (measured on gfx950: one tile per
        // wave at 8 targets beats two tiles at one wave per SIMD)
        case 1: launch_mm<1, 2>(m, P.n_ctiles, st); break;
        case 2: launch_mm<2, 2>(m, P.n_ctiles, st); break;
        case 4: launch_mm<4, 1>(m, P.n_ctiles, st); break;
        case 8: launch_mm<8, 1>(m, P.n_ctiles, st); break;
        default: launch_mm<16, 1>(m, P.n_ctiles, st); break;
        }
        check_launch("k_r3_mm");
    }
    if (P.n_as_work) {
        double* bm = (double*)((char*)a.bmat + r3_as_offset(P, a.TP, a.n));
        double* pc = a.pstat + 2 * P.pe;
        k_r3_pconst<<<(unsigned)P.pe, 256, 0, st>>>(a.n, a.ldn, a.TP, a.Vf, a.Yn, pc);
        check_launch("k_r3_pconst");
        const int64_t tot = (int64_t)P.n_as_ctiles * (a.TP + 2) * NQ * 64;
        k_r3_bmat<<<(unsigned)std::min<int64_t>(cdiv(tot, 256), 16384), 256, 0, st>>>(
            a.n, a.ldn, a.TP, NQ, P.n_as_ctiles, P.as_coldesc, a.Vf, a.Rf, a.Yn, bm);
        check_launch("k_r3_bmat");
        double* yb = (double*)((char*)a.bmat + r3_asy_offset(P, a.TP, a.n));
        k_r3_ybmat<<<(unsigned)std::min<int64_t>(cdiv((int64_t)NQ * 64, 256), 4096), 256, 0, st>>>(
            a.n, a.ldn, a.TP, NQ, a.Yn, yb);
        check_launch("k_r3_ybmat");
        R3mArgs m{};
        m.grec = P.as_grec; m.n_grec = P.n_as_grec; m.work = P.as_work; m.n_work = P.n_as_work;
        m.pconst = pc; m.coldesc = P.as_coldesc; m.n_gct = 0; m.ybmat = yb;
        m.NQ = NQ; m.n = a.n; m.T = a.T; m.mode = a.mode; m.ldn = a.ldn; m.bmat = bm;
        m.Vf = a.Vf; m.Rf = a.Rf; m.pstat = a.pstat; m.pe = P.pe; m.ops = P.ops;
        m.valid = a.valid; m.mat_raw = a.mat_raw; m.r2v = a.r2v; m.ysum = a.ysum; m.sd = a.sd;
        m.sm = a.sm; m.N = a.N; m.scores = a.scores; m.nscored = a.nscored; m.fix_ids = a.fix_ids;
        m.fix_cnt = a.fix_cnt; m.fix_cap = a.fix_cap;
        KTimer kt(ctx, st, "screen_r3_addsub");
        switch (a.TP) {
        case 1: launch_as<1>(m, st); break;
        case 2: launch_as<2>(m, st); break;
        case 4: launch_as<4>(m, st); break;
        case 8: launch_as<8>(m, st); break;
        default: launch_as<16>(m, st); break;
        }
        check_launch("k_r3_mm(add/sub)");
    }
}

R3Plan::~R3Plan() {
    for (void* p : allocs)
        if (hipFree(p) != hipSuccess) { /* nothing to do */ }
}

}  // namespace dsc
