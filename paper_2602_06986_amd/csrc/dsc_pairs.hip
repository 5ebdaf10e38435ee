// The matrix form of the streamed pair screen: moments and numerators of
// every pair of operand features as FP64 matrix products over samples (see
// dsc_pairs.h for the products and their limits).
//
// v_mfma_f64_16x16x4f64 takes A[i][k] from lane i + 16 k and B[k][j] from
// lane j + 16 k and leaves D[i][j] in lane j + 16 (i mod 4), register i / 4.
// The sum over samples may run in any order, so lane l takes samples
// 4 (l / 16) + e at step e of a 16-sample chunk: its four samples of a
// feature are one 32-byte load.
#include "dsc_internal.h"
#include "dsc_pairs.h"

namespace dsc {
namespace {

typedef double pr_v4d __attribute__((ext_vector_type(4)));

// A wave forms the (2 + T) products of RT x CT tiles of 16 rows i and 16
// columns j for one operator set: a and b (or 1/a, 1/b) are read once per
// tile row and column, their squares and a y_t formed on the way; with KS =
// 4 the waves of a block share one tile, each a run of the samples, and add
// their partial tiles in LDS in wave order.  Bound by the matrix cores: (2
// + T) 2 n flop per candidate of mul, div and rdiv (add and sub take the
// mul tile's sums); the operands of a chunk are a few KB against thousands
// of cycles of products, so nothing is staged in LDS, and the next chunk's
// operands are loaded while this one's products run.  Measured against the
// vector form, which issues 3 + T FP64 instructions per sample and
// operator (7.5 cycles each, its loads exposed at three waves per SIMD),
// both with their launches: 20 features without units, n = 1999: 8 targets
// 3280 -> 1380 us (72 % of the FP64 matrix rate), 1 target 1098 -> 425 us;
// 24 features with units, n = 2000, 8 targets: 1850 -> 1360 us.
template <int TP, int RT, int CT, int KS>
__global__ __launch_bounds__(256, 2) void k_pairs_mm(ctab<PairArgs> A, const int4* __restrict__ work, int64_t n_work) {
    constexpr int TK = TP + 2;
    static_assert(KS == 1 || (RT == 1 && CT == 1), "waves that share a tile share one of 16 x 16");
    const int wv = wave_id();
    const int64_t w = KS == 1 ? (int64_t)blockIdx.x * 4 + wv : (int64_t)blockIdx.x;
    if (w >= n_work) return;
    const int4 wk = work[w];
    const PairArgs& g = tab(A, wk.x);
    if (*g.route == 0) return;
    DSC_GLOBAL(g.Vf); DSC_GLOBAL(g.Rf); DSC_GLOBAL(g.mu); DSC_GLOBAL(g.valid); DSC_GLOBAL(g.mat_raw); DSC_GLOBAL(g.Yn);
    DSC_GLOBAL(g.ysum); DSC_GLOBAL(g.scores); DSC_GLOBAL(g.nscored); DSC_GLOBAL(g.fix_ids); DSC_GLOBAL(g.fix_cnt);
    DSC_GLOBAL(g.msq); DSC_GLOBAL(g.cls); DSC_GLOBAL(g.ex); DSC_GLOBAL(g.fy);
    const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
    const int i0 = wk.y, j0 = wk.z, sel = wk.w;
    const int64_t ldn = g.ldn;
    const double* __restrict__ Va = sel == 2 ? g.Rf : g.Vf;
    const double* __restrict__ Vb = sel == 1 ? g.Rf : g.Vf;
    const double* pa[RT];
    const double* pb[CT];
    double sa[RT], sb[CT];                       // the features' scales
#pragma unroll
    for (int u = 0; u < RT; u++) {
        const int i = min(i0 + 16 * u + r16, g.Mc - 1);
        pa[u] = Va + (int64_t)i * ldn + 4 * kq;
        sa[u] = ldexp(1.0, -(sel == 2 ? g.ex[i].y : g.ex[i].x));
    }
#pragma unroll
    for (int v = 0; v < CT; v++) {
        const int j = min(j0 + 16 * v + r16, g.Mc - 1);
        pb[v] = Vb + (int64_t)j * ldn + 4 * kq;
        sb[v] = ldexp(1.0, -(sel == 1 ? g.ex[j].y : g.ex[j].x));
    }
    const double* __restrict__ py = g.Yn + 4 * kq;
    pr_v4d acc[RT][CT][TK];
#pragma unroll
    for (int u = 0; u < RT; u++)
#pragma unroll
        for (int v = 0; v < CT; v++)
#pragma unroll
            for (int t = 0; t < TK; t++) acc[u][v][t] = pr_v4d{0.0, 0.0, 0.0, 0.0};
    // this wave's run of 16-sample chunks
    const int nch = (g.n + 15) / 16;
    const int first = KS == 1 ? 0 : 16 * ((nch * wv) / KS);
    const int last = 16 * (KS == 1 ? nch : (nch * (wv + 1)) / KS) - 16;
    pr_v4d a[RT], b[CT];
#pragma unroll
    for (int u = 0; u < RT; u++) a[u] = *(const pr_v4d*)(pa[u] + first) * sa[u];
#pragma unroll
    for (int v = 0; v < CT; v++) b[v] = *(const pr_v4d*)(pb[v] + first) * sb[v];
    for (int s = first; s <= last; s += 16) {
        const int sn = min(s + 16, last);
        pr_v4d an[RT], bn[CT];
#pragma unroll
        for (int u = 0; u < RT; u++) an[u] = *(const pr_v4d*)(pa[u] + sn);
#pragma unroll
        for (int v = 0; v < CT; v++) bn[v] = *(const pr_v4d*)(pb[v] + sn);
#pragma unroll
        for (int u = 0; u < RT; u++) {
            const pr_v4d a2 = a[u] * a[u];
#pragma unroll
            for (int v = 0; v < CT; v++) {
                const pr_v4d b2 = b[v] * b[v];
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    acc[u][v][TP] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u][e], b[v][e], acc[u][v][TP], 0, 0, 0);
                    acc[u][v][TP + 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a2[e], b2[e], acc[u][v][TP + 1], 0, 0, 0);
                }
            }
#pragma unroll
            for (int t = 0; t < TP; t++) {
                const pr_v4d ay = a[u] * *(const pr_v4d*)(py + (int64_t)t * ldn + s);
#pragma unroll
                for (int v = 0; v < CT; v++)
#pragma unroll
                    for (int e = 0; e < 4; e++)
                        acc[u][v][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(ay[e], b[v][e], acc[u][v][t], 0, 0, 0);
            }
        }
        // (an empty asm takes the loaded operands here, so that the compiler
        // does not move their loads to the top of the next chunk)
#pragma unroll
        for (int u = 0; u < RT; u++) {
            asm("" : "+v"(an[u].x), "+v"(an[u].y), "+v"(an[u].z), "+v"(an[u].w));
            a[u] = an[u] * sa[u];
        }
#pragma unroll
        for (int v = 0; v < CT; v++) {
            asm("" : "+v"(bn[v].x), "+v"(bn[v].y), "+v"(bn[v].z), "+v"(bn[v].w));
            b[v] = bn[v] * sb[v];
        }
    }

    const double nn = (double)g.n;
    unsigned cnt = 0;
    // one candidate: score from its numerators and n times its variance, or
    // the fix-up list
    auto emit = [&](int op, int64_t ri, int64_t rj, double varn, double kappa, bool sure, double mean, double msq,
                    const double (&num)[TP]) {
        const int64_t id = pair_id(g.sd, g.r, op, ri, rj);
        if (!sure || !(kappa <= g.kappa)) {
            const unsigned long long slot = wave_slot(g.fix_cnt);
            if ((int64_t)slot < g.fix_cap) g.fix_ids[slot] = id;
            return;
        }
        const double isd = 1.0 / sqrt(varn);
        cnt++;
        if (g.r2v) {
            g.r2v[id - g.sd.off[2]] = 1;
            g.r2m[id - g.sd.off[2]] = mean;
            g.r2q[id - g.sd.off[2]] = msq;
        }
        if (g.mode == DISCOVER_SCORE_MAX) {
            double best = 0.0;
#pragma unroll
            for (int t = 0; t < TP; t++)
                if (t < g.T) best = fmax(best, fabs(num[t] * isd));
            g.scores[id] = best;
        } else {
#pragma unroll
            for (int t = 0; t < TP; t++)
                if (t < g.T) g.scores[(int64_t)t * g.N + id] = fabs(num[t] * isd);
        }
    };
    double ys[TP];
#pragma unroll
    for (int t = 0; t < TP; t++) ys[t] = g.ysum[t] / nn;
    // the pair (i, j) with this operator set's sums P_t, S1, S2 in m
    auto pair = [&](int i, int j, const double (&m)[TK]) {
        if (!(j < g.jc_end && i < g.i_end && i < j) || !g.valid[i] || !g.valid[j]) return;
        const int64_t ri = g.mat_raw[i], rj = g.mat_raw[j];
        const uint8_t ci = g.cls[i], cj = g.cls[j];
        const short2 xi = g.ex[i], xj = g.ex[j];
        const int ei = sel == 2 ? xi.y : xi.x, ej = sel == 1 ? xj.y : xj.x;
        const double back = ldexp(1.0, ei + ej);     // undoes the scales
        const double S1 = m[TP], S2 = m[TP + 1];
        double num[TP];
        // the product of this operator set; a zero divisor makes every
        // quotient non-finite (the slot stays invalid)
        const int op = sel == 0 ? OP_MUL : sel == 1 ? OP_DIV : OP_RDIV;
        const uint8_t cd = sel == 0 ? 0 : sel == 1 ? cj : ci;
        if (((g.opmask >> (op - OP_ADD)) & 1u) && !(cd & PC_ZERO)) {
            const bool sure = !(cd & PC_RCP) && ei + ej >= PC_EMIN && ei + ej <= PC_EMAX && S2 >= PC_S2MIN;
            const double varn = S2 - S1 * (S1 / nn);
            const double kappa = varn > 0.0 ? S2 / varn : INFINITY;
            const double mean = S1 / nn * back;
#pragma unroll
            for (int t = 0; t < TP; t++) num[t] = m[t] - S1 * ys[t];
            emit(op, ri, rj, varn, kappa, sure, mean, S2 / nn * back * back, num);
        }
        if (sel != 0 || !(g.opmask & 3u)) return;
        const double ma = g.mu[i], mb = g.mu[j], M1 = S1 * back;
        const double B = nn * (g.msq[i] + g.msq[j]);
        const bool sure = max(xi.x, xj.x) <= PC_EMAX && max(xi.x, xj.x) >= PC_EMIN;
#pragma unroll
        for (int o = 0; o < 2; o++) {
            if (!((g.opmask >> o) & 1u)) continue;
            const double sg = o == 0 ? 1.0 : -1.0;
            const double mean = fma(sg, mb, ma);
            const double q = fma(2.0 * sg, M1, B);
            const double varn = q - nn * mean * mean;
            const double kappa = varn > 0.0 ? B / varn : INFINITY;
#pragma unroll
            for (int t = 0; t < TP; t++) num[t] = fma(sg, g.fy[(int64_t)j * TP + t], g.fy[(int64_t)i * TP + t]);
            emit(OP_ADD + o, ri, rj, varn, kappa, sure, mean, q / nn, num);
        }
    };
    if constexpr (KS > 1) {
        // wave r sums register r of the partial tiles in wave order and
        // finishes its rows
        __shared__ double part[KS][4][64];
        double m[TK];
#pragma unroll
        for (int t = 0; t < TK; t++) {
#pragma unroll
            for (int r = 0; r < 4; r++) part[wv][r][lane] = acc[0][0][t][r];
            __syncthreads();
            m[t] = ((part[0][wv][lane] + part[1][wv][lane]) + part[2][wv][lane]) + part[3][wv][lane];
            __syncthreads();
        }
        pair(i0 + kq + 4 * wv, j0 + r16, m);
    } else {
#pragma unroll
        for (int v = 0; v < CT; v++)
#pragma unroll
            for (int u = 0; u < RT; u++)
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    double m[TK];
#pragma unroll
                    for (int t = 0; t < TK; t++) m[t] = acc[u][v][t][r];
                    pair(i0 + 16 * u + kq + 4 * r, j0 + 16 * v + r16, m);
                }
    }
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor((int)cnt, o, 64);
    if (lane == 0 && cnt) atomicAdd(g.nscored, (unsigned long long)cnt);
}

template <int TP>
void launch(ctab<PairArgs> A, const int4* work, int64_t n, int shape, hipStream_t st) {
    constexpr int RT = TP == 1 ? 2 : 1, CT = TP == 1 || TP == 8 ? 2 : 1;
    if (CT > 1 && shape == 2) k_pairs_mm<TP, RT, CT, 1><<<(unsigned)cdiv(n, 4), 256, 0, st>>>(A, work, n);
    else if (shape) k_pairs_mm<TP, 1, 1, 1><<<(unsigned)cdiv(n, 4), 256, 0, st>>>(A, work, n);
    else k_pairs_mm<TP, 1, 1, 4><<<(unsigned)n, 256, 0, st>>>(A, work, n);
}

}  // namespace

void pairs_mm_tile(int TP, int shape, int& rows, int& cols) {
    rows = cols = 16;
    if (shape < 2) return;
    rows *= TP == 1 ? 2 : 1;
    cols *= TP == 1 || TP == 8 ? 2 : 1;
}

void launch_pairs_mm(ctab<PairArgs> A, const int4* work, int64_t n, int TP, int shape, hipStream_t st) {
    if (n == 0) return;
    switch (TP) {
    case 1: launch<1>(A, work, n, shape, st); break;
    case 2: launch<2>(A, work, n, shape, st); break;
    case 4: launch<4>(A, work, n, shape, st); break;
    case 8: launch<8>(A, work, n, shape, st); break;
    default: launch<16>(A, work, n, shape, st); break;
    }
    check_launch("k_pairs_mm");
}

}  // namespace dsc
