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

#include <type_traits>

namespace dsc {
namespace {

typedef double pr_v4d __attribute__((ext_vector_type(4)));

// A wave forms the (3 + T) products of a tile of 16 rows i and 16 columns j
// for one operator set: a and b (or 1/a, 1/b) are read once and centred,
// squared and multiplied by y_t on the way; with KS = 4 the waves of a block
// share one tile, each a run of the samples, and add their partial tiles in
// LDS in wave order.  Bound by the matrix cores: (3 + T) 2 n flop per
// candidate of mul, div and rdiv (add and sub take the mul tile's sums); the
// operands of a chunk are a few KB against thousands of cycles of products,
// so nothing is staged in LDS; the next chunk's operands and the next two
// targets are loaded while products run (each target's load waited for before
// its products: 125 us instead of 66 for 6 features, 8 targets, n = 2000).
// Measured against the vector form, which issues 3 + T FP64 instructions per
// sample and operator (7.5 cycles each, its loads exposed at three waves per
// SIMD), both with their launches: 20 features without units, n = 1999: 8
// targets 3170 -> 1370 us (76 % of the FP64 matrix rate that a large product
// reaches), 1 target 1070 -> 530 us (FP64 vector instructions take another
// fifth of the cycles, which the matrix cores then stand still).  Without the
// centring (2 + T products, scores off by up to 6e-9 where columns vary by
// 1 %, here 2e-15) 1420 and 420 us.
template <int TP, int KS>
__global__ __launch_bounds__(256, 2) void k_pairs_mm(ctab<PairArgs> A, const int4* __restrict__ work, int64_t n_work) {
    constexpr int TK = TP + 3, G = TP >= 2 ? 2 : 1;      // products; targets in step
    const int wv = wave_id();
    const int64_t w = KS == 1 ? (int64_t)blockIdx.x * 4 + wv : (int64_t)blockIdx.x;
    if (w >= n_work) return;
    const int4 wk = work[w];
    const PairArgs& g = tab(A, wk.x);
    if (*g.bad > PROBE_MAX) return;
    DSC_GLOBAL(g.Vf); DSC_GLOBAL(g.Rf); DSC_GLOBAL(g.mu); DSC_GLOBAL(g.valid); DSC_GLOBAL(g.mat_raw); DSC_GLOBAL(g.Yn);
    DSC_GLOBAL(g.ysum); DSC_GLOBAL(g.scores); DSC_GLOBAL(g.nscored); DSC_GLOBAL(g.fix_ids); DSC_GLOBAL(g.fix_cnt);
    DSC_GLOBAL(g.msq); DSC_GLOBAL(g.cls); DSC_GLOBAL(g.ex); DSC_GLOBAL(g.fy); DSC_GLOBAL(g.mur); DSC_GLOBAL(g.css); DSC_GLOBAL(g.cssr);
    const int lane = threadIdx.x & 63, r16 = lane & 15, kq = lane >> 4;
    const int i0 = wk.y, j0 = wk.z, sel = wk.w;
    const int64_t ldn = g.ldn;
    const int ir = min(i0 + r16, g.Mc - 1), jr = min(j0 + r16, g.Mc - 1);
    const double* pa = (sel == 2 ? g.Rf : g.Vf) + (int64_t)ir * ldn + 4 * kq;
    const double* pb = (sel == 1 ? g.Rf : g.Vf) + (int64_t)jr * ldn + 4 * kq;
    // the features' scales and scaled means
    const double sa = ldexp(1.0, -(sel == 2 ? g.ex[ir].y : g.ex[ir].x)), ca = (sel == 2 ? g.mur[ir] : g.mu[ir]) * sa;
    const double sb = ldexp(1.0, -(sel == 1 ? g.ex[jr].y : g.ex[jr].x)), cb = (sel == 1 ? g.mur[jr] : g.mu[jr]) * sb;
    const double* __restrict__ py = g.Yn + 4 * kq;
    pr_v4d acc[TK];
#pragma unroll
    for (int t = 0; t < TK; t++) acc[t] = pr_v4d{0.0, 0.0, 0.0, 0.0};
    // this wave's run of 16-sample chunks
    const int nch = (g.n + 15) / 16;
    const int first = KS == 1 ? 0 : 16 * ((nch * wv) / KS);
    const int last = 16 * (KS == 1 ? nch : (nch * (wv + 1)) / KS) - 16;
    // DIV: the columns' operand is centred and the rows' enters as it is
    auto run = [&](auto div_c) {
        constexpr bool DIV = decltype(div_c)::value;
        pr_v4d a = *(const pr_v4d*)(pa + first) * sa, b = *(const pr_v4d*)(pb + first) * sb;
        for (int s = first; s <= last; s += 16) {
            const int sn = min(s + 16, last);
            // loads return in order: the first targets' before the next chunk's
            pr_v4d y[G];
#pragma unroll
            for (int q = 0; q < G; q++) y[q] = *(const pr_v4d*)(py + (int64_t)q * ldn + s);
            pr_v4d an = *(const pr_v4d*)(pa + sn), bn = *(const pr_v4d*)(pb + sn);
            __builtin_amdgcn_sched_barrier(0);
            const pr_v4d ac = a - ca;            // 0 past the last sample, as b - cb and y
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const double x = a[e], xc = ac[e], z = b[e], zc = z - cb;
                const double p = DIV ? x : xc, q = DIV ? zc : z;
                acc[TP] = __builtin_amdgcn_mfma_f64_16x16x4f64(xc, zc, acc[TP], 0, 0, 0);
                acc[TP + 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(p * p, q * q, acc[TP + 1], 0, 0, 0);
                acc[TP + 2] = DIV ? __builtin_amdgcn_mfma_f64_16x16x4f64(x * xc, zc, acc[TP + 2], 0, 0, 0)
                                  : __builtin_amdgcn_mfma_f64_16x16x4f64(xc, z * zc, acc[TP + 2], 0, 0, 0);
            }
            const pr_v4d ya = DIV ? a : ac, yb = DIV ? b - cb : b;
#pragma unroll
            for (int t = 0; t < TP; t += G) {
                pr_v4d yn[G];
                if (t + G < TP) {
#pragma unroll
                    for (int q = 0; q < G; q++) yn[q] = *(const pr_v4d*)(py + (int64_t)(t + G + q) * ldn + s);
                }
                __builtin_amdgcn_sched_barrier(0);
                pr_v4d ay[G];
#pragma unroll
                for (int q = 0; q < G; q++) ay[q] = ya * y[q];
#pragma unroll
                for (int e = 0; e < 4; e++)
#pragma unroll
                    for (int q = 0; q < G; q++)
                        acc[t + q] = __builtin_amdgcn_mfma_f64_16x16x4f64(ay[q][e], yb[e], acc[t + q], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (t + G < TP) {
#pragma unroll
                    for (int q = 0; q < G; q++) y[q] = yn[q];
                }
            }
            // (an empty asm takes the loaded operands here, so that the compiler
            // does not move their loads to the top of the next chunk)
            asm("" : "+v"(an.x), "+v"(an.y), "+v"(an.z), "+v"(an.w));
            asm("" : "+v"(bn.x), "+v"(bn.y), "+v"(bn.z), "+v"(bn.w));
            a = an * sa;
            b = bn * sb;
        }
    };
    if (sel == 1) run(std::true_type{});
    else run(std::false_type{});

    const double nn = (double)g.n;
    unsigned cnt = 0;
    // one candidate: score from its numerators and n times its variance, or
    // the fix-up list
    auto emit = [&](int op, int64_t ri, int64_t rj, double varn, double kappa, bool sure, double mean, double msq,
                    const double (&num)[TP]) {
        const int64_t id = pair_id(g.sd, g.r, op, ri, rj);
        if (!sure || !(kappa <= PAIR_KAPPA)) {
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
    // the pair (i, j) with this operator set's sums P_t, C, G1, G2 in m
    auto pair = [&](int i, int j, const double (&m)[TK]) {
        if (!(j < g.jc_end && i < g.i_end && i < j) || !g.valid[i] || !g.valid[j]) return;
        const int64_t ri = g.mat_raw[i], rj = g.mat_raw[j];
        const uint8_t ci = g.cls[i], cj = g.cls[j];
        const short2 xi = g.ex[i], xj = g.ex[j];
        const int ei = sel == 2 ? xi.y : xi.x, ej = sel == 1 ? xj.y : xj.x;
        const double back = ldexp(1.0, ei + ej);     // undoes the scales
        const double C = m[TP];
        double num[TP];
        // the product of this operator set; a zero divisor makes every
        // quotient non-finite (the slot stays invalid)
        const int op = sel == 0 ? OP_MUL : sel == 1 ? OP_DIV : OP_RDIV;
        const uint8_t cd = sel == 0 ? 0 : sel == 1 ? cj : ci;
        if (((g.opmask >> (op - OP_ADD)) & 1u) && !(cd & PC_ZERO)) {
            // A, B: the means of the centred operand and of the other one
            const int ka = sel == 1 ? j : i, kb = sel == 1 ? i : j;
            const double wa = ldexp(1.0, -(sel == 1 ? ej : ei)), wb = ldexp(1.0, -(sel == 1 ? ei : ej));
            const double A = (sel ? g.mur : g.mu)[ka] * wa, B = g.mu[kb] * wb;
            const double qa = (sel ? g.cssr : g.css)[ka] * wa * wa, qb = g.css[kb] * wb * wb;
            const double t1 = A * A * qb, G1 = m[TP + 1];
            const double varn = t1 + G1 + 2.0 * A * m[TP + 2] - C * (C / nn);
            const double mean = fma(A, B, C / nn);
            const bool sure = !(cd & PC_RCP) && pair_range(ei, ej) && t1 + G1 >= PC_S2MIN &&
                              varn > 4.0 * PAIR_CONST * PAIR_CONST * (varn + nn * mean * mean);
            const double kappa = varn > 0.0 ? (t1 + G1 + fabs(C) / nn * sqrt(qa) * sqrt(qb)) / varn : INFINITY;
            const double* fb = g.fy + (int64_t)kb * TP;
#pragma unroll
            for (int t = 0; t < TP; t++) num[t] = fma(A, fb[t] * wb, m[t]) - C / nn * g.ysum[t];
            const double mb = mean * back;
            emit(op, ri, rj, varn, kappa, sure, mb, varn / nn * back * back + mb * mb, num);
        }
        if (sel != 0 || !(g.opmask & 3u)) return;
        const double ma = g.mu[i], mb = g.mu[j], Q = g.css[i] + g.css[j], C1 = C * back;
        const double ab = nn * (g.msq[i] + g.msq[j]);
        const bool range = max(xi.x, xj.x) <= PC_EMAX && max(xi.x, xj.x) >= PC_EMIN;
#pragma unroll
        for (int o = 0; o < 2; o++) {
            if (!((g.opmask >> o) & 1u)) continue;
            const double sg = o == 0 ? 1.0 : -1.0;
            const double mean = fma(sg, mb, ma);
            const double varn = fma(2.0 * sg, C1, Q), ff = varn + nn * mean * mean;
            // (one that may have cancelled to rounding noise is decided exactly as well)
            const bool sure = range && ff > 1e-12 * ab && varn > 4.0 * PAIR_CONST * PAIR_CONST * ff;
            const double kappa = varn > 0.0 ? Q / varn : INFINITY;
#pragma unroll
            for (int t = 0; t < TP; t++) num[t] = fma(sg, g.fy[(int64_t)j * TP + t], g.fy[(int64_t)i * TP + t]);
            emit(OP_ADD + o, ri, rj, varn, kappa, sure, mean, ff / nn, num);
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
            for (int r = 0; r < 4; r++) part[wv][r][lane] = acc[t][r];
            __syncthreads();
            m[t] = ((part[0][wv][lane] + part[1][wv][lane]) + part[2][wv][lane]) + part[3][wv][lane];
            __syncthreads();
        }
        pair(i0 + kq + 4 * wv, j0 + r16, m);
    } else {
#pragma unroll
        for (int r = 0; r < 4; r++) {
            double m[TK];
#pragma unroll
            for (int t = 0; t < TK; t++) m[t] = acc[t][r];
            pair(i0 + kq + 4 * r, j0 + r16, m);
        }
    }
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor((int)cnt, o, 64);
    if (lane == 0 && cnt) atomicAdd(g.nscored, (unsigned long long)cnt);
}

template <int TP>
void launch(ctab<PairArgs> A, const int4* work, int64_t n, bool split, hipStream_t st) {
    if (split) k_pairs_mm<TP, 4><<<(unsigned)n, 256, 0, st>>>(A, work, n);
    else k_pairs_mm<TP, 1><<<(unsigned)cdiv(n, 4), 256, 0, st>>>(A, work, n);
}

}  // namespace

void launch_pairs_mm(ctab<PairArgs> A, const int4* work, int64_t n, int TP, bool split, hipStream_t st) {
    if (n == 0) return;
    switch (TP) {
    case 1: launch<1>(A, work, n, split, st); break;
    case 2: launch<2>(A, work, n, split, st); break;
    case 4: launch<4>(A, work, n, split, st); break;
    case 8: launch<8>(A, work, n, split, st); break;
    default: launch<16>(A, work, n, split, st); break;
    }
    check_launch("k_pairs_mm");
}

}  // namespace dsc
