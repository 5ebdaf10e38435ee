// Arguments of the streamed pair screens (candidates op(f_i, f_j) of the
// rung above the materialised operand features) and their matrix form.
//
// With A, B the means of a and b, a' = a - A and b' = b - B, a product
// shifted by the product of the means is ab - AB = A b' + a' b, whose
// moments are matrix products over samples:
//   C  = sum a' b',  G1 = sum a'^2 b^2,  G2 = sum a' (b b'),  P_t = sum (a' y_t) b
//   sum (ab - AB) = C,  sum (ab - AB)^2 = A^2 sum b'^2 + G1 + 2 A G2,
//   sum (ab - AB) y_t = A sum b' y_t + P_t;
// rdiv is the same with 1/a in place of a; div with 1/b in the place of a
// and a in that of b (a reciprocal's mean often comes from a few large
// values, which A b' + a' b then cancels least); a sum or difference follows
// from C and the features' own sums.  The matrix form (k_pairs_mm) computes
// them on the FP64 matrix cores; the vector form (k_screen_pairs) forms every
// shifted value itself, and takes data whose pairs cancel in those sums.
#pragma once

#include "dsc_common.h"
#include "dsc_space.h"

namespace dsc {

struct PairArgs {
    const int2* tiles;        // precision form: (jc, ic0) per wave
    const int32_t* ilist;     // explicit partner lists (list mode) or NULL
    int64_t n_tiles;
    int n, ldm, ldn, Mc, jc_end, i_end;   // i_end: end of the partner pool
    const double *Vs, *Rs, *Cs, *Vf, *Rf, *Cf, *mu, *mur;
    const uint8_t* valid;
    const int64_t* mat_raw;
    const double* Yn;
    const double* ysum;
    int T, mode, r;
    uint32_t opmask;          // runtime enabled subset of OPS (bits as above)
    SpaceDev sd;
    int64_t N;
    double* scores;
    unsigned long long* nscored;
    int64_t* fix_ids;         // candidates whose moments are ill-conditioned
    unsigned long long* fix_cnt;
    int64_t fix_cap;
    uint8_t* r2v;             // rung-2 operand statistics for a streamed rung 3 (or NULL)
    double* r2m;
    double* r2q;
    const double* msq;        // mean square of every operand feature
    const uint8_t* cls;       // range class of every operand feature (PC_*)
    const short2* ex;         // binary exponents of max |f| and max |1/f|
    const double *css, *cssr; // [Mc] sums of squares of f and of 1/f about their means
    const double* fy;         // [Mc][TP] sum of (f - mean) y_t
    const unsigned* bad;      // weight of the probes that cancel: above PROBE_MAX the vector form takes the problem
};

// Conditioning the matrix form trusts: K = (A^2 sum b'^2 + G1 + |C| sqrt(sum
// a'^2 sum b'^2) / n) / V for products and (sum a'^2 + sum b'^2) / V for sums
// and differences, V the candidate's centred sum of squares.  Rounding moves
// a score by at most g (K + 1.5 sqrt K), g = (n + 10) eps; K <= 128 keeps
// that below 4 n eps 64, the bound of the vector form at its own limit.  A
// candidate beyond goes to the exact fix-up.
constexpr double PAIR_KAPPA = 128.0;
// A candidate whose standard deviation lies within twice this share of its
// root mean square is decided exactly as well (the rule's own limit is 1e-8).
constexpr double PAIR_CONST = 1e-8;

// Range classes of an operand feature f.
enum : uint8_t {
    PC_RCP = 4,               // 1/f overflows though f has no zero
    PC_ZERO = 8               // f has a zero
};
// The matrix form scales every feature by a power of two so that its
// largest value lies in [1, 2) (correlations do not change), so squares
// neither overflow nor vanish; a product of which an operand, or the largest
// possible value, lies outside [2^-480, 2^498] goes to the exact fix-up,
// which knows whether its values and their squares are finite, and so does
// one whose scaled square sum is small enough for subnormal squares to
// matter.
constexpr int PC_EMIN = -480, PC_EMAX = 498;
constexpr double PC_S2MIN = 1e-250;

__host__ __device__ inline bool pair_range(int ei, int ej) {
    return ei >= PC_EMIN && ej >= PC_EMIN && ei + ej >= PC_EMIN && ei <= PC_EMAX && ej <= PC_EMAX && ei + ej <= PC_EMAX;
}

// Which form takes a problem's dense pairs: the matrix form unless more than
// 1 in 64 of its candidates would go to the exact fix-up, estimated from up
// to PAIR_PROBES of them.  The fix-up decides 73 candidates a microsecond at
// n = 2000 with 8 targets, 126 with one, 400 at n = 500, and the matrix form
// saves 1600, 500 and 45 us of 2.9, 2.9 and 1.2 million: as much as the
// fix-up of 1 in 25, 45 and 67 costs.  Data beyond it (columns that are
// nearly multiples of one another, whose quotients cancel) takes the vector
// form.  Decided on the device: it depends on the data and must hold for a
// captured call.  The probes of a problem weigh PAIR_PROBES together.
constexpr int PAIR_PROBES = 1024;
constexpr unsigned PROBE_MAX = PAIR_PROBES / 64;

// Samples padded to whole 16-sample chunks are read: Vf and Rf hold the
// feature's mean from n to ldn (a multiple of 64), Yn zeros, so that every
// product has a factor 0 there.
// Work items (problem, first row i0, first column j0, operator set: 0 mul,
// add and sub, 1 div, 2 rdiv) of 16 x 16 pairs; split: the four waves of a
// block share an item, else each takes one.
void launch_pairs_mm(ctab<PairArgs> A, const int4* work, int64_t n, int TP, bool split, hipStream_t st);

// One slot of a counter-indexed list for every active lane of the wave
// (lane order), with a single atomic: for appends made inside divergent
// code, where the active lanes are exactly those that append.
__device__ __forceinline__ unsigned long long wave_slot(unsigned long long* ctr) {
    const uint64_t m = __builtin_amdgcn_ballot_w64(true);
    const int lane = threadIdx.x & 63;
    const int leader = __ffsll((long long)m) - 1;
    unsigned long long base = 0;
    if (lane == leader) base = atomicAdd(ctr, (unsigned long long)__popcll(m));
    base = __shfl(base, leader, 64);
    return base + (unsigned long long)__popcll(m & ((1ull << lane) - 1ull));
}

}  // namespace dsc
