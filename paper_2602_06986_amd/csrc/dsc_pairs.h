// Arguments of the streamed pair screens (candidates op(f_i, f_j) of the
// rung above the materialised operand features) and their matrix form.
//
// With unshifted moments the products of all pairs of operand features are
// matrix products over samples:
//   mul   S1 = sum a b,      S2 = sum a^2 b^2,      P_t = sum (a y_t) b
//   div   the same with 1/b in place of b, rdiv with 1/a in place of a
// and a sum or difference follows from sum a b and the features' own sums.
// The matrix form (k_pairs_mm) computes them on the FP64 matrix cores; the
// vector form (k_screen_pairs) shifts every candidate by an estimate of its
// mean, and takes the data that unshifted moments cannot carry (see
// pair_kappa and k_pair_route).
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
    double kappa;             // conditioning the matrix form's moments are trusted to (pair_kappa)
    const double* fy;         // [Mc][TP] sum of (f - mean) y_t
    const int* route;         // form of the problem's dense pairs: 1 matrix, 0 vector
};

// Conditioning S2 / (S2 - S1^2 / n) up to which the matrix form's unshifted
// moments are trusted: a score's error stays below 4 n eps kappa, and this
// keeps it within PAIR_MARGIN, which the selection margin covers (some
// hundred more pool entries among 10^8 candidates).  A candidate beyond
// goes to the exact fix-up.  At n = 2000 that is 2e6, the product of two
// columns with a spread of 0.1 % of their means; 64, the vector form's
// limit, would send products of columns with one of 13 % there.
constexpr double PAIR_MARGIN = 2e-6;
inline double pair_kappa(int n) { return PAIR_MARGIN / (4.0 * n * 1.1102230246251565e-16); }

// Range classes of an operand feature f.
enum : uint8_t {
    PC_NARROW = 1,            // variance below 4 / pair_kappa of the mean square
    PC_RCP = 4,               // 1/f overflows though f has no zero
    PC_ZERO = 8               // f has a zero
};
// The matrix form scales every feature by a power of two so that its
// largest value lies in [1, 2) (correlations do not change), so squares
// neither overflow nor vanish; a product whose largest possible value lies
// outside [2^-480, 2^498] goes to the exact fix-up, which knows whether its
// values and their squares are finite, and so does one whose scaled square
// sum is small enough for subnormal squares to matter.
constexpr int PC_EMIN = -480, PC_EMAX = 498;
constexpr double PC_S2MIN = 1e-250;

// Samples padded to whole 16-sample chunks are read: Vf, Rf and Yn hold
// zeros from n to ldn (a multiple of 64).
// Tile shapes: 0: 16 x 16, its samples split over the four waves of a block,
// 1: 16 x 16 per wave, 2: per wave 32 x 32 for one target, 16 x 32 for
// eight.  Rows and columns for padded target count TP:
void pairs_mm_tile(int TP, int shape, int& rows, int& cols);

// Work items (problem, first row i0, first column j0, operator set: 0 mul,
// add and sub, 1 div, 2 rdiv).
void launch_pairs_mm(ctab<PairArgs> A, const int4* work, int64_t n, int TP, int shape, hipStream_t st);

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
