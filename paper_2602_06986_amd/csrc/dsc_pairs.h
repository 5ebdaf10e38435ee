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
// PAIR_KAPPA and k_pair_route).
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
    const double* fy;         // [Mc][TP] sum of (f - mean) y_t
    const int* route;         // the problem's dense pairs: 1 matrix form, 0 vector form; NULL: vector form
};

// Conditioning S2 / (S2 - S1^2 / n) up to which the matrix form's unshifted
// moments are trusted.  The score's error stays below 4 n eps kappa, which
// the selection margin covers (7e-9 at n = 2000); a candidate beyond goes
// to the exact fix-up.  64, the vector form's limit, would send products of
// features with a relative spread below 13 % there.
constexpr double PAIR_KAPPA = 4096.0;

// Range classes of an operand feature f.
enum : uint8_t {
    PC_NARROW = 1,            // variance below 1/2048 of the mean square
    PC_VAL = 2,               // max |f| outside [1e-40, 1e50]
    PC_RCP = 4,               // max |1/f| outside it
    PC_ZERO = 8               // f has a zero
};
constexpr double PC_MAX = 1e50, PC_MIN = 1e-40;
// With the classes' limits a product's square sum has lost at most n 2e-208
// to subnormal squares, nothing of one above this.
constexpr double PC_S2MIN = 1e-180;

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
