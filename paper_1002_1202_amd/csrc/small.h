#pragma once
#include "kernels.h"

namespace gsc {

// One column of a small system iterated by one workgroup (small.hip): what the
// kernel takes over from a tile after its set-up (r, r'_0, p, rho and the
// shifts' state in place) and hands back when every column is finished.
struct SmallSolve {
    const int32_t *rowptr, *colidx;
    const double *S, *H;
    int N, nb, B, K, R, Rp, m;
    const c128 *p, *r, *rp;          // [N][Rp]: p_0, r_0, r'_0
    ColState cs;
    ShiftState ss;
    // Chebyshev iteration of the inner solve: interval, steps, tolerance
    double theta, delta, rho, inner_tol;
    int steps;
    double tol;
    int max_iter;
    // full carry (X != nullptr): x^k and p^k, the ring of r' by columns
    c128 *X, *P, *ringT;
    size_t ldx, ldp;
    // projected carry: unit projections, the S e_a row, h and g (or the
    // z-derivative carry's dh, weights and sums)
    int Mu, srow;
    const int64_t *rhs;
    const int32_t *pidx;
    c128 *h, *g, *dh, *acc;
    const double *wE;
    double *packed;                  // workspace of small_packed() values: S and H by lanes
    int nj;                          // small_lane_blocks()
    int *switches;                   // seed switches and restarts, summed over columns
};

// whether one workgroup a column is the way for R columns of M projections, or of
// the full carry of K shifts
bool small_fits(const Pair &pr, int K, bool full, int M, int R, int num_cu);
// stored blocks a lane takes of the longest block row
int small_lane_blocks(const Pair &pr);
size_t small_packed(const Pair &pr, int nj);
void launch_small_solve(hipStream_t st, const Pair &pr, const SmallSolve &a);

}  // namespace gsc
