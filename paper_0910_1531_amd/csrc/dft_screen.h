// Launch interface of the RFD screening-operator kernels (host side).
#pragma once

#include "dft_kernels.h"

namespace dft {

// Per-block minima and maxima of r[0 .. n) and counts of entries that are not positive and
// finite; returns the number of blocks written (at most cap).
int rsc_range(long long n, const double *r, double *pmin, double *pmax, int *pbad, int cap, hipStream_t s);

// Barycentric interpolation in the radius on the M first-kind Chebyshev points
// R_j = cc + dd cos((2 j + 1) pi / (2 M)) with weights (-1)^j sin((2 j + 1) pi / (2 M)):
// per point the reciprocal of sum_j w_j / (r - R_j), or the index j where r equals R_j.  The points
// are computed once on the host: every kernel has to subtract the same R_j from r.
struct ChebNodes {
    double R[DFT_RFD_MAX_NODES], w[DFT_RFD_MAX_NODES];
};
void cheb_prep(long long n, const double *r, int M, const ChebNodes &nd, double *inv_den, int *hit, hipStream_t s);
// out[i][x] (=, first node; += otherwise) l_m(r(x)) part[i][x] for the S fields.
void cheb_accum(long long n, int S, int m, const ChebNodes &nd, const double *r, const double *inv_den, const int *hit,
                const double *part, double *out, bool first, hipStream_t s);

// One batch of radii on the compiled z lengths: the fields' full spectra in specA -> ball averages of radii
// m0 .. m0 + nodes - 1 in specB slots (nodes S of them; ball_averages, after the inverse y pass) -> on the
// compiled x lengths, their interpolation at every point's R_SC written (first) or added to out
// (ball_interpolate; other x lengths transform and accumulate the slots one radius at a time).
constexpr int kBallSlots = DFT_NALPHA;   // slots of specB
struct BallArgs {
    const void *specA;
    void *specB;
    int nodes, m0, first;
    double R[kBallSlots], w[kBallSlots];   // radii and barycentric weights of the batch
    const double *rsc, *inv_den;           // [N]
    const int *hit;                        // [N]
    double *out;                           // [S][N]
};
void ball_averages(const Geo &g, const BallArgs &a, hipStream_t s);
void ball_interpolate(const Geo &g, const BallArgs &a, hipStream_t s);

}  // namespace dft
