// Launchers of the compiled-length passes of the RFD screening operator.
#include "ct_screen.h"

namespace dft {

template <int L>
static void launch_ball_len(const Geo &g, const BallArgs &a, hipStream_t s) {
    constexpr int P = ball_width(L), NTB = z_one_threads<double, L>(P);
    const dim3 grid((unsigned)ct_cdiv(g.ny * g.Kx, P), 1, (unsigned)((g.S + 1) / 2));   // flattened (y, kx) columns
    hipLaunchKernelGGL((k_ballc<L, P, NTB>), grid, dim3(NTB), 0, s, g, a);
    ct_check("ball averages");
}

template <int L>
static void launch_ballx_len(const Geo &g, const BallArgs &a, hipStream_t s) {
    const long long waves = ct_cdiv(((long long)g.ny * g.nz + 1) / 2, XRow<L>::PW);
    const int wpb = waves >= 2048 ? 4 : 1;   // few row pairs: blocks of one wave reach more CUs
    const dim3 grid((unsigned)ct_cdiv(waves, wpb), (unsigned)((g.S + 1) / 2), 1);
    hipLaunchKernelGGL((k_ballx<L>), grid, dim3(64 * wpb), 0, s, g, a);
    ct_check("interpolation in the radius");
}

void ball_averages(const Geo &g, const BallArgs &a, hipStream_t s) {
    switch (g.nz) {
#define DFT_CASE(n) case n: launch_ball_len<n>(g, a, s); break;
        DFT_X_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: throw std::runtime_error("ball averages: no compiled kernel for this z length");
    }
    YArgs y{a.specB, a.nodes * g.S, 1, nullptr};
    launch_y<double>(g, y, s);
}

void ball_interpolate(const Geo &g, const BallArgs &a, hipStream_t s) {
    switch (g.nx) {
#define DFT_CASE(n) case n: launch_ballx_len<n>(g, a, s); break;
        DFT_X_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: throw std::runtime_error("interpolation in the radius: no compiled kernel for this x length");
    }
}

}  // namespace dft
