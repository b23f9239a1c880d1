// Launchers of the compiled-length x passes X1 and X3.
#include "ct_rows.h"

namespace dft {

// Waves per block, each with its own row pairs: four, or one where the point has so few row pairs
// that blocks of one wave reach more CUs.  By the point's own size only, so that the order of the
// residual sums is the same alone and in a batch.
template <int L>
static int waves_per_block(const Geo &g) {
    const long long npairs = ((long long)g.ny * g.nz + 1) / 2;
    return ct_cdiv(npairs, XRow<L>::PW) * g.S >= 2048 ? 4 : 1;
}

template <int L>
static long long x_blocks(const Geo &g) {
    return ct_cdiv(((long long)g.ny * g.nz + 1) / 2, (long long)XRow<L>::PW * waves_per_block<L>(g));
}

template <typename T, int L>
static void launch_x1c_len(const Geo &g, const XFwdArgs &a, hipStream_t s) {
    const dim3 grid((unsigned)x_blocks<L>(g), (unsigned)a.nfield, (unsigned)g.nprob);
    hipLaunchKernelGGL((k_x1c<T, L>), grid, dim3(64 * waves_per_block<L>(g)), 0, s, g, a);
    ct_check("x1 (compiled length)");
}

template <typename T, int L>
static void launch_x3c_len(const Geo &g, const X3Args &a, hipStream_t s) {
    const long long nb = x_blocks<L>(g);
    if (!a.raw && nb * a.nfield > a.red.cap) throw std::runtime_error("x3: reduction buffer too small");
    const dim3 grid((unsigned)nb, (unsigned)a.nfield, (unsigned)g.nprob);
    hipLaunchKernelGGL((k_x3c<T, L>), grid, dim3(64 * waves_per_block<L>(g)), 0, s, g, a);
    ct_check("x3 (compiled length)");
}

template <typename T>
bool launch_x1_ct(const Geo &g, const XFwdArgs &a, hipStream_t s) {
    switch (g.nx) {
#define DFT_CASE(n) case n: launch_x1c_len<T, n>(g, a, s); return true;
        DFT_X_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return false;
    }
}

template <typename T>
bool launch_x3_ct(const Geo &g, const X3Args &a, hipStream_t s) {
    switch (g.nx) {
#define DFT_CASE(n) case n: launch_x3c_len<T, n>(g, a, s); return true;
        DFT_X_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return false;
    }
}

// Blocks per field of the compiled-length X3 (0: the length has none); each writes one partial.
long long x3_ct_blocks(const Geo &g) {
    switch (g.nx) {
#define DFT_CASE(n) case n: return x_blocks<n>(g);
        DFT_X_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return 0;
    }
}

template bool launch_x1_ct<double>(const Geo &, const XFwdArgs &, hipStream_t);
template bool launch_x1_ct<float>(const Geo &, const XFwdArgs &, hipStream_t);
template bool launch_x3_ct<double>(const Geo &, const X3Args &, hipStream_t);
template bool launch_x3_ct<float>(const Geo &, const X3Args &, hipStream_t);

}  // namespace dft
