// Launchers of the compiled-length x passes X1 and X3, and the choice of X2's launcher.
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

// Row pairs per block of the length's X2 kernel (0: none): bounds the number of n3-maximum partials.
int x2_ct_min_pairs(int nx) {
    switch (nx) {
#define DFT_CASE(n) case n: return XRow<n>::PW;
        DFT_X_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return 0;
    }
}

// Group of a row length (-1: no compiled kernel).
static int x_group(int nx) {
    switch (nx) {
#define DFT_CASE(n) case n:
        DFT_X_GROUP_0(DFT_CASE) return 0;
        DFT_X_GROUP_1(DFT_CASE) return 1;
        DFT_X_GROUP_2(DFT_CASE) return 2;
        DFT_X_GROUP_3(DFT_CASE) return 3;
        DFT_X_GROUP_4(DFT_CASE) return 4;
        DFT_X_GROUP_5(DFT_CASE) return 5;
#undef DFT_CASE
        default: return -1;
    }
}

template <typename T, int CLASS, int GROUP = 0>
static int launch_x2_class(int group, const Geo &g, const X2Args &a, hipStream_t s) {
    if constexpr (GROUP == kXGroups) return 0;
    else return group == GROUP ? launch_x2_unit<T, CLASS, GROUP>(g, a, s) : launch_x2_class<T, CLASS, GROUP + 1>(group, g, a, s);
}

// Launches the pass; returns the number of blocks (each writes one n3-maximum partial; 0: no compiled kernel).
template <typename T>
int launch_x2_ct(const Geo &g, const X2Args &a, hipStream_t s) {
    constexpr bool F32 = std::is_same<T, float>::value;
    const int group = x_group(g.nx);
    if (group < 0) return 0;
    if (a.mode == X2_N3_ONLY) return launch_x2_class<T, X2C_PLAIN>(group, g, a, s);
    if (a.hs != DFT_HS_RSLT) {
        if (a.mode != X2_HESS) return launch_x2_class<T, X2C_ALT>(group, g, a, s);
        if constexpr (!F32) return launch_x2_class<T, X2C_HESS_ALT>(group, g, a, s);
        throw std::runtime_error("x2: the Hessian mode has FP64 transforms");
    }
    if constexpr (F32) {
        if (a.mode != X2_FULL || !a.nref || a.n_out || a.dphi_out || a.nref_out)
            throw std::runtime_error("x2: FP32 transforms need the reference densities");
    } else {
        if (a.mode == X2_HESS) return launch_x2_class<T, X2C_HESS>(group, g, a, s);
    }
    return launch_x2_class<T, X2C_PLAIN>(group, g, a, s);
}

template int launch_x2_ct<double>(const Geo &, const X2Args &, hipStream_t);
template int launch_x2_ct<float>(const Geo &, const X2Args &, hipStream_t);
template bool launch_x1_ct<double>(const Geo &, const XFwdArgs &, hipStream_t);
template bool launch_x1_ct<float>(const Geo &, const XFwdArgs &, hipStream_t);
template bool launch_x3_ct<double>(const Geo &, const X3Args &, hipStream_t);
template bool launch_x3_ct<float>(const Geo &, const X3Args &, hipStream_t);

}  // namespace dft
