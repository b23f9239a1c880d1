// Launchers of the compiled-length X2 pass.
#include "ct_x2.h"

namespace dft {

// Launches the pass; returns the number of blocks (each writes one n3-maximum partial).
template <typename T, int L>
static int launch_x2_len(const Geo &g, const X2Args &a, hipStream_t s) {
    constexpr int PW = XWide<L>::PW;
    const long long npairs = ((long long)g.ny * g.nz + 1) / 2;
    const bool n3only = a.mode == X2_N3_ONLY;
    const long long nb = ct_cdiv(npairs, n3only ? 4 * PW : PW);
    if (nb > a.red.cap) throw std::runtime_error("x2: reduction buffer too small");
    const dim3 grid((unsigned)nb, 1, (unsigned)g.nprob);
    if (n3only) {
        hipLaunchKernelGGL((k_x2n<T, L>), grid, dim3(256), 0, s, g, a);
    } else if (a.hs != DFT_HS_RSLT) {
        // other functionals: FP64 nodewise work, kernels of their own (launch_x2_alt_ct)
        const int nba = launch_x2_alt_ct<T>(g, a, s);
        if (!nba) throw std::runtime_error("x2: no kernel for this functional");
        return nba;
    } else if constexpr (std::is_same<T, float>::value) {
        // FP32 transforms act on differences from the reference, with FP32 nodewise work
        if (a.mode != X2_FULL || !a.nref || a.n_out || a.dphi_out || a.nref_out)
            throw std::runtime_error("x2: FP32 transforms need the reference densities");
        return launch_x2_form<T, L, X2N_D32>(g, a, s);
    } else if (a.mode == X2_HESS) {
        return launch_x2_form<T, L, X2N_HESS>(g, a, s);
    } else {
        return launch_x2_form<T, L, X2N_FP64>(g, a, s);
    }
    ct_check("x2 (compiled length)");
    return (int)nb;
}

template <typename T>
int launch_x2_ct(const Geo &g, const X2Args &a, hipStream_t s) {
    switch (g.nx) {
#define DFT_CASE(n) case n: return launch_x2_len<T, n>(g, a, s);
        DFT_CT_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return 0;
    }
}

// Row pairs per block of the length's X2 kernel (0: none): bounds the number of n3-maximum partials.
int x2_ct_min_pairs(int nx) {
    switch (nx) {
#define DFT_CASE(n) case n: return XWide<n>::PW;
        DFT_CT_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return 0;
    }
}

template int launch_x2_ct<double>(const Geo &, const X2Args &, hipStream_t);
template int launch_x2_ct<float>(const Geo &, const X2Args &, hipStream_t);

}  // namespace dft
