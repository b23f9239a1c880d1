// Launchers of the compiled-length X2 pass for the alternative hard-sphere functionals
// (Rosenfeld's original vector form, White Bear): FP64 nodewise work in kernels of their own,
// so the kernels of eq. (Phi) keep their register budget.
#include "ct_x2.h"

namespace dft {

template <typename T, int L>
static int launch_x2_alt_len(const Geo &g, const X2Args &a, hipStream_t s) {
    if constexpr (std::is_same<T, double>::value) {
        if (a.mode == X2_HESS) return launch_x2_form<T, L, X2N_HESS_ALT>(g, a, s);
    } else if (a.mode == X2_HESS) {
        throw std::runtime_error("x2: the Hessian mode has FP64 transforms");
    }
    return launch_x2_form<T, L, X2N_ALT>(g, a, s);
}

template <typename T>
int launch_x2_alt_ct(const Geo &g, const X2Args &a, hipStream_t s) {
    switch (g.nx) {
#define DFT_CASE(n) case n: return launch_x2_alt_len<T, n>(g, a, s);
        DFT_CT_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return 0;
    }
}

template int launch_x2_alt_ct<double>(const Geo &, const X2Args &, hipStream_t);
template int launch_x2_alt_ct<float>(const Geo &, const X2Args &, hipStream_t);

}  // namespace dft
