// Launchers of the compiled-length X2 pass: one precision (DFT_X2_T), class (DFT_X2_CLASS) and group of row
// lengths (DFT_X2_GROUP) a translation unit.
#include "ct_x2.h"

#define DFT_PASTE_(a, b) a##b
#define DFT_PASTE(a, b) DFT_PASTE_(a, b)

namespace dft {

template <>
int launch_x2_unit<DFT_X2_T, DFT_X2_CLASS, DFT_X2_GROUP>(const Geo &g, const X2Args &a, hipStream_t s) {
    switch (g.nx) {
#define DFT_CASE(n) case n: return launch_x2_len<DFT_X2_T, DFT_X2_CLASS, n>(g, a, s);
        DFT_PASTE(DFT_X_GROUP_, DFT_X2_GROUP)(DFT_CASE)
#undef DFT_CASE
        default: throw std::runtime_error("x2: row length of another group");
    }
}

}  // namespace dft
