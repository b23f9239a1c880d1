// Launchers of the compiled-length y passes (and plain z transforms) in precision double.
#include "ct_y.h"

namespace dft {

// Number of y shapes for a length (0: no compiled kernel).  A shape whose tile does not
// fit the LDS runs as shape 0.
int y_ct_variants(int L, bool) {
    switch (L) {
#define DFT_CASE(n) case n: return kYVariants;
        DFT_CT_LENGTHS(DFT_CASE)
#undef DFT_CASE
#define DFT_CASE(n) case n: return 1;
        DFT_CT_MORE_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return 0;
    }
}

template bool launch_y_ct<double>(const Geo &, const YArgs &, hipStream_t);

}  // namespace dft
