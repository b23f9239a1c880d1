// Launchers of the compiled-length X2 pass in precision double.
#include "ct_x2.h"

namespace dft {

// Row pairs per block of the length's X2 kernel (0: none): bounds the number of n3-maximum partials.
int x2_ct_min_pairs(int nx) {
    switch (nx) {
#define DFT_CASE(n) case n: return XRow<n>::PW;
        DFT_X_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return 0;
    }
}

template int launch_x2_ct<double>(const Geo &, const X2Args &, hipStream_t);

}  // namespace dft
