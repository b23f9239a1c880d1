// Launchers of the compiled-length Z1 pass in precision float: the lengths compiled in one shape.
#include "ct_z1.h"

namespace dft {

template <>
bool launch_z1_more<float>(const Geo &g, const Z1Args &a, int es, hipStream_t s) {
    return launch_z1_more_lengths<float>(g, a, es, s);
}

}  // namespace dft
