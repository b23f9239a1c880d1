// Launchers of the compiled-length Z1 pass in precision double.
#include "ct_z1.h"

namespace dft {

template <>
bool launch_z1_ct<double>(const Geo &g, const Z1Args &a, int es, hipStream_t s) {
    if (!g.tab64) return false;   // no spectral tables (or S > 4 with electrostatics): run-time kernel
    return launch_z1_lengths<double>(g, a, es, s);
}

}  // namespace dft
