// Launchers of the compiled-length Z1 pass in precision float.
#include "ct_z1.h"

namespace dft {

template <>
bool launch_z1_ct<float>(const Geo &g, const Z1Args &a, int es, hipStream_t s) {
    if (!g.tab64) return false;   // no spectral tables (or S > 4 with electrostatics): run-time kernel
    // the on-the-fly pair factors take sin and cos of k (R_i + R_j) by the addition theorem, so a
    // screening cutoff at lambda_i + lambda_j runs the run-time-length kernel
    if (es && g.cut_lambda) return false;
    return launch_z1_lengths<float>(g, a, es, s);
}

}  // namespace dft
