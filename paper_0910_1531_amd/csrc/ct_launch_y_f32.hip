// Launchers of the compiled-length y passes (and plain z transforms) in precision float.
#include "ct_y.h"

namespace dft {

template bool launch_y_ct<float>(const Geo &, const YArgs &, hipStream_t);

}  // namespace dft
