// Launchers of the compiled-length X2 pass in precision float.
#include "ct_x2.h"

namespace dft {

template int launch_x2_ct<float>(const Geo &, const X2Args &, hipStream_t);

}  // namespace dft
