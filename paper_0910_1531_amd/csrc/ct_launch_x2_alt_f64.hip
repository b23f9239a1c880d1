// Launchers of the compiled-length X2 pass of the alternative functionals, transforms in precision double.
#include "ct_x2.h"

namespace dft {

template int launch_x2_alt_ct<double>(const Geo &, const X2Args &, hipStream_t);

}  // namespace dft
