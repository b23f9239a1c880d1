// Launchers of Z1 and Z2 with one wave per transform, in precision float.
#include "ct_zwide.h"

namespace dft {

template bool z1_is_wide<float>(const Geo &);
template bool z2_is_wide<float>(const Geo &);
template bool launch_z1_wide<float>(const Geo &, const Z1Args &, int, hipStream_t);
template bool launch_z2_wide<float>(const Geo &, const Z2Args &, hipStream_t);

}  // namespace dft
